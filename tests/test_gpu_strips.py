"""The streaming kernels at widths, leading dimensions and base addresses that are multiples of nothing, and
the kernels that hold whole columns of B for a short inner dimension: every integer stage against the
oracle, bit for bit, at the edges of their shapes."""
import numpy as np
import pytest

from oracle import srq_oracle as o

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
F32 = np.float32


@pytest.fixture(scope="module")
def srq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_06924_amd import binding as b
    h = b.Srq(device=0)
    yield h
    h.close()


@pytest.fixture(scope="module")
def b():
    from paper_2403_06924_amd import binding
    return binding


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def host(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("cols", [1, 3, 6, 61, 1025, 2050])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("layout", [0, 1])
def test_windows_that_start_anywhere(srq, b, cols, axis, layout):
    """X as a window one element into rows of odd length: codes and scales against the oracle, residual codes
    and selection against the same call on a contiguous copy."""
    rng = np.random.default_rng(cols + axis)
    big = (rng.standard_normal((77, cols + 4 - (cols + 1) % 2)) * np.exp(rng.standard_normal((77, 1)))).astype(F32)
    big[3] = 0
    big[5, :] = F32(1e-38)                                   # qmax / amax overflows there (rows), or nearly so
    W = dev(big)[:, 1:cols + 1]
    assert W.stride(0) % 2 == 1 and W.data_ptr() % 16 == 4    # (rows start at every multiple of 4 bytes)
    X = big[:, 1:cols + 1]
    name = "row" if axis == 0 else "col"
    with np.errstate(all="ignore"):
        q_ref, s_ref, lam_ref = o.quantize_vectors(np.delete(X, 5, axis=0), name)
    keep = [i for i in range(77) if i != 5]
    Q, s, lam = srq.quantize(dev(big[keep])[:, 1:cols + 1], axis, layout=layout)
    vm = q_ref if axis == 0 else q_ref.T
    assert (host(s) == s_ref).all() and (host(lam) == lam_ref).all()
    assert (host(Q) == (vm if layout == 0 else vm.T)).all()
    Q, s, lam = srq.quantize(W, axis, layout=layout)
    Y = W.contiguous()
    Q2, s2, lam2 = srq.quantize(Y, axis, layout=layout)
    assert torch.equal(Q, Q2) and torch.equal(s, s2) and torch.equal(lam, lam2)
    thresh = Y.abs().mean(dim=1 - axis).contiguous()
    r = srq.build_sparse_residual(W, axis, s, lam, thresh, r_layout=layout)
    r2 = srq.build_sparse_residual(Y, axis, s, lam, thresh, r_layout=layout)
    n = int(r["nnz"].item())
    mask = Y.abs() > (thresh.view(-1, 1) if axis == 0 else thresh.view(1, -1))
    assert n == int(mask.sum())
    for key in ("Rq", "rscale", "ptr", "nnz"):
        assert torch.equal(r[key], r2[key]), key
    assert torch.equal(r["idx"][:n], r2["idx"][:n]) and torch.equal(r["val"][:n], r2["val"][:n])


# K at the edges of the strip shapes (256, 512, 1024, 2048, 4096, 8192) and of the padded length, M and N around strips of
# 8 and 16 columns, many vectors
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 17, 2), (33, 9, 63), (130, 15, 255), (65, 33, 256), (64, 70, 257), (31, 129, 512),
                                   (40, 24, 513), (129, 65, 1023), (24, 40, 1024), (33, 31, 1025), (50, 63, 2047), (16, 8, 2048),
                                   (20, 12, 2049), (35, 50, 4095), (17, 9, 4097),
                                   (9, 17, 8192), (5, 6, 8193), (6001, 8, 1100), (10, 6001, 2047), (4097, 40, 100), (40, 4097, 100), (4096, 24, 130)])
@pytest.mark.parametrize("terms", ["both", "a", "b", "dense"])
def test_short_inner_dimension(srq, b, shape, terms):
    M, N, K = shape
    rng = np.random.default_rng(M + 3 * N + 5 * K)
    A = (rng.standard_normal((M, K)) * np.exp(rng.standard_normal((M, 1)))).astype(F32)
    B = (rng.standard_normal((K, N)) * np.exp(rng.standard_normal((1, N)))).astype(F32)
    if M > 2:
        A[1] = 0
    if N > 2:
        B[:, 2] = 0
    theta = 1.5 / K ** 0.5
    ta, tb = (theta if terms != "b" else np.inf), (theta if terms != "a" else np.inf)
    Cin = rng.standard_normal((M, N)).astype(F32)
    stats = b.stats_tensor()
    s = 0.0 if terms == "dense" else 2.0
    C, _, _ = srq.compensated_gemm(dev(A), dev(B), ta, tb, strategy=b.STRATEGY_CSR_MFMA, dense_fallback_density=s, stats=stats,
                                   alpha=0.5, beta=-0.75, C_in=dev(Cin))
    torch.cuda.synchronize()
    im, st = srq.intermediates(M, N, K), b.read_stats(stats)
    ref = o.compensated_gemm(A, B, ta, tb, alpha=0.5, beta=-0.75, C_in=Cin, dense_fallback_density=s,
                             thresh_a=host(im["t_a"]) if terms != "b" else None,
                             thresh_b=host(im["t_b"]) if terms != "a" else None)
    assert (host(im["A_int"]) == ref.A_int).all() and (host(im["B_int"]) == ref.B_int.T).all()
    for key in ("s_a", "s_b", "lam_a", "lam_b", "s_ra", "s_rb"):
        assert (host(im[key]) == getattr(ref, key)).all(), key
    np.testing.assert_allclose(host(im["drow"]), ref.drow, rtol=1e-6)
    np.testing.assert_allclose(host(im["dcol"]), ref.dcol, rtol=1e-6)
    if terms != "a":
        assert (host(im["RA_int"]) == ref.RA_int).all()
        assert st["nnz_b"] == ref.csc_b.nnz and (host(im["b_ptr"]) == ref.csc_b.ptr).all()
    if terms != "b":
        assert (host(im["RB_int"]) == ref.RB_int.T).all()
        assert st["nnz_a"] == ref.csr_a.nnz and (host(im["a_ptr"]) == ref.csr_a.ptr).all()
    if terms in ("both", "a"):
        assert (host(im["a_idx"]) == ref.csr_a.idx).all() and (host(im["a_val"]) == ref.csr_a.val).all()
    if terms in ("both", "b"):
        assert (host(im["b_idx"]) == ref.csc_b.idx).all() and (host(im["b_val"]) == ref.csc_b.val).all()
    assert o.error_rel(ref.C, host(C)) <= 1e-5              # the FP32 output's tolerance everywhere


# more than 2048 vectors together: a wave of the compaction has a whole vector; vectors at the edges of its shapes, and
# counts of vectors that are no multiple of four; the limit on vectors (16384) of a compaction without a scan
@pytest.mark.parametrize("shape", [(1502, 549, 256), (2043, 6, 257), (7, 2042, 1024), (2041, 9, 1025), (9, 2041, 2048), (2049, 1, 3), (2043, 14, 2049), (14, 2043, 3001), (2050, 7, 4095), (5853, 5, 4096),
                                   (16384, 5, 40), (16385, 5, 40), (3, 16385, 130)])
def test_a_wave_per_vector(srq, b, shape):
    test_short_inner_dimension(srq, b, shape, "both")


@pytest.mark.parametrize("shape", [(1, 1), (77, 61), (9, 255), (256, 33), (257, 7), (512, 40), (1023, 9), (1025, 18), (2049, 5),
                                   (4095, 11), (4097, 10), (8192, 6), (8193, 6), (100, 4100)])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("bits", [8, 4])
def test_reduction_of_one_operand(srq, b, shape, axis, bits):
    """Codes, residual codes and compressed form against the definitions, one FP32 rounding per step; shape is
    (vector length, vectors), the operand a window of odd leading dimension."""
    K, nvec = shape
    rng = np.random.default_rng(K + nvec + axis)
    big = (rng.standard_normal((nvec, K) if axis == 0 else (K, nvec))).astype(F32)
    width = big.shape[1]
    W = dev(np.pad(big, ((0, 0), (1, 2 + width % 2))))[:, 1:width + 1]
    V = host(W) if axis == 0 else host(W).T                   # one vector per row
    assert V.shape == (nvec, K)
    Q, s, lam = srq.quantize(W, axis, bits=bits)
    qmax = F32(2 ** (bits - 1) - 1)
    amax = np.abs(V).max(axis=1)
    assert (host(s) == amax / qmax).all() and (host(lam) == qmax / amax).all()
    q = np.clip(np.rint(V * host(lam)[:, None]), -qmax, qmax)
    assert (host(Q) == q).all()
    t = (amax * rng.random(nvec).astype(F32)).astype(F32)
    r = srq.build_sparse_residual(W, axis, s, lam, dev(t), bits=bits)
    res = V - q.astype(F32) * host(s)[:, None]
    ramax = np.abs(res).max(axis=1)
    with np.errstate(all="ignore"):                       # (a residual of zeros)
        rlam = np.where(ramax > 0, qmax / ramax, F32(0)).astype(F32)
    assert (host(r["rscale"]) == ramax / qmax).all()
    assert (host(r["Rq"]) == np.clip(np.rint(res * rlam[:, None]), -qmax, qmax)).all()
    vec, k = np.nonzero(np.abs(V) > t[:, None])
    n = int(r["nnz"].item())
    assert n == len(k) and (host(r["ptr"]) == np.searchsorted(vec, np.arange(nvec + 1))).all()
    assert (host(r["idx"][:n]) == k).all() and (host(r["val"][:n]) == q[vec, k]).all()


@pytest.mark.parametrize("shape", [(4096, 4100), (2049, 6000), (1027, 12300), (2048, 4099), (4096, 10241)])
@pytest.mark.parametrize("axis", [0, 1])
def test_reduction_of_many_vectors(srq, b, shape, axis):
    test_reduction_of_one_operand(srq, b, shape, axis, 8)


@pytest.mark.parametrize("n", [1, 255, 257, 4095, 8192, 16385, 20001])
def test_scan_of_many_counts(srq, b, n):
    """Row pointers over piece, wave and block boundaries of the scan (one and two vectors a launch)."""
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 5)).astype(F32)
    Q, s, lam = srq.quantize(dev(X), 0)
    t = rng.random(n).astype(F32)
    r = srq.build_sparse_residual(dev(X), 0, s, lam, dev(t))
    counts = (np.abs(X) > t[:, None]).sum(axis=1)
    assert (host(r["ptr"]) == np.concatenate([[0], np.cumsum(counts)])).all() and int(r["nnz"].item()) == counts.sum()


@pytest.mark.parametrize("cols", [1, 2, 3, 5, 61, 1023, 2047, 4098, 8191, 8193, 16382, 16385])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("residual", [False, True])
def test_negative_thresholds_keep_what_exists(srq, b, cols, axis, residual):
    """A threshold below zero keeps every entry of its vector, zeros among them, and none of the columns or rows
    past the end of a ragged operand; with and without the residual (which go different ways)."""
    rng = np.random.default_rng(cols)
    X = rng.standard_normal((5, cols)).astype(F32)
    X[:, ::3] = 0
    if axis == 1:
        X = X.T.copy()
    Q, s, lam = srq.quantize(dev(X), axis)
    t = np.array([-1.0, 0.5, -0.0, -np.inf, 0.0], dtype=F32)
    r = srq.build_sparse_residual(dev(X), axis, s, lam, dev(t), want_residual=residual)
    V = X if axis == 0 else X.T
    vec, k = np.nonzero(np.abs(V) > t[:, None])
    assert (vec == 0).sum() == (vec == 3).sum() == cols
    n = int(r["nnz"].item())
    assert n == len(k) and (host(r["ptr"]) == np.searchsorted(vec, np.arange(6))).all()
    assert (host(r["idx"][:n]) == k).all() and (host(r["val"][:n]) == host(Q)[vec, k]).all()


def powers(n):
    """1, 2^-24 and then 2^-54 in every 64th place: added up one after the other in double the small ones are
    lost and 1 + 2^-24 rounds to 1 in FP32; added to each other first, they push it to 1 + 2^-23."""
    x = np.zeros(n, F32)
    x[0], x[1], x[64::64] = 1.0, 2.0 ** -24, 2.0 ** -54
    return x


@pytest.mark.parametrize("shape", [(1024, 1024, 128), (1024, 2048, 512), (512, 1024, 2048), (4096, 4352, 128)])
def test_thresholds_do_not_depend_on_the_execution(srq, b, shape):
    """The same call with either sparse execution, or with either expectation of what the device will decide,
    takes different selection passes; means and thresholds are the same bits.  Two-bit codes of vectors of one
    value make D_F the outer product of `powers`, exactly, so that any difference in the order of the
    additions shows."""
    M, N, K = shape
    A, B = dev(np.repeat(powers(M)[:, None], K, axis=1)), dev(np.repeat(powers(N)[None, :], K, axis=0))
    inf = float("inf")

    def sums(ta, tb, strategy, hint):
        srq.set_auto_hint(*hint)
        srq.compensated_gemm(A, B, ta, tb, bits=2, strategy=strategy)
        torch.cuda.synchronize()
        im = srq.intermediates(M, N, K)
        return [host(im[k]).copy() for k in ("drow", "dcol", "t_a", "t_b")]

    try:
        for ta, tb in ((0.5, 0.5), (0.5, inf), (inf, 0.5)):
            ways = [sums(ta, tb, b.STRATEGY_CSR_MFMA, (0, 0)), sums(ta, tb, b.STRATEGY_CSR_VALU, (0, 0)),
                    sums(ta, tb, b.STRATEGY_AUTO, (2, 2)), sums(ta, tb, b.STRATEGY_AUTO, (1, 1))]
            assert abs(float(ways[0][0][0]) * N / K - 1) < 1e-6 and abs(float(ways[0][1][0]) * M / K - 1) < 1e-6
            for w in ways[1:]:
                for x, y in zip(w, ways[0]):
                    assert x.tobytes() == y.tobytes()
    finally:
        srq.set_auto_hint(0, 0)


# The two launches for K up to 256, at the edges of their 64 x 64 tiles, chunks of sixteen vectors and K-tiles, against the
# same call with its stages as launches of their own (every stage timed): the same bits everywhere
@pytest.mark.parametrize("shape", [(1, 16, 1), (15, 17, 3), (16, 64, 64), (63, 65, 127), (64, 1, 128), (129, 48, 129), (960, 896, 64),
                                   (1000, 1023, 250), (17, 1024, 256), (1024, 33, 192), (1024, 1024, 256)])
@pytest.mark.parametrize("odd", [False, True])
def test_two_launches_are_the_separate_ones(srq, b, shape, odd):
    M, N, K = shape
    gen = torch.Generator(device="cuda").manual_seed(M + 3 * N + 5 * K)
    wide = 3 if odd else 0
    A, B, Cin = (torch.randn((r, c + wide), generator=gen, device="cuda")[:, wide // 2:wide // 2 + c] for r, c in ((M, K), (K, N), (M, N)))
    A[M // 2] = 0
    B[:, N // 2] = 0
    for ta, tb, beta, bits, rounding in ((0.02, 0.02, 0.0, 8, b.ROUND_NEAREST_EVEN), (0.01, np.inf, -0.75, 4, b.ROUND_TRUNC),
                                         (np.inf, 0.0, 0.5, 8, b.ROUND_NEAREST_EVEN), (np.inf, np.inf, 0.5, 5, b.ROUND_TRUNC)):
        got = []
        for separate in (False, True):
            srq.profile_enable(separate)
            stats, out = b.stats_tensor(), torch.full((M, N + wide), -5.0, device="cuda")
            try:
                srq.compensated_gemm(A, B, ta, tb, bits=bits, rounding=rounding, strategy=b.STRATEGY_CSR_MFMA, alpha=1.5, beta=beta,
                                     C_in=Cin, out=out[:, :N], stats=stats)
                torch.cuda.synchronize()
            finally:
                srq.profile_enable(False)
            im = srq.intermediates(M, N, K)
            got.append((out, stats, {k: v.clone() for k, v in im.items() if torch.is_tensor(v)}))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
        assert got[0][2].keys() == got[1][2].keys()
        for key, value in got[0][2].items():               # (bits: a threshold of an infinite factor and a zero mean is no number)
            assert torch.equal(value.contiguous().view(torch.uint8), got[1][2][key].contiguous().view(torch.uint8)), key


@pytest.mark.parametrize("rows,cols,axis", [(0, 5, 1), (5, 0, 0)] + [(*s, a) for s in ((3, 7), (900, 33), (70, 5000), (5000, 70)) for a in (0, 1)])
def test_count_of_nothing_kept(srq, b, rows, cols, axis):
    """The count is written by every call that has entries to look at, and zero where there are none."""
    n = rows if axis == 0 else cols
    X, one, t = torch.ones(rows, cols, device="cuda"), torch.ones(n, device="cuda"), torch.full((n,), float("inf"), device="cuda")
    stale = [torch.full((1,), 7, dtype=torch.int64, device="cuda") for _ in range(64)]
    del stale                                                # what a count that nobody writes would hold
    r = srq.build_sparse_residual(X, axis, one, one, t, want_residual=rows * cols > 0)
    assert int(r["nnz"].item()) == 0 and not host(r["ptr"]).any()


def test_short_calls_on_several_streams(b):
    """Calls in two launches on six streams at once, a handle each: the workgroups that compact wait for those of their own
    call alone.  Every call's result, counts and row pointers are those of the same call by itself."""
    shapes = [(1024, 1024, 256), (1000, 1023, 250), (256, 256, 256), (960, 896, 64), (1024, 33, 192), (513, 1024, 129)]
    gen = torch.Generator(device="cuda").manual_seed(41)
    calls = []
    for M, N, K in shapes:
        h = b.Srq(device=0)
        h.ensure_workspace(b.workspace_bytes(M, N, K, 1.0))
        A, B = torch.randn((M, K), generator=gen, device="cuda"), torch.randn((K, N), generator=gen, device="cuda")
        outs = [torch.empty((M, N), device="cuda") for _ in range(8)]
        stats = [b.stats_tensor() for _ in outs]
        ref, ref_stats = torch.empty((M, N), device="cuda"), b.stats_tensor()
        kw = dict(strategy=b.STRATEGY_CSR_MFMA, max_density=1.0)
        h.compensated_gemm(A, B, 0.03, out=ref, stats=ref_stats, **kw)
        torch.cuda.synchronize()
        im = h.intermediates(M, N, K)
        calls.append((h, A, B, outs, stats, ref, ref_stats, {k: im[k].clone() for k in ("a_ptr", "a_idx", "b_ptr", "b_idx")}, kw,
                      torch.cuda.Stream()))
    torch.cuda.synchronize()
    try:
        for i in range(8):
            for h, A, B, outs, stats, _, _, _, kw, stream in calls:
                with torch.cuda.stream(stream):
                    h.compensated_gemm(A, B, 0.03, out=outs[i], stats=stats[i], **kw)
        torch.cuda.synchronize()
        for (M, N, K), (h, _, _, outs, stats, ref, ref_stats, kept, _, _) in zip(shapes, calls):
            assert b.read_stats(ref_stats)["nnz_a"] > 0
            for out, st in zip(outs, stats):
                assert torch.equal(out, ref) and torch.equal(st, ref_stats)
            im = h.intermediates(M, N, K)
            for key, value in kept.items():
                assert torch.equal(im[key], value), key
    finally:
        for c in calls:
            c[0].close()


# without compensation C may take the place of an operand: both are quantized before it is written, also where workgroups
# start one after the other because another stream keeps the compute units busy
@pytest.mark.parametrize("n", [64, 250, 256])
def test_product_in_place_of_an_operand(srq, b, n):
    gen = torch.Generator(device="cuda").manual_seed(n)
    inf, side, load = float("inf"), torch.cuda.Stream(), torch.ones(1 << 26, device="cuda")
    for M, N in ((n, n), (1000, n), (n, 1000)):
        for place in ("a", "b", "rows of b"):
            A, B = torch.randn((M, n), generator=gen, device="cuda"), torch.randn((n, N), generator=gen, device="cuda")
            ref = torch.empty((M, N), device="cuda")
            srq.compensated_gemm(A, B, inf, out=ref)
            if place == "a" and N == n:
                out = A
            elif place == "b" and M == n:
                out = B
            else:                                            # B lies within C
                out = torch.empty(M + n, N, device="cuda")
                out[M // 2:M // 2 + n] = B
                out, B = out[:M], out[M // 2:M // 2 + n]
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                for _ in range(4):
                    load.mul_(1.0)
            srq.compensated_gemm(A, B, inf, out=out)
            torch.cuda.synchronize()
            assert torch.equal(out, ref), (M, N, place)


# (M, N, K): one tile and one over 256 of them, more than 512; one, two, four and eight pieces of a vector; vectors that are no
# whole group of four, K no multiple of 16; both selections (FP32 up to 1024)
@pytest.mark.parametrize("shape", [(65, 70, 260), (300, 401, 1000), (1024, 1024, 1024), (1029, 1020, 515), (1500, 1501, 700), (2100, 63, 257),
                                   (333, 270, 1025), (513, 515, 2049), (90, 1111, 4100)])
@pytest.mark.parametrize("alpha,beta", [(1.0, 0.0), (-0.5, 0.25)])
@pytest.mark.parametrize("bits,share", [(8, 2.0), (8, 0.2), (4, 2.0)])   # (share: a few percent, most of the entries)
def test_compaction_behind_the_tiles(srq, b, shape, alpha, beta, bits, share):
    """The corrections that compact their operands in the same launch against separate launches (a call with debug
    outputs): the same bits in C, CSR / CSC and statistics, also where a vector keeps nothing or everything."""
    M, N, K = shape
    rng = np.random.default_rng(sum(shape))
    A, B = rng.standard_normal((M, K)).astype(F32), rng.standard_normal((K, N)).astype(F32)
    A[2] = 0
    A[5] *= 10
    A[6, 3] = np.nan
    B[:, -1] *= 10
    B[::2, 1] = 2.0 ** -140
    C_in = dev(rng.standard_normal((M, N)).astype(F32)) if beta else None
    theta, got = share / K ** 0.5, []
    for debug in (False, True):
        stats = b.stats_tensor()
        C, _, _ = srq.compensated_gemm(dev(A), dev(B), theta, theta, bits=bits, strategy=b.STRATEGY_CSR_MFMA, alpha=alpha, beta=beta, C_in=C_in,
                                       stats=stats, debug=debug)
        torch.cuda.synchronize()
        im = srq.intermediates(M, N, K)
        got.append([host(C)] + [host(im[s + n]).copy() for s in "ab" for n in ("_ptr", "_idx", "_val")] + [b.read_stats(stats)])
    for x, y in zip(got[0][:-1], got[1][:-1]):
        assert np.array_equal(x, y, equal_nan=x.dtype.kind == "f")
    assert got[0][-1] == got[1][-1] and got[0][-1]["nnz_a"] == len(got[0][2]) > 0 and got[0][-1]["nnz_b"] == len(got[0][5]) > 0
