"""Columns of a matrix quantized in one read (workgroups that exchange maxima) and the selection from codes and residual
codes, against the definitions, bit for bit, at the edges of pieces, strips and vectors."""
import numpy as np
import pytest

from test_gpu_strips import F32, dev, host, test_reduction_of_one_operand as reduction

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def b():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_06924_amd import binding
    return binding


@pytest.fixture(scope="module")
def srq(b):
    h = b.Srq(device=0)
    yield h
    h.close()


@pytest.fixture(scope="module", params=["20000", "0"])
def exchanging(b, request):
    """A handle whose workgroups wait for each other, and one where whoever does not find a maximum at once works it out
    alone."""
    with pytest.MonkeyPatch.context() as m:
        m.setenv("SRQ_EXCHANGE_WAIT_TICKS", request.param)
        h = b.Srq(device=0)
    yield h
    h.close()


# (rows, columns): pieces of 512 rows, patches of 16, strips of 32 columns, the last columns no whole patch
@pytest.mark.parametrize("shape", [(4097, 4), (4100, 5), (4111, 31), (4607, 33), (4608, 34), (4609, 67), (8704, 98), (16385, 6), (32768, 9)])
@pytest.mark.parametrize("bits", [8, 3])
def test_columns_in_one_read(exchanging, b, shape, bits):
    reduction(exchanging, b, shape, 1, bits)


@pytest.mark.parametrize("shape", [(1100, 1030, 4099), (40, 2050, 8192), (2100, 37, 16385)])
@pytest.mark.parametrize("bits,trunc", [(8, 0), (5, 1)])
def test_columns_in_one_read_of_a_whole_call(exchanging, b, shape, bits, trunc):
    """Codes, scales, residual codes and residual scales of B against those of the rows of its transpose, which nothing is
    exchanged for."""
    M, N, K = shape
    rng = np.random.default_rng(K + bits)
    A, B = rng.standard_normal((M, K)).astype(F32), rng.standard_normal((K, N)).astype(F32)
    B[:, 3], B[:, 4], B[7, 5], B[-1, 6] = 0, F32(1e-39), np.nan, 1e38
    rounding = b.ROUND_TRUNC if trunc else b.ROUND_NEAREST_EVEN
    exchanging.compensated_gemm(dev(A), dev(B), 0.03, bits=bits, rounding=rounding)
    torch.cuda.synchronize()
    im = {key: t.clone() for key, t in exchanging.intermediates(M, N, K).items() if key in ("B_int", "s_b", "lam_b", "RB_int", "s_rb")}
    V = dev(B.T.copy())
    Q, s, lam = exchanging.quantize(V, b.AXIS_ROW, bits=bits, rounding=rounding)
    r = exchanging.build_sparse_residual(V, b.AXIS_ROW, s, lam, None, bits=bits, rounding=rounding, want_selection=False)
    for key, ref in (("B_int", Q), ("s_b", s), ("lam_b", lam), ("RB_int", r["Rq"]), ("s_rb", r["rscale"])):
        assert torch.equal(im[key], ref), key


def test_columns_in_one_read_on_several_streams(b):
    """Calls on four streams at once, a handle each, with more workgroups than the chip holds: those that exchange maxima may be
    kept from starting by the others' for as long as they wait.  Every call's outputs are those of the same call by itself."""
    gen = torch.Generator(device="cuda").manual_seed(43)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    def quantize(h, X):
        return h.quantize(X, b.AXIS_COL)

    def reduction(h, X):
        Q, s, lam = h.quantize(X, b.AXIS_COL)
        r = h.build_sparse_residual(X, b.AXIS_COL, s, lam, 50 * s)
        n = X.numel() // 20                                   # (some 12 % are kept)
        return [r["Rq"], r["rscale"], r["ptr"], r["nnz"], r["idx"][:n], r["val"][:n]]

    def whole(h, X):
        return [h.compensated_gemm(X[:1500], X[1500:6500, :2000], 0.03)[0]] if X.shape == (6500, 5000) else \
               [h.compensated_gemm(X[:, :9000], X[:, 9000:].reshape(9000, -1), 0.03)[0]]

    calls = [(quantize, normal(16385, 3000)), (reduction, normal(8192, 4096)), (whole, normal(6500, 5000)), (whole, normal(1800, 18000))]
    calls = [(b.Srq(device=0), torch.cuda.Stream(), run, X) for run, X in calls]
    try:
        refs = [[t.clone() for t in run(h, X)] for h, _, run, X in calls]
        torch.cuda.synchronize()
        outs = [[] for _ in calls]
        for _ in range(6):
            for (h, stream, run, X), out in zip(calls, outs):
                with torch.cuda.stream(stream):
                    out.append(run(h, X))
        torch.cuda.synchronize()
        for ref, out in zip(refs, outs):
            for got in out:
                assert all(torch.equal(x, y) for x, y in zip(got, ref))
    finally:
        for h, _, _, _ in calls:
            h.close()


@pytest.mark.parametrize("shape", [(4099, 37), (4608, 32)])
def test_other_layouts_and_parts_of_the_reduction(exchanging, b, shape):
    X = torch.randn(shape, generator=torch.Generator(device="cuda").manual_seed(shape[1]), device="cuda")
    X[:, 3] = 0
    X[:, 4] = 1e-39                                           # (qmax / amax overflows)
    t = X.abs().mean(dim=0).contiguous()
    for rounding in (b.ROUND_NEAREST_EVEN, b.ROUND_TRUNC):
        Q, s, lam = exchanging.quantize(X, b.AXIS_COL, rounding=rounding)
        Qt, st, lamt = exchanging.quantize(X.t().contiguous(), b.AXIS_ROW, rounding=rounding)
        assert torch.equal(Q, Qt) and torch.equal(s, st) and torch.equal(lam, lamt)
        r = exchanging.build_sparse_residual(X, b.AXIS_COL, s, lam, t, rounding=rounding)
        rt = exchanging.build_sparse_residual(X.t().contiguous(), b.AXIS_ROW, s, lam, t, rounding=rounding)
        em = exchanging.build_sparse_residual(X, b.AXIS_COL, s, lam, t, rounding=rounding, r_layout=b.LAYOUT_ELEMENT_MAJOR)
        n = int(r["nnz"].item())
        for key in ("Rq", "rscale", "ptr", "nnz"):
            assert torch.equal(r[key], rt[key]), key
            assert torch.equal(r[key], em[key].t() if key == "Rq" else em[key]), key
        assert torch.equal(r["idx"][:n], rt["idx"][:n]) and torch.equal(r["val"][:n], rt["val"][:n])


def operand(rng, kind, nvec, K):
    """nvec vectors of K entries, special ones among them."""
    if kind == "normal":
        V = rng.standard_normal((nvec, K))
    elif kind == "outliers":                                  # most codes are 0 or 1: the residual codes decide
        V = rng.standard_normal((nvec, K))
        V[:, rng.integers(0, K, 7)] *= 300.0
    else:                                                     # few values: bins full of ties, residuals of zeros
        V = rng.integers(-3, 4, (nvec, K)).astype(np.float64)
        V[::2, 0] = 127.0
    V = V.astype(F32)
    V[0] = 0
    V[1] = F32(2.0 ** -140) * np.sign(V[1])                    # scales that are not ordinary numbers
    V[2, 1::2] = -1.0
    V[2, ::2] = 1.0                                           # one magnitude: the topmost code alone
    V[3, 5] = np.nan
    return V


def assert_selection(srq, A, B):
    """The compressed operands of the last call are the entries above its thresholds and their codes."""
    im = srq.intermediates(A.shape[0], B.shape[1], A.shape[1])
    for V, t, ptr, idx, val, codes in ((A, im["t_a"], im["a_ptr"], im["a_idx"], im["a_val"], im["A_int"]),
                                       (B.T, im["t_b"], im["b_ptr"], im["b_idx"], im["b_val"], im["B_int"])):
        with np.errstate(invalid="ignore"):
            vec, k = np.nonzero(np.abs(V) > host(t)[:, None])
        assert (host(ptr) == np.searchsorted(vec, np.arange(len(V) + 1))).all()
        assert (host(idx)[:len(k)] == k).all() and (host(val)[:len(k)] == host(codes)[vec, k]).all()


# (M, N, K): one wave, two and four of them per vector, a last piece that is no whole sixteen; the operands' thresholds
# put exactly on an entry of some vectors
@pytest.mark.parametrize("shape", [(300, 1800, 4099), (40, 2100, 8192), (1030, 1029, 8205), (20, 2040, 16384)])
@pytest.mark.parametrize("kind", ["normal", "outliers", "ties"])
@pytest.mark.parametrize("bits,trunc", [(8, 0), (8, 1), (7, 0), (4, 0)])
def test_selection_from_codes(srq, b, shape, kind, bits, trunc):
    M, N, K = shape
    rng = np.random.default_rng(M + N + K + bits)
    A, B = operand(rng, kind, M, K), operand(rng, kind, N, K).T.copy()
    theta = 1.0 / K ** 0.5
    for _ in range(2):
        srq.compensated_gemm(dev(A), dev(B), theta, theta, bits=bits, rounding=b.ROUND_TRUNC if trunc else b.ROUND_NEAREST_EVEN,
                             strategy=b.STRATEGY_CSR_MFMA, max_density=1.0)
        torch.cuda.synchronize()
        assert_selection(srq, A, B)
        # once more with the threshold of row 7 on (or next to) an entry
        theta = float(np.sort(np.abs(A[7]))[-K // 10] / host(srq.intermediates(M, N, K)["drow"])[7])


# (M, N, K): both operands' vectors by one to four waves, columns by workgroups of their own (from 1280 on) or not, their last sixteen,
# four and eight rows not whole; with means formed in the same launch and after them; kept codes written on the side (the first two) or
# not.  Thresholds within the lowest bins of most vectors, and beyond them.
@pytest.mark.parametrize("shape", [(300, 400, 1100), (90, 1290, 4100), (1283, 1301, 1503), (40, 1450, 2052), (700, 60, 3001), (100, 1900, 7001),
                                   (530, 2050, 4501), (20, 2030, 16385)])
@pytest.mark.parametrize("kind,sigmas", [("wide", 0.0002), ("wide", 0.5), ("far", 0.2), ("far", 3.0)])
@pytest.mark.parametrize("bits,trunc", [(8, 0), (7, 1), (4, 0)])
def test_selection_with_thresholds_in_the_lowest_bins(srq, b, shape, kind, sigmas, bits, trunc):
    M, N, K = shape
    rng = np.random.default_rng(M + N + K + bits)

    def vectors(nvec):
        if kind == "wide":
            V = np.ldexp(rng.choice([-1.0, 1.0], (nvec, K)) * (1 + rng.random((nvec, K))), rng.integers(-10, 11, (nvec, K)))
        else:                                                 # a few outliers that set the scales
            V = rng.standard_normal((nvec, K))
            V[::2, rng.integers(0, K, 3)] *= 1000.0
        V = V.astype(F32)
        V[0] = 0
        V[1] = F32(2.0 ** -140) * np.sign(V[1])
        V[3, 5], V[3, K - 1], V[8, 6] = np.nan, np.nan, np.nan
        return V

    A, B = vectors(M), vectors(N).T.copy()
    # the means of |D_F| go with the vectors' own size: thresholds about `sigmas` times what most entries are
    theta = sigmas / (K ** 0.5 * (40.0 if kind == "far" else 150.0))
    stats = b.stats_tensor()
    for strategy in (b.STRATEGY_CSR_MFMA, b.STRATEGY_AUTO):
        srq.compensated_gemm(dev(A), dev(B), theta, theta, bits=bits, rounding=b.ROUND_TRUNC if trunc else b.ROUND_NEAREST_EVEN,
                             strategy=strategy, stats=stats, max_density=1.0, debug=strategy == b.STRATEGY_AUTO)
        torch.cuda.synchronize()
        assert_selection(srq, A, B)
        st = b.read_stats(stats)
        im = srq.intermediates(M, N, K)
        assert st["nnz_a"] == int(im["a_ptr"][-1]) > 0 and st["nnz_b"] == int(im["b_ptr"][-1]) > 0


# at 8 bits the code of FLT_MAX times its scale is infinite, and with it the largest residual of the vector, whose lambda becomes
# zero as if there were none
@pytest.mark.parametrize("shape", [(300, 400, 1100), (300, 1800, 4099)])
@pytest.mark.parametrize("side", ["a", "b"])
@pytest.mark.parametrize("bits,trunc", [(8, 0), (8, 1), (7, 0)])
def test_selection_with_an_infinite_residual(srq, b, shape, side, bits, trunc):
    M, N, K = shape
    rng = np.random.default_rng(K + bits)
    A, B = rng.standard_normal((M, K)), rng.standard_normal((K, N))
    V, W = (A, B) if side == "a" else (B.T, A)
    W /= K ** 0.5                                             # (means of |D_F| as large as the entries of V)
    for row, sigma, top in ((4, 2e37, 1.0), (5, 1e37, -1.0), (6, 5e36, 1.0)):
        V[row] *= sigma
        V[row, 7] = top * np.finfo(F32).max
    A, B = A.astype(F32), B.astype(F32)
    srq.compensated_gemm(dev(A), dev(B), 1.0, 1.0, bits=bits, rounding=b.ROUND_TRUNC if trunc else b.ROUND_NEAREST_EVEN,
                         strategy=b.STRATEGY_CSR_MFMA, max_density=1.0)
    torch.cuda.synchronize()
    im = srq.intermediates(M, N, K)
    kept = np.diff(host(im[side + "_ptr"]))[4:7]
    assert np.isfinite(host(im["t_" + side])[4:7]).all() and (kept > 0).all() and (kept < K).all()
    assert_selection(srq, A, B)


# (the last three: columns in one read; a wave and a workgroup per row)
@pytest.mark.parametrize("shape", [(5, 9, 3), (65, 70, 250), (100, 1001, 1024), (129, 65, 1500), (40, 30, 4500), (1100, 1000, 4099), (2100, 37, 8192),
                                   (70, 2100, 16384)])
def test_counts_of_operands_that_are_not_compacted(srq, b, shape):
    """The dense branch whatever the counts, thresholds of zero: every entry that is not zero counts, and none where the
    threshold is no number (0 times a mean that has overflowed)."""
    M, N, K = shape
    rng = np.random.default_rng(K)
    A, B = rng.standard_normal((M, K)).astype(F32), rng.standard_normal((K, N)).astype(F32)
    A[rng.random((M, K)) < 0.3] = 0
    B[rng.random((K, N)) < 0.6] = 0
    A[1], B[:, 2] = 0, 0
    A[3, 0], B[0, 4] = np.nan, np.nan
    A[4] = 1e38                                               # |D_F| overflows in this row
    stats = b.stats_tensor()
    srq.compensated_gemm(dev(A), dev(B), 0.0, 0.0, dense_fallback_density=0.0, stats=stats)
    torch.cuda.synchronize()
    im, st = srq.intermediates(M, N, K), b.read_stats(stats)
    with np.errstate(invalid="ignore"):
        counts = [(np.abs(V) > host(t)[:, None]).sum(axis=1) for V, t in ((A, im["t_a"]), (B.T, im["t_b"]))]
    assert (host(im["a_ptr"]) == np.concatenate([[0], np.cumsum(counts[0])])).all()
    assert (host(im["b_ptr"]) == np.concatenate([[0], np.cumsum(counts[1])])).all()
    assert st["nnz_a"] == counts[0].sum() and st["nnz_b"] == counts[1].sum() and counts[0][0] > 0


# (M, N, K): vectors that are no whole group of four, one and one over a sum's 256; two to sixteen pieces of a vector.  Kept shares on
# either side of where a term changes its execution.
@pytest.mark.parametrize("shape", [(2301, 1030, 1700), (257, 2100, 4099), (100, 2001, 4300), (256, 255, 8200), (1030, 70, 16384)])
@pytest.mark.parametrize("kept", [(0.0005, 0.0003), (0.05, 0.0003), (0.0005, 0.05), (0.05, 0.05), (0.05, None), (None, 0.0003),
                                  (0.9, 0.2)])
def test_decision_and_compaction_in_one_launch(srq, b, shape, kept):
    """SRQ_STRATEGY_AUTO decided on the device (debug outputs keep it from taking the matrix cores outright): compressed operands,
    statistics and both terms against the definitions and a call with the execution given, bit for bit."""
    M, N, K = shape
    rng = np.random.default_rng(sum(shape))
    A, B = rng.standard_normal((M, K)).astype(F32), rng.standard_normal((K, N)).astype(F32)
    A[1], B[:, 2], A[3, 5] = 0, 0, np.nan
    def theta(share):                                         # |x| over the mean of |D_F|, about 0.8 sqrt(K)
        if share is None:
            return float("inf")
        return float(np.quantile(np.abs(B[:, -1 - min(N, 64):-1]), 1 - share)) / (0.8 * K ** 0.5)
    ta, tb = theta(kept[0]), theta(kept[1])
    out = []
    for hint in (1, 2):
        srq.set_auto_hint(hint, hint)
        stats = b.stats_tensor()
        C, _, dbg = srq.compensated_gemm(dev(A), dev(B), ta, tb, stats=stats, debug=True)
        torch.cuda.synchronize()
        im, st = srq.intermediates(M, N, K), b.read_stats(stats)
        for term, V, s, codes in ((0, A, "a", im["A_int"]), (1, B.T, "b", im["B_int"])):
            if kept[term] is None:
                assert st["path_" + s] == 0 and st["nnz_" + s] == 0
                continue
            with np.errstate(invalid="ignore"):
                vec, k = np.nonzero(np.abs(V) > host(im["t_" + s])[:, None])
            assert (host(im[s + "_ptr"]) == np.searchsorted(vec, np.arange(len(V) + 1))).all()
            assert (host(im[s + "_idx"]) == k).all() and (host(im[s + "_val"]) == host(codes)[vec, k]).all()
            assert st["nnz_" + s] == len(k) > 0 and st["path_" + s] == (2 if kept[term] > 0.01 else 1)
        out.append([host(C)] + [host(dbg[x]) for x in ("DR1_int", "DR2_int")])
    C, _, dbg = srq.compensated_gemm(dev(A), dev(B), ta, tb, strategy=b.STRATEGY_CSR_MFMA, debug=True)
    torch.cuda.synchronize()
    ref = [host(C)] + [host(dbg[x]) for x in ("DR1_int", "DR2_int")]
    for got in out:
        assert all(np.array_equal(x, y, equal_nan=x.dtype.kind == "f") for x, y in zip(got, ref))


# one, two, four and eight pieces of a vector, a last one that is partly there; vectors that are no whole group of four
@pytest.mark.parametrize("shape", [(701, 1024), (203, 1500), (150, 4096), (61, 8190)])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("room", [1.0, 0.37])
def test_compaction_of_crowded_vectors(b, shape, axis, room):
    """Vectors that keep nothing to everything, pieces on either side of the number of entries from which on they go through
    LDS; room for all entries, or for some that end within a vector."""
    nvec, K = shape
    rng = np.random.default_rng(K)
    V = np.argsort(rng.random((nvec, K)), axis=1).astype(F32) + 1             # 1 .. K in any order
    count = (np.arange(nvec) * 7919 % (K + 1)).astype(np.int64)
    count[:24] = np.minimum(K, np.r_[0, 1, 3, 157:167, 255:258, 511:514, K - 3:K + 1, 160 * (-(-K // 1024))])
    V *= rng.choice([-1.0, 1.0], V.shape).astype(F32)
    X, t = dev(V if axis == 0 else V.T.copy()), dev((K - count + 0.5).astype(F32))
    capacity = int(room * count.sum())
    h = b.Srq(device=0)
    try:
        Q, scale, lam = h.quantize(X, axis)
        r = h.build_sparse_residual(X, axis, scale, lam, t, capacity=capacity)
        vec, k = np.nonzero(np.abs(V) > host(t)[:, None])
        assert int(r["nnz"].item()) == count.sum() and (host(r["ptr"]) == np.r_[0, np.cumsum(count)]).all()
        assert (host(r["idx"]) == k[:capacity]).all() and (host(r["val"]) == host(Q)[vec, k][:capacity]).all()
    finally:
        h.close()
