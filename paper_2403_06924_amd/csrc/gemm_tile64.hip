// INT8 GEMM for problems whose time is latency or the traffic of C rather than matrix-core work: few
// output tiles, or a short inner dimension (operands K-contiguous, 16-byte aligned, K a multiple of 64,
// any M and N).
//
// One 64 x 64 output tile per workgroup of four waves (32 x 32 each, v_mfma_i32_16x16x64_i8), K staged
// 128 bytes at a time from global memory straight into LDS as in the persistent kernel (unpadded rows,
// XOR swizzle of the 16-byte pieces), through a ring of NST stages of 16 KiB with NST - 1 K-tiles in
// flight and one barrier per K-tile.  What a stage costs is the CU's vector-memory path, 256 clocks
// for 16 KiB against 128 of matrix-core time; that is why larger tiles take over where there are
// enough of them to fill the chip and K is long.
//
//  * few tiles (at most one per compute unit): eight stages, so that the round trips of a long K
//    overlap seven deep;
//  * more: four or three stages, two or three workgroups per compute unit, whose loads, products and
//    accesses to C overlap each other's;
//  * corrections whose launch also compacts the operands (CompactTail): four or three, so that compacting workgroups fit beside.
//
// Both corrections go through one launch (DirectProducts) as one stream of K-tiles, each product with
// accumulators of its own: they are added to C in registers, in the order of Algorithm 1, and C is read and
// written once.
//
// (Fragments read straight from global memory, without LDS, were slower: the 64 lanes of such a load
// touch sixteen rows and the vector-memory path takes 64 clocks for it instead of 16.  8192 x 8192 x
// 256: 262 us.)
#include "srq_internal.h"
#include "compact.h"
#include "gemm_tiles.h"
#include "gemm_tile64.h"

namespace srq {
namespace {

constexpr int BT = 64, BK = kKTile;
constexpr int kOperand = BT * BK;                    // 8 KiB
constexpr int kStage = 2 * kOperand;                 // A tile then B tile
constexpr int kLoads = 4;                            // per wave and K-tile: 2 for A, 2 for B

struct NoTail {};

template <int NP, int NST, bool SUMS, class Tail, int NV>   // NV: pieces of 1024 elements that the tail compacts
__global__ __launch_bounds__(256, NST >= 8 ? 1 : 12 / NST) void gemm_i8_tile64_kernel(int64_t M, int64_t N, int K, int64_t lda,
                                                                                    int64_t ldb, int tiles_m, int tiles_n,
                                                                                    DirectProducts pr, GemmEpilogue ep, Tail more) {
  static_assert(!SUMS || NP == 1, "");
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  __shared__ double rowx[SUMS ? 2 * BT : 1], colx[SUMS ? 2 * BT : 1];
  if (guard_tripped(ep)) return;                     // the whole grid leaves together
  if constexpr (std::is_same_v<Tail, CompactTail>) {
    if ((int)blockIdx.x >= more.tiles) {
      __shared__ int64_t before[4];
      __shared__ int count[4];
      static_assert(NST * kStage >= 4 * kGatherWave, "the stages' LDS gathers the entries of crowded vectors");
      const int group = (int)blockIdx.x - more.tiles;
      const bool second = group >= more.groups_a;
      compact_four<NV>(second ? more.b : more.a, second ? group - more.groups_a : group, more.K, K, before, count,
                       reinterpret_cast<uint8_t*>(lds));
      return;
    }
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) int8_t*)lds);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w >> 1, wn = w & 1;
  const int quad = lane >> 4, rl = lane & 15;
  int tile_m, tile_n;
  tile_of((int)blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
  const int64_t m0 = (int64_t)tile_m * BT, n0 = (int64_t)tile_n * BT;
  const uint32_t rows_a = (uint32_t)(M - m0 < BT ? M - m0 : BT), rows_b = (uint32_t)(N - n0 < BT ? N - n0 : BT);
  const bool full = rows_a == BT && rows_b == BT;

  // ---- loader: wave w fetches rows 16w .. 16w+15 of each operand tile, eight rows per load.  Lane l of
  // load j covers row 16w + 8j + l/8 and LDS piece l%8, which holds the logical piece (l%8) ^
  // ((row >> 1) & 7).  The descriptor ends with the operand's last row: rows past it read as zero.
  const int nk = (K + BK - 1) / BK;
  uint32_t voff_a[2], voff_b[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t row = 16 * w + 8 * j + (lane >> 3), piece = 16 * ((lane & 7) ^ ((row >> 1) & 7));
    voff_a[j] = row * (uint32_t)lda + piece;
    voff_b[j] = row * (uint32_t)ldb + piece;
  }
  int cur_kt = 0, cur_p = 0, cur_g = 0;              // cursor of the fetches
  v4i ra, rb;
  auto point = [&](int p) __attribute__((always_inline)) {
    const uint64_t pa = (uint64_t)(uintptr_t)(pr.p[p].Qa + m0 * lda), pb = (uint64_t)(uintptr_t)(pr.p[p].Qb + n0 * ldb);
    ra = v4i{(int)(uint32_t)pa, (int)(uint32_t)(pa >> 32), (int)((rows_a - 1) * (uint32_t)lda + (uint32_t)K), 0x00020000};
    rb = v4i{(int)(uint32_t)pb, (int)(uint32_t)(pb >> 32), (int)((rows_b - 1) * (uint32_t)ldb + (uint32_t)K), 0x00020000};
  };
  auto issue = [&](uint32_t dst, v4i rsrc, uint32_t voff, uint32_t soff) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 : : "s"(dst), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
  };
  auto fetch = [&](int stage) __attribute__((always_inline)) {
    const uint32_t dst = lds0 + stage * kStage + 16 * w * BK, soff = (uint32_t)ktile_start(cur_kt, K);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      issue(dst + 8 * j * BK, ra, voff_a[j], soff);
      issue(dst + kOperand + 8 * j * BK, rb, voff_b[j], soff);
    }
    ++cur_g;
    if (++cur_kt == nk) {
      cur_kt = 0;
      if (NP > 1 && cur_p + 1 < NP) ++cur_p;
      if (NP > 1) point(cur_p);
    }
  };
  // ---- C, fetched ahead of the products (and older than their loads, see the counted wait).  It is
  // accessed after an exchange of the two blocks of a row block between the half rows of lanes.
  const TileAccess<4> tile = {32 * wm + (rl & 7), 32 * wn + 16 * (rl >> 3) + 4 * quad, rows_a, rows_b, full};
  v4f out[4], cin[4];
  const bool read_c = ep.mode == kGemmAccum, has_beta = ep.final_scale && ep.beta != 0.f;
  if (read_c) tile.load(out, ep.C + m0 * ep.ldc + n0, (uint32_t)ep.ldc);
  if (has_beta) tile.load(cin, ep.Cin + m0 * ep.ldcin + n0, (uint32_t)ep.ldcin);
  point(0);
  const int total = NP * nk;
#pragma unroll
  for (int g = 0; g < NST - 1; ++g)
    if (g < total) fetch(g);

  // ---- fragments: lane (rl, quad) reads logical piece 4 step + quad of its rows
  const int key = (rl >> 1) & 7;
  const int a_row = (32 * wm + rl) * BK, b_row = kOperand + (32 * wn + rl) * BK;
  const int xoff[2] = {16 * (quad ^ key), 16 * ((4 + quad) ^ key)};
  v4i acc[NP][2][2];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[p][a][b] = v4i{0, 0, 0, 0};
  const int head = last_ktile_mask(K, 0), tail = last_ktile_mask(K, 1), masked = (K & 64) ? nk - 1 : -1;
  int stage = 0;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    for (int kt = 0; kt < nk; ++kt) {
      // this K-tile has landed: everything but the NST - 2 K-tiles after it (near the end: everything)
      if (p * nk + kt + NST - 2 < total) wait_loads_but<(NST - 2) * kLoads>();
      else wait_loads();
      __syncthreads();                               // ... for every wave; and the stage before it is free
      const int8_t* base = lds + stage * kStage;
      v4i fa[2][2], fb[2][2];
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          fb[s][i] = *reinterpret_cast<const v4i*>(base + b_row + xoff[s] + i * 16 * BK);
          fa[s][i] = *reinterpret_cast<const v4i*>(base + a_row + xoff[s] + i * 16 * BK);
        }
      if (cur_g < total) fetch(stage == 0 ? NST - 1 : stage - 1);
      if (kt == masked) {
#pragma unroll
        for (int a = 0; a < 2; ++a) { fa[0][a] &= head; fa[1][a] &= tail; }
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[p][a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[s][b], fa[s][a], acc[p][a][b], 0, 0, 0);
      stage = stage == NST - 1 ? 0 : stage + 1;
    }
  }

  // ================= epilogue
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const __amdgpu_buffer_rsrc_t rsr = buf_rsrc(pr.p[p].s_row + m0, 4 * rows_a), rsc = buf_rsrc(pr.p[p].s_col + n0, 4 * rows_b);
    float srow[2];
    v4f scol[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      srow[i] = buf_load_f32(rsr, 4u * (uint32_t)(32 * wm + 16 * i + rl));
      scol[i] = buf_load_4(rsc, 4u * (uint32_t)(32 * wn + 16 * i + 4 * quad), full);
    }
    tile64_product<SUMS>(acc[p], srow, scol, p || read_c, out, wm, wn, quad, rl, rowx, colx);
    if (SUMS) {
      __syncthreads();
      tile64_store_sums(ep, tid, M, N, tile_m, tile_n, rows_a, rows_b, rowx, colx);
    }
  }
  if (ep.final_scale) tile64_scale(ep, has_beta, out, cin);
  tile.store(out, ep.C + m0 * ep.ldc + n0, (uint32_t)ep.ldc);
}

template <int NP, bool SUMS>
hipError_t launch(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, const DirectProducts& pr,
                  const GemmEpilogue& ep, hipStream_t st) {
  const int64_t tm = (M + BT - 1) / BT, tn = (N + BT - 1) / BT;
  const int64_t ktiles = NP * ((K + BK - 1) / BK);
  // stages: as many as the stream has K-tiles, at most 8 where a compute unit has one tile, 4 where it has
  // two, else 3
  const int cap = tm * tn <= 256 ? 8 : tm * tn <= 512 ? 4 : 3;
  void (*kern)(int64_t, int64_t, int, int64_t, int64_t, int, int, DirectProducts, GemmEpilogue, NoTail);
  int nst;
  if (cap == 8 && ktiles > 4) { kern = gemm_i8_tile64_kernel<NP, 8, SUMS, NoTail, 0>; nst = 8; }
  else if (cap >= 4 && ktiles > 3) { kern = gemm_i8_tile64_kernel<NP, 4, SUMS, NoTail, 0>; nst = 4; }
  else { kern = gemm_i8_tile64_kernel<NP, 3, SUMS, NoTail, 0>; nst = 3; }
  const int bytes = nst * kStage;
  if (bytes > 48 * 1024) {
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(tm * tn)), dim3(256), bytes, st, M, N, (int)K, lda, ldb, (int)tm, (int)tn, pr, ep, NoTail{});
  return hipGetLastError();
}

}  // namespace

// A compute unit holds a tile of C (or two) and compacting workgroups beside it, which take the place of a launch of their own
// between the selection and the corrections: 64 KiB of LDS for each (with 80 KiB and 48 bytes two do not fit, and the compaction
// begins where the tiles end: 1024^3 35 us a call, as with 128 KiB), 48 KiB where there is more than one tile for a compute unit.
// Calls at 5 % kept, us, separate launches / this: 300 x 400 x 1000 31.4 / 27.9, 512^3 26.0 / 22.4, 700 x 900 x 800 35.2 / 31.4, 1024^3
// 34.8 / 30.8, 2000 x 400 x 300 28.3 / 25.5, 1400^2 x 1000 41.9 / 38.2, 1500^2 x 1200 51.3 / 46.9, 1000^2 x 3000 59.0 / 53.4, 500 x 600 x
// 4000 62.4 / 57.0, 640^2 x 5000 76.3 / 69.2, 300^2 x 8000 92.8 / 85.1.  Compacted by the workgroups of the tiles after their stores 1024^3 takes 34.7, 512^3 28.7.  Larger
// tiles leave no LDS for a second workgroup.
bool gemm_tile64_tail_ok(int64_t M, int64_t N, int64_t K) { return K <= kStripsMaxK && ((M + BT - 1) / BT) * ((N + BT - 1) / BT) <= 640; }

hipError_t launch_gemm_i8_tile64_tail(int64_t M, int64_t N, int64_t K, int64_t ld, const DirectProducts& pr, const GemmEpilogue& ep,
                                      const CompactTail& with, hipStream_t st) {
  const int64_t tm = (M + BT - 1) / BT, tn = (N + BT - 1) / BT;
  CompactTail tail = with;
  tail.tiles = (int)(tm * tn);
  tail.groups_a = (tail.a.nvec + 3) / 4;
  const int nst = tail.tiles <= 256 ? 4 : 3;
  void (*kern)(int64_t, int64_t, int, int64_t, int64_t, int, int, DirectProducts, GemmEpilogue, CompactTail);
#define SRQ_TAIL(NV) kern = nst == 4 ? gemm_i8_tile64_kernel<2, 4, false, CompactTail, NV> : gemm_i8_tile64_kernel<2, 3, false, CompactTail, NV>
  if (K <= 1024) SRQ_TAIL(1);
  else if (K <= 2048) SRQ_TAIL(2);
  else if (K <= 4096) SRQ_TAIL(4);
  else SRQ_TAIL(8);
#undef SRQ_TAIL
  const int bytes = nst * kStage;
  const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(tail.tiles + tail.groups_a + (tail.b.nvec + 3) / 4)), dim3(256), bytes, st, M, N, (int)K, ld, ld,
                     (int)tm, (int)tn, pr, ep, tail);
  return hipGetLastError();
}

hipError_t launch_gemm_i8_tile64(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, const DirectProducts& pr,
                                 const GemmEpilogue& ep, hipStream_t st) {
  if (ep.row_part) return launch<1, true>(M, N, K, lda, ldb, pr, ep, st);
  if (pr.n == 2) return launch<2, false>(M, N, K, lda, ldb, pr, ep, st);
  return launch<1, false>(M, N, K, lda, ldb, pr, ep, st);
}

}  // namespace srq
