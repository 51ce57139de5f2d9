// Persistent variant of the INT8 GEMM for large problems with K-contiguous, 16-byte aligned
// operands: the products of every large workload.
//
// One 256 x 256 output tile per 4-wave workgroup at a time (128 x 128 per wave), one workgroup per
// compute unit:
//
//  * v_mfma_i32_16x16x64_i8, not 32x32x32: at the same rate per clock it moves 8 KiB instead of
//    10 KiB through the registers per 65536 operations (the accumulators of a 32 x 32 block are
//    read and written twice as often per operation as its operands are saved), and the launch runs
//    at the chip's power limit.  A register-resident loop on random operand bytes: 4.27 POP/s at
//    2.07 GHz against 3.54 POP/s at 1.72 GHz.
//  * operand tiles go from global memory straight into LDS (buffer_load_dwordx4 ... lds): no
//    staging registers and no ds_write instructions.  The hardware writes the 64 lanes of one
//    load to 1 KiB of consecutive LDS bytes, so the tile rows are unpadded (128 B) and bank
//    conflicts of the 16-byte fragment reads are avoided by an XOR swizzle instead: the 16-byte
//    piece s of row r sits at position s ^ ((r >> 1) & 7), applied on the global-address side
//    when loading and on the LDS-address side when reading;
//  * a workgroup walks over several output tiles and the stream of staged K-tiles never drains
//    between them: while one tile's epilogue runs, the first K-tiles of the next are already
//    landing in LDS (they need no registers), and the epilogue's stores retire while the next
//    tile is multiplied;
//  * LDS holds three buffers for the tiles of A and two for the tiles of B (5 x 32 KiB, all of a
//    CU's LDS).  The fragments of a step are read a whole step (64 MFMAs) ahead, so both buffers
//    of a K-tile are free at its one barrier, half-way through it; the sixteen loads a wave issues
//    per K-tile go out one after every eighth MFMA: in the first half of K-tile g the A tile of
//    K-tile g+2 (into the buffer that K-tile g-1 left), in the second half its B tile.  (The CU's
//    vector-memory path takes a 1 KiB load about every 20 clocks, and a wave whose load cannot be
//    accepted yet also holds back the MFMAs behind it.)
//  * the first operand of an MFMA is the B fragment, so that a lane ends up with four consecutive
//    columns of one row of C, in 16-row x 16-column blocks; two neighbouring blocks are exchanged
//    between the half rows of 8 lanes (one DPP move per element), so that every access to C is
//    16 bytes per lane and whole 128-byte lines per row.  (All compute units store at once: with
//    64-byte pieces a round of 64 MiB leaves at 3.0 TB/s, with whole lines at 5.9 TB/s.)
//
// What bounds it: on operands that toggle, the power limit (1.86 GHz in a loop of products on random
// bytes); on zeros about 2300 clocks per K-tile against 2048 of matrix-core time; and the epilogue, in which all compute
// units access C at once: 64 MiB a round written in first mode, read and written in accumulate mode.
// 8192^3, us, with 32x32x32 and 64 dwords per row block / now: product without sums, random codes 472 / 389-404,
// zeros 322 / 309; normal operands with outliers, 5 % kept, in a call: first product 443 / 367, both corrections in
// one launch 968 / 781, of which 592 are the K loops and 190 eight epilogues: 14 us each for loading C, converting and
// adding, 10 for the stores, together 5.5 TB/s.
//
// The epilogues spill no vector register, inside and outside the K loop (scalar ones go to lanes of vector registers: 10 to 79 in
// most variants, about 250 in the accumulating edge kernels with alpha and beta), because (a) the accumulators are read one by one through
// assembly: otherwise the conversions that the copies of an epilogue have in common are all computed ahead of the
// branch between them; (b) C is accessed through buffer descriptors with running scalar row pointers and one lane
// offset, not 64-bit addresses per access; (c) accesses on the edge are cut off by the descriptor's range, not
// branched around; (d) sums are pinned where they are formed.  Before / after, calls at 5 % kept, us: 2999 x 4097 x
// 3001 319 / 294 (first product 67 / 60, corrections 135 / 106), 5000^2 x 2000 with beta 475 / 424, 4096 x 14336 x 4096
// 972 / 938, 8192^3 1576 / 1535, 4096 x 8192 x 1024 with beta 327 / 295.
// The order in which the accumulating epilogue visits its blocks (JN): down the 128 rows of 32 columns, then the next
// 32; on the edge, where rows of C seldom start on the same channels of memory, along the row unless the pitch is a
// multiple of 4 KiB (corrections, us, down / along: pitch 32 KiB 781 / 858, 56 KiB 456 / 456, 16388 bytes 122 / 106,
// 20000 bytes 236 / 222; edge with 32 KiB 191 / 208).  8, 12, 16 or 20 blocks ahead are the same time.
//
// Where M or N is no multiple of the tile C goes through the caches, also in whole tiles, so that parts of a line which
// two rows or tiles share leave together (around them / through them, calls, us: 2999 x 4097 x 3001 279 / 266, 5000^2 x 2000
// 330 / 313, 9000^2 x 3000 1187 / 1147, 4001 x 14001 x 4000 1246 / 1206); whole tiles of a last product go around them.
//
// M and N need not be multiples of the tile: rows past the end are cut off by the range check of the
// buffer descriptor (whatever lands in LDS for them feeds elements that are never stored), and the
// epilogue of a tile on the edge checks every access.
#include <atomic>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>
#include "srq_internal.h"
#include "gemm_tiles.h"
#include "gemm_lanes.h"

namespace srq {
namespace {

// four consecutive floats at any 4-byte aligned address (rows of C may start anywhere)

constexpr int BM = 256, BN = 256, BK = kKTile;
constexpr int kOperand = BM * BK;                   // 32 KiB per operand tile
constexpr int TM = 8, TN = 8;                       // 16 x 16 MFMA tiles per wave
constexpr int kABufs = 3, kBBufs = 2;               // LDS buffers of the A tiles and of the B tiles
constexpr int kLdsB = kABufs * kOperand;            // the B buffers follow the A buffers
constexpr int kLdsBytes = kLdsB + kBBufs * kOperand;   // 160 KiB; the epilogue's scales borrow a free A buffer
constexpr int kLoads = 8;                           // loads per wave, operand and K-tile
enum { kFirst, kMiddle, kLast };                    // K-tiles of an output tile

// the lane's number, computed where it is wanted: nothing derived from it can be computed ahead of the
// K loop and kept (or spilled) through it
__device__ __forceinline__ int fresh_lane() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// EDGE: M or N is no multiple of 256.  JN: neighbouring blocks of a row of C that an accumulating epilogue visits before
// the next row.
template <int MODE, bool SUMS, bool SCALE, bool EDGE, int JN>
__global__ __launch_bounds__(256) void gemm_i8_persistent_kernel(int64_t M, int64_t N, int64_t K,
                                                                 const int8_t* __restrict__ Qa, int64_t lda,
                                                                 const int8_t* __restrict__ Qb, int64_t ldb,
                                                                 int tiles_m, int tiles_n,
                                                                 GemmEpilogue ep, GemmSecond sec) {
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  if (MODE == kGemmAccum && guard_tripped(ep)) return;   // the whole grid leaves together
  // LDS byte address of the first stage (an address-space-3 pointer is a 32-bit offset)
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) int8_t*)lds);

  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));                     // keeps per-thread offsets from being hoisted out of the tile loop
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w >> 1, wn = w & 1;
  const int total = tiles_m * tiles_n, G = gridDim.x;
  const int nk = (int)((K + BK - 1) / BK);
  // (where K is an odd multiple of 64 the first K-tile counts for 64 alone, and the second starts there)
  const int half = (K & 64) ? 0 : -1;
  // accumulate mode may carry a second product over the same tiles (sec.Qa != null): a workgroup
  // then runs product 0 and product 1 of a tile back to back, so that the tile of C written by
  // the first is still in the caches when the second adds to it
  const int nprod = (MODE == kGemmAccum && sec.Qa) ? 2 : 1;
  int p_lo, p_hi;                                   // the products this launch runs (device-side decision)
  pair_range(ep, nprod, p_lo, p_hi);

  // ---- loader: wave w fetches rows 64w .. 64w+63 of each operand tile, eight rows per load.
  // Lane l of load j covers row 64w + 8j + l/8 and LDS piece l%8, which holds the logical piece
  // (l%8) ^ ((row >> 1) & 7); (row >> 1) & 7 = ((l >> 4) + 4j) & 7 depends on j only through
  // its parity.
  const uint32_t la32 = (uint32_t)lda, lb32 = (uint32_t)ldb;
  uint32_t voff_a[2], voff_b[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const uint32_t piece = 16 * ((lane & 7) ^ (((lane >> 4) + 4 * e) & 7));
    voff_a[e] = (64 * w + (lane >> 3)) * la32 + piece;
    voff_b[e] = (64 * w + (lane >> 3)) * lb32 + piece;
  }
  // Cursor over the stream of K-tiles: output tile, K-tile within it, product; base address and
  // remaining bytes of the rows of that K-tile in A and B (uniform: all of it in scalar registers)
  int cur_vb = blockIdx.x, cur_kt = 0, cur_prod = p_lo;
  uint64_t base_a = 0, base_b = 0;
  uint32_t bytes_a = 0, bytes_b = 0;
  const uint32_t first_step = (uint32_t)first_ktile_step((int)K);
  auto point = [&]() {
    int tm, tn;
    tile_of(cur_vb, tiles_m, tiles_n, tm, tn);
    const int64_t ra = (int64_t)tm * BM, rb = (int64_t)tn * BN;
    const int64_t left_a = M - ra < BM ? M - ra : BM, left_b = N - rb < BN ? N - rb : BN;
    base_a = (uint64_t)(uintptr_t)((cur_prod ? sec.Qa : Qa) + ra * lda);
    base_b = (uint64_t)(uintptr_t)((cur_prod ? sec.Qb : Qb) + rb * ldb);
    bytes_a = (uint32_t)((left_a - 1) * lda + K);
    bytes_b = (uint32_t)((left_b - 1) * ldb + K);
  };
  auto advance = [&]() {
    if (cur_kt + 1 < nk) {
      ++cur_kt;
      const uint32_t step = cur_kt == 1 ? first_step : (uint32_t)BK;
      base_a += step;
      base_b += step;
      bytes_a -= step;
      bytes_b -= step;
    } else if (cur_prod < p_hi) {
      ++cur_prod;
      cur_kt = 0;
      point();
    } else if (cur_vb + G < total) {
      cur_vb += G;
      cur_prod = p_lo;
      cur_kt = 0;
      point();
    }                                               // else stay on the last K-tile (harmless re-fetch)
  };
  // One load in as few issue slots as possible (an MFMA leaves three until the next one): where it goes
  // (M0) is set one MFMA ahead, which also keeps the one instruction between the two that the
  // hardware asks for (nothing the compiler puts there uses M0); the row offset 8 j ld is the scalar
  // offset, which needs no vector instruction.  The range check is not relied upon to count it: whole tiles
  // load nothing past their rows, and on the edges it is added to the lane's offset instead (inside the
  // assembly: as ordinary code the sixteen sums would be hoisted out of the loops, into registers that are not
  // there).
  auto target = [&](uint32_t lds_addr, int j) __attribute__((always_inline)) {
    asm volatile("s_add_i32 m0, %0, %1" : : "s"(lds_addr), "i"(j * 8 * BK) : "m0", "scc");
  };
  auto issue = [&](uint64_t base, uint32_t bytes, uint32_t voff, uint32_t rows) __attribute__((always_inline)) {
    const v4i rsrc = {(int)(uint32_t)base, (int)(uint32_t)(base >> 32), (int)bytes, 0x00020000};
    if (EDGE) {
      uint32_t tmp;
      asm volatile("v_add_u32 %0, %1, %3\n\tbuffer_load_dwordx4 %0, %2, 0 offen lds"
                   : "=&v"(tmp) : "v"(voff), "s"(rsrc), "s"(rows) : "memory");
    } else {
      asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" : : "v"(voff), "s"(rsrc), "s"(rows) : "memory");
    }
  };
  const uint32_t lds_a = lds0 + (64 * w) * BK, lds_b = lds_a + kLdsB;
  auto target_a = [&](int buf, int j) __attribute__((always_inline)) { target(lds_a + buf * kOperand, j); };
  auto target_b = [&](int buf, int j) __attribute__((always_inline)) { target(lds_b + buf * kOperand, j); };
  auto issue_a = [&](int j) __attribute__((always_inline)) { issue(base_a, bytes_a, voff_a[j & 1], 8 * j * la32); };
  auto issue_b = [&](int j) __attribute__((always_inline)) { issue(base_b, bytes_b, voff_b[j & 1], 8 * j * lb32); };
  auto issue_ktile = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      target_a(buf, j);
      asm volatile("s_nop 0");
      issue_a(j);
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      target_b(buf, j);
      asm volatile("s_nop 0");
      issue_b(j);
    }
  };

  // ---- fragment reads: lane (frow, kq) reads logical piece 4*step + kq of its rows; read r of a
  // step's sixteen: 0..7 -> B blocks, 8..15 -> A blocks
  const int frow = lane & 15, kq = lane >> 4, key = (frow >> 1) & 7;
  const int a_row = (wm * (BM / 2) + frow) * BK;
  const int b_row = kLdsB + (wn * (BN / 2) + frow) * BK;
  const int xoff[2] = {16 * (kq ^ key), 16 * ((4 + kq) ^ key)};
  v4i fa[2][TM], fb[2][TN];
  auto fread = [&](int abuf, int bbuf, int step, int r) {
    if (r < TN)
      fb[step][r] = *reinterpret_cast<const v4i*>(lds + bbuf * kOperand + b_row + xoff[step] + r * 16 * BK);
    else
      fa[step][r - TN] = *reinterpret_cast<const v4i*>(lds + abuf * kOperand + a_row + xoff[step] + (r - TN) * 16 * BK);
  };

  // ---- the output tile being multiplied
  int vb = blockIdx.x, tile_m, tile_n;
  tile_of(vb, tiles_m, tiles_n, tile_m, tile_n);

  // K-tiles 0 and 1
  point();
  issue_ktile(0);
  advance();
  issue_ktile(1);
  advance();
  wait_loads();                                     // both have landed
  __syncthreads();

  v4i acc[TM][TN];
  const int my_tiles = (total - (int)blockIdx.x + G - 1) / G;
  int g = 0;                                        // position in the K-tile stream across tiles
  int abuf = 0;                                     // A buffer of K-tile g (g mod 3)
  int prod = p_lo;                                  // product being multiplied (pairs: 0, 1, 0, 1, ...)
  const bool two = p_lo != p_hi;
  for (int tile = 0; tile < my_tiles * (p_hi - p_lo + 1); ++tile) {
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    const bool full = !EDGE || (m0 + BM <= M && n0 + BN <= N);
    const float* srow_g = prod ? sec.s_row : ep.s_row;
    const float* scol_g = prod ? sec.s_col : ep.s_col;
    // where the scales of this tile go: the A buffer of its last K-tile, free from that K-tile's
    // barrier until the second K-tile of the next tile
    int sbuf = 0;
    // KIND: first K-tile of the tile (the accumulators start at zero), one in the middle, the last one
    auto ktile = [&](auto kind_tag) {
      constexpr int KIND = decltype(kind_tag)::value;
      constexpr bool FIRST = KIND == kFirst, LAST = KIND == kLast;
      const int bbuf = g & 1;
      const int anext = abuf == kABufs - 1 ? 0 : abuf + 1;
      const int aprev = abuf == 0 ? kABufs - 1 : abuf - 1;
      // first half: the A tile of K-tile g+2 follows (into the buffer that K-tile g-1 left), and the
      // fragments of the second half are read
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
          const v4i zero = {0, 0, 0, 0};
          acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[0][b], fa[0][a], FIRST ? zero : acc[a][b], 0, 0, 0);
          const int n = a * TN + b;
          if (n < 48 && n % 3 == 0) fread(abuf, bbuf, 1, n / 3);
          if (n % 8 == 5) target_a(aprev, n / 8);
          if (n % 8 == 6) issue_a(n / 8);
          __builtin_amdgcn_sched_barrier(0);
        }
      if (FIRST) {
#pragma unroll
        for (int a = 0; a < TM; ++a) fa[1][a] &= half;
      }
      // K-tile g+1 must have landed: everything but the eight loads just issued.  After the barrier everybody has the fragments of this K-tile in
      // registers: its buffers are free.  (In the first K-tile of a tile nothing is left to wait for:
      // the prologue resp. the epilogue before it has waited for every load before its first store,
      // so that the stores, which the counter counts as well, may still be on their way.)
      if (!FIRST) wait_loads_but<kLoads>();
      __syncthreads();
      if (LAST) {
        sbuf = abuf;
        const int64_t rb = (M - m0 < BM ? M - m0 : BM) * 4, cbytes = (N - n0 < BN ? N - n0 : BN) * 4;
        const uint64_t pr = (uint64_t)(uintptr_t)(srow_g + m0), pc = (uint64_t)(uintptr_t)(scol_g + n0);
        const v4i rr = {(int)(uint32_t)pr, (int)(uint32_t)(pr >> 32), (int)rb, 0x00020000};
        const v4i rc = {(int)(uint32_t)pc, (int)(uint32_t)(pc >> 32), (int)cbytes, 0x00020000};
        const uint32_t dst = lds0 + sbuf * kOperand + 256 * w, off = 256 * w + 4 * fresh_lane();
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                     : : "s"(dst), "v"(off), "s"(rr) : "memory", "m0");
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                     : : "s"(dst + 4 * BM), "v"(off), "s"(rc) : "memory", "m0");
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
          acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[1][b], fa[1][a], acc[a][b], 0, 0, 0);
          const int n = a * TN + b;
          if (!LAST && n < 48 && n % 3 == 0) fread(anext, bbuf ^ 1, 0, n / 3);
          if (n % 8 == 5) target_b(bbuf, n / 8);
          if (n % 8 == 6) issue_b(n / 8);
          __builtin_amdgcn_sched_barrier(0);
        }
      advance();
      abuf = anext;
      ++g;
    };
    // (read here and not ahead of the last epilogue, which needs the registers)
#pragma unroll
    for (int r = 0; r < TM + TN; ++r) fread(abuf, g & 1, 0, r);
    ktile(std::integral_constant<int, kFirst>());
    for (int kt = 1; kt < nk - 1; ++kt) ktile(std::integral_constant<int, kMiddle>());
    ktile(std::integral_constant<int, kLast>());

    // ================= epilogue of tile (tile_m, tile_n): acc[a][b][v] is element
    // (16 a + rl, 16 b + 4 quad + v) of the wave's 128 x 128 block
    wait_loads_but<kLoads>();                       // the scales (older than the last eight loads)
    __syncthreads();
    // (the accumulators are read through assembly, where the compiler does not see to the distance from the last MFMA)
    asm volatile("s_nop 15\n\ts_nop 15" : : : "memory");
    const int ln = fresh_lane();
    const int quad = ln >> 4, rl = ln & 15;         // the lane's columns 4*quad.. and its row of a 16 x 16 block
    const float* sc_row = reinterpret_cast<const float*>(lds + sbuf * kOperand) + wm * (BM / 2) + rl;
    const float* sc_col = reinterpret_cast<const float*>(lds + sbuf * kOperand) + BM + wn * (BN / 2) + 4 * quad;
    const bool do_scale = SCALE && prod == nprod - 1;
    // (alpha, beta and the strides are read here, not kept in registers through the K loop)
    const float alpha = SCALE ? ep.alpha : 1.f, beta = SCALE ? ep.beta : 0.f;
    const bool has_beta = SCALE && do_scale && beta != 0.f;
    const int64_t ldcin = SCALE ? ep.ldcin : 0;
    auto left = [](int64_t n) { return (int)(n < BM ? n : BM); };
    // elements of block (a, j), scaled, in the layout C is stored in
    auto block_of = [&](int a, int j, float sr, v4f c0, v4f c1, v4f (&t)[2]) __attribute__((always_inline)) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        t[0][v] = acc_value(acc[a][2 * j][v]) * (sr * c0[v]);
        t[1][v] = acc_value(acc[a][2 * j + 1][v]) * (sr * c1[v]);
      }
      exchange_half_rows(t[0], t[1]);
    };
    const int64_t ldc4 = 4 * ep.ldc;
    auto lane_bytes = [&](int64_t ld4) { return (uint32_t)(ln & 7) * (uint32_t)ld4 + 64u * ((ln >> 3) & 1) + 16u * quad; };
    auto first_row = [&](const float* base, int64_t ld) { return (uint64_t)(uintptr_t)(base + (m0 + wm * (BM / 2)) * ld + n0 + wn * (BN / 2)); };
    // ---- accumulate mode, a whole tile: the tile's C goes through a ring of kRing blocks of 16 x 32 (two accesses
    // of eight rows each), loaded kRing blocks ahead of their turn.  Block i is column j_of(i) of row a_of(i) of
    // the blocks; row addresses are running (scalar) pointers.  CACHED: the first product of a pair leaves its
    // tile of C cached for the second; the last one goes around the caches (it would evict the FP32 operands
    // the next stages stream)
    auto add_to_c = [&](auto cached_tag, auto scaled_tag, auto beta_tag) {
      constexpr bool CACHED = decltype(cached_tag)::value, SCALED = decltype(scaled_tag)::value, BETA = decltype(beta_tag)::value;
      constexpr int kBlocks = TM * TN / 2, kRing = EDGE ? 8 : 12, kIn = 4;   // kIn: blocks of Cin ahead
      auto a_of = [](int i) constexpr { return i / JN % TM; };
      auto j_of = [](int i) constexpr { return i / (TM * JN) * JN + i % JN; };
      // from a block's rows to the next one's
      auto next = [&](uint64_t& p, int i, int64_t ld4) __attribute__((always_inline)) {
        if (i % JN != JN - 1) return;
        p += a_of(i) == TM - 1 ? -(TM - 1) * 16 * ld4 : 16 * ld4;
        asm volatile("" : "+s"(p));
      };
      const uint32_t lane = lane_bytes(ldc4), in_lane = BETA ? lane_bytes(4 * ldcin) : 0;
      uint64_t c_next = first_row(ep.C, ep.ldc), c_out = c_next, in_next = BETA ? first_row(ep.Cin, ldcin) : 0;
      v4f cx[kRing][2], cin[BETA ? kIn : 1][2];
      auto load_c = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) cx[i % kRing][h] = row_load(c_next, lane + 128 * j_of(i), h * 8 * (uint32_t)ldc4);
        next(c_next, i, ldc4);
      };
      auto load_in = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) cin[BETA ? i % kIn : 0][h] = row_load(in_next, in_lane + 128 * j_of(i), h * 32 * (uint32_t)ldcin);
        next(in_next, i, 4 * ldcin);
      };
#pragma unroll
      for (int i = 0; i < kRing; ++i) load_c(i);
      if (BETA) {
#pragma unroll
        for (int i = 0; i < kIn; ++i) load_in(i);
      }
      float srow[TM];
      v4f sc[2 * JN];
#pragma unroll
      for (int a = 0; a < TM; ++a) srow[a] = sc_row[16 * a];
#pragma unroll
      for (int i = 0; i < kBlocks; ++i) {
        const int a = a_of(i), j = j_of(i), jl = i % JN;
        if (a == 0) {
#pragma unroll
          for (int e = 0; e < 2; ++e) sc[2 * jl + e] = *reinterpret_cast<const v4f*>(sc_col + 32 * j + 16 * e);
        }
        v4f t[2];
        block_of(a, j, srow[a], sc[2 * jl], sc[2 * jl + 1], t);
        // (the K-tiles in flight, before the first store: they are older than the loads issued here)
        if (i == 0) wait_loads_but<2 * kRing + (BETA ? 2 * kIn : 0)>();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          v4f out;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            out[v] = cx[i % kRing][h][v] + t[h][v];
            if (SCALED) out[v] = alpha * out[v];
            if (BETA) out[v] = out[v] + beta * cin[BETA ? i % kIn : 0][h][v];
          }
          row_store<CACHED || EDGE>(out, c_out, lane + 128 * j, h * 8 * (uint32_t)ldc4);
        }
        next(c_out, i, ldc4);
        if (i + kRing < kBlocks) load_c(i + kRing);
        if (BETA && i + kIn < kBlocks) load_in(i + kIn);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // ---- accumulate mode, a tile on the edge: sixteen rows at a time (a ring through the branches spills)
    auto add_to_edge = [&](auto elems_tag, int rows, int cols) {
      constexpr bool ELEMS = decltype(elems_tag)::value;
      const int r8 = ln & 7, c16 = 16 * ((ln >> 3) & 1) + 4 * quad;
      uint64_t c_row = first_row(ep.C, ep.ldc), in_row = has_beta ? first_row(ep.Cin, ldcin) : 0;
      wait_loads();                                  // (the K-tiles in flight, before the first store)
#pragma unroll
      for (int a = 0; a < TM; ++a) {
        if (16 * a < rows) {
          const float sr = sc_row[16 * a];
          v4f x[TN / 2][2];
#pragma unroll
          for (int j = 0; j < TN / 2; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) x[j][h] = edge_load<ELEMS>(c_row, ldc4, 8 * h + r8, 32 * j + c16, rows - 16 * a, cols);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < TN / 2; ++j) {
            v4f t[2];
            block_of(a, j, sr, *reinterpret_cast<const v4f*>(sc_col + 32 * j), *reinterpret_cast<const v4f*>(sc_col + 32 * j + 16), t);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              v4f out, cin = {0.f, 0.f, 0.f, 0.f};
              if (SCALE && has_beta) cin = edge_load<ELEMS>(in_row, 4 * ldcin, 8 * h + r8, 32 * j + c16, rows - 16 * a, cols);
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                out[v] = x[j][h][v] + t[h][v];
                if (SCALE && do_scale) {
                  out[v] = alpha * out[v];
                  if (has_beta) out[v] = out[v] + beta * cin[v];
                }
              }
              edge_store<ELEMS>(out, c_row, ldc4, 8 * h + r8, 32 * j + c16, rows - 16 * a, cols);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        c_row += 16 * ldc4;
        in_row += 64 * ldcin;
        asm volatile("" : "+s"(c_row), "+s"(in_row));
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // ---- first mode.  EDGES: 0 a whole tile, 1 a tile on the edge, 2 one whose last columns are not a whole access
    // (rows x cols of the wave's block exist)
    auto write_c = [&](auto edges_tag, int rows, int cols) {
      constexpr int EDGES = decltype(edges_tag)::value;
      const int r8 = ln & 7, c16 = 16 * ((ln >> 3) & 1) + 4 * quad;
      uint64_t c_row = first_row(ep.C, ep.ldc), in_row = has_beta ? first_row(ep.Cin, ldcin) : 0;
      const uint32_t lane = lane_bytes(ldc4), in_lane = SCALE ? lane_bytes(4 * ldcin) : 0;
      // |D_F| is added up in FP32 over a lane's 16 columns of 64 resp. 4 rows of 64 and in double from there
      float srow[TM], r1[TM], r2[TM];                // row scales; the lane's sums of the columns 0-63 and 64-127
#pragma unroll
      for (int a = 0; a < TM; ++a) srow[a] = sc_row[16 * a];
      const int64_t me = m0 + wm * (BM / 2) + rl, ne = n0 + wn * (BN / 2) + 4 * quad;
#pragma unroll
      for (int j = 0; j < TN / 2; ++j) {
        v4f sc[2], q1[2], q2[2], q4[2];              // column scales; column sums of 2, 2 and 4 rows
        double col8[8];                              // ... of 8 rows
#pragma unroll
        for (int e = 0; e < 2; ++e) sc[e] = *reinterpret_cast<const v4f*>(sc_col + 32 * j + 16 * e);
#pragma unroll
        for (int a = 0; a < TM; ++a) {
          // (the comparisons are made afresh in every step: kept, their masks spill scalar registers)
          if (EDGES) asm volatile("" : "+s"(rows), "+s"(cols));
          v4f cin[2];
          if (SCALE && has_beta) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
              cin[h] = EDGES ? edge_load<EDGES == 2>(in_row, 4 * ldcin, 8 * h + r8, 32 * j + c16, rows - 16 * a, cols)
                             : row_load(in_row, in_lane + 128 * j, h * 32 * (uint32_t)ldcin);
          }
          v4f d[2];
          float rs[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              d[e][v] = acc_value(acc[a][2 * j + e][v]) * (srow[a] * sc[e][v]);
              if (EDGES && SUMS && !(16 * a + rl < rows && 32 * j + 16 * e + 4 * quad + v < cols)) d[e][v] = 0.f;
            }
            if (SUMS) {
              rs[e] = (fabsf(d[e][0]) + fabsf(d[e][1])) + (fabsf(d[e][2]) + fabsf(d[e][3]));
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                q1[e][v] = (a & 1) == 0 ? fabsf(d[e][v]) : q1[e][v] + fabsf(d[e][v]);
                if ((a & 3) == 1) q2[e][v] = q1[e][v];
                if (a == 3) q4[e][v] = q2[e][v] + q1[e][v];
                if (a == TM - 1) col8[4 * e + v] = (double)q4[e][v] + (double)(q2[e][v] + q1[e][v]);
              }
            }
          }
          if (SUMS) {
            // (the sums are formed here: nothing but this keeps the compiler from putting them off, with all they add
            // up, to the end)
#pragma unroll
            for (int e = 0; e < 2; ++e) asm volatile("" : "+v"(rs[e]), "+v"(q1[e][0]), "+v"(q1[e][1]), "+v"(q1[e][2]), "+v"(q1[e][3]));
            const float r = rs[0] + rs[1];
            if (j == 0) r1[a] = r;
            if (j == 1) r1[a] += r;
            if (j == 2) r2[a] = r;
            if (j == 3) r2[a] += r;
          }
          exchange_half_rows(d[0], d[1]);
          if (j == 0 && a == 0) wait_loads();        // the K-tiles in flight, before the first store
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            v4f out;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              out[v] = d[h][v];
              if (SCALE && do_scale) {
                out[v] = alpha * out[v];
                if (has_beta) out[v] = out[v] + beta * cin[h][v];
              }
            }
            if (EDGES) edge_store<EDGES == 2>(out, c_row, ldc4, 8 * h + r8, 32 * j + c16, rows - 16 * a, cols);
            else row_store<EDGE>(out, c_row, lane + 128 * j, h * 8 * (uint32_t)ldc4);
          }
          c_row += a == TM - 1 ? -(TM - 1) * 16 * ldc4 : 16 * ldc4;
          if (SCALE) in_row += a == TM - 1 ? -(TM - 1) * 64 * ldcin : 64 * ldcin;
          asm volatile("" : "+s"(c_row), "+s"(in_row));
          __builtin_amdgcn_sched_barrier(0);
        }
        if (SUMS) {
          // the 16 rows of a block: lane rl gets the sum of its value rl >> 1
          const double c = column_sum8(col8, rl);
          const int at = 32 * j + 16 * (rl >> 3) + ((rl >> 1) & 3);
          if (!(rl & 1) && (!EDGES || at + 4 * quad < cols))
            ep.col_part[(int64_t)(2 * tile_m + wm) * N + ne + at] = c;
        }
      }
      if (SUMS) {
#pragma unroll
        for (int a = 0; a < TM; ++a) {
          double r = (double)r1[a] + (double)r2[a];
          r += __shfl_xor(r, 16, 64);
          r += __shfl_xor(r, 32, 64);
          if (quad == 0 && (!EDGES || 16 * a + rl < rows))
            ep.row_part[(int64_t)(2 * tile_n + wn) * M + me + 16 * a] = r;
        }
      }
    };
    if (EDGE && !full) {
      const int rows = left(M - m0 - wm * (BM / 2)), cols = left(N - n0 - wn * (BN / 2));
      const bool whole = cols >= BN / 2 || (cols & 3) == 0;
      if (rows <= 0 || cols <= 0) wait_loads();
      else if constexpr (MODE == kGemmFirst) {
        if (whole) write_c(std::integral_constant<int, 1>(), rows, cols);
        else write_c(std::integral_constant<int, 2>(), rows, cols);
      } else {
        if (whole) add_to_edge(std::false_type(), rows, cols);
        else add_to_edge(std::true_type(), rows, cols);
      }
    } else if constexpr (MODE == kGemmFirst) {
      write_c(std::integral_constant<int, 0>(), BM, BN);
    } else if (SCALE ? !do_scale : two && prod == 0) {   // (another product or kernel adds to this tile)
      add_to_c(std::true_type(), std::false_type(), std::false_type());
    } else if (has_beta) {
      add_to_c(std::false_type(), std::integral_constant<bool, SCALE>(), std::integral_constant<bool, SCALE>());
    } else {
      add_to_c(std::false_type(), std::integral_constant<bool, SCALE>(), std::false_type());
    }
    // everybody has read its scales: the A buffer that held them may be loaded again (a bare
    // barrier: the stores of C stay in flight)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");
    // next product of this tile, or the next output tile of this workgroup
    if (prod < p_hi) {
      prod = 1;
    } else {
      prod = p_lo;
      vb += G;
      if (vb < total) tile_of(vb, tiles_m, tiles_n, tile_m, tile_n);
    }
  }
  wait_loads();                                     // nothing may still be writing LDS when the wave ends
}

}  // namespace

bool gemm_persistent_ok(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda, const int8_t* Qb,
                        int64_t ldb, const GemmEpilogue& ep) {
  if (ep.D_int || ep.D_F_copy) return false;                 // parity-check outputs use the plain kernel
  if (M <= 0 || N <= 0 || K <= 0 || K <= BK || (K % 64)) return false;   // (two K-tiles at least)
  if (lda >= (1 << 23) || ldb >= (1 << 23)) return false;    // byte offsets within a tile are 32-bit
  if (ep.ldc >= (1 << 25) || (ep.final_scale && ep.beta != 0.f && ep.ldcin >= (1 << 25))) return false;   // ... and within 16 rows of C
  if (((reinterpret_cast<uintptr_t>(Qa) | reinterpret_cast<uintptr_t>(Qb)) & 15) || (lda % 16) || (ldb % 16))
    return false;
  return ((M + BM - 1) / BM) * ((N + BN - 1) / BN) < (1 << 30);
}

// Compute units of the current device, looked up once per device (srq_create primes it, so
// that no property query happens inside a caller's stream capture).
hipError_t gemm_device_cus(int* cus) {
  static std::atomic<int> cached[64];               // zero-initialised; a racing first query stores the same value
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  int n = (dev >= 0 && dev < 64) ? cached[dev].load(std::memory_order_relaxed) : 0;
  if (!n) {
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, dev);
    if (e != hipSuccess) return e;
    n = prop.multiProcessorCount;
    if (dev >= 0 && dev < 64) cached[dev].store(n, std::memory_order_relaxed);
  }
  *cus = n;
  return hipSuccess;
}

hipError_t ensure_dynamic_lds(const void* kernel, int bytes) {
  static std::mutex mu;
  static std::vector<std::pair<int, const void*>> done;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  for (const auto& d : done)
    if (d.first == dev && d.second == kernel) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.emplace_back(dev, kernel);
  return e;
}

hipError_t launch_gemm_i8_persistent(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda,
                                     const int8_t* Qb, int64_t ldb, const GemmEpilogue& ep, hipStream_t st,
                                     const GemmSecond* second) {
  int num_cu = 0;
  hipError_t e = gemm_device_cus(&num_cu);
  if (e != hipSuccess) return e;
  const int64_t tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
  int64_t wgs = num_cu / 8 * 8;                              // one workgroup per CU, a multiple of the 8 XCDs
  if (wgs < 8) wgs = 8;
  if (wgs > tm * tn) wgs = tm * tn;
  const bool sums = ep.mode == kGemmFirst && ep.row_part != nullptr;
  const bool scale = ep.final_scale != 0, edge = (M % BM) || (N % BN);
  void (*kern)(int64_t, int64_t, int64_t, const int8_t*, int64_t, const int8_t*, int64_t, int, int, GemmEpilogue,
               GemmSecond);
  GemmSecond sec = {nullptr, nullptr, 0, 0, nullptr, nullptr};
  if (second && ep.mode == kGemmAccum) sec = *second;
#define SRQ_KERN(MODE, SUMS, SCALE)                                                  \
  (!edge                                                                           \
       ? gemm_i8_persistent_kernel<MODE, SUMS, SCALE, false, 1>                    \
       : MODE == kGemmAccum && ep.ldc % 1024 ? gemm_i8_persistent_kernel<MODE, SUMS, SCALE, true, MODE == kGemmAccum ? 4 : 1> \
                                             : gemm_i8_persistent_kernel<MODE, SUMS, SCALE, true, 1>)
  // (sums come with a correction after this product, alpha and beta with the last one)
  if (sums && scale) return hipErrorInvalidValue;
  kern = ep.mode != kGemmFirst ? (scale ? SRQ_KERN(kGemmAccum, false, true) : SRQ_KERN(kGemmAccum, false, false))
         : sums                ? SRQ_KERN(kGemmFirst, true, false)
                               : (scale ? SRQ_KERN(kGemmFirst, false, true) : SRQ_KERN(kGemmFirst, false, false));
#undef SRQ_KERN
  e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kLdsBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(256), kLdsBytes, st, M, N, K, Qa, lda, Qb, ldb, (int)tm,
                     (int)tn, ep, sec);
  return hipGetLastError();
}

}  // namespace srq
