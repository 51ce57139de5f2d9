// Operand with strided vectors (B, columns of a row-major matrix) in ONE read: maxima, scales, codes, residual scales
// and residual codes, where the passes of fused.hip read it once for each of the maxima, the codes and the residual codes.
//
// A workgroup holds 512 rows x 32 columns in registers (sixteen rows by four columns per thread, as cols_pass_kernel:
// 128 contiguous bytes of a row, 512 of a column of codes).  The workgroups of a strip of 32 columns exchange what a
// column's scale needs, the maxima of their pieces, through memory: each publishes a line of 32 words and reads the lines
// of the others.  The columns of the residual follow in the same way.
//
// What bounds it: 4 bytes read and 2 written per element, and the residence of a workgroup, whose two exchanges take
// about 3 us each (one trip of a line from one XCD to another) while its registers hold data: three or four
// workgroups per compute unit keep 48 to 64 MiB of the operand on chip, enough to cover that.
//
// Measured (rocprofv3, us), the passes of fused.hip / this: 8192 x 8192 maxima + codes + (residual codes and mask) 61 + 63 + 68 /
// 93 (4.3 TB/s), 4096 x 14336 41 + 50 + 50 / 79, scales given and mask 48 + 50 / 73, codes alone 41 + 50 / 57; 4096 x 4096 27.
//
// Every wait ends: a workgroup waits for a bounded time in each exchange (exchange_wait.h), and what has not been published by then (others may be kept
// from starting by whatever else runs) it works out from memory by itself, which is slower and gives the same
// bits: maxima do not depend on an order.
#include <type_traits>
#include "exchange_wait.h"
#include "gemm_lanes.h"
#include "stream.h"

namespace srq {
namespace {

constexpr int CG = 8, BC = 4 * CG, BR = kColsOnceRows;   // column groups, columns and rows of a workgroup
static_assert(BC == kColsOnceCols && BR == 256 / CG * 16, "a workgroup's patch");

constexpr uint32_t kPublished = 0x80000000u;          // (maxima are not negative)

__device__ __forceinline__ void put_word(uint32_t* p, uint32_t w) {
  __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class There>
__device__ __forceinline__ uint32_t wait_for(ExchangeWait& wait, const uint32_t* p, There there) {
  return wait.word([p]() { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }, there,
                   []() { return (uint64_t)wall_clock64(); }, []() { __builtin_amdgcn_s_sleep(4); });
}

// max |x|, or max |x - fl(code * s)|, of the four columns of a column group over all rows
template <bool TRUNC, bool RESIDUAL>
__device__ __forceinline__ void strip_maxima(const float* X, int64_t rows, int64_t ldx, int64_t col0, int ncol, int rb,
                                             const float (&lam)[4], const float (&sc)[4], float qmax, float (&m)[4]) {
#pragma unroll 1
  for (int64_t r = rb; r < rows; r += 256 / CG) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float x = X[r * ldx + col0 + (c < ncol ? c : 0)];
      m[c] = fmaxf(m[c], fabsf(RESIDUAL ? x - code_value(biased_code(x, lam[c], qmax, TRUNC)) * sc[c] : x));
    }
  }
}

template <bool TRUNC, bool GIVEN, bool RESID, bool MASK, bool EM>   // EM: residual codes element-major
__global__ __launch_bounds__(256, EM ? 3 : 4) void cols_once_kernel(ColsOnce g, int64_t rows, int64_t cols, float qmax, int pieces) {
  __shared__ uint32_t red[BC], kept[BC];
  const int tid = threadIdx.x, cg = tid & (CG - 1), rb = tid / CG;
  const int64_t strip = blockIdx.x / (unsigned)pieces;
  const int piece = (int)(blockIdx.x - strip * pieces);
  const int64_t col0 = strip * BC + cg * 4, row0 = (int64_t)piece * BR + rb * 16;
  const int ncol = col0 + 4 <= cols ? 4 : col0 < cols ? (int)(cols - col0) : 0;   // columns of the patch
  if (tid < BC) { red[tid] = 0; kept[tid] = 0; }
  // (no branch around a load: what does not exist gets an offset outside the descriptor and reads as zero; the last
  // columns of a row that are not four are read with those before them)
  float4 v[16];
  {
    const __amdgpu_buffer_rsrc_t rs = buf_rsrc(g.X + (int64_t)piece * BR * g.ldx, kRecords);
    const uint32_t ld4 = 4u * (uint32_t)g.ldx, at = 4u * (uint32_t)(ncol == 4 ? col0 : cols - 4) + (uint32_t)(rb * 16) * ld4;
    const int here = ncol ? (int)(rows - row0) : 0;    // rows of the patch, or more
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const v4i t = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, i < here ? at + i * ld4 : kOutside, 0, 2 /* non-temporal */));
      v[i] = make_float4(__int_as_float(t.x), __int_as_float(t.y), __int_as_float(t.z), __int_as_float(t.w));
    }
    if (ncol > 0 && ncol < 4) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float4 x = v[i];
        v[i] = make_float4(ncol == 3 ? x.y : ncol == 2 ? x.z : x.w, ncol == 3 ? x.z : ncol == 2 ? x.w : 0.f, ncol == 3 ? x.w : 0.f, 0.f);
      }
    }
  }
  const bool writer = piece == 0 && rb == 0 && ncol > 0;
  float lam[4] = {0.f, 0.f, 0.f, 0.f}, sc[4] = {0.f, 0.f, 0.f, 0.f};
  // red gets what this workgroup cannot wait for from memory
  auto alone = [&](auto residual_tag, float (&m)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = 0.f;
    if (ncol) strip_maxima<TRUNC, decltype(residual_tag)::value>(g.X, rows, g.ldx, col0, ncol, rb, lam, sc, qmax, m);
#pragma unroll
    for (int c = 0; c < 4; ++c) atomicMax(&red[cg * 4 + c], __float_as_uint(m[c]));
    __syncthreads();
  };
  // the maxima m of the patch become those of the whole columns; `lines`: where this exchange publishes
  auto exchange = [&](uint32_t* lines, auto residual_tag, float (&m)[4]) __attribute__((always_inline)) {
    __syncthreads();                                   // red is clear
#pragma unroll
    for (int c = 0; c < 4; ++c) atomicMax(&red[cg * 4 + c], __float_as_uint(m[c]));
    __syncthreads();
    if (pieces > 1) {
      uint32_t* const mine = lines + strip * pieces * BC;
      // (what other pieces have added to red in the meantime belongs to the same column)
      if (tid < BC) put_word(mine + piece * BC + tid, red[tid] | kPublished);
      bool late = false;
      ExchangeWait wait{g.wait_ticks};
      for (int i = tid; i < pieces * BC; i += 256) {
        const uint32_t w = wait_for(wait, mine + i, [](uint32_t x) { return x != 0; });
        if (w) atomicMax(&red[i & (BC - 1)], w & ~kPublished);
        else late = true;
      }
      if (__syncthreads_or(late)) alone(residual_tag, m);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = __uint_as_float(red[cg * 4 + c]);
  };
  // The same without memory of its own, for a call that may use none: the maxima gather in `scale`, and the first word
  // of the strip's lambdas counts the pieces that have added theirs (low half) and those that have read the
  // result (high half); the last one of these puts the scales and lambdas there.
  auto exchange_in_place = [&](float (&m)[4]) __attribute__((always_inline)) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) atomicMax(&red[cg * 4 + c], __float_as_uint(m[c]));
    __syncthreads();
    const bool has = tid < BC && strip * BC + tid < cols;
    uint32_t* const maxima = reinterpret_cast<uint32_t*>(g.scale) + strip * BC;
    uint32_t* const state = reinterpret_cast<uint32_t*>(g.lambda) + strip * BC;
    if (pieces > 1) {
      bool late = false;
      if (tid < 64) {                                  // (one wave: what it has done before a count is complete by then)
        uint32_t done = 0;
        if (has) done = __hip_atomic_fetch_max(maxima + tid, red[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(done) : : "memory");
        if (tid == 0) {
          __hip_atomic_fetch_add(state, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const uint32_t all = (uint32_t)pieces;
          ExchangeWait wait{g.wait_ticks};
          const uint32_t w = wait_for(wait, state, [all](uint32_t x) { return (x & 0xffffu) == all; });
          late = (w & 0xffffu) != all;
        }
        if (has) {
          const uint32_t w = __hip_atomic_load(maxima + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          atomicMax(&red[tid], w);
          done = w;
        }
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(done) : : "memory");
      }
      if (__syncthreads_or(late)) alone(std::false_type(), m);
    }
    // (the count of readers after the barrier: everything above has been read by then)
    if (tid < 64) {
      uint32_t before = (uint32_t)(pieces - 1) << 16;
      if (pieces > 1 && tid == 0) before = __hip_atomic_fetch_add(state, 1u << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      before = __builtin_amdgcn_readfirstlane(before);
      if (has && (before >> 16) + 1 == (uint32_t)pieces) {
        const float top = __uint_as_float(red[tid]);
        g.scale[strip * BC + tid] = top > 0.f ? top / qmax : 0.f;
        g.lambda[strip * BC + tid] = top > 0.f ? qmax / top : 0.f;
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = __uint_as_float(red[cg * 4 + c]);
  };
  if (GIVEN) {
    const float4 l4 = load_part(g.lambda + col0, ncol), s4 = load_part(g.scale + col0, ncol);
    lam[0] = l4.x; lam[1] = l4.y; lam[2] = l4.z; lam[3] = l4.w;
    sc[0] = s4.x; sc[1] = s4.y; sc[2] = s4.z; sc[3] = s4.w;
  } else {
    float m[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      m[0] = fmaxf(m[0], fabsf(v[i].x)); m[1] = fmaxf(m[1], fabsf(v[i].y));
      m[2] = fmaxf(m[2], fabsf(v[i].z)); m[3] = fmaxf(m[3], fabsf(v[i].w));
    }
    if (RESID) exchange(g.lines, std::false_type(), m);
    else exchange_in_place(m);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (m[c] > 0.f) { lam[c] = qmax / m[c]; sc[c] = m[c] / qmax; }
    if (RESID && writer) {
      store_part(g.scale + col0, sc, ncol);
      store_part(g.lambda + col0, lam, ncol);
    }
  }
  if (MASK) {
    const float4 t4 = load_part(g.thresh + col0, ncol);
    const float tt[4] = {t4.x, t4.y, t4.z, t4.w};
    unsigned bits[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const bool ok = ncol > 0 && row0 + i < rows;
      const float xv[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) bits[c] |= (ok && fabsf(xv[c]) > tt[c]) ? (1u << i) : 0u;
    }
    if (row0 < g.mask_stride * 8) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (c < ncol) *reinterpret_cast<uint16_t*>(g.mask + (col0 + c) * g.mask_stride + (row0 >> 3)) = (uint16_t)bits[c];
    }
    if (GIVEN) __syncthreads();                        // kept is clear
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (bits[c]) atomicAdd(&kept[cg * 4 + c], (uint32_t)__popc(bits[c]));
    __syncthreads();
    if (tid < BC && strip * BC + tid < cols && kept[tid]) atomicAdd(&g.counts[strip * BC + tid], (int32_t)kept[tid]);
  }
  if (RESID && !GIVEN && !MASK && g.counts) {
    // (kept was cleared before the barriers of the exchange)
    int n[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      n[0] += fabsf(v[i].x) > 0.f; n[1] += fabsf(v[i].y) > 0.f;
      n[2] += fabsf(v[i].z) > 0.f; n[3] += fabsf(v[i].w) > 0.f;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) atomicAdd(&kept[cg * 4 + c], (uint32_t)n[c]);
    __syncthreads();
    if (tid < BC && strip * BC + tid < cols && kept[tid]) atomicAdd(&g.counts[strip * BC + tid], (int32_t)kept[tid]);
  }
  // sixteen codes of each of the patch's columns
  auto put = [&](int8_t* Qvm, int64_t ldvm, const unsigned (&packed)[4][4]) __attribute__((always_inline)) {
    if (row0 >= (g.pad_to ? g.pad_to : rows)) return;
    const int here = row0 + 16 <= rows ? 16 : rows > row0 ? (int)(rows - row0) : 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c >= ncol) break;
      int8_t* dst = Qvm + (col0 + c) * ldvm + row0;
      if (here == 16) {
        const u4u pk = {packed[c][0], packed[c][1], packed[c][2], packed[c][3]};
        *reinterpret_cast<u4u*>(dst) = pk;
      } else {
        // the last rows, without a loop (one of single bytes took 11 us of 26 at 4000 x 1200).  Zeros come after them where rows are
        // padded: the code of what does not exist is another one where lambda overflowed.
        unsigned x[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int n = here - 4 * w;
          x[w] = packed[c][w] & (n >= 4 ? ~0u : n > 0 ? (1u << (8 * n)) - 1u : 0u);
        }
        if (g.pad_to) {
          *reinterpret_cast<u4u*>(dst) = u4u{x[0], x[1], x[2], x[3]};
        } else {
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int n = here - 4 * w;
            if (n >= 4) {
              *reinterpret_cast<u1u*>(dst + 4 * w) = x[w];
            } else {
#pragma unroll
              for (int i = 0; i < 3; ++i)
                if (i < n) dst[4 * w + i] = (int8_t)(x[w] >> (8 * i));
            }
          }
        }
      }
    }
  };
  float rm[4] = {0.f, 0.f, 0.f, 0.f};
  {
    unsigned packed[4][4];                             // [column][word]
#pragma unroll
    for (int i = 0; i < 16; i += 4) {
      float z[4][4];                                   // [row][column]
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float xv[4] = {v[i + r].x, v[i + r].y, v[i + r].z, v[i + r].w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          z[r][c] = biased_code(xv[c], lam[c], qmax, TRUNC);
          if (RESID) {
            xv[c] = xv[c] - code_value(z[r][c]) * sc[c];
            // (one register per element, through the exchange that follows: the maximum is formed here)
            asm volatile("" : "+v"(xv[c]));
            rm[c] = fmaxf(rm[c], fabsf(xv[c]));
            asm volatile("" : "+v"(rm[c]));
          }
        }
        if (RESID) v[i + r] = make_float4(xv[0], xv[1], xv[2], xv[3]);   // the residual in place of x
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        packed[c][i / 4] = pack_codes(z[0][c], z[1][c], z[2][c], z[3][c], 4);
        asm volatile("" : "+v"(packed[c][i / 4]));     // (packed here, or the biased codes stay in as many registers as x)
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    put(g.Q, g.ldq, packed);
  }
  if (!RESID) return;
  if (row0 + 16 > rows) {
    // (places past the last row hold 0, but 0 * lam is not 0 where lam overflowed: they stay out of the maxima)
#pragma unroll
    for (int c = 0; c < 4; ++c) rm[c] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (row0 + i >= rows) v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      rm[0] = fmaxf(rm[0], fabsf(v[i].x)); rm[1] = fmaxf(rm[1], fabsf(v[i].y));
      rm[2] = fmaxf(rm[2], fabsf(v[i].z)); rm[3] = fmaxf(rm[3], fabsf(v[i].w));
    }
  }
  __syncthreads();                                     // (red has been read)
  if (tid < BC) red[tid] = 0;
  exchange(g.lines + (GIVEN ? 0 : (int64_t)(gridDim.x * BC)), std::true_type(), rm);
  float rlam[4] = {0.f, 0.f, 0.f, 0.f}, rs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (rm[c] > 0.f) { rlam[c] = qmax / rm[c]; rs[c] = rm[c] / qmax; }
  if (writer) {
    store_part(g.rscale + col0, rs, ncol);
    if (g.rlambda) store_part(g.rlambda + col0, rlam, ncol);
  }
  unsigned packed[4][4];
#pragma unroll
  for (int i = 0; i < 16; i += 4) {
    float z[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float xv[4] = {v[i + r].x, v[i + r].y, v[i + r].z, v[i + r].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) z[r][c] = biased_code(xv[c], rlam[c], qmax, TRUNC);
      if (EM && ncol && row0 + i + r < rows) {
        int8_t* dst = g.Rem + (row0 + i + r) * g.ldem + col0;
        const unsigned p = pack_codes(z[r][0], z[r][1], z[r][2], z[r][3], 4);
        if (ncol == 4) {
          *reinterpret_cast<u1u*>(dst) = p;
        } else {
#pragma unroll
          for (int c = 0; c < 3; ++c)
            if (c < ncol) dst[c] = (int8_t)(p >> (8 * c));
        }
      }
    }
    if (!EM) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        packed[c][i / 4] = pack_codes(z[0][c], z[1][c], z[2][c], z[3][c], 4);
        asm volatile("" : "+v"(packed[c][i / 4]));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if (!EM) put(g.Rvm, g.ldr, packed);
}

}  // namespace

// (the rows of a piece are reached by 32-bit offsets)
bool cols_once_ok(int64_t rows, int64_t cols, int64_t ldx) {
  return rows > 0 && rows <= 32768 && cols >= 4 && cols <= ((int64_t)1 << 24) && ldx < ((int64_t)1 << 20);
}

hipError_t launch_cols_once(const ColsOnce& g, int64_t rows, int64_t cols, int qmax, int trunc, bool given, hipStream_t st) {
  const int64_t pieces = (rows + BR - 1) / BR, strips = (cols + BC - 1) / BC;
  const dim3 grid((unsigned)(strips * pieces));
  const bool resid = g.rscale != nullptr, mask = g.mask != nullptr;
  // (what no call asks for: a mask with scales yet to be formed, codes alone with scales given, both layouts, k-major codes of a
  // whole call, which are copied)
  if ((mask && !given) || (!resid && given) || (resid && (!g.Rvm == !g.Rem)) || (g.Rem && !given)) return hipErrorInvalidValue;
#define SRQ_ONCE(GIVEN, RESID, MASK, EM)                                                                                       \
  hipLaunchKernelGGL((trunc ? cols_once_kernel<true, GIVEN, RESID, MASK, EM> : cols_once_kernel<false, GIVEN, RESID, MASK, EM>), \
                     grid, dim3(256), 0, st, g, rows, cols, (float)qmax, (int)pieces)
  if (!resid) SRQ_ONCE(false, false, false, false);
  else if (g.Rem) {
    if (mask) SRQ_ONCE(true, true, true, true);
    else SRQ_ONCE(true, true, false, true);
  } else {
    if (mask) SRQ_ONCE(true, true, true, false);
    else if (given) SRQ_ONCE(true, true, false, false);
    else SRQ_ONCE(false, true, false, false);
  }
#undef SRQ_ONCE
  return hipGetLastError();
}

}  // namespace srq
