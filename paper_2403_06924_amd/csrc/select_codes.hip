// Keep-masks of Eq. avgQuan with their counts per vector, of both operands in one launch, from the codes and residual codes
// that the quantize passes have left, where the mask passes of fused.hip and strips.hip read the FP32 operands again: 2
// bytes per element instead of 4.  Where strips.hip would take the selection, with the means and thresholds as it does.
//
// |x| -> (code, residual code) is monotone: fl(x * lambda), the rounding and the clamp are, and for one code so are
// fl(x - fl(code * s)) and its code in turn; all of them are odd.  With key(x) = |256 code + residual code| therefore
//     key(x) > key(t)  =>  |x| > t,       key(x) < key(t)  =>  |x| < t,
// and only the elements of the threshold's own key (one bin in some 16000 of the vector's range) are read in FP32.  So are
// those of the topmost key, which NaN shares, and whole vectors whose scales are not ordinary numbers.
//
// What bounds it: 2 bytes per element (4.8 TB/s on two operands of 8192 x 8192).  Both operands, us, from FP32 / from codes:
// 8192 x 8192 each 46 + (68 with the residual codes of B) / 54 to 56; 4096 x 4096 and 4096 x 14336 12 + 50 / 36 with a wave per
// vector (55 with a workgroup for each, which has too few bytes on their way).
// On the side: the zero-filled codes (16 bytes per lane, what is in registers already) where the corrections follow at once, and the
// counts of every 256 vectors where the compaction wants them.
#include "compact.h"
#include "stream.h"

namespace srq {
namespace {

typedef short s2 __attribute__((ext_vector_type(2)));
typedef unsigned u4a __attribute__((ext_vector_type(4)));

__device__ __forceinline__ s2 both(int x) { return s2{(short)x, (short)x}; }

// One bit of each of sixteen elements out of the signs of eight pairs: pushed in from the top two places at a time, the even
// elements end in the odd bits of the low half, the odd ones in those of the high half.
struct Bits16 {
  unsigned acc = 0;
  __device__ __forceinline__ void take(unsigned w) { acc = (w & 0x80008000u) | (acc >> 2); }
  __device__ __forceinline__ unsigned get() const { return (acc >> 1 & 0x5555u) | (acc >> 16 & 0xaaaau); }
};

// |256 code + residual code| - key of elements 2 j and 2 j + 1 of the sixteen in q and r (residual codes plus 128); the
// differences are at least -32767
__device__ __forceinline__ s2 above_key(const unsigned (&q)[4], const unsigned (&r)[4], int j, s2 hi, s2 lo) {
  const s2 w = __builtin_bit_cast(s2, __builtin_amdgcn_perm(q[j >> 1], r[j >> 1], j & 1 ? 0x07030602u : 0x05010400u));
  return __builtin_elementwise_max(__builtin_elementwise_sub_sat(w, hi), __builtin_elementwise_sub_sat(lo, w));
}

// sixteen elements: bits of those above the threshold's key, and of those that have to be looked at (that key's own and the
// topmost one's).  Bound by vector instructions as much as by memory: eleven for two elements (with other pairs, whose bits
// took two more and the topmost key eight, 62 us instead of 54 for two operands of 8192 x 8192, calls of 2048^3 67.6 instead of 65.8).
__device__ __forceinline__ void compare16(u4a q, u4a r, int tk, int top, unsigned& above, unsigned& open) {
  const unsigned qw[4] = {q.x, q.y, q.z, q.w};
  const unsigned rw[4] = {r.x ^ 0x80808080u, r.y ^ 0x80808080u, r.z ^ 0x80808080u, r.w ^ 0x80808080u};
  const s2 hi = both(tk + 128), lo = both(128 - tk), none = both(0);
  Bits16 gt, lt;
  s2 most = both(-32767);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const s2 d = above_key(qw, rw, j, hi, lo);
    gt.take(__builtin_bit_cast(unsigned, (s2)(none - d)));
    lt.take(__builtin_bit_cast(unsigned, d));
    most = __builtin_elementwise_max(most, d);
  }
  above = gt.get();
  open = ~lt.get() & ~above & 0xffffu;
  if (most.x == top - tk || most.y == top - tk) {      // (none is above the topmost key)
    const s2 last = both(top - tk), one = both(1);
    Bits16 at;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const s2 e = above_key(qw, rw, j, hi, lo) ^ last;
      at.take(__builtin_bit_cast(unsigned, (s2)(e - one)) & ~__builtin_bit_cast(unsigned, e));   // (the sign of e == 0)
    }
    open |= at.get();
  }
}

__device__ __forceinline__ bool ordinary(float x) { return x > 0.f && x < INFINITY; }

template <int TH, int NV, bool TRUNC>   // TH threads per vector, NV pieces of 16 elements for each
__global__ __launch_bounds__(256) void select_codes_kernel(CodesSelect a, CodesSelect b, int64_t veclen, int64_t ld, float qmax, int64_t groups_a) {
  constexpr int VECS = 256 / TH, STEP = 16 * TH;
  __shared__ int sm[4];
  const bool first = (int64_t)blockIdx.x < groups_a;
  const CodesSelect& o = first ? a : b;
  const int tid = threadIdx.x & (TH - 1);
  const int sub = TH >= 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / TH) : 0;
  int64_t group = first ? blockIdx.x : blockIdx.x - groups_a;
  if (o.elem_step != 1) {
    // 32 neighbouring columns, which share lines of X, on one XCD: what has to be looked at is found in its L2
    constexpr int64_t kNear = 32 / VECS;
    const int64_t groups = (o.nvec + VECS - 1) / VECS, q = group >> 3;
    if (group < groups / (8 * kNear) * (8 * kNear)) group = ((q / kNear) * 8 + (group & 7)) * kNear + q % kNear;
  }
  int64_t v = group * VECS + sub;
  const bool exists = v < o.nvec;
  if (!exists) v = o.nvec - 1;                         // (does the last vector's work again and writes nothing)
  const int8_t *const q = o.Q + v * ld, *const r = o.R + v * ld;
  u4a qv[NV], rv[NV];
  if (o.mask) {                                        // (on their way while the threshold is formed)
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int64_t e = 16 * tid + STEP * i, at = e < ld ? e : 0;
      qv[i] = *reinterpret_cast<const u4a*>(q + at);
      rv[i] = *reinterpret_cast<const u4a*>(r + at);
    }
  }
  float t;
  if (o.part) {
    // line 7: the mean.  Every 64th partial sum by a lane, the lanes as a tree: the order in which strips.hip adds them, too
    double sum = 0.0;
    for (int64_t p = threadIdx.x & 63; p < o.nparts; p += 64) sum += o.part[p * o.nvec + v];
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    const float mean = (float)(sum / o.count);
    t = o.theta * mean;
    if (tid == 0 && exists) { o.mean[v] = mean; o.thresh[v] = t; }
  } else {
    t = o.thresh[v];
  }
  if (!o.mask) return;
  const float lam = o.lambda[v], s = o.scale[v], rlam = o.rlambda[v];
  const int64_t words = (veclen + 63) / 64;
  uint16_t* const out = reinterpret_cast<uint16_t*>(o.mask + v * words);
  const float* const x = o.X + v * o.vec_step;
  // elements e .. e + 15 that exist
  auto present = [&](int64_t e) -> unsigned { return e + 16 <= veclen ? 0xffffu : e < veclen ? (1u << (veclen - e)) - 1u : 0u; };
  // sixteen elements in FP32; those past the end are read in the last one's place
  auto look_all = [&](int64_t e) -> unsigned {
    float y[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) y[j] = x[(e + j < veclen ? e + j : veclen - 1) * o.elem_step];
    unsigned m = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) m |= fabsf(y[j]) > t ? 1u << j : 0u;
    return m;
  };
  // the elements of `open`: as a rule one in a few hundred lanes
  auto look = [&](int64_t e, unsigned open) -> unsigned {
    if (__any(__popc(open) > 4)) return look_all(e) & open;
    unsigned m = 0;
    while (open) {
      const int j = __ffs((int)open) - 1;
      open &= open - 1u;
      if (fabsf(x[(e + j) * o.elem_step]) > t) m |= 1u << j;
    }
    return m;
  };
  int total = 0;
  auto put = [&](int64_t e, unsigned m, u4a code) {
    if (exists && e < words * 64) {
      out[e >> 4] = (uint16_t)m;
      if (o.D) {
        u4a d;
#pragma unroll
        for (int j = 0; j < 4; ++j) d[j] = code[j] & bytes_of(m >> (4 * j) & 15u);
        *reinterpret_cast<u4a*>(o.D + v * ld + e) = d;
      }
    }
    total += __popc(m);
  };
  const bool none = !(t < INFINITY) || (s == 0.f && lam == 0.f && t >= 0.f);   // (nothing is above NaN, infinity or the maximum of a zero vector)
  if (none) {
    for (int64_t e = 16 * tid; e < words * 64; e += STEP) put(e, 0u, u4a{0, 0, 0, 0});
  } else if (!(ordinary(lam) && ordinary(s) && qmax * s < INFINITY && rlam < INFINITY && t >= 0.f)) {
    // (qmax * s overflows where the scale of a maximum next to FLT_MAX is rounded up: that element's residual is infinite, and
    // rlam zero as where every residual is)
#pragma unroll 1
    for (int64_t e = 16 * tid; e < words * 64; e += STEP) put(e, look_all(e) & present(e), *reinterpret_cast<const u4a*>(q + e));
  } else {
    const float zc = biased_code(t, lam, qmax, TRUNC), tc = code_value(zc);
    const int tk = (int)tc * 256 + (int)code_value(biased_code(t - tc * s, rlam, qmax, TRUNC));
    const int top = 257 * (int)qmax;
    // a residual that is zero everywhere: x is fl(code * s) itself
    const bool exact = rlam == 0.f, equal = tc * s > t;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int64_t e = 16 * tid + STEP * i;
      unsigned m, open;
      compare16(qv[i], rv[i], tk, top, m, open);
      const unsigned here = present(e);
      m &= here & ~open;
      open &= here;
      if (exact) {
        // (only the topmost key is looked at: its residual code is not zero unless x is NaN)
        unsigned above, t1;
        compare16(qv[i], rv[i], top, top, above, t1);
        if (equal) m |= open & ~t1;
        open &= t1;
      }
      if (open) m |= look(e, open);
      put(e, m, qv[i]);
    }
  }
  for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
  if (TH > 64) {
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = total;
    __syncthreads();
    total = 0;
#pragma unroll
    for (int i = 0; i < TH / 64; ++i) total += sm[sub * (TH / 64) + i];
  }
  if (tid == 0 && exists) {
    o.counts[v] = total;
    if (o.sums && total) atomicAdd(o.sums + (v >> 8) * kSumStride, total);
  }
}

}  // namespace

// (With few codes the threshold's bin is wide, and most of it is looked at in FP32 where outliers set the scale: calls, us, the passes
// over FP32 / from the codes, 4 bits 384 x 5952 x 8576 329 / 422, 5000 x 4000 x 3000 341 / 432, without outliers 336 / 310; 7 bits 315 /
// 271, 8 bits 320 / 277.  On the path of strips.hip most of what is looked at is found in the caches, and the compaction may go
// behind the tiles: with outliers / normal, 4 bits, 96 x 128 x 3371 57.4 / 51.5 and 52.3 / 46.0, 640^2 x 4000 74.2 / 68.8 and 69.1 / 58.4,
// 2000^3 70.9 / 66.6 and 73.1 / 69.6, 100 x 1900 x 7000 170 / 176 and 126 / 103.  3 bits have 49 keys.  A threshold of zero leaves every
// zero to be looked at.  What stays slower, 4096^3 with 80 % kept of numbers over twenty binades 425 / 495, is where the threshold
// is in the lowest of 65000 bins.)
bool select_codes_ok(int qmax, float theta, bool strips) { return qmax >= (strips ? 7 : 63) && theta > 0.f; }

hipError_t launch_select_codes(const CodesSelect& a, const CodesSelect& b, int64_t veclen, int64_t ld, int qmax, int trunc, hipStream_t st) {
  if (a.nvec + b.nvec <= 0 || veclen <= 0) return hipSuccess;
#define SRQ_MASK(TH, NV)                                                                                                   \
  do {                                                                                                                     \
    const int64_t ga = (a.nvec + 256 / TH - 1) / (256 / TH), gb = (b.nvec + 256 / TH - 1) / (256 / TH);                     \
    hipLaunchKernelGGL((trunc ? select_codes_kernel<TH, NV, true> : select_codes_kernel<TH, NV, false>), dim3((unsigned)(ga + gb)), \
                       dim3(256), 0, st, a, b, veclen, ld, (float)qmax, ga);                                                \
  } while (0)
  if (veclen <= 1024) SRQ_MASK(64, 1);
  else if (veclen <= 2048) SRQ_MASK(64, 2);
  else if (veclen <= 4096) SRQ_MASK(64, 4);
  else if (veclen <= 8192) SRQ_MASK(128, 4);
  else if (veclen <= 16384) SRQ_MASK(256, 4);
  else SRQ_MASK(256, 8);
#undef SRQ_MASK
  return hipGetLastError();
}

}  // namespace srq
