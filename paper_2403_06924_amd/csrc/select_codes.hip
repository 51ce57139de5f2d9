// Keep-masks of Eq. avgQuan with their counts per vector, of both operands in one launch, from the codes and residual codes
// that the quantize passes have left, where the mask passes of fused.hip and strips.hip read the FP32 operands again: 2
// bytes per element instead of 4.  Where strips.hip would take the selection, with the means and thresholds as it does.
//
// |x| -> (code, residual code) is monotone: fl(x * lambda), the rounding and the clamp are, and for one code so are
// fl(x - fl(code * s)) and its code in turn; all of them are odd.  With key(x) = |256 code + residual code| therefore
//     key(x) > key(t)  =>  |x| > t,       key(x) < key(t)  =>  |x| < t,
// and only the elements of the threshold's own key (one bin in some 16000 of the vector's range) are read in FP32.  So are
// those of the topmost key, which NaN shares, and whole vectors whose scales are not ordinary numbers or whose threshold
// lies in one of the lowest bins.
//
// What bounds it: 2 bytes per element (5.7 TB/s on two operands of 8192 x 8192).  Both operands, us, from FP32 / from codes:
// 8192 x 8192 each 46 + (68 with the residual codes of B) / 47 to 51; 4096 x 4096 and 4096 x 14336 12 + 50 / 32 with a wave per
// vector (with a workgroup for each, which has too few bytes on their way, 55 against 36 at the time).
// On the side: the zero-filled codes (16 bytes per lane, what is in registers already) where the corrections follow at once, and the
// counts of every 256 vectors where the compaction wants them.
#include "compact.h"
#include "gemm_lanes.h"
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
  if (most.x == top - tk || most.y == top - tk) {    const s2 last = both(top - tk), one = both(1);
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

// How a vector is decided.  In FP32 altogether where a scale is no ordinary number, and where the threshold's key is below kLowKeys:
// the lowest bins are the fullest where a few outliers have set the scales, and most of the elements would be looked at one by
// one.  (Calls, us, never / 2 / 4 / 16: 1500^3, 4 bits, outliers 69 / 68 / 62 / 62, 4096^3 over twenty binades at 95 % kept 405 / 333 / 333 /
// 333, but with outliers, 8 bits, 95 % kept 305 / 305 / 305 / 332.)
constexpr int kLowKeys = 4;
enum Way { kNothing, kByCodes, kInFloats };
template <bool TRUNC>
__device__ __forceinline__ Way way_of(float t, float lam, float s, float rlam, float qmax, int low, int& key, float& at_code) {
  if (!(t < INFINITY) || (s == 0.f && lam == 0.f && t >= 0.f)) return kNothing;   // (nothing is above NaN, infinity or the maximum of a zero vector)
  // (qmax * s overflows where the scale of a maximum next to FLT_MAX is rounded up: that element's residual is infinite, and
  // rlam zero as where every residual is)
  if (!(ordinary(lam) && ordinary(s) && qmax * s < INFINITY && rlam < INFINITY && t >= 0.f)) return kInFloats;
  const float code = code_value(biased_code(t, lam, qmax, TRUNC));
  at_code = code * s;
  key = (int)code * 256 + (int)code_value(biased_code(t - at_code, rlam, qmax, TRUNC));
  return rlam > 0.f && key < low ? kInFloats : kByCodes;   // (without residuals a key is one magnitude, and nothing is looked at)
}

// Every 64th partial sum by a lane, the lanes as a tree: the order in which strips.hip adds them, too
__device__ __forceinline__ double sum_of(const CodesSelect& o, int64_t v) {
  double sum = 0.0;
  for (int64_t p = threadIdx.x & 63; p < o.nparts; p += 64) sum += o.part[p * o.nvec + v];
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
  return sum;
}

// The columns among sixteen neighbouring ones that are decided in FP32: eight rows by four columns per thread, 64 contiguous bytes of
// a row, where a wave with a column to itself fetches a line for each element.  Bound by the serial trips of a workgroup (512 rows
// each) where columns are few: there the waves read them by themselves.  Calls with a low key in every column, us, by the waves /
// this: 100 x 1900 x 7000 (4 bits, outliers) 155 / 140, 3000 x 3000 x 2000 at 95 % kept 168 / 147, 8192 x 8192 x 4096 1155 / 994, but
// 300 x 1024 x 8000 125 / 130, 300 x 512 x 8000 100 / 121.  Workgroups that find no such column cost 0.3 to 1 us of these calls.
constexpr int64_t kColumnsApart = 1280;                // columns from which on there are such workgroups
template <bool TRUNC>
__device__ __forceinline__ void columns_in_floats(const CodesSelect& o, int64_t col16, int64_t veclen, int64_t ld, float qmax) {
  __shared__ float above[16];                          // thresholds
  __shared__ int kept[16];
  __shared__ unsigned wanted;                          // a bit per column
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (o.part) {
    // (as sum_of, four columns at a time)
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    const double* from[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) from[c] = o.part + (col16 + 4 * w + c < o.nvec ? col16 + 4 * w + c : o.nvec - 1);
    for (int64_t p = lane; p < o.nparts; p += 64) {
#pragma unroll
      for (int c = 0; c < 4; ++c) sum[c] += from[c][p * o.nvec];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      for (int off = 32; off > 0; off >>= 1) sum[c] += __shfl_xor(sum[c], off, 64);
      const float mean = (float)(sum[c] / o.count);
      if (lane == 0) above[4 * w + c] = o.theta * mean;
    }
    __syncthreads();
  }
  if (tid < 64) {
    bool mine = false;
    if (tid < 16) {
      const int64_t v = col16 + tid < o.nvec ? col16 + tid : o.nvec - 1;
      const float t = o.part ? above[tid] : o.thresh[v];
      int key;
      float at_code;
      mine = col16 + tid < o.nvec && way_of<TRUNC>(t, o.lambda[v], o.scale[v], o.rlambda[v], qmax, kLowKeys, key, at_code) == kInFloats;
      above[tid] = t;
      kept[tid] = 0;
    }
    const uint64_t all = __ballot(mine);
    if (tid == 0) wanted = (unsigned)all;
  }
  __syncthreads();
  const unsigned columns = wanted;
  if (!columns) return;
  typedef unsigned u2a __attribute__((ext_vector_type(2)));
  const int cg = tid & 3, four = columns >> (4 * cg) & 15;
  const int64_t col0 = col16 + 4 * cg, words = (veclen + 63) / 64;
  const float t[4] = {above[4 * cg], above[4 * cg + 1], above[4 * cg + 2], above[4 * cg + 3]};
  int n[4] = {0, 0, 0, 0};
  if (four) {
    const int ncol = col0 + 4 <= o.nvec ? 4 : (int)(o.nvec - col0);
    const uint32_t ld4 = 4u * (uint32_t)o.elem_step, at = 4u * (uint32_t)(ncol == 4 ? col0 : o.nvec - 4) + (uint32_t)(tid >> 2) * 8 * ld4;
#pragma unroll 1
    for (int row = 0; row < (int)words * 64; row += 512) {
      // (no branch around a load: what does not exist reads as zero and is not above; the last columns that are not four are
      // read with those before them)
      const __amdgpu_buffer_rsrc_t rs = buf_rsrc(o.X + (int64_t)row * o.elem_step, kRecords);
      const int row0 = row + 8 * (tid >> 2), here = (int)veclen - row0;
      v4i x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, i < here ? at + i * ld4 : kOutside, 0, 0));
      if (ncol < 4) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          x[i] = v4i{ncol == 3 ? x[i].y : ncol == 2 ? x[i].z : x[i].w, ncol == 3 ? x[i].z : x[i].w, x[i].w, 0};
      }
      unsigned bits[4] = {0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int c = 0; c < 4; ++c) bits[c] |= fabsf(__int_as_float(x[i][c])) > t[c] ? 1u << i : 0u;
      }
      if (row0 >= (int)words * 64) break;
      // (offsets formed here, or each of the addresses holds two registers through the loop)
      uint32_t mask_at = 4 * cg * (uint32_t)words * 8 + (row0 >> 3), code_at = 4 * cg * (uint32_t)ld + row0;
      asm volatile("" : "+v"(mask_at), "+v"(code_at));
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (four >> c & 1) {
          n[c] += __popc(bits[c]);
          reinterpret_cast<uint8_t*>(o.mask + col16 * words)[mask_at] = (uint8_t)bits[c];
          if (o.D) {
            const u2a code = *reinterpret_cast<const u2a*>(o.Q + col16 * ld + code_at);
            *reinterpret_cast<u2a*>(o.D + col16 * ld + code_at) = u2a{code.x & bytes_of(bits[c] & 15u), code.y & bytes_of(bits[c] >> 4)};
          }
        }
        mask_at += (uint32_t)words * 8;
        code_at += (uint32_t)ld;
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (n[c]) atomicAdd(&kept[4 * cg + c], n[c]);
  }
  __syncthreads();
  if (tid < 16 && (columns >> tid & 1)) {
    const int64_t v = col16 + tid;
    o.counts[v] = kept[tid];
    if (o.sums && kept[tid]) atomicAdd(o.sums + (v >> 8) * kSumStride, kept[tid]);
  }
}

struct CodesPair {
  CodesSelect op[2];
};

template <int TH, int NV, bool TRUNC>   // TH threads per vector, NV pieces of 16 elements for each
__global__ __launch_bounds__(256, NV <= 4 ? 7 : 4) void select_codes_kernel(CodesPair g, int64_t veclen, int64_t ld, float qmax, int floats, int groups_a) {
  constexpr int VECS = 256 / TH, STEP = 16 * TH;
  __shared__ int sm[4];
  if ((int)blockIdx.x < floats) {
    // (two neighbouring sixteens, which share lines, on one XCD)
    const int at = blockIdx.x, pair = at < (floats & ~15) ? (at & ~15) + 2 * (at & 7) + (at >> 3 & 1) : at;
    columns_in_floats<TRUNC>(g.op[1], (int64_t)pair * 16, veclen, ld, qmax);
    return;
  }
  const int block = (int)blockIdx.x - floats;
  const bool first = block < groups_a;
  // (by an index that the compiler does not look through, and all of it now: otherwise each field is chosen and fetched by
  // itself where it is wanted, a trip each)
  const CodesSelect& o = g.op[(unsigned)(groups_a - 1 - block) >> 31];
  asm volatile("" : : "s"(o.part), "s"(o.nparts), "s"(o.count), "s"(o.theta), "s"(o.mean), "s"(o.thresh), "s"(o.X), "s"(o.vec_step), "s"(o.elem_step),
               "s"(o.Q), "s"(o.R), "s"(o.scale), "s"(o.lambda), "s"(o.rlambda), "s"(o.mask), "s"(o.counts), "s"(o.nvec), "s"(o.D), "s"(o.sums));
  const int tid = threadIdx.x & (TH - 1);
  const int sub = TH >= 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / TH) : 0;
  int64_t group = first ? block : block - groups_a;
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
  float lam = 0.f, s = 0.f, rlam = 0.f;
  if (o.mask) {                                        // (on their way while the threshold is formed)
    lam = o.lambda[v];
    s = o.scale[v];
    rlam = o.rlambda[v];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int64_t e = 16 * tid + STEP * i, at = e < ld ? e : 0;
      qv[i] = *reinterpret_cast<const u4a*>(q + at);
      rv[i] = *reinterpret_cast<const u4a*>(r + at);
    }
  }
  float t;
  if (o.part) {
    const float mean = (float)(sum_of(o, v) / o.count);   // line 7
    t = o.theta * mean;
    if (tid == 0 && exists) { o.mean[v] = mean; o.thresh[v] = t; }
  } else {
    t = o.thresh[v];
  }
  if (!o.mask) return;
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
  // (vectors in FP32: columns by workgroups of their own, if there are any)
  const bool elsewhere = !first && floats > 0;
  int tk;
  float at_code;
  const Way way = way_of<TRUNC>(t, lam, s, rlam, qmax, elsewhere || first ? kLowKeys : 0, tk, at_code);
  if (way == kNothing) {
    for (int64_t e = 16 * tid; e < words * 64; e += STEP) put(e, 0u, u4a{0, 0, 0, 0});
  } else if (way == kInFloats) {
    if (!elsewhere) {
      // 64 neighbouring elements by the lanes of a wave, a word of the mask for each load
      const int lane = threadIdx.x & 63;
#pragma unroll 1
      for (int64_t e0 = 16 * (tid - lane); e0 < words * 64; e0 += STEP) {
        float y[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) y[j] = x[(e0 + 64 * j + lane < veclen ? e0 + 64 * j + lane : veclen - 1) * o.elem_step];
        unsigned m = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const uint64_t word = __ballot(fabsf(y[j]) > t);
          if (lane >> 2 == j) m = (unsigned)(word >> (16 * (lane & 3))) & 0xffffu;
          asm volatile("" : "+v"(m));                // (one word at a time: two scalar registers for each)
        }
        const int64_t e = e0 + 16 * lane;
        put(e, m & present(e), *reinterpret_cast<const u4a*>(q + (e < ld ? e : 0)));
      }
    }
  } else {
    const int top = 257 * (int)qmax;
    // a residual that is zero everywhere: x is fl(code * s) itself
    const bool exact = rlam == 0.f, equal = at_code > t;
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
  if (tid == 0 && exists && !(way == kInFloats && elsewhere)) {
    o.counts[v] = total;
    if (o.sums && total) atomicAdd(o.sums + (v >> 8) * kSumStride, total);
  }
}

}  // namespace

// (With few codes the threshold's bin is wide, and most of it is looked at in FP32 where outliers set the scale: calls, us, the passes
// over FP32 / from the codes, 4 bits 384 x 5952 x 8576 329 / 422, 5000 x 4000 x 3000 341 / 432, without outliers 336 / 310; 7 bits 315 /
// 271, 8 bits 320 / 277.  On the path of strips.hip the compaction may go behind the tiles: 4 bits, with outliers / normal, 300 x 128 x
// 4000 60.5 / 58.1 and 59.2 / 53.8, 600^2 x 4000 73 / 71 and 68 / 59, 1500^3 60.9 / 62.4 (65 / 62 where more is kept), 100 x 1900 x 7000 143 / 140.
// 3 bits have 49 keys.  A threshold of zero leaves every zero to be looked at.)
bool select_codes_ok(int qmax, float theta, bool strips) { return qmax >= (strips ? 7 : 63) && theta > 0.f; }

hipError_t launch_select_codes(const CodesSelect& a, const CodesSelect& b, int64_t veclen, int64_t ld, int qmax, int trunc, hipStream_t st) {
  if (a.nvec + b.nvec <= 0 || veclen <= 0) return hipSuccess;
  const int64_t floats = b.mask && b.nvec >= kColumnsApart && b.elem_step < ((int64_t)1 << 20) ? (b.nvec + 15) / 16 : 0;   // (32-bit offsets)
#define SRQ_MASK(TH, NV)                                                                                                   \
  do {                                                                                                                     \
    const int64_t ga = (a.nvec + 256 / TH - 1) / (256 / TH), gb = (b.nvec + 256 / TH - 1) / (256 / TH);                     \
    hipLaunchKernelGGL((trunc ? select_codes_kernel<TH, NV, true> : select_codes_kernel<TH, NV, false>), dim3((unsigned)(floats + ga + gb)), \
                       dim3(256), 0, st, CodesPair{{a, b}}, veclen, ld, (float)qmax, (int)floats, (int)ga);                             \
  } while (0)
  // Few vectors by more waves each, up to six vectors for a compute unit.  Calls, us, a wave or two per vector / these: 64^2 x 4000 48.1 /
  // 46.5, 300 x 128 x 4000 54.3 / 52.9 (outliers, 4 bits 69 / 58), 1000 x 400 x 4000 57.1 / 57.0 (72 / 66), 900 x 1000 x 4000 60.9 / 61.3 (79 / 84).
  const bool few = a.nvec + b.nvec <= 1536;
  if (few && veclen > 2048 && veclen <= 4096) SRQ_MASK(256, 1);
  else if (few && veclen > 4096 && veclen <= 8192) SRQ_MASK(256, 2);
  else if (few && veclen > 1024 && veclen <= 2048) SRQ_MASK(128, 1);
  else if (veclen <= 1024) SRQ_MASK(64, 1);
  else if (veclen <= 2048) SRQ_MASK(64, 2);
  else if (veclen <= 4096) SRQ_MASK(64, 4);
  else if (veclen <= 8192) SRQ_MASK(128, 4);
  else if (veclen <= 16384) SRQ_MASK(256, 4);
  else SRQ_MASK(256, 8);
#undef SRQ_MASK
  return hipGetLastError();
}

}  // namespace srq
