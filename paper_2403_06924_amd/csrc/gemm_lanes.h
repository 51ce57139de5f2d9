// Register-level pieces of the 16 x 16 x 64 matrix-core kernels: buffer accesses with range checks, the
// exchange that turns two 16 x 16 blocks into whole 128-byte lines, sums over the lanes of a block.
#ifndef SRQ_GEMM_LANES_H_
#define SRQ_GEMM_LANES_H_
#include "srq_internal.h"

namespace srq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// buffer descriptor of `bytes` bytes at a wave-uniform address: accesses take a 32-bit lane offset, reads
// past the end return zero and writes are dropped
static __device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
static __device__ __forceinline__ v4i buf_load16(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff) {
  const v4u t = __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0);
  return v4i{(int)t.x, (int)t.y, (int)t.z, (int)t.w};
}
static __device__ __forceinline__ float buf_load_f32(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
// four consecutive floats; `whole`: none of them is past the end
static __device__ __forceinline__ v4f buf_load_4(__amdgpu_buffer_rsrc_t r, uint32_t off, bool whole) {
  v4f x;
  if (whole) {
    const v4i t = buf_load16(r, off, 0);
    x = v4f{__int_as_float(t.x), __int_as_float(t.y), __int_as_float(t.z), __int_as_float(t.w)};
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = buf_load_f32(r, off + 4u * v);
  }
  return x;
}

// an accumulator as a number, read where it is wanted (several copies of an epilogue follow the K loop: what they
// have in common the compiler computes before it branches to one of them, all conversions at once; nor does it keep
// accumulators in ordinary registers and move them there and back in every K-tile).  Two s_nop 15 stand between the
// last MFMA and the first of these.
static __device__ __forceinline__ float acc_value(int x) {
  int y;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(y) : "a"(x));
  return (float)y;
}

// 16 bytes of a row of C (at any 4-byte aligned address): uniform base and offset, the lane's offset
static __device__ __forceinline__ v4f row_load(uint64_t base, uint32_t lane, uint32_t off) {
  const v4i t = buf_load16(buf_rsrc(reinterpret_cast<const void*>(base), 0xffffffffu), lane, off);
  return v4f{__int_as_float(t.x), __int_as_float(t.y), __int_as_float(t.z), __int_as_float(t.w)};
}
template <bool CACHED>
static __device__ __forceinline__ void row_store(v4f x, uint64_t base, uint32_t lane, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b128(
      v4u{__float_as_uint(x.x), __float_as_uint(x.y), __float_as_uint(x.z), __float_as_uint(x.w)},
      buf_rsrc(reinterpret_cast<const void*>(base), 0xffffffffu), lane, off, CACHED ? 0 : 2 /* non-temporal */);
}

// Accesses without branches (a load behind one is waited for before the next is issued): what does not exist gets an
// offset past the end of its descriptor, where a load brings zero and a store is dropped.
constexpr uint32_t kOutside = 0xfffffff0u, kRecords = 0x7fffffffu;
// the same on the edge: row `row`, columns col .. col + 3 of the rows that start at `base`, of which rows x cols
// exist.  ELEMS: the last columns are not a whole access.
static __device__ __forceinline__ uint32_t edge_offset(int64_t ld4, int row, int col, int rows, int cols) {
  return row < rows && col < cols ? (uint32_t)row * (uint32_t)ld4 + 4u * (uint32_t)col : kOutside;
}
template <bool ELEMS>
static __device__ __forceinline__ v4f edge_load(uint64_t base, int64_t ld4, int row, int col, int rows, int cols) {
  const __amdgpu_buffer_rsrc_t rs = buf_rsrc(reinterpret_cast<const void*>(base), kRecords);
  if (!ELEMS) return buf_load_4(rs, edge_offset(ld4, row, col, rows, cols), true);
  v4f x;
#pragma unroll
  for (int v = 0; v < 4; ++v) x[v] = buf_load_f32(rs, edge_offset(ld4, row, col + v, rows, cols));
  return x;
}
template <bool ELEMS>
static __device__ __forceinline__ void edge_store(v4f x, uint64_t base, int64_t ld4, int row, int col, int rows, int cols) {
  const __amdgpu_buffer_rsrc_t rs = buf_rsrc(reinterpret_cast<const void*>(base), kRecords);
  if (!ELEMS) {
    __builtin_amdgcn_raw_buffer_store_b128(
        v4u{__float_as_uint(x.x), __float_as_uint(x.y), __float_as_uint(x.z), __float_as_uint(x.w)}, rs,
        edge_offset(ld4, row, col, rows, cols), 0, 0);
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[v]), rs, edge_offset(ld4, row, col + v, rows, cols), 0, 0);
  }
}

// A lane's N accesses of four consecutive floats of a tile of C: access i covers row row + 8 (i & 1) +
// 16 (i >> 1), columns col .. col + 3; rows x cols of the tile exist (full: all of it).
template <int N>
struct TileAccess {
  int row, col;
  uint32_t rows, cols;
  bool full;
  __device__ __forceinline__ uint32_t row_of(int i) const { return (uint32_t)(row + 8 * (i & 1) + 16 * (i >> 1)); }
  // outside the tile: past every descriptor's end
  __device__ __forceinline__ uint32_t offset(int i, int v, uint32_t ld) const {
    return row_of(i) < rows && (uint32_t)(col + v) < cols ? 4u * (row_of(i) * ld + (uint32_t)(col + v)) : 0xfffffff0u;
  }
  __device__ __forceinline__ void load(v4f (&x)[N], const float* tile, uint32_t ld) const {
    const __amdgpu_buffer_rsrc_t r = buf_rsrc(tile, 0x7fffffffu);
    if (full) {
#pragma unroll
      for (int i = 0; i < N; ++i) x[i] = buf_load_4(r, 4u * (row_of(i) * ld + (uint32_t)col), true);
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) x[i][v] = buf_load_f32(r, offset(i, v, ld));
    }
  }
  __device__ __forceinline__ void store(const v4f (&x)[N], float* tile, uint32_t ld) const {
    const __amdgpu_buffer_rsrc_t r = buf_rsrc(tile, 0x7fffffffu);
    if (full) {
#pragma unroll
      for (int i = 0; i < N; ++i)
        __builtin_amdgcn_raw_buffer_store_b128(
            v4u{__float_as_uint(x[i].x), __float_as_uint(x[i].y), __float_as_uint(x[i].z), __float_as_uint(x[i].w)}, r,
            4u * (row_of(i) * ld + (uint32_t)col), 0, 2 /* non-temporal */);
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[i][v]), r, offset(i, v, ld), 0, 0);
    }
  }
};

// Two neighbouring 16 x 16 blocks, four consecutive columns of a row per lane: lanes 8-15 of a row of
// sixteen trade their part of the first for lanes 0-7's part of the second.  Afterwards x0 holds rows
// 0-7 and x1 rows 8-15 of both blocks, the first block in lanes 0-7, the second in lanes 8-15.
static __device__ __forceinline__ void exchange_half_rows(v4f& x0, v4f& x1) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int d0 = __float_as_int(x0[v]), d1 = __float_as_int(x1[v]);
    x0[v] = __int_as_float(__builtin_amdgcn_update_dpp(d0, d1, 0x128, 0xf, 0xc, false));
    x1[v] = __int_as_float(__builtin_amdgcn_update_dpp(d1, d0, 0x128, 0xf, 0x3, false));
  }
}

// Sums over the 16 lanes of a row of sixteen, which hold 8 values each: lane rl ends with the sum of value
// rl >> 1.  Reduce-scatter by DPP with partners lane ^ 15, ^ 7, ^ 3 (each differs in one more bit of the
// half that is kept), then lane ^ 1.
template <int CTRL>
static __device__ __forceinline__ double dpp_f64(double x) {
  const int2 b = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, b.x, CTRL, 0xf, 0xf, true),
                                              __builtin_amdgcn_update_dpp(0, b.y, CTRL, 0xf, 0xf, true)));
}
template <int N, int CTRL>
static __device__ __forceinline__ void halve8(double (&x)[8], bool up) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double send = up ? x[i] : x[i + N], keep = up ? x[i + N] : x[i];
    x[i] = keep + dpp_f64<CTRL>(send);
  }
}
static __device__ __forceinline__ double column_sum8(double (&x)[8], int rl) {
  halve8<4, 0x140>(x, rl & 8);                       // row_mirror
  halve8<2, 0x141>(x, rl & 4);                       // row_half_mirror
  halve8<1, 0x1b>(x, rl & 2);                        // quad_perm 3 2 1 0
  return x[0] + dpp_f64<0xb1>(x[0]);                 // quad_perm 1 0 3 2
}

}  // namespace srq

#endif  // SRQ_GEMM_LANES_H_
