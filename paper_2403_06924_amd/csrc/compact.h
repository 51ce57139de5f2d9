// Compaction of keep-bits and codes to CSR / CSC, for kernels of 256 threads.
#pragma once
#include "srq_internal.h"
#include "stream.h"

namespace srq {

// all bits of the bytes whose bit is set
static __device__ __forceinline__ unsigned bytes_of(unsigned nib) { return ((nib * 0x00204081u) & 0x01010101u) * 0xffu; }

// A vector by a wave, sixteen elements per lane and piece: the place of a lane's first kept entry is the number of entries of
// earlier vectors, pieces and lanes (the last from five ballots of its own count, 0..16).  Codes and zero-filled copy have rows
// of Kc bytes (a multiple of 16) with zeros past K.  One 16-byte load and store per 1024 elements, and as many stores of entries
// as the lane with most of them has: with four elements per lane, us, 2999 x 4097 x 3001 26 / 16, calls 226 / 216, 2048^3 70.6 / 67.5,
// 2000 x 1500 x 6000 161 / 154, reduction of 2000 x 15000 124 / 112.
// Vectors with many entries by way of LDS, us, all entries as above / all by way of LDS: reduction of 4096 x 14336 at 5 % kept 157 / 161,
// 10 % 162 / 162, 20 % 175 / 164, 45 % 255 / 174, of 6000 x 2000 at 5 % 34.1 / 35.0, 15 % 36.5 / 35.8, 45 % 55 / 38; calls of 2048^3 at 10 %
// 64.2 / 64.8, 30 % 68.8 / 65.8, 95 % 106 / 69, 4096^3 at 5 % 270 / 275, 20 % 281 / 280, 50 % 329 / 287, 95 % 452 / 306.  (A workgroup and a
// wave per vector with four elements per lane, two and four times as many stores: 2048^3 at 95 % 80, 4096^3 486.)
constexpr int kCrowded = 160;                          // entries of 1024 elements from which on a vector's go by way of LDS
constexpr int kGatherWave = 3072;                      // bytes of LDS for a wave: places and codes of a piece's entries
template <int NV>                                      // pieces of 1024 elements
struct CompactFour {
  typedef unsigned u4a __attribute__((ext_vector_type(4)));
  typedef int i4a __attribute__((ext_vector_type(4)));
  u4a code[NV];
  unsigned m[NV];
  int v;
  bool ok;

  // vectors 4 group .. + 3, one for a wave
  __device__ __forceinline__ void load(const StripCompact& s, int group, int K, int Kc) {
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    v = 4 * group + w;
    ok = v < s.nvec;
    const int words = (K + 63) / 64, last = 4 * words - 1;
    const uint16_t* mv = reinterpret_cast<const uint16_t*>(s.mask + (int64_t)(ok ? v : 0) * words);
    const int8_t* qv = s.Q + (int64_t)(ok ? v : 0) * Kc;
#pragma unroll
    for (int i = 0; i < NV; ++i) {                     // (without branches: what is not wanted is read where something is)
      const int e = 1024 * i + 16 * lane;
      m[i] = mv[e >> 4 < last ? e >> 4 : last];
      code[i] = *reinterpret_cast<const u4a*>(qv + (e < Kc ? e : 0));
    }
  }
  // The n entries of piece i from place p on, by way of the wave's part of LDS: stored as they come, the entries of neighbouring lanes
  // lie as far apart as a lane has, and every store is as many lines as there are lanes.  (Reads follow writes of the same wave: no
  // barrier.)
  __device__ __forceinline__ void store_crowded(const StripCompact& s, int i, int64_t p, int n, int at, uint8_t* part) {
    typedef unsigned short u4h __attribute__((ext_vector_type(4), may_alias));
    typedef unsigned u1a __attribute__((may_alias));
    const int lane = threadIdx.x & 63;
    uint8_t* const vals = part + 2048;
    unsigned short* const places = reinterpret_cast<unsigned short*>(part);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (m[i] >> j & 1u) {
        places[at] = (unsigned short)(1024 * i + 16 * lane + j);
        vals[at] = (uint8_t)(code[i][j >> 2] >> (8 * (j & 3)));
        ++at;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (p + n > s.capacity) n = s.capacity > p ? (int)(s.capacity - p) : 0;
    for (int t = 4 * lane; t < n; t += 256) {
      const u4h e = *reinterpret_cast<const u4h*>(places + t);
      const unsigned four = *reinterpret_cast<const u1a*>(vals + t);
      if (t + 4 <= n) {
        *reinterpret_cast<u4u*>(s.idx + p + t) = u4u{e.x, e.y, e.z, e.w};
        *reinterpret_cast<u1u*>(s.val + p + t) = four;
      } else {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          if (t + j < n) {
            s.idx[p + t + j] = e[j];
            s.val[p + t + j] = (int8_t)(four >> (8 * j));
          }
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  // before: kept entries of the vectors before the workgroup's, in four parts, behind no barrier yet
  __device__ __forceinline__ void store(const StripCompact& s, int8_t* dense, int K, int Kc, const int64_t (&before)[4], int (&count)[4],
                                        uint8_t* gather, bool around = false) {   // (zero-filled codes around the caches)
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t lower = (1ull << lane) - 1ull;
    int at[NV], at_piece[NV], mine = 0;                // (the latter the same for all lanes)
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int e = 1024 * i + 16 * lane;
      if (!ok || e >= K) m[i] = 0;                     // (bits past K are zero)
      if (dense && ok && e < Kc) {
        u4a o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = code[i][j] & bytes_of(m[i] >> (4 * j) & 15u);
        if (around) __builtin_nontemporal_store(o, reinterpret_cast<u4a*>(dense + (int64_t)v * Kc + e));
        else *reinterpret_cast<u4a*>(dense + (int64_t)v * Kc + e) = o;
      }
      at_piece[i] = mine;
      const int cnt = __popc(m[i]);
      const uint64_t b0 = __ballot(cnt & 1), b1 = __ballot(cnt & 2), b2 = __ballot(cnt & 4), b3 = __ballot(cnt & 8), b4 = __ballot(cnt & 16);
      at[i] = mine + __popcll(b0 & lower) + 2 * __popcll(b1 & lower) + 4 * __popcll(b2 & lower) + 8 * __popcll(b3 & lower) +
              16 * __popcll(b4 & lower);
      mine += __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2) + 8 * __popcll(b3) + 16 * __popcll(b4);
      asm volatile("" : "+v"(at[i]));                  // (formed here, or ten scalar registers hold the ballots of each piece)
    }
    if (lane == 0) count[w] = mine;
    __syncthreads();
    int64_t first = before[0] + before[1] + before[2] + before[3];
    for (int j = 0; j < w; ++j) first += count[j];
    if (__builtin_expect(mine * 1024 < kCrowded * K, 1)) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        int64_t p = first + at[i];
        unsigned left = m[i];
        while (left) {
          const int j = __ffs((int)left) - 1;
          left &= left - 1u;
          if (p < s.capacity) {
            const unsigned word = (j & 8) ? ((j & 4) ? code[i][3] : code[i][2]) : ((j & 4) ? code[i][1] : code[i][0]);
            s.idx[p] = 1024 * i + 16 * lane + j;
            s.val[p] = (int8_t)(word >> (8 * (j & 3)));
          }
          ++p;
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int from = i ? at_piece[i] : 0, n = (i + 1 < NV ? at_piece[i + 1 < NV ? i + 1 : 0] : mine) - from;
        store_crowded(s, i, first + from, n, at[i] - from, gather + w * kGatherWave);
      }
    }
    if (lane == 0 && ok) {
      s.ptr[v] = (int32_t)first;
      if (v == s.nvec - 1) {
        s.ptr[s.nvec] = (int32_t)(first + mine);
        if (s.nnz) *s.nnz = first + mine;
      }
    }
  }
};

template <int NV>
static __device__ __forceinline__ void compact_four(const StripCompact& s, int group, int K, int Kc, int64_t (&before)[4], int (&count)[4],
                                                    uint8_t* gather) {
  CompactFour<NV> f;
  f.load(s, group, K, Kc);
  // kept entries of the vectors before the workgroup's
  int64_t sum = 0;
  for (int i = 4 * (int)threadIdx.x; i < 4 * group; i += 1024) {
    const auto c = *reinterpret_cast<const typename CompactFour<NV>::i4a*>(s.counts + i);
    sum += (int64_t)c.x + c.y + c.z + c.w;
  }
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
  if ((threadIdx.x & 63) == 0) before[threadIdx.x >> 6] = sum;
  f.store(s, s.dense, K, Kc, before, count, gather);
}

}  // namespace srq
