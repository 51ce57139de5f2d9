// Internal declarations shared by the translation units of libsrq (not part of the ABI).
#ifndef SRQ_INTERNAL_H_
#define SRQ_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "srq.h"

struct srq_context {
  int device;            // -1: no device (validation only)
  void* ws;              // caller-owned device workspace
  size_t ws_bytes;
  int last_hip_error;
  int64_t* host_nnz;     // pinned host buffer for the two counters read back in synchronising modes
  srq_intermediates_t last;
  int prof_enabled;
  unsigned prof_mask;                       // bit i: stage i is timed
  // stage events of the last kProfRing calls (slot = call number mod kProfRing)
  unsigned prof_used[64];                   // bit i: stage i ran in that call
  hipEvent_t prof_ev[64][2 * SRQ_NUM_STAGES];   // start/stop per stage, created on enable
  int prof_slot;                            // slot of the call being recorded
  int64_t prof_calls;                       // calls recorded since the last read
  int prof_created;
  int scale_mode;        // srq_scale_t of the next srq_compensated_gemm calls
  int last_path_a;       // execution the caller expects SRQ_STRATEGY_AUTO to pick for term 1 (srq_set_auto_hint;
  int last_path_b;       // 0: none given, the matrix cores are assumed), resp. for term 2
  uint32_t wait_ticks;   // how long workgroups that exchange maxima wait for each other (100 MHz, cols_once.hip)
};

namespace srq {

inline int qmax_of_bits(int bits) { return (1 << (bits - 1)) - 1; }

// A launch that only matters for some outcomes of a decision taken on the device (which execution
// SRQ_STRATEGY_AUTO picks for a term): the kernel reads *value and does nothing unless bit *value
// of ok_mask is set.  value == null: unconditional.
struct RunIf {
  const int32_t* value;
  uint32_t ok_mask;
};
static __device__ __forceinline__ bool run_if_ok(const RunIf& r) { return !r.value || ((r.ok_mask >> *r.value) & 1u); }
constexpr RunIf kAlways = {nullptr, 0u};

constexpr int kSelChunk = 256;      // elements of a vector handled by one wave in count/scatter

// epilogue modes of the INT8 GEMM
enum GemmMode { kGemmFirst = 0, kGemmAccum = 1 };

struct GemmEpilogue {
  int mode;               // GemmMode
  const float* s_row;     // [M] scale paired with rows of the output
  const float* s_col;     // [N] scale paired with columns
  float* C;               // output / accumulator, row-major
  int64_t ldc;
  int32_t* D_int;         // optional raw INT32 product (ld = ldd), may be null
  int64_t ldd;
  float* D_F_copy;        // optional copy of the dequantized product before alpha/beta (ld = ldd)
  double* row_part;       // kGemmFirst: [tiles_n][M] partial sums of |D_F| (may be null)
  double* col_part;       // kGemmFirst: [tiles_m][N]
  int final_scale;        // apply alpha/beta after this term
  float alpha, beta;
  const float* Cin;
  int64_t ldcin;
  // Overflow guard of the non-synchronising modes: when set, a kernel that adds a correction
  // term (or applies alpha / beta after one) does nothing if the selection kept more entries
  // than the compressed arrays hold (guard_nnz[0] > guard_cap_a or guard_nnz[1] > guard_cap_b),
  // so that C stays the uncorrected first product instead of receiving a truncated correction.
  const int64_t* guard_nnz;   // device int64[2]: kept entries of A' and B' (null: no guard)
  int64_t guard_cap_a, guard_cap_b;
  // a product that only matters when a device-side count is non-zero (the dense strip of the
  // column-block execution): when set and *run_if_nonzero == 0 the kernel does nothing
  const int32_t* run_if_nonzero;
  int dint_add;               // vector-ALU kernels: add the raw sums to D_int instead of storing them
  // executions chosen on the device (SRQ_STRATEGY_AUTO): paths[0] / paths[1] hold the execution of
  // term 1 / term 2; the kernel runs only if both are among those it was launched for
  const int32_t* paths;       // device int32[2] (null: unconditional)
  uint32_t ok_a, ok_b;        // bit p set: path p of term 1 resp. term 2 is acceptable
  // paired launches only: the two products are decided one by one (product t runs iff the path of
  // term t+1 is acceptable) instead of both or none; alpha / beta go with the second product only
  int each_product;
  // the kernel that leaves partial sums per 64 columns / rows is not to be used (the buffers are sized
  // for one per 128)
  int no_tile64;
};

// true when the epilogue's overflow guard is set and tripped (wave-uniform: scalar loads)
static __device__ __forceinline__ bool guard_tripped(const GemmEpilogue& ep) {
  if (ep.run_if_nonzero && *ep.run_if_nonzero == 0) return true;
  if (ep.paths) {
    const bool run_a = (ep.ok_a >> ep.paths[0]) & 1u, run_b = (ep.ok_b >> ep.paths[1]) & 1u;
    if (ep.each_product ? !(run_a || run_b) : !(run_a && run_b)) return true;
  }
  return ep.guard_nnz && (ep.guard_nnz[0] > ep.guard_cap_a || ep.guard_nnz[1] > ep.guard_cap_b);
}

// first and last product (0 or 1) a paired launch runs (guard_tripped has dealt with "none")
static __device__ __forceinline__ void pair_range(const GemmEpilogue& ep, int nprod, int& lo, int& hi) {
  lo = 0;
  hi = nprod - 1;
  if (nprod == 2 && ep.paths && ep.each_product) {
    if (!((ep.ok_a >> ep.paths[0]) & 1u)) lo = 1;
    if (!((ep.ok_b >> ep.paths[1]) & 1u)) hi = 0;
  }
}

// Second product of a paired accumulate-mode launch of the persistent kernel: C += dequant(Qa.Qb^T)
// with its own scales, right after the first product of the same output tile (Qa == null: none).
// alpha / beta of the epilogue, if any, are applied after the second product.
struct GemmSecond {
  const int8_t* Qa;
  const int8_t* Qb;
  int64_t lda, ldb;
  const float* s_row;
  const float* s_col;
};

// ---- launchers (each returns the hipError_t of its launches) --------------------------
hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st);

// amax of |x| per vector as float bits in amax_bits[nvec] (must be zero-filled for AXIS_COL)
hipError_t launch_amax(const float* X, int64_t rows, int64_t cols, int64_t ldx, int axis,
                       uint32_t* amax_bits, hipStream_t st);
// in place: amax bits -> scale = amax/qmax; lambda = qmax/amax (lambda may be null)
// every entry of the vector of non-negative float bit patterns becomes their maximum
hipError_t launch_broadcast_max(uint32_t* bits, int64_t n, hipStream_t st);
hipError_t launch_scales(uint32_t* amax_bits_then_scale, float* lambda, int64_t nvec, int qmax,
                         hipStream_t st);
// codes of X in `layout`; if ramax_bits != null also accumulates max|residual| per vector
hipError_t launch_quantize_tiles(const float* X, int64_t rows, int64_t cols, int64_t ldx, int axis,
                                 const float* scale, const float* lambda, int qmax, int trunc,
                                 int layout, int8_t* Q, int64_t ldq, uint32_t* ramax_bits,
                                 hipStream_t st);
// residual codes in up to two layouts (either output may be null)
hipError_t launch_residual_tiles(const float* X, int64_t rows, int64_t cols, int64_t ldx, int axis,
                                 const float* scale, const float* lambda, const float* rlambda,
                                 int qmax, int trunc, int8_t* R_vm, int64_t ld_vm, int8_t* R_em,
                                 int64_t ld_em, hipStream_t st, RunIf run = kAlways);

// selection: counts per (chunk, vector) -> offsets -> compacted arrays
hipError_t launch_select_count(const float* X, int64_t rows, int64_t cols, int64_t ldx, int axis,
                               const float* thresh, int32_t* cnt, hipStream_t st);
hipError_t launch_select_scan(int32_t* cnt_then_off, int64_t nvec, int64_t nchunks, int32_t* totals,
                              int32_t* ptr, int64_t* nnz_dev, hipStream_t st);
hipError_t launch_select_scatter(const float* X, int64_t rows, int64_t cols, int64_t ldx, int axis,
                                 const float* thresh, const float* lambda, int qmax, int trunc,
                                 const int32_t* ptr, const int32_t* off, int32_t* idx, int8_t* val,
                                 int64_t capacity, hipStream_t st);
inline int64_t select_chunks(int64_t veclen) { return (veclen + kSelChunk - 1) / kSelChunk; }

// ---- streaming fast paths (fused.hip); the *_ok predicates say whether shapes/alignment allow them
inline int64_t mask_words(int64_t veclen) { return (veclen + 63) / 64; }
bool rows_fused_ok(int64_t cols);
// (rscale == null: no residual at all; Rq == null with rscale given: residual scales only;
//  given_scale / given_lambda: use these per-row values instead of deriving them from the row's
//  maximum, and leave scale / lambda unwritten; rlambda may be null)
// up to three arrays of 32-bit words that launch_rows_fused zeroes on the side
struct ClearList {
  uint32_t* a; int64_t na;
  uint32_t* b; int64_t nb;
  uint32_t* c; int64_t nc;
};
bool rows_fused_can_clear(int64_t rows, const ClearList& c);   // one word per thread and array
hipError_t launch_rows_fused(const float* X, int64_t rows, int64_t cols, int64_t ldx, int qmax, int trunc,
                             int8_t* Q, int64_t ldq, float* scale, float* lambda, int8_t* Rq, int64_t ldr,
                             float* rscale, float* rlambda, hipStream_t st, const float* given_scale = nullptr,
                             const float* given_lambda = nullptr,
                             const ClearList* clear = nullptr,
                             int32_t* nonzero = nullptr,    // entries that are not zero, per row
                             int pad = 0);   // zeros (less than 256) past the end of the rows of both code matrices
bool rows_resid_em_ok(const float* X, int64_t rows, int64_t cols, int64_t ldx, const float* scale,
                      const float* lambda, const float* rlambda, const int8_t* Rem, int64_t ldem);
hipError_t launch_rows_resid_em(const float* X, int64_t rows, int64_t cols, int64_t ldx, int qmax, int trunc,
                                const float* scale, const float* lambda, const float* rlambda, int8_t* Rem,
                                int64_t ldem, hipStream_t st, RunIf run = kAlways);
// that pass doubling as the selection pass of the operand (mask and counts as launch_rows_mask)
bool rows_mask_resid_em_ok(const float* X, int64_t rows, int64_t cols, int64_t ldx, const float* scale,
                           const float* lambda, const float* rlambda, const int8_t* Rem, int64_t ldem,
                           const float* thresh);
hipError_t launch_rows_mask_resid_em(const float* X, int64_t rows, int64_t cols, int64_t ldx, int qmax, int trunc,
                                     const float* scale, const float* lambda, const float* rlambda, int8_t* Rem,
                                     int64_t ldem, const float* thresh, uint64_t* mask, int32_t* counts,
                                     hipStream_t st);
hipError_t launch_cols_amax(const float* X, int64_t rows, int64_t cols, int64_t ldx, uint32_t* amax_bits,
                            hipStream_t st);
hipError_t launch_cols_codes(const float* X, int64_t rows, int64_t cols, int64_t ldx, int qmax, int trunc,
                             const float* scale, const float* lambda, int8_t* Qvm, int64_t ldvm, int8_t* Qem,
                             int64_t ldem, uint32_t* ramax_bits, hipStream_t st);
hipError_t launch_cols_codes_from_amax(const float* X, int64_t rows, int64_t cols, int64_t ldx, int qmax,
                                       int trunc, const uint32_t* amax_bits, float* scale, float* lambda,
                                       int8_t* Qvm, int64_t ldvm, uint32_t* ramax_bits, hipStream_t st);
hipError_t launch_cols_resid_from_amax(const float* X, int64_t rows, int64_t cols, int64_t ldx, int qmax,
                                       int trunc, const float* scale, const float* lambda,
                                       const uint32_t* ramax_bits, float* rscale, float* rlambda, int8_t* Rvm,
                                       int64_t ldvm, int8_t* Rem, int64_t ldem, hipStream_t st);
// columns in one read (cols_once.hip).  With a residual, `lines`: cols_once_words(rows, cols) words of zeros for each
// exchange (the maxima of X unless its scales are given, those of the residual).  Without, scale and lambda start
// at zero.
constexpr int kColsOnceRows = 512, kColsOnceCols = 32;
struct ColsOnce {
  const float* X;
  int64_t ldx;
  float *scale, *lambda;       // written, or given
  int8_t* Q;                   // codes, vector-major
  int64_t ldq;
  float *rscale, *rlambda;     // null: no residual; rlambda may be null by itself
  int8_t* Rvm;                 // residual codes in one layout or the other (k-major: with scales given)
  int64_t ldr;
  int8_t* Rem;
  int64_t ldem;
  int64_t pad_to;              // zeros in Q and Rvm from the last row on up to here (a multiple of 16; 0: none)
  const float* thresh;         // with mask: keep-bits (mask_stride bytes per column) and counts, which start at zero;
                               // counts alone (with a residual, scales not given): of the entries that are not zero
  uint8_t* mask;
  int64_t mask_stride;
  int32_t* counts;
  uint32_t* lines;
  uint32_t wait_ticks;
};
bool cols_once_ok(int64_t rows, int64_t cols, int64_t ldx);
inline int64_t cols_once_words(int64_t rows, int64_t cols) {
  const int64_t pieces = (rows + kColsOnceRows - 1) / kColsOnceRows, strips = (cols + kColsOnceCols - 1) / kColsOnceCols;
  return pieces > 1 ? pieces * strips * kColsOnceCols : 0;
}
hipError_t launch_cols_once(const ColsOnce& g, int64_t rows, int64_t cols, int qmax, int trunc, bool given, hipStream_t st);
// Sums of counts (of 256 vectors each) that a selection leaves lie this many words apart: atomics on one line are served one
// after the other, 5 ns each (next to each other: selection of two operands of 8192 x 8192 129 us, 54 to 56 like this and without sums)
constexpr int kSumStride = 64;
// Keep-masks and counts of one or two operands from codes and residual codes (select_codes.hip), with the means of |D_F| and
// the thresholds or after them
struct CodesSelect {
  const double* part;          // partial sums of |D_F|: nparts for each vector; null: the thresholds are there
  int64_t nparts;
  double count;
  float theta;
  float *mean, *thresh;
  const float* X;              // element e of vector v: X[v * vec_step + e * elem_step]
  int64_t vec_step, elem_step;
  const int8_t *Q, *R;         // rows of ld bytes, 16-byte aligned, ld a multiple of 128
  const float *scale, *lambda, *rlambda;
  uint64_t* mask;              // null: the mean and the threshold only
  int32_t* counts;
  int64_t nvec;                // 0: no such operand
  int8_t* D;                   // the kept codes, zeros elsewhere, laid out as Q (zeros past the end are there); null: not wanted
  int32_t* sums;               // the counts of every 256 vectors are added up here (kSumStride), on top of what is there; null: not wanted
};
// (veclen at most 32768)
bool select_codes_ok(int qmax, float theta, bool strips);   // strips: the call is on the path of strips.hip
hipError_t launch_select_codes(const CodesSelect& a, const CodesSelect& b, int64_t veclen, int64_t ld, int qmax, int trunc, hipStream_t st);
// k-major copies of one or two residual code matrices (codes_em.hip): nvec rows of ld bytes (16-byte aligned, ld a multiple of
// 16) to veclen rows of nvec bytes
struct CodesEm {
  const int8_t* R;
  int8_t* Rem;
  int64_t nvec;                // 0: no such matrix
  RunIf run;
};
hipError_t launch_codes_em(const CodesEm& a, const CodesEm& b, int64_t veclen, int64_t ld, hipStream_t st);
// zeroes columns [cols, ld) of up to six row-major byte matrices of `rows[i]` rows each (null: skipped)
hipError_t launch_zero_pad(int8_t* const* mats, const int64_t* rows, int n, int64_t cols, int64_t ld,
                           hipStream_t st);
// zero-fills up to three arrays of 32-bit words in one launch (null pointers are skipped)
hipError_t launch_fill3_u32(uint32_t* a, int64_t na, uint32_t* b, int64_t nb, uint32_t* c, int64_t nc,
                            hipStream_t st);
hipError_t launch_cols_resid(const float* X, int64_t rows, int64_t cols, int64_t ldx, int qmax, int trunc,
                             const float* scale, const float* lambda, const float* rlambda, int8_t* Rvm,
                             int64_t ldvm, int8_t* Rem, int64_t ldem, hipStream_t st, RunIf run = kAlways);
hipError_t launch_cols_mask(const float* X, int64_t rows, int64_t cols, int64_t ldx, const float* thresh,
                            uint64_t* mask, int32_t* counts, hipStream_t st);
hipError_t launch_cols_mask_resid(const float* X, int64_t rows, int64_t cols, int64_t ldx, int qmax, int trunc,
                                  const float* scale, const float* lambda, const uint32_t* ramax_bits,
                                  float* rscale, float* rlambda, int8_t* Rvm, int64_t ldvm, int8_t* Rem,
                                  int64_t ldem, const float* thresh, uint64_t* mask, int32_t* counts,
                                  hipStream_t st);
hipError_t launch_rows_mask(const float* X, int64_t rows, int64_t cols, int64_t ldx, const float* thresh,
                            uint64_t* mask, int32_t* counts, hipStream_t st);
// compaction from mask + codes; dense != null also writes the vector zero-filled to dense[v*ldd + e];
// nnz_hint: the number of kept entries if the host knows it (picks the variant for very sparse
// operands), else -1; dense_if: the expansion is written only if the device-side decision allows
hipError_t launch_scatter_mask(const uint64_t* mask, int64_t nvec, int64_t veclen, const int8_t* Q, int64_t ldq,
                               const int32_t* ptr, int32_t* idx, int8_t* val, int64_t capacity, int8_t* dense,
                               int64_t ldd, int64_t nnz_hint, hipStream_t st, RunIf dense_if = kAlways);
// two exclusive scans in one launch; a null totals pointer skips that half
// decide != null (paths set): one block scans both vectors, then writes SRQ_STRATEGY_AUTO's choice per
// term (paths[t] = 0 if its totals pointer is null, i.e. the term does not exist, else the matrix cores (2) if the
// total z0 / z1 reaches min_mfma, else the vector ALUs (1); seen, optional: host-visible words that
// receive the decision of each term that exists) and, if stats != null, the call's statistics
struct ScanDecision {
  int32_t* paths;             // device int32[2]
  int32_t* seen;              // host-visible int32[2] or null
  int64_t min_mfma_a, min_mfma_b;
  srq_stats_t* stats;         // device, or null
  int64_t cap_a, cap_b;       // capacities the totals are compared with for stats->overflow
};
hipError_t launch_scan_pair(const int32_t* t0, int64_t n0, int32_t* p0, int64_t* z0, const int32_t* t1,
                            int64_t n1, int32_t* p1, int64_t* z1, hipStream_t st,
                            const ScanDecision* decide = nullptr);

// ---- both operands of a small call, or one with a short inner dimension, at once (strips.hip).  Code matrices have rows
// of Kc bytes (K rounded up to a multiple of 128) and come out with zeros past K.
constexpr int64_t kStripsMaxK = 8192;        // columns of B that a workgroup can hold
constexpr int64_t kStripsMaxScan = 16384;    // vectors whose counts every workgroup of the compaction adds up
struct StripOperand {
  const float* X;
  int64_t ldx;
  int8_t* Q;
  float *scale, *lambda;
  int8_t* Rq;                  // residual codes; null: no residual (and no D)
  float *rscale, *rlambda;
  int8_t* D;                   // zero-filled codes: only the places past K are written here
  int32_t* nonzero;            // entries that are not zero, per vector; null: not wanted
};
struct StripSelect {
  const float* X;
  int64_t ldx;
  const double* part;          // partial sums of |D_F|: nparts for each vector
  int64_t nparts;
  double count;
  float theta;
  float *mean, *thresh;
  uint64_t* mask;              // null: the mean and the threshold only, and with counts a zero there if no entry is above
  int32_t* counts;             // the threshold (of zero, unless it is no number)
  const int8_t* Q;             // with D (K <= 1024): codes, rows of ldq bytes (a multiple of 128) with zeros past K
  int8_t* D;                   // zero-filled codes, the same layout; null: not wanted
  int ldq;
};
struct StripCompact {
  int nvec;
  const uint64_t* mask;
  const int32_t* counts;
  const int8_t* Q;
  int32_t *ptr, *idx;
  int8_t* val;
  int64_t capacity;
  int8_t* dense;               // null: not wanted
  int64_t* nnz;                // null: not wanted
};
// Both operands of a call whose executions are decided on the device (codes_em.hip): K <= 16384, fewer than 2^24 vectors
constexpr int64_t kCompactDecideMaxK = 16384;
struct CompactDecide {
  StripCompact a, b;           // nvec 0: no such term; dense: written where the term goes to the matrix cores
  const int32_t* sums;         // counts of every 256 vectors of a, then of b (kSumStride)
  ScanDecision dec;
  CodesEm em_a, em_b;          // copies for a term on the vector ALUs (em_a: term 2), or in any case; nvec 0: none.  `run` is not read
  int always_a, always_b;
  int groups_a, groups_b, around;   // set by the launch
};
hipError_t launch_compact_decide(const CompactDecide& g, int64_t K, int64_t Kc, hipStream_t st);
struct StripReduce {
  const float* X;
  int64_t ldx;
  const float *scale, *lambda, *thresh;
  int8_t* Q;                   // codes, rows of Kc bytes
  int8_t* Rq;
  int64_t ldr;
  float* rscale;
  uint64_t* mask;
  int32_t* counts;
};
bool strips_ok(int64_t M, int64_t N, int64_t K);
bool strips_one_ok(int axis, int64_t nvec, int64_t veclen);      // the staged entry points, one operand
bool strips_compact_ok(int64_t M, int64_t N);
hipError_t launch_quant_pair(const StripOperand& a, const StripOperand& b, int64_t M, int64_t N, int64_t K, int64_t Kc, int qmax,
                             int trunc, hipStream_t st);
hipError_t launch_select_pair(const StripSelect& a, const StripSelect& b, int64_t M, int64_t N, int64_t K, hipStream_t st);
// one operand: N columns of K codes into Q (leading dimension ldq, any alignment); its reduction (Kc: K rounded up
// to a multiple of 16)
hipError_t launch_quant_strips(const StripOperand& s, int64_t N, int64_t K, int64_t ldq, int qmax, int trunc, hipStream_t st);
hipError_t launch_reduce_rows(const StripReduce& s, int64_t M, int64_t K, int64_t Kc, int qmax, int trunc, hipStream_t st);
hipError_t launch_reduce_cols(const StripReduce& s, int64_t N, int64_t K, int64_t Kc, int qmax, int trunc, hipStream_t st);
hipError_t launch_compact_pair(const StripCompact& a, const StripCompact& b, int64_t K, int64_t Kc, hipStream_t st);

// ---- an inner dimension of at most 256 and few tiles of C: the whole call in two launches (short.hip).  Code matrices
// have rows of K rounded up to 128.  state_a / state_b: a word per sixteen rows of A / columns of B; ticket: one.
struct ShortCompact {
  int32_t *ptr, *idx;
  int8_t* val;
  int64_t capacity, *nnz;
};
struct ShortCall {
  const float *A, *B;
  int64_t lda, ldb;
  int M, N, K, trunc;
  float qmax, theta_a, theta_b;
  bool term_a, term_b;
  int8_t *Qa, *Qb, *Ra, *Rb;
  float *s_a, *lam_a, *s_ra, *s_b, *lam_b, *s_rb;
  double *row_part, *col_part;
  float *drow, *dcol, *t_a, *t_b;
  int32_t *state_a, *state_b, *ticket;
  ShortCompact ca, cb;
};
bool short_ok(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, const GemmEpilogue& ep);
hipError_t launch_short_first(const ShortCall& g, bool comp, const GemmEpilogue& ep, hipStream_t st);
hipError_t launch_short_second(const ShortCall& g, const GemmEpilogue& ep, hipStream_t st);

// thresholds from the partial sums of the GEMM epilogue; counts0 / counts1: a zero for vectors whose threshold is no number
hipError_t launch_reduce_means_pair(const double* part0, int64_t nparts0, int64_t n0, int64_t count0, float theta0,
                                    float* mean0, float* thresh0, const double* part1, int64_t nparts1,
                                    int64_t n1, int64_t count1, float theta1, float* mean1, float* thresh1,
                                    hipStream_t st, int32_t* counts0 = nullptr, int32_t* counts1 = nullptr);

// INT8 GEMM, both operands K-contiguous
constexpr int kGemmPart = 64;                 // fewest rows / columns of C per partial sum of |D_F| (sizes the buffers)
constexpr int kGemmPartLarge = 128;        // ... of the kernels with larger tiles
// number of partial sums launch_gemm_i8 leaves per row (parts_n) and per column (parts_m) of D_F
// for this problem: what the reduction after it has to add up
void gemm_sum_parts(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda, const int8_t* Qb, int64_t ldb,
                    const GemmEpilogue& ep, int64_t* parts_n, int64_t* parts_m);
int64_t gemm_tiles_m(int64_t M, int64_t N);  // tile counts of the configuration launch_gemm_i8 picks
int64_t gemm_tiles_n(int64_t M, int64_t N);
hipError_t launch_gemm_i8(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda,
                          const int8_t* Qb, int64_t ldb, const GemmEpilogue& ep, hipStream_t st);
// compute units of the current device
hipError_t gemm_device_cus(int* cus);
// raises a kernel's dynamic-LDS limit to `bytes` once per (device, kernel); safe to call from
// several host threads
hipError_t ensure_dynamic_lds(const void* kernel, int bytes);
// persistent-workgroup variant for aligned, large problems: whether it can take one (chosen inside launch_gemm_i8)
bool gemm_persistent_ok(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda, const int8_t* Qb,
                        int64_t ldb, const GemmEpilogue& ep);
// (second: accumulate mode only; both products must pass gemm_persistent_ok)
hipError_t launch_gemm_i8_persistent(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda,
                                     const int8_t* Qb, int64_t ldb, const GemmEpilogue& ep, hipStream_t st,
                                     const GemmSecond* second = nullptr);
// the kernel for the aligned problems that the two others leave (gemm_small.hip); same contract
bool gemm_small_ok(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda, const int8_t* Qb, int64_t ldb,
                   const GemmEpilogue& ep);
hipError_t launch_gemm_i8_small(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda, const int8_t* Qb,
                                int64_t ldb, const GemmEpilogue& ep, hipStream_t st,
                                const GemmSecond* second = nullptr);
bool gemm_few_large_tiles(int64_t M, int64_t N);   // fewer than 256 tiles of 256 x 256
// the kernel for few output tiles or a short K (gemm_tile64.hip), partial sums per 64 columns / rows.  One
// product or two of one shape and one pair of leading dimensions, added up in this order; in first mode C is
// not read.
struct DirectProduct {
  const int8_t *Qa, *Qb;
  const float *s_row, *s_col;
};
struct DirectProducts {
  DirectProduct p[2];
  int n;
};
bool gemm_tile64_ok(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda, const int8_t* Qb, int64_t ldb,
                    const GemmEpilogue& ep);
hipError_t launch_gemm_i8_tile64(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, const DirectProducts& pr,
                                 const GemmEpilogue& ep, hipStream_t st);
// The pair of corrections with the compaction of both operands in the same launch, behind the tiles (its operands are
// the zero-filled codes, which the selection has written).  True where that is the better way, for a pair that goes to this kernel.
struct CompactTail {
  StripCompact a, b;
  int groups_a, K, tiles;      // groups of four vectors of a; elements of a vector; tiles of C (the first and the last: set by the launch)
};
bool gemm_tile64_tail_ok(int64_t M, int64_t N, int64_t K);
hipError_t launch_gemm_i8_tile64_tail(int64_t M, int64_t N, int64_t K, int64_t ld, const DirectProducts& pr, const GemmEpilogue& ep,
                                      const CompactTail& tail, hipStream_t st);
// at most 32 rows, 64 of a narrower product, and no sums (gemm_skinny.hip)
hipError_t launch_gemm_i8_skinny(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda, const int8_t* Qb,
                                 int64_t ldb, const GemmEpilogue& ep, hipStream_t st);
// Both correction products in one accumulate-mode launch (first Qa.Qb^T with ep's scales, then sec):
// possible when both products fit the same one of the two kernels above.
bool gemm_pair_ok(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda, const int8_t* Qb, int64_t ldb,
                  const GemmSecond& sec, const GemmEpilogue& ep);
hipError_t launch_gemm_i8_pair(int64_t M, int64_t N, int64_t K, const int8_t* Qa, int64_t lda, const int8_t* Qb,
                               int64_t ldb, const GemmSecond& sec, const GemmEpilogue& ep, hipStream_t st);

// CSR (vector-major) -> zero-filled dense vector-major codes
hipError_t launch_densify(const int32_t* ptr, const int32_t* idx, const int8_t* val, int64_t nvec,
                          int64_t veclen, int64_t capacity, int8_t* dense, int64_t ld, hipStream_t st,
                          RunIf run = kAlways);

// VALU SpMM.  out[v, e] = sum_p val[p] * R[idx[p]*ldr + e];  side 0: C[v, e], side 1: C[e, v].
// Vector v owns the pairs [ptr[v], ptr_end[v]); ptr_end == null means plain CSR (ptr + 1).
hipError_t launch_spmm_valu(int side, int64_t nvec, int64_t nelem, int64_t K, const int32_t* ptr,
                            const int32_t* ptr_end, const int32_t* idx, const int8_t* val, int64_t capacity,
                            const int8_t* R, int64_t ldr, const GemmEpilogue& ep, hipStream_t st,
                            const uint32_t* kflag = nullptr);   // kflag: bitmap over k of entries to skip

// ---- column-block execution (colblock.hip): the k kept in at least min_keep_ratio of the vectors
// (at most kStripK of them) become a dense strip.  count: int32[mask_words(K) * 64] scratch;
// klist: int32[kStripK]; kflag: uint32[mask_words(K) * 2]; nstrip: int32[1]
constexpr int kStripK = 128;
hipError_t launch_colblock_pick(const uint64_t* mask, int64_t nvec, int64_t K, double min_keep_ratio,
                                int32_t* count, int32_t* klist, uint32_t* kflag, int32_t* nstrip,
                                hipStream_t st);
// strip[v][c] = Q[v][klist[c]] (only where the keep-bit is set, if a mask is given), zero-padded
// to kStripK columns
hipError_t launch_strip_gather(const int8_t* Q, int64_t ldq, const uint64_t* mask, int64_t K, int64_t nvec,
                               const int32_t* klist, int8_t* strip, hipStream_t st);

// ---- 2:4-structured execution (sparse24.hip, gemm_sparse24.hip)
// A reduced operand in 2:4 form: P1 (first two codes of a group of four k) and P2 (third and
// fourth), each as code bytes + position nibbles in the K-tile-major layout of sparse24.hip, and
// one flag word per (block of 256 vectors, K-tile) telling where P2 holds anything; plus the
// dense operand it is multiplied with, and (second product of a paired launch only) the scales
// paired with the rows and columns of C.
struct Sparse24Operand {
  const int8_t *vals1, *vals2;
  const uint8_t *nib1, *nib2;
  const uint32_t* flags;
  const int8_t* Qb;           // dense operand, K-contiguous
  int64_t ldb;
  const float *s_row, *s_col;
};
constexpr int kSparse24MaxKTiles = 256;      // K / 128 may not exceed this (one flag row = one wave-wide load)
// flag words per block of 256 vectors (a multiple of 4: rows start 16-byte aligned), and of a whole
// operand including the padding that lets the product kernel read 256 words from any row start
__host__ __device__ inline int64_t sparse24_flag_stride(int64_t kc) { return ((kc >> 7) + 3) & ~(int64_t)3; }
inline int64_t sparse24_flag_words(int64_t nvec, int64_t kc) {
  return ((nvec + 255) / 256) * sparse24_flag_stride(kc) + kSparse24MaxKTiles;
}
// compaction pass that also writes the 2:4 form (flags must be zero on entry)
bool scatter24_ok(int64_t nvec, int64_t kc, const int8_t* Q, int64_t ldq);
hipError_t launch_scatter24(const uint64_t* mask, int64_t nvec, int64_t veclen, int64_t kc, const int8_t* Q,
                            int64_t ldq, const int32_t* ptr, int32_t* idx, int8_t* val, int64_t capacity,
                            int8_t* vals1, uint8_t* nib1, int8_t* vals2, uint8_t* nib2, uint32_t* flags,
                            hipStream_t st);
// C (M x N) += dequant(product).  One product (second == null): `op` with its sparse vectors along
// the rows of C (trans false) or along its columns (trans true; scales from the epilogue either
// way).  Two products: op = term 1 (rows), *second = term 2 (columns, with its own scales).
bool gemm_sparse24_ok(int64_t M, int64_t N, int64_t K, const Sparse24Operand& op, bool trans, const GemmEpilogue& ep);
hipError_t launch_gemm_i8_sparse24(int64_t M, int64_t N, int64_t K, const Sparse24Operand& op, bool trans,
                                   const Sparse24Operand* second, const GemmEpilogue& ep, hipStream_t st);

hipError_t launch_stats(const int64_t* nnz_a, const int64_t* nnz_b, int path_a, int path_b, int64_t cap_a,
                        int64_t cap_b, srq_stats_t* out, hipStream_t st);
hipError_t launch_scale_only(int64_t M, int64_t N, const GemmEpilogue& ep, hipStream_t st);

}  // namespace srq
#endif
