// Shared declarations of the HIP implementation (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/llc.h"

namespace llc {

constexpr int kBlock = 256;        // threads of a workgroup: four 64-wide wavefronts, or two or four times that
constexpr int kMaxThreads = 1024;  // of a scan's workgroup

// Variants of the scan kernel held to 128 registers (four wavefronts per SIMD, up to 1024 threads);
// the others get 256 (two wavefronts per SIMD, up to 512 threads).
constexpr bool lean_variant(bool shared, int pairs, bool lse) { return (shared || pairs <= 2) && !(lse && !shared); }
constexpr int kListCap = 1024;     // candidate records a workgroup can hold in LDS

// Four consecutive elements of a row wherever the row starts: the alignment stated is the element's,
// so rows of an odd length or with an odd offset take the same full-width loads as aligned ones (the
// hardware splits a load that straddles cache lines).  Rows that are not 16-byte aligned used to be
// read element by element: 300 rows of 50 257 fp32 logits, K = 5, with keys 106 -> 97 us a call.
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t uint2_any __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t uint_any __attribute__((aligned(1)));
__device__ __forceinline__ float4 load_four(const float *p) {
  const float4_any t = *reinterpret_cast<const float4_any *>(p);
  return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ uint2 load_four(const uint16_t *p) {
  const uint2_any t = *reinterpret_cast<const uint2_any *>(p);
  return make_uint2(t.x, t.y);
}

// Partial result of one reduction: the smallest exact key and where it sits.
// Keys are fp64; for the logit / log-weight kinds they are ln(S) - x/T (a
// monotone image of S/p that cannot overflow), for the probability kind S/p.
struct Partials {
  double *keyX;   // [B][K][n_chunks]
  int32_t *idxX;  // [B][K][n_chunks]
  double *keyY;   // [B][n_kgroups][n_chunks]
  int32_t *idxY;  // [B][n_kgroups][n_chunks]
  int32_t *kY;    // [B][n_kgroups][n_chunks]
  double *secX;   // [B][K][n_chunks] runner-up keys: the smallest key at an index other than the
  double *secY;   // [B][n_kgroups][n_chunks] winner's (+inf if none was seen within the band)
  double *lse;    // [B][K+1]: ln sum exp(x/T) of draft k (k < K) and of the target (k == K)
  double *lse_part;  // [B][K+1][n_chunks] per-chunk shares to merge into lse first, or nullptr
  int lse_part_target;  // the shares include the target row's (slot K); else lse[.][K] is in place
};

// Rows may be a two-level index b = outer * inner_count + inner (sequences x positions in
// the verifier); plain batches have inner_count = 1.
struct RowMap {
  long long inner_count;
  long long draft_outer, draft_inner;    // element strides of the draft tensor
  long long target_outer, target_inner;  // element strides of the target tensor
  long long row_outer, row_inner;        // strides of the random stream's row number
  __host__ __device__ long long draft_off(long long b) const {
    return (b / inner_count) * draft_outer + (b % inner_count) * draft_inner;
  }
  __host__ __device__ long long target_off(long long b) const {
    return (b / inner_count) * target_outer + (b % inner_count) * target_inner;
  }
};

struct FinalizeParams {
  long long B;
  int K, n_chunks, n_kgroups;
  int log_kind;        // keys are in the log domain and need the normaliser
  Partials in;
  int need_norm;       // the keys' normalisers are wanted ...
  int store_norm;      // ... and, of the drafts, also kept in in.lse
  int32_t *X, *Y, *match_k;  // Y, accept may be null (draft side only)
  int y_given;               // Y holds the pool's index already: only the accept test is taken
  const uint8_t *bins;       // optional: message[b] = bin of candidate Y[b]
  long long bins_stride_b;
  int32_t *message;
  uint8_t *accept;
  float *keyX, *keyY;  // optional
  double *log_keyX;    // optional [B][K]: ln of the normalised winning key (log kinds)
  double *log_secX;    // optional [B][K]: the same for the runner-up (another index) of that reduction
  // optional decoder outputs of the compression scheme (Appendix C, Appendix D.2): W_k = cand[X_k],
  // the estimate g(W_k, T_k) = (vz W_k + ve T_k) / (ve + vz + ve vz), the best squared error
  const float *cand;         // [B][V'] candidates U_i, or nullptr
  long long cand_stride_b;
  const float *side;         // [B][K] side information T_k
  long long side_stride_b;
  const float *source;       // [B] the source sample A (known to an evaluation only), or nullptr
  double var_e, var_z;       // variance of W given A, of T given A
  float *W, *A_hat;          // [B][K] optional
  float *sq_err;             // [B] optional: min_k (g(W_k, T_k) - A)^2
  int count_draft;     // count the draft side's reductions in stats->degenerate
  int count_pool;      // count the pool's
  int count_near;      // also count the near-ties of the sides that are counted
  llc_stats *stats;
};

struct ScanParams {
  const void *draft;
  const void *target;
  RowMap map;
  long long draft_stride_k;  // elements
  long long B;
  int n_each;            // rows (draft_stride_k apart) that each price all K drafts: B x n_each rows of results; else 1
  int K, V;
  int threads;           // of a workgroup
  int finish;            // a row is one workgroup, which also takes the finalize step (fin)
  int form_lse;          // the scan also forms the rows' normalisers (into lse_part unless it finishes them)
  int n_chunks;          // workgroups a row's V is split over
  int groups_per_chunk;  // 4-element groups per chunk (a multiple of the threads)
  int n_kgroups;         // ceil(K / KT)
  unsigned seed_lo, seed_hi;
  unsigned long long row_offset;
  float temp_target, temp_draft_all;
  const float *temp_draft;  // device, K entries, or nullptr
  int force_exact;
  int no_pool;              // draft-side reductions only: the target is never read
  int no_draft;             // pool only: the draft rows are never read, X comes out as -1
  int same_race;            // every draft uses draft 0's race times (binned / pool-only variant only)
  const uint8_t *bins;      // optional [B][V] bins of the candidates (bins_stride_b bytes per row):
  long long bins_stride_b;  // on the draft side only candidates in the bin of index bin_of[b] count
  const int32_t *bin_of;    // [B]
  double *lse_part;         // [B][K+1][n_chunks] or nullptr: the scan also forms the rows' normalisers,
                            // ln of every chunk's sum of exp(x/T) (merged by the finalize kernel)
  const long long *draft_row_off;  // optional [B]: elements added to row b's draft offset; a negative
                            // entry means the row is not wanted (its partial results come out empty)
  Partials out;
  llc_stats *stats;
  FinalizeParams fin;       // used if finish is set
};


// Algorithm 2's sequential epilogue over the per-(position, draft) target-side argmins.
struct VerifyParams {
  long long S;
  int L, K;
  const int32_t *cand;       // [S][L+1][K] argmin_i S_i^(j,k) / q_i^(j,k)
  const double *cand_key;    // [S][L+1][K] ln of its normalised key
  const double *cand_sec;    // [S][L+1][K] ln of the normalised runner-up key of the same reduction
  const int32_t *tokens;     // draft tokens
  long long tok_stride_s, tok_stride_j;
  int32_t *Y;                // [S][L+1]
  int32_t *n_out;            // [S]
  uint8_t *active;           // [S][K] optional
  float *keyY;               // [S][L+1] optional
  llc_stats *stats;          // optional: near_ties of the emitted positions
};

struct LseParams {
  const void *draft;
  const void *target;
  RowMap map;
  long long draft_stride_k;
  long long B;
  int K, V;
  int dtype;
  float temp_target, temp_draft_all;
  const float *temp_draft;
  int is_logits;  // divide by the temperature
  int per_k;      // every draft has its own row (else one row serves the K drafts)
  int with_target;  // also the target row's normaliser
  int with_drafts;  // the draft rows' normalisers (0: the scan kernel forms them itself)
  const uint8_t *bins;      // as in ScanParams: masks the draft rows
  long long bins_stride_b;
  const int32_t *bin_of;
  const long long *draft_row_off;  // as in ScanParams (rows that are not wanted are skipped)
  double *lse;    // [B][K+1]
};

// One position of Algorithm 2's loop in its strongly drafter-invariant form (Appendix B): the pool
// runs over all K drafts' race times; a viable draft is priced with its own target row, a dropped
// one with the row of the first viable draft.
struct StrongStepParams {
  long long S;
  int L, K, j;               // position j of 0..L
  const int32_t *cand;       // [S][L+1][K] own-row argmins (viable drafts)
  const double *cand_key;    // [S][L+1][K] ln of their normalised keys
  const double *cand_sec;    // [S][L+1][K] ln of the normalised runner-up keys
  // this position priced with the first viable draft's row, as the scan left it: per-chunk
  // partial argmins (only read for dropped drafts; unused at j == 0)
  const double *part_key;    // [S][K][n_chunks] ln-domain keys before the normaliser is added
  const int32_t *part_idx;   // [S][K][n_chunks]
  const double *part_sec;    // [S][K][n_chunks] runner-up keys of the same partial reductions
  int n_chunks;
  const int32_t *tokens;
  long long tok_stride_s, tok_stride_j;
  long long stride_k;        // of the target tensor, for the next position's row offsets
  uint8_t *viable;           // [S][K] state, set up at j == 0
  int32_t *running;          // [S] state
  long long *next_off;       // [S] out: stride_k * (first viable draft) if the next position needs
                             // dropped drafts priced, else -1
  const double *lse;         // [S][L+1][K+1] normalisers of every (position, draft) row
  double *lse_sel;           // [S][K+1] out: the normaliser of the row that prices the next position
  int32_t *Y;                // [S][L+1]
  int32_t *n_out;            // [S]
  uint8_t *active;           // [S][K] optional
  float *keyY;               // [S][L+1] optional
  llc_stats *stats;          // optional: near_ties of the emitted positions
};

// The same loop where every position's K rows have been scanned for all K drafts at once.
struct StrongParams {
  long long S;
  int L, K;
  const int32_t *cand;       // [S][L+1][K][K] argmin of draft (last) priced with a row
  const double *cand_key;    // [S][L+1][K][K] ln of their normalised keys
  const int32_t *tokens;
  long long tok_stride_s, tok_stride_j;
  int32_t *Y;                // [S][L+1]
  int32_t *n_out;            // [S]
  uint8_t *active;           // [S][K] optional
  float *keyY;               // [S][L+1] optional
};

// Algorithm 1 on candidate lists: one workgroup per row, exact keys for the entries an fp32 key lets through.
struct TopmParams {
  long long B;
  int K, Md, Mt;
  int dtype, kind;
  const int32_t *draft_ids;
  const void *draft_val;
  long long draft_stride_b, draft_stride_k;
  const int32_t *target_ids;
  const void *target_val;
  long long target_stride_b;
  float temp_target, temp_draft_all;
  const float *temp_draft;
  unsigned seed_lo, seed_hi;
  unsigned long long row_offset;
  int32_t *X, *Y, *match_k;
  uint8_t *accept;
  float *keyX, *keyY;
  llc_stats *stats;
  int at_once;  // drafts whose candidates share the list (launcher)
};

// Theorem 1's bound per row (diagnostics): one workgroup sums a row, by cells of ln(q/p) or by sorting.
constexpr int kLmlMaxK = LLC_LML_MAX_K;
constexpr int kLmlSlots = 512;  // (sorting runs two workgroups on each of 256 CUs, cells run one: more cannot be resident)
struct LmlParams {
  long long B;
  int V;
  int dtype;
  int probs;        // inputs are probabilities (else logits / log-weights)
  const void *draft;
  const void *target;
  long long draft_stride_b, target_stride_b;
  float temp_draft, temp_target;  // 1 for log-weights and probabilities
  int n_k;
  int k[kLmlMaxK];  // list sizes
  double kd[kLmlMaxK];
  double *bound;    // [B][n_k]
  double *relaxed;  // [B][n_k] or nullptr
  double *tv;       // [B] or nullptr
  char *work;       // workspace: 24 V bytes per slot (see the kernels)
  int slots;        // rows the workspace holds at a time (= rows per launch; a call is ceil(B / slots) launches)
  long long row0;   // first row of this launch (set by the launcher)
  int only_flagged; // the sorting kernel takes only the rows that the cell kernel left (launcher)
};

// One launcher per (element type, draft layout); defined in scan_*.hip.
// kt: drafts per workgroup pass (2, 4, 8; one word per (index, draft) and a shared proposal also 6); probs: inputs are probabilities.
hipError_t launch_scan_f32_shared(int kt, bool probs, unsigned grid, hipStream_t s, const ScanParams &p);
hipError_t launch_scan_f32_perk(int kt, bool probs, unsigned grid, hipStream_t s, const ScanParams &p);
hipError_t launch_scan_bf16_shared(int kt, bool probs, unsigned grid, hipStream_t s, const ScanParams &p);
hipError_t launch_scan_bf16_perk(int kt, bool probs, unsigned grid, hipStream_t s, const ScanParams &p);
// the same with the race times drawn min-first (no binned or pool-only passes)
hipError_t launch_scan_f32_shared_minf(int kt, bool probs, unsigned grid, hipStream_t s, const ScanParams &p);
hipError_t launch_scan_f32_perk_minf(int kt, bool probs, unsigned grid, hipStream_t s, const ScanParams &p);
hipError_t launch_scan_bf16_shared_minf(int kt, bool probs, unsigned grid, hipStream_t s, const ScanParams &p);
hipError_t launch_scan_bf16_perk_minf(int kt, bool probs, unsigned grid, hipStream_t s, const ScanParams &p);

// llc_couple on a given workspace (api.hip).
int couple_on(const llc_couple_args *a, void *workspace, size_t workspace_bytes);

hipError_t launch_finalize(hipStream_t s, const FinalizeParams &p);
hipError_t launch_lse(hipStream_t s, const LseParams &p);
hipError_t launch_verify(hipStream_t s, const VerifyParams &p);
hipError_t launch_strong_step(hipStream_t s, const StrongStepParams &p);
hipError_t launch_strong(hipStream_t s, const StrongParams &p);
hipError_t launch_topm(hipStream_t s, const TopmParams &p);
hipError_t launch_lml(hipStream_t s, const LmlParams &p);

}  // namespace llc
