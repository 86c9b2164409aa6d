// Algorithm 1 on candidate lists (paper Section 4.4: with top-K sampling only M << N tokens
// per distribution survive).  A row is a few hundred (token id, value) pairs: one workgroup per row,
// one wavefront per draft list at a time, all (draft, target entry) pairs over the workgroup for the pool.
// Every entry draws the upper half of its random word (the block it is in also holds the half of the entry's
// other draft of the pair) and bounds its key from both sides in fp32; those whose lower bound is within a band
// of their reduction's smallest upper bound go to a list in LDS, where the lower half is drawn, and are evaluated exactly, in fp64, all at
// once: ln S - x/T for logits and log-weights, S/p for probabilities, reduced with the usual tie rule
// (smaller key, then smaller token id, then smaller k).  The band covers the approximation's error on both
// sides with room for every key within 1e-6 of the winner's, so nothing that could win, or make the winner a
// near-tie, is left out.  Where there are many drafts they go through the list in parts, so that it holds their
// candidates however many there are; what overflows it all the same is evaluated exactly entry by entry.
#include <cmath>

#include "scan.hpp"

namespace llc {
namespace {

constexpr int kCandidates = 512;  // entries of the list in LDS

__device__ __forceinline__ float widen_at(const void *base, int dtype, long long off) {
  if (dtype == LLC_F32) return reinterpret_cast<const float *>(base)[off];
  return __uint_as_float((uint32_t) reinterpret_cast<const uint16_t *>(base)[off] << 16);
}

// does the entry carry mass?  (empty slot, NaN, +inf, and for probabilities <= 0: no)
__device__ __forceinline__ bool has_mass(int id, float v, bool probs) {
  if (id < 0) return false;
  if (probs) return v > 0.0f && v < __builtin_huge_valf();
  return v < __builtin_huge_valf() && v > -__builtin_huge_valf();
}

// The word of a block that holds the half-words of `id`.
__device__ __forceinline__ uint32_t pick(const uint32_t (&w)[4], uint32_t id) {
  const int j = (int)(id & 3u);
  return j == 0 ? w[0] : j == 1 ? w[1] : j == 2 ? w[2] : w[3];
}
__device__ __forceinline__ uint32_t word_of(uint32_t id, uint32_t k, uint32_t row_lo, uint32_t row_hi,
                                            uint32_t k0, uint32_t k1) {
  uint32_t up[4], lo[4];
  philox_block(row_lo, id >> 2, row_hi, k >> 1, k0, k1, up);
  philox_block(row_lo, id >> 2, row_hi, (k >> 1) | kLowBlock, k0, k1, lo);
  return element_word(pick(up, id), pick(lo, id), (int)(k & 1u));
}

// The upper half-words of (id, draft pair): the even draft's in the lower 16 bits, the odd one's in the upper.
__device__ __forceinline__ uint32_t upper_of(uint32_t id, uint32_t pair, uint32_t row_lo, uint32_t row_hi,
                                             uint32_t k0, uint32_t k1) {
  uint32_t up[4];
  philox_block(row_lo, id >> 2, row_hi, pair, k0, k1, up);
  return pick(up, id);
}

// One of a row's K + 1 reductions (drafts, then the pool), in LDS.
struct Race {
  unsigned long long best, where, second;  // ordered images of the keys; where = (id, k)
};

// The same in registers (id -1: nothing yet); fold takes one more entry, or what others found, into it.
struct Best {
  double key;
  int id, k;
  double sec;
};
__device__ __forceinline__ void fold(Best &v, const Best &c) {
  if (c.id < 0) return;
  const bool wins = v.id < 0 || c.key < v.key || (c.key == v.key && (c.id < v.id || (c.id == v.id && c.k < v.k)));
  double sec = fmin(v.sec, c.sec);
  if (v.id >= 0 && v.id != c.id) sec = fmin(sec, wins ? v.key : c.key);
  if (wins) v = c;
  v.sec = sec;
}
__device__ __forceinline__ Best wave_best(Best v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    Best o;
    o.key = __shfl_xor(v.key, d);
    o.id = __shfl_xor(v.id, d);
    o.k = __shfl_xor(v.k, d);
    o.sec = __shfl_xor(v.sec, d);
    fold(v, o);
  }
  return v;
}
__device__ __forceinline__ void store_best(Race &r, const Best &v) {
  if (v.id < 0) return;
  r.best = ord64(v.key);
  r.where = ((unsigned long long)(uint32_t)v.id << 32) | (uint32_t)v.k;
  r.second = ord64(v.sec);
}

enum Form {
  kPairs,   // two drafts that share their blocks at a time, in the pool and, where all drafts have one list, there
  kHalves,  // the same, and two wavefronts take a list, 64 entries each in turn
  kSingle   // one draft at a time
};

// What bounds it: the latency of its phases (reductions across lanes, the exact keys' logarithms), then
// instruction issue.  Exact keys for all entries took more than half of all instructions; both halves of every
// entry's word, two blocks for each draft, most of the rest: 1024 rows, K = 8, one list of 50, with keys 13.0 us, now
// 10.9; lists of 256, own for each draft 36.1, 30.3, shared 28.4, 21.0.  (Fetching every round's entries a
// round ahead, beyond the first ones that are, and a shorter exponential for the normalisers, changed nothing.)
// WHOLE: what is near by its upper half-word is looked at again with the whole word; FORM: how lists and the pool's
// entries are shared out (both: see launch_topm).
template <bool PROBS, bool MANY, bool WHOLE, int FORM>
__global__ void __launch_bounds__(kBlock, 4) topm_kernel(const TopmParams p) {
  __shared__ double c_key[kCandidates];
  __shared__ int c_id[kCandidates], c_k[kCandidates];  // c_k: the draft, K more for a pool entry
  __shared__ float c_v[kCandidates];
  __shared__ uint32_t c_x[kCandidates];  // the upper half of its word
  __shared__ double s_lse_draft, s_lse_target;
  __shared__ int s_count, s_match;
  __shared__ unsigned long long s_evals;
  __shared__ unsigned s_degenerate, s_near;
  extern __shared__ __align__(16) char s_dyn[];
  const int K = p.K;
  Race *race = reinterpret_cast<Race *>(s_dyn);              // [K + 1]
  double *s_lse = reinterpret_cast<double *>(race + K + 1);  // [K]: where every draft has its own list

  const long long b = blockIdx.x;
  const int waves = blockDim.x >> 6, nt = blockDim.x;
  int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool logits = p.kind == LLC_LOGITS;
  const unsigned long long row = p.row_offset + (unsigned long long)b;
  const uint32_t row_lo = (uint32_t)row, row_hi = (uint32_t)(row >> 32);
  const long long t_off = b * p.target_stride_b;
  const int32_t *t_ids = p.target_ids + t_off;
  const float inf = __builtin_huge_valf();
  const bool one_list = p.draft_stride_k == 0 && p.temp_draft == nullptr;
  auto draft_off = [&](const int k) { return b * p.draft_stride_b + (long long)k * p.draft_stride_k; };
  auto draft_temp = [&](const int k) { return logits ? (p.temp_draft != nullptr ? p.temp_draft[k] : p.temp_draft_all) : 1.0f; };
  const float Tq = logits ? p.temp_target : 1.0f;

  // The first entries of a wavefront's first list and of its share of the pool leave before anything is set up.
  // A wavefront takes a draft's list, or where all drafts have one list, a pair of drafts', which share their blocks.
  const int step = FORM != kSingle && one_list ? 2 : 1;  // drafts whose list a wavefront takes
  const int my_list = FORM == kHalves ? wave >> 1 : wave;
  const int e_first = FORM == kHalves ? __builtin_amdgcn_readfirstlane((wave & 1) * 64) : 0;
  constexpr int kStepE = FORM == kHalves ? 128 : 64;
  // ((draft pair or draft, target entry); below 2^25)
  const unsigned pool_items = (unsigned)(FORM == kSingle ? K : (K + 1) >> 1) * (unsigned)p.Mt;
  struct Slot { int id; float v; };
  auto draft_slot = [&](const int k, const int e) {
    Slot x = {-1, 0.0f};
    if (e < p.Md) { const long long off = draft_off(k) + e; x.id = p.draft_ids[off]; x.v = widen_at(p.draft_val, p.dtype, off); }
    return x;
  };
  auto pool_slot = [&](const unsigned it) {
    Slot x = {-1, 0.0f};
    if (it < pool_items) { const int e = (int)(it % (unsigned)p.Mt); x.id = t_ids[e]; x.v = widen_at(p.target_val, p.dtype, t_off + e); }
    return x;
  };
  Slot first_draft = {-1, 0.0f}, first_pool = {-1, 0.0f};
  if (!MANY) {
    if (my_list * step < K) first_draft = draft_slot(my_list * step, e_first + lane);
    first_pool = pool_slot((unsigned)((waves - 1 - wave) * 64 + lane));
  }

  for (int k = tid; k <= K; k += nt) { race[k].best = kOrdInf64; race[k].where = ~0ull; race[k].second = kOrdInf64; }
  if (tid == 0) { s_count = 0; s_match = 0x7FFFFFFF; s_evals = 0; s_degenerate = 0; s_near = 0; }
  __syncthreads();

  // the entries of one round of a wavefront, a pair of drafts' half-words at a time: the smallest upper bound of
  // a key so far (tau), and onto the list with whatever may be below it or near it (what comes later can only
  // lower it)
  unsigned long long evals = 0;
  struct Bounds { float low, high; };
  auto bounds = [&](const bool has, const float v, const uint32_t half, const float c) {
    Bounds a = {inf, inf};
    float ell;
    if (has && approx_log2_mass<PROBS>(v, c, ell)) {  // (the race time falls as the word grows)
      a.low = approx_log2_race_time((half << 16) | 0xFFFFu) - ell;
      a.high = approx_log2_race_time(half << 16) - ell;
    }
    return a;
  };
  auto lower_tau = [&](float &tau, const float a) {
    tau = fminf(tau, unord32(__builtin_amdgcn_readlane(wave_min_to_last(ord32(a)), 63)));
  };
  auto is_near = [&](const float a, const float tau) {
    // (far values: the fp32 product's rounding grows with them; beyond all measure every entry goes)
    const float band = kEps2 + (fabsf(tau) + 64.0f) * 0x1p-20f;
    return a <= tau + band || !(fabsf(tau) < 1e30f);
  };
  auto list = [&](const bool has, const int id, const float v, const uint32_t half, const float c, const int tag, const float low,
                  float &tau) {
    bool near = is_near(low, tau);
    if (WHOLE && __ballot(has && near) != 0ull) {  // uniform
      float a = inf, ell;
      if (has && near && approx_log2_mass<PROBS>(v, c, ell)) {
        const uint32_t k = (uint32_t)(tag >= K ? tag - K : tag);
        uint32_t lo[4];
        philox_block(row_lo, (uint32_t)id >> 2, row_hi, (k >> 1) | kLowBlock, p.seed_lo, p.seed_hi, lo);
        const uint32_t lw = pick(lo, (uint32_t)id);
        a = approx_log2_race_time((half << 16) | ((k & 1u) ? lw >> 16 : lw & 0xFFFFu)) - ell;
      }
      lower_tau(tau, a);
      near = near && is_near(a, tau);
    }
    if (has) ++evals;
    if (has && near) {
      const int pos = atomicAdd(&s_count, 1);
      if (pos < kCandidates) { c_id[pos] = id; c_v[pos] = v; c_x[pos] = half; c_k[pos] = tag; }
    }
  };

  const double huge = __builtin_huge_val();
  auto offer = [&](const int round, const int tag, const int id, const double key) {
    if (!(key < huge)) return;
    Race &r = race[min(tag, K)];
    const unsigned long long o = ord64(key);
    if (round == 0) {
      atomicMin(&r.best, o);
    } else if (round == 1) {
      if (o == r.best) atomicMin(&r.where, ((unsigned long long)(uint32_t)id << 32) | (uint32_t)(tag >= K ? tag - K : tag));
    } else if ((uint32_t)id != (uint32_t)(r.where >> 32)) {
      atomicMin(&r.second, o);
    }
  };
  // entry e of list (k, or the target's for all k): its exact key as a reduction of its own
  auto exact_entry = [&](const bool pool, const int k, const int e) {
    const long long off = (pool ? t_off : draft_off(k)) + e;
    const int id = pool ? p.target_ids[off] : p.draft_ids[off];
    const float v = widen_at(pool ? p.target_val : p.draft_val, p.dtype, off);
    const float T = pool ? Tq : draft_temp(k);
    Best c = {huge, -1, k, huge};
    if (has_mass(id, v, PROBS) && T > 0.0f && T < inf) {
      const uint32_t x = word_of((uint32_t)id, (uint32_t)k, row_lo, row_hi, p.seed_lo, p.seed_hi);
      c.key = exact_key<PROBS>(exact_race_time(x), v, (double)T);
      c.id = id;
    }
    return c;
  };
  int k0 = 0;
  do {
    if (MANY) {  // (or what is formed from them for every part below is kept, and spills, across the whole loop)
      asm volatile("" : "+v"(tid));
      lane = tid & 63;
      wave = tid >> 6;
    }
    const int k1 = MANY ? min(k0 + p.at_once, K) : K;
    const bool last = !MANY || k1 == K;  // with the pool and the normalisers
    // ---- draft side: one wavefront per list, lanes over its entries
    for (int k = k0 + (FORM == kHalves ? my_list : wave) * step; k < k1; k += waves * step) {
      const float T = draft_temp(k);
      const bool t_ok = T > 0.0f && T < inf;
      const bool two = FORM != kSingle && one_list && k + 1 < k1;  // uniform
      const float c = kLog2e / T;
      float tau[2] = {inf, inf};
      for (int e0 = e_first; e0 < p.Md; e0 += kStepE) {
        const Slot x = !MANY && e0 == e_first && k == my_list * step ? first_draft : draft_slot(k, e0 + lane);
        const bool has = t_ok && has_mass(x.id, x.v, PROBS);
        const uint32_t halves = upper_of((uint32_t)x.id, (uint32_t)(k >> 1), row_lo, row_hi, p.seed_lo, p.seed_hi);
        const uint32_t mine = (k & 1) ? halves >> 16 : halves & 0xFFFFu;
        const Bounds a = bounds(has, x.v, mine, c);
        lower_tau(tau[0], a.high);
        list(has, x.id, x.v, mine, c, k, a.low, tau[0]);
        if (two) {  // (k is even)
          const Bounds o = bounds(has, x.v, halves >> 16, c);
          lower_tau(tau[1], o.high);
          list(has, x.id, x.v, halves >> 16, c, k + 1, o.low, tau[1]);
        }
      }
    }
    if (last) {
      // ---- pool: all (k, target entry) pairs over the workgroup, two drafts at a time, the last wavefronts
      // first (the first ones have had the more lists)
      {
        const float c = kLog2e / Tq;
        float tau = inf;
        for (unsigned i0 = (unsigned)(waves - 1 - wave) * 64; i0 < pool_items; i0 += (unsigned)nt) {
          const unsigned it = i0 + (unsigned)lane;
          const Slot x = !MANY && i0 < (unsigned)nt ? first_pool : pool_slot(it);
          const int k = it < pool_items ? (FORM == kSingle ? 1 : 2) * (int)(it / (unsigned)p.Mt) : 0;
          const bool has = has_mass(x.id, x.v, PROBS), two = has && k + 1 < K;
          const uint32_t halves = upper_of((uint32_t)x.id, (uint32_t)(k >> 1), row_lo, row_hi, p.seed_lo, p.seed_hi);
          if (FORM == kSingle) {
            const uint32_t mine = (k & 1) ? halves >> 16 : halves & 0xFFFFu;
            const Bounds a = bounds(has, x.v, mine, c);
            lower_tau(tau, a.high);
            list(has, x.id, x.v, mine, c, K + k, a.low, tau);
            continue;
          }
          const Bounds a = bounds(has, x.v, halves & 0xFFFFu, c), o = bounds(two, x.v, halves >> 16, c);
          lower_tau(tau, fminf(a.high, o.high));
          list(has, x.id, x.v, halves & 0xFFFFu, c, K + k, a.low, tau);
          list(two, x.id, x.v, halves >> 16, c, K + k + 1, o.low, tau);
        }
      }
      // ---- normalisers, only for reported keys (the argmins and near-ties need none): one wavefront per list
      if (!PROBS && (p.keyX != nullptr || p.keyY != nullptr)) {
        for (int l = waves - 1 - wave; l <= (one_list ? 1 : K); l += waves) {
          const bool target = l == 0;  // list 0 the target's, l > 0 draft l - 1's
          const int M = target ? p.Mt : p.Md;
          const long long off = target ? t_off : draft_off(l - 1);
          const int32_t *ids = target ? t_ids : p.draft_ids + off;
          const void *val = target ? p.target_val : p.draft_val;
          const float T = target ? Tq : draft_temp(l - 1);
          float m = -inf;
          for (int e = lane; e < M; e += 64) {
            const float v = widen_at(val, p.dtype, off + e);
            if (has_mass(ids[e], v, false)) m = fmaxf(m, v);
          }
#pragma unroll
          for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d));
          double sum = 0.0;
          if (m > -inf) {
            for (int e = lane; e < M; e += 64) {
              const float v = widen_at(val, p.dtype, off + e);
              if (has_mass(ids[e], v, false)) sum += exp(((double)v - (double)m) / (double)T);
            }
          }
#pragma unroll
          for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
          if (lane == 0) {
            const bool ok = m > -inf && T > 0.0f && T < inf;
            const double lse = ok ? (double)m / (double)T + log(sum) : -__builtin_huge_val();
            if (target) s_lse_target = lse;
            else if (one_list) s_lse_draft = lse;
            else s_lse[l - 1] = lse;
          }
        }
      }
    }
    __syncthreads();

    // ---- exact keys of the list, in three rounds: the smallest key, the smallest (id, k) that holds it, the
    // smallest key at another id
    const int n = s_count;
    if (n <= kCandidates) {  // uniform
      for (int c = tid; c < n; c += nt) {
        const int tag = c_k[c];
        const uint32_t k = (uint32_t)(tag >= K ? tag - K : tag), id = (uint32_t)c_id[c];
        uint32_t lo[4];
        philox_block(row_lo, id >> 2, row_hi, (k >> 1) | kLowBlock, p.seed_lo, p.seed_hi, lo);
        const uint32_t lw = pick(lo, id);
        const uint32_t x = (c_x[c] << 16) | ((k & 1u) ? lw >> 16 : lw & 0xFFFFu);
        c_key[c] = exact_key<PROBS>(exact_race_time(x), c_v[c], (double)(tag >= K ? Tq : draft_temp(tag)));
        offer(0, tag, c_id[c], c_key[c]);
      }
      __syncthreads();
      for (int c = tid; c < n; c += nt) offer(1, c_k[c], c_id[c], c_key[c]);
      __syncthreads();
      for (int c = tid; c < n; c += nt) offer(2, c_k[c], c_id[c], c_key[c]);
    } else {
      // more candidates than the list holds (one id over and over, or values beyond fp32's measure): every entry
#pragma unroll 1
      for (int k = k0 + wave; k < k1; k += waves) {
        Best v = {huge, -1, k, huge};
#pragma unroll 1
        for (int e = lane; e < p.Md; e += 64) fold(v, exact_entry(false, k, e));
        v = wave_best(v);
        if (lane == 0) store_best(race[k], v);
      }
      if (last) {  // uniform
        Best v = {huge, -1, 0, huge};
        const unsigned items = (unsigned)K * (unsigned)p.Mt;
#pragma unroll 1
        for (unsigned it = tid; it < items; it += nt) fold(v, exact_entry(true, (int)(it / (unsigned)p.Mt), (int)(it % (unsigned)p.Mt)));
        v = wave_best(v);
        if (lane == 0) { c_key[2 * wave] = v.key; c_key[2 * wave + 1] = v.sec; c_id[wave] = v.id; c_k[wave] = v.k; }
        __syncthreads();
        if (tid == 0) {
          for (int w = 1; w < waves; ++w) fold(v, Best{c_key[2 * w], c_id[w], c_k[w], c_key[2 * w + 1]});
          store_best(race[K], v);
        }
      }
    }
    __syncthreads();
    if (MANY) {
      if (tid == 0) s_count = 0;
      __syncthreads();
      k0 = k1;
    }
  } while (MANY && k0 < K);

  // ---- outputs
  const int y = race[K].where != ~0ull ? (int)(race[K].where >> 32) : -1;
  for (int k = tid; k <= K; k += nt) {
    const Race r = race[k];
    const int id = r.where != ~0ull ? (int)(r.where >> 32) : -1;
    const double key = unord64(r.best), sec = unord64(r.second);
    float *out = k < K ? p.keyX : p.keyY;
    const long long at = k < K ? b * K + k : b;
    (k < K ? p.X : p.Y)[at] = id;
    if (out != nullptr) {
      const double lse = PROBS ? 0.0 : k == K ? s_lse_target : one_list ? s_lse_draft : s_lse[k];
      out[at] = id >= 0 ? (float)(PROBS ? key : exp(key + lse)) : inf;
    }
    if (k < K && id >= 0 && id == y) atomicMin(&s_match, k);
    if (p.stats != nullptr) {
      // the winner and the runner-up within 1e-6 (relative, in S/p; log-domain keys differ by the log of the ratio)
      if (id < 0) atomicAdd(&s_degenerate, 1u);
      else if (sec < huge &&
               (!PROBS ? expm1(sec - key) < 1e-6 : key > 0.0 ? (sec - key) / key < 1e-6 : !(sec > 0.0))) atomicAdd(&s_near, 1u);
    }
  }
  if (p.stats != nullptr && evals) atomicAdd(&s_evals, evals);
  __syncthreads();
  if (tid == 0) {
    const bool hit = s_match != 0x7FFFFFFF;
    p.accept[b] = hit ? 1 : 0;
    if (p.match_k != nullptr) p.match_k[b] = hit ? s_match : -1;
    if (p.stats != nullptr) {
      if (s_evals) atomicAdd(&p.stats->exact_evals, s_evals);
      if (s_degenerate) atomicAdd(&p.stats->degenerate, (unsigned long long)s_degenerate);
      if (s_near) atomicAdd(&p.stats->near_ties, (unsigned long long)s_near);
    }
  }
}

}  // namespace

hipError_t launch_topm(hipStream_t s, const TopmParams &params) {
  if (params.B == 0) return hipSuccess;
  TopmParams p = params;
  // How many drafts share the list at a time: a list of r rounds of 64 entries leaves 1 + 1/2 + .. + 1/r
  // candidates on average, and the list has room for the pool's few dozen besides.  All at once up to 400 drafts
  // of 64 entries, 167 of 256, 50 of the longest.  (K = 512, lists of 50, 1024 rows, where all at once overflows:
  // 1874 us, now 350; K = 256 in parts of 64 measured 182 against 166.)
  // (an even number: a pair of drafts is not divided)
  p.at_once = (int)(400.0 / (1.0 + std::log((double)((p.Md + 63) / 64)))) & ~1;
  // Half-words tell race times apart by 2^-16 only, where the smallest of n is about 1 / n: a flat reduction leaves some n / 30 000 more
  // candidates by them than by whole words (a list of 65 536 9.7 and not 7.3, a pool of 2^24 524 and not 42; values apart
  // leave less).  Where that would fill the list, what is near is looked at again with the whole word, which would cost others 2
  // to 8 %.  (Flat lists, 64 rows, ms, both halves of every word, half-words alone, now: 50 lists of 65 536 and as long a target's 22.0,
  // 45.1, 17.8; K = 256, the target's of 65 536 46.0, 88.7, 27.9; K = 128, lists of 8 192, just beyond the line 5.56, 3.44, 3.71.)
  const double at_a_time = p.K < p.at_once ? p.K : p.at_once, pairs = (double)p.K * p.Mt;
  const double by_halves = at_a_time * (1.0 + std::log((p.Md + 63) / 64) + p.Md / 30000.0) +
                           4.0 * (1.0 + std::log(std::ceil(pairs / 512.0))) + pairs / 30000.0;
  const bool whole = by_halves > 440.0;  // (of 512: sums vary by twenty)
  // (four wavefronts a row: 1024 rows are resident at once; eight, with half as many rows resident, measured
  // 26.4 against 25.1 us a call at 1024 rows, K = 8, lists of 256)
  const unsigned lds = (unsigned)((p.K + 1) * sizeof(Race) + p.K * sizeof(double));
  const bool probs = p.kind == LLC_PROBS, many = p.K > p.at_once;
  // Few drafts: pairs leave wavefronts idle, and a lone wavefront's second draft, or the other half of a long list, is what the
  // row then waits for.  One draft at a time where there is a wavefront for every 64 (draft, entry) pairs, and for one
  // draft, which has no other to share with; two wavefronts to a long list where there are two for every pair of drafts.
  // Kernel us (whole words and a wavefront a list, pairs everywhere, now): K = 2, a list of 2000, 256 rows 25.7, 30.7, 19.2;
  // K = 4, 660, 4 rows 19.2, 17.8, 13.6, 4096 rows 97.6, 76.2, 65.2; K = 3, 20, 4 rows 4.72, 5.25, 4.80; K = 1, 50, 4 rows 4.67, 4.92,
  // 4.77.  (As run-time choices in one kernel they cost others 3 to 5 %; halves of a list of 50 are one half and nothing, K = 4
  // 18.9 -> 23.0 at 4096 rows.)
  constexpr int kWaves = kBlock / 64;
  const bool one_list = p.draft_stride_k == 0 && p.temp_draft == nullptr;
  const bool single = !whole && (p.K == 1 || (long long)p.K * ((p.Md + 63) / 64) + ((long long)p.K * p.Mt + 63) / 64 <= kWaves);
  const bool halves = !whole && one_list && p.Md > 64 && (p.K + 1) / 2 * 2 <= kWaves;
  auto *kernel = topm_kernel<false, false, false, kPairs>;
  if (single) kernel = probs ? topm_kernel<true, false, false, kSingle> : topm_kernel<false, false, false, kSingle>;
  else if (halves) kernel = probs ? topm_kernel<true, false, false, kHalves> : topm_kernel<false, false, false, kHalves>;
  else if (probs) kernel = many ? (whole ? topm_kernel<true, true, true, kPairs> : topm_kernel<true, true, false, kPairs>)
                                : (whole ? topm_kernel<true, false, true, kPairs> : topm_kernel<true, false, false, kPairs>);
  else kernel = many ? (whole ? topm_kernel<false, true, true, kPairs> : topm_kernel<false, true, false, kPairs>)
                     : (whole ? topm_kernel<false, false, true, kPairs> : topm_kernel<false, false, false, kPairs>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)p.B), dim3(kBlock), lds, s, p);
  return hipGetLastError();
}

}  // namespace llc
