// The list matching lemma's lower bound on the matching probability (paper Theorem 1,
// eq. (1)), its relaxed form (the display that follows the theorem's proof sketch) and the total
// variation distance behind the two-party bound of the introduction, evaluated per row on the
// device so that a serving stack can choose the list size K from the distributions it has.
//
// Eq. (1) for K drafts drawn from p and a target q:
//   sum_j K / sum_i ( max{q_i/q_j, p_i/p_j} + (K - 1) q_i/q_j ).
// max{q_i/q_j, p_i/p_j} is q_i/q_j exactly when q_i/p_i >= q_j/p_j, so with the indices sorted by
// r = q/p the inner sum is (the q-mass from j on)/q_j + (the p-mass before j)/p_j + (K-1) Q/q_j:
// an order by r and running sums per row.  One workgroup does a whole row.  Two forms:
//
//  by buckets (rows of about 10^4 to 2 10^5 entries): no entry is moved more than once.  A sample of the row
//  gives splitters of ln r, a first pass counts the entries of every bucket between them, a second
//  forms the normalisers, a third writes every entry's two masses (rounded to fp32) and its place (the fp32
//  image of ln r) into its bucket's part of the workspace; then groups of up to 4096 entries are ordered in
//  LDS (a counting sort on a linear map of ln r inside every bucket, entries of one cell compared one by
//  one, or the whole group sorted where cells are long) and walked with running sums in fp64.  Entries that share a place may form a bucket of any size,
//  which needs no order.
//  by sorting (other rows, and a row in which a bucket came out larger than a group): four passes of a
//  stable 8-bit radix sort on the fp32 image of ln r, in which the two masses travel with their key
//  through two buffers in the workspace.
//
// Indices whose r agree to fp32 precision may come out in either order, which together with the rounding of
// the masses moves a result by a relative 2^-22 at most.
// Entries without mass on one side follow the limits: p_j = 0 or q_j = 0 gives term j = 0; as a
// summand i such an entry still counts with the mass it has on the other side.
#include "common.hpp"

#include <type_traits>

namespace llc {
namespace {

constexpr int kThreads = 512;         // eight wavefronts share a row
constexpr int kWaves = kThreads / 64;
constexpr int kRounds = 8;            // elements a thread holds per tile of the sort
constexpr int kTile = kThreads * kRounds;

template <typename E>
__device__ __forceinline__ float elem(const E *row, int i);
template <>
__device__ __forceinline__ float elem<float>(const float *row, int i) { return row[i]; }
template <>
__device__ __forceinline__ float elem<uint16_t>(const uint16_t *row, int i) {
  return __uint_as_float((uint32_t)row[i] << 16);
}

// Sum / maximum over the workgroup; every thread gets the result.  `scratch` holds a double per wavefront.
__device__ double block_sum(double v, double *scratch) {
  const int waves = blockDim.x >> 6;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
  __syncthreads();  // scratch may still be read from the previous reduction
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
  for (int w = 0; w < waves; ++w) r += scratch[w];  // a fixed order
  return r;
}
__device__ double block_max(double v, double *scratch) {
  const int waves = blockDim.x >> 6;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = fmax(v, __shfl_xor(v, d));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = scratch[0];
  for (int w = 1; w < waves; ++w) r = fmax(r, scratch[w]);
  return r;
}

// ln of the normalised mass of one entry.  Logits and log-weights: (x - m)/T - ln z with m the
// row's largest finite value; probabilities: ln x - ln z.  NaN, +inf (and for probabilities
// anything not > 0) carry no mass.
struct Side {
  double m, inv_t, ln_z;
  int probs;
  __device__ __forceinline__ double log_mass(float x) const {
    const double ninf = -__builtin_huge_val();
    if (probs) return (x > 0.0f && x < __builtin_huge_valf()) ? log((double)x) - ln_z : ninf;
    return (x < __builtin_huge_valf() && x > -__builtin_huge_valf()) ? ((double)x - m) * inv_t - ln_z : ninf;
  }
};

template <typename E>
__device__ Side normalise(const E *row, int V, int probs, float temp, double *scratch) {
  Side s;
  s.probs = probs;
  s.inv_t = 1.0 / (double)temp;
  double m = -__builtin_huge_val();
  if (!probs) {
    for (int i = threadIdx.x; i < V; i += kThreads) {
      const float x = elem<E>(row, i);
      if (x < __builtin_huge_valf()) m = fmax(m, (double)x);  // (NaN compares false)
    }
    m = block_max(m, scratch);
  }
  s.m = m;
  double z = 0.0;
  for (int i = threadIdx.x; i < V; i += kThreads) {
    const float x = elem<E>(row, i);
    if (probs) {
      if (x > 0.0f && x < __builtin_huge_valf()) z += (double)x;
    } else if (x < __builtin_huge_valf() && x > -__builtin_huge_valf()) {
      z += exp(((double)x - m) * s.inv_t);
    }
  }
  z = block_sum(z, scratch);
  s.ln_z = log(z);  // z == 0: no mass at all, every log_mass is -inf or NaN-free below
  return s;
}

// Where the bucket kernel tells the sorting one, launched behind it, that it left a row: behind the
// masses in the row's part of the workspace.
__device__ __forceinline__ int *flag_of(char *work, int V) { return reinterpret_cast<int *>(work + 16u * (size_t)V); }

// order-preserving image of a float in the unsigned integers
__device__ __forceinline__ uint32_t sort_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

template <typename E>
__global__ void __launch_bounds__(kThreads) lml_sort_kernel(const LmlParams p) {
  __shared__ double s_red[kWaves];
  __shared__ unsigned short s_cnt[kWaves][256];  // per wavefront and digit of a tile: counts, then starts
  __shared__ int s_goff[256];          // where a digit's run continues in the output
  __shared__ int s_tstart[256];        // where a digit's run starts inside the tile
  __shared__ int s_gbase[256];         // s_goff - s_tstart of the tile at hand
  __shared__ uint32_t st_key[kTile];   // the tile in digit order, on its way out
  __shared__ float2 st_mass[kTile];
  __shared__ double s_seg[kWaves][2];
  __shared__ int s_total[4][256];      // how often every digit of every pass occurs in the row
  // while the keys are made the staging area holds the counters: per pass, wavefront and digit
  static_assert(sizeof(st_mass) >= 4 * kWaves * 256 * sizeof(int), "the counters do not fit");
  int (*hist)[kWaves][256] = reinterpret_cast<int (*)[kWaves][256]>(st_mass);

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const long long b = p.row0 + blockIdx.x;
  const int V = p.V;
  const E *prow = reinterpret_cast<const E *>(p.draft) + b * p.draft_stride_b;
  const E *qrow = reinterpret_cast<const E *>(p.target) + b * p.target_stride_b;
  // A launch takes as many rows as the workspace has slots (two key buffers, then two buffers of
  // (p-mass, q-mass) each); the launches of one call follow each other on the stream, so the
  // workspace is as large as the workgroups that can be resident need, not as the batch.
  char *work = p.work + (size_t)blockIdx.x * 24u * (size_t)V;
  if (p.only_flagged && *flag_of(work, V) == 0) return;  // (uniform) the other kernel has done the row
  uint32_t *key_a = reinterpret_cast<uint32_t *>(work), *key_b = key_a + V;
  float2 *mass_a = reinterpret_cast<float2 *>(work + 8u * (size_t)V), *mass_b = mass_a + V;

  const Side sp = normalise<E>(prow, V, p.probs, p.temp_draft, s_red);
  const Side sq = normalise<E>(qrow, V, p.probs, p.temp_target, s_red);

  // ---- sort keys with the masses that travel with them, how often every digit occurs (the
  // arithmetic around them hides the counters' collisions), and the sums that need no order
  for (int j = tid; j < 4 * kWaves * 256; j += kThreads) (&hist[0][0][0])[j] = 0;
  __syncthreads();
  double tv = 0.0, relaxed[kLmlMaxK];
#pragma unroll
  for (int kk = 0; kk < kLmlMaxK; ++kk) relaxed[kk] = 0.0;
  for (int i = tid; i < V; i += kThreads) {
    const double lp = sp.log_mass(elem<E>(prow, i)), lq = sq.log_mass(elem<E>(qrow, i));
    const bool hp = lp > -__builtin_huge_val(), hq = lq > -__builtin_huge_val();
    float lr = -__builtin_huge_valf();           // no target mass (or none at all): sorts first
    if (hq) lr = hp ? (float)(lq - lp) : __builtin_huge_valf();
    const double pm = hp ? exp(lp) : 0.0, qm = hq ? exp(lq) : 0.0;
    const uint32_t key = sort_key(lr);
    key_a[i] = key;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) atomicAdd(&hist[pass][wv][(key >> (8 * pass)) & 255u], 1);
    mass_a[i] = make_float2((float)pm, (float)qm);
    tv += fabs(pm - qm);
    if (hp && hq) {
#pragma unroll
      for (int kk = 0; kk < kLmlMaxK; ++kk)
        if (kk < p.n_k) {  // q / (1 + q / (K p)) with one division
          const double kp = (double)p.k[kk] * pm;
          relaxed[kk] += kp * qm / (kp + qm);
        }
    }
  }
  tv = block_sum(tv, s_red);
#pragma unroll
  for (int kk = 0; kk < kLmlMaxK; ++kk)
    if (kk < p.n_k) {  // uniform
      const double r = block_sum(relaxed[kk], s_red);
      if (tid == 0 && p.relaxed != nullptr) p.relaxed[b * p.n_k + kk] = r;
    }
  if (tid == 0 && p.tv != nullptr) p.tv[b] = 0.5 * tv;
  // (block_sum has synchronised since the last counter was bumped)
  for (int j = tid; j < 4 * 256; j += kThreads) {
    int total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) total += hist[j >> 8][w][j & 255];
    s_total[j >> 8][j & 255] = total;
  }

  // ---- stable radix sort, 8 bits a pass.  A pass takes the row a tile of kTile entries at a
  // time: wavefront w holds the w-th part of the tile,
  // ranks them among the tile's entries of the same digit (within the wavefront by ballots, in
  // order; across wavefronts by a prefix over their counts), the tile is laid out in digit order
  // in LDS, and is written from there so that neighbouring threads write neighbouring addresses
  // (a digit's entries of one tile are contiguous in the output).
  uint32_t *kin = key_a, *kout = key_b;
  float2 *min_ = mass_a, *mout = mass_b;
#pragma unroll 1
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 8 * pass;
    __syncthreads();  // the previous pass's (or the key loop's) stores are done and visible
    if (wv == 0) {
      // lane l takes digits l, 64 + l, 128 + l, 192 + l: the start of every digit's run
      int carry = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int d = q * 64 + lane;
        const int total = s_total[pass][d];
        int incl = total;
#pragma unroll
        for (int dd = 1; dd < 64; dd <<= 1) {
          const int up = __shfl_up(incl, dd);
          if (lane >= dd) incl += up;
        }
        s_goff[d] = carry + incl - total;
        carry += __shfl(incl, 63);
      }
    }
    // (FULL: every entry of the tile exists, nothing is checked)
    auto sort_tile = [&](auto full_tag, const int t0) {
      constexpr bool FULL = decltype(full_tag)::value;
      __syncthreads();  // the tile before is on its way out of LDS; s_goff is in place
      for (int j = tid; j < kWaves * 256; j += kThreads) (&s_cnt[0][0])[j] = 0;
      __syncthreads();
      uint32_t key[kRounds];
      float2 mass[kRounds];
      int where[kRounds];  // rank among the wavefront's entries of the same digit
#pragma unroll
      for (int e = 0; e < kRounds; ++e) {
        const int i = t0 + wv * (64 * kRounds) + e * 64 + lane;
        const bool valid = FULL || i < V;
        key[e] = valid ? kin[i] : 0u;
        mass[e] = valid ? min_[i] : make_float2(0.0f, 0.0f);
      }
#pragma unroll
      for (int e = 0; e < kRounds; ++e) {
        const bool valid = FULL || t0 + wv * (64 * kRounds) + e * 64 + lane < V;
        const uint32_t d = (key[e] >> shift) & 255u;
        // lanes of this round with the same digit: bit by bit, keep those whose bit is like mine
        const unsigned long long live = __ballot(valid);
        uint32_t peers_lo = (uint32_t)live, peers_hi = (uint32_t)(live >> 32);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
          const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe((int)d, bit, 1);  // all ones if the bit is set
          const unsigned long long have = __ballot(mine != 0u);
          peers_lo &= ~((uint32_t)have ^ mine);
          peers_hi &= ~((uint32_t)(have >> 32) ^ mine);
        }
        where[e] = 0;
        if (valid) {
          const int rank = (int)__builtin_amdgcn_mbcnt_hi(peers_hi, __builtin_amdgcn_mbcnt_lo(peers_lo, 0u));
          const int seen = s_cnt[wv][d];
          if (rank == 0) s_cnt[wv][d] = (unsigned short)(seen + __popc(peers_lo) + __popc(peers_hi));
          where[e] = seen + rank;
        }
        __builtin_amdgcn_wave_barrier();
      }
      __syncthreads();
      if (wv == 0) {
        // per digit: every wavefront's start inside the digit's part of the tile, the part's start
        // inside the tile, and where the part goes in the output
        int carry = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int d = q * 64 + lane;
          int total = 0;
#pragma unroll
          for (int w = 0; w < kWaves; ++w) {
            const int c = s_cnt[w][d];
            s_cnt[w][d] = (unsigned short)total;
            total += c;
          }
          int incl = total;
#pragma unroll
          for (int dd = 1; dd < 64; dd <<= 1) {
            const int up = __shfl_up(incl, dd);
            if (lane >= dd) incl += up;
          }
          const int start = carry + incl - total;
          carry += __shfl(incl, 63);
          const int g = s_goff[d];
          s_tstart[d] = start;
          s_gbase[d] = g - start;
          s_goff[d] = g + total;
        }
      }
      __syncthreads();
#pragma unroll
      for (int e = 0; e < kRounds; ++e) {
        if (FULL || t0 + wv * (64 * kRounds) + e * 64 + lane < V) {
          const uint32_t d = (key[e] >> shift) & 255u;
          const int pos = s_tstart[d] + s_cnt[wv][d] + where[e];
          st_key[pos] = key[e];
          st_mass[pos] = mass[e];
        }
      }
      __syncthreads();
      const int n_tile = FULL ? kTile : min(kTile, V - t0);
#pragma unroll
      for (int e = 0; e < kRounds; ++e) {
        const int pos = e * kThreads + tid;
        if (FULL || pos < n_tile) {
          const uint32_t k = st_key[pos];
          const int g = s_gbase[(k >> shift) & 255u] + pos;
          kout[g] = k;
          mout[g] = st_mass[pos];
        }
      }
    };
    int t0 = 0;
#pragma unroll 1
    for (; t0 + kTile <= V; t0 += kTile) sort_tile(std::true_type(), t0);
    if (t0 < V) sort_tile(std::false_type(), t0);
    { uint32_t *t = kin; kin = kout; kout = t; }
    { float2 *t = min_; min_ = mout; mout = t; }
  }
  __syncthreads();
  // after four passes the sorted order is back in the first buffers (min_ == mass_a)

  // ---- running sums over the sorted order.  Wavefront w takes the w-th part of the row: first
  // every part's masses are added up, then every wavefront walks its part with the masses of the
  // parts before it as the carry.
  const int seg = (V + kWaves - 1) / kWaves;
  const int seg_begin = min(wv * seg, V), seg_end = min(seg_begin + seg, V);
  const float2 *mass = min_;
  double seg_p = 0.0, seg_q = 0.0;
  for (int j = seg_begin + lane; j < seg_end; j += 64) {
    const float2 m = mass[j];
    seg_p += (double)m.x;
    seg_q += (double)m.y;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) { seg_p += __shfl_xor(seg_p, d); seg_q += __shfl_xor(seg_q, d); }
  if (lane == 0) { s_seg[wv][0] = seg_p; s_seg[wv][1] = seg_q; }
  __syncthreads();
  double p_before = 0.0, q_before = 0.0, q_total = 0.0;
  for (int w = 0; w < kWaves; ++w) {
    if (w < wv) { p_before += s_seg[w][0]; q_before += s_seg[w][1]; }
    q_total += s_seg[w][1];
  }
  double acc[kLmlMaxK];
#pragma unroll
  for (int kk = 0; kk < kLmlMaxK; ++kk) acc[kk] = 0.0;
  for (int j0 = seg_begin; j0 < seg_end; j0 += 64) {
    const int j = j0 + lane;
    double pm = 0.0, qm = 0.0;
    if (j < seg_end) {
      const float2 m = mass[j];
      pm = (double)m.x;
      qm = (double)m.y;
    }
    double pin = pm, qin = qm;  // inclusive sums over the lanes of this tile
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const double up_p = __shfl_up(pin, d), up_q = __shfl_up(qin, d);
      if (lane >= d) { pin += up_p; qin += up_q; }
    }
    if (pm > 0.0 && qm > 0.0) {
      const double p_pre = p_before + (pin - pm);             // mass of p strictly before j
      const double q_suf = q_total - (q_before + (qin - qm));  // mass of q from j on
      // K / (q_suf/q_j + p_pre/p_j + (K - 1) Q/q_j), numerator and denominator times q_j
      const double common = q_suf + p_pre * (qm / pm);
#pragma unroll
      for (int kk = 0; kk < kLmlMaxK; ++kk)
        if (kk < p.n_k) {
          const double K = (double)p.k[kk];
          acc[kk] += K * qm / (common + (K - 1.0) * q_total);
        }
    }
    p_before += __shfl(pin, 63);
    q_before += __shfl(qin, 63);
  }
#pragma unroll
  for (int kk = 0; kk < kLmlMaxK; ++kk)
    if (kk < p.n_k) {  // uniform
      const double r = block_sum(acc[kk], s_red);
      if (tid == 0) p.bound[b * p.n_k + kk] = r;
    }
}

// ---- the form by buckets

// The rows it takes.  Shorter ones are quicker sorted (fewer fixed steps), from about 40 000 entries on if the
// inputs are bf16, whose many ties cost the ordering in LDS (us a call, buckets against sorting: fp32 8 192
// entries, 1 row 114 : 102, 12 288: 136 : 140, 32 000: 274 : 347; bf16 40 960, 64 rows 473 : 484, 512 rows 662 :
// 895, 128 256: 64 rows 1219 : 1555, 512 rows 1740 : 2885; 1024 rows x 128 256 fp32 3150 : 7515).
constexpr int kBucketMinV = 12288, kBucketMinVNarrow = 40960, kBucketMaxV = 1 << 18;
// The sample, and the buckets that its quantiles make.  A row is left to the sorting kernel if one bucket
// outgrows a group, and one such row costs the call a whole sort: with 127 buckets of 16 samples each the
// largest of a row's is about twice the average, which from kWideV entries on is too near a group's 4096.
// Those rows take twice the sample and 190 buckets (512 rows of 200 064: 5047 us : 2711, 64 of 262 144 5383 :
// 2109; 512 of 152 064, where it never happened, 1854 : 1904).
constexpr int kSamples = 2048, kQuantiles = 127;
constexpr int kWideV = 160000, kWideSamples = 4096, kWideQuantiles = 190;
constexpr int kGroup = 4096;          // entries of a tile, and of a group that is ordered in LDS
constexpr int kR = kGroup / kThreads; // what a thread holds of it
constexpr int kMaxBuckets = 255;
constexpr int kNoBucket = 255;        // of an entry that lacks mass on a side
// Entries of one cell up to which they are compared with each other; a group with a larger cell (equal ratios
// that the sample did not show, a far outlier in its bucket) is sorted whole.  512 rows of 128 256 bf16
// probabilities: 5.6 ms with comparing alone, 4.1 sorting from 256 on, 3.1 from 96, 3.2 from 32; fp32 rows
// without such a group 1.57 either way.
constexpr int kLongCell = 96;
constexpr float kFar = 512.0f;         // entries farther from the row's centre in ln r have no place
// An entry with both masses above zero in fp32 (2^-150 or more: ln >= -104) lies within this of the centre
// that the rows' largest entries make, in ln r: each mass is an entry's distance to its row's largest, less
// ln z, which is at most ln 2^18.  So an entry without a place, from a centre that is near that one, has no
// mass on one side, and which of such entries comes first is of no account.
constexpr double kReach = 120.0;

__device__ __forceinline__ float4 widen(const float4 &r) { return r; }
__device__ __forceinline__ float4 widen(const uint2 &r) {
  return make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xFFFF0000u), __uint_as_float(r.y << 16),
                     __uint_as_float(r.y & 0xFFFF0000u));
}
// Entries i..i+3 of a row; `fill` (which carries no mass) stands for those past the end.
template <typename E>
__device__ __forceinline__ float4 four(const E *row, int i, int V, float fill) {
  if (i + 3 < V) return widen(load_four(row + i));
  return make_float4(i < V ? elem<E>(row, i) : fill, i + 1 < V ? elem<E>(row, i + 1) : fill,
                     i + 2 < V ? elem<E>(row, i + 2) : fill, fill);
}
__device__ __forceinline__ float at(const float4 &v, int j) { return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w; }

// Exclusive prefix sum over the workgroup; *total gets the sum.  `scratch` holds an element per wavefront.
template <typename N>
__device__ __forceinline__ N block_prefix(N v, N *scratch, N *total) {
  const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  N incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const N up = __shfl_up(incl, d);
    if (lane >= d) incl += up;
  }
  __syncthreads();  // scratch may still be read from the previous call
  if (lane == 63) scratch[threadIdx.x >> 6] = incl;
  __syncthreads();
  N before = N(0), sum = N(0);
  for (int w = 0; w < waves; ++w) {
    if (w == (int)(threadIdx.x >> 6)) before = sum;
    sum += scratch[w];
  }
  *total = sum;
  return before + incl - v;
}

// A value that is the same in all lanes, held in scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) { return __int_as_float(uniform(__float_as_int(v))); }
__device__ __forceinline__ double uniform(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)uniform((int)(uint32_t)b), hi = (uint32_t)uniform((int)(uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The same for two sums at once, in place.
__device__ __forceinline__ void block_prefix2(double &a, double &b, double *scratch_a, double *scratch_b, double *total_a,
                                              double *total_b) {
  const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  double ia = a, ib = b;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double ua = __shfl_up(ia, d), ub = __shfl_up(ib, d);
    if (lane >= d) { ia += ua; ib += ub; }
  }
  __syncthreads();
  if (lane == 63) { scratch_a[threadIdx.x >> 6] = ia; scratch_b[threadIdx.x >> 6] = ib; }
  __syncthreads();
  double before_a = 0.0, before_b = 0.0, sum_a = 0.0, sum_b = 0.0;
  for (int w = 0; w < waves; ++w) {
    if (w == (int)(threadIdx.x >> 6)) { before_a = sum_a; before_b = sum_b; }
    sum_a += scratch_a[w];
    sum_b += scratch_b[w];
  }
  *total_a = sum_a;
  *total_b = sum_b;
  a = before_a + ia - a;
  b = before_b + ib - b;
}

// 1 / x to about an ulp, for normal x: the hardware's estimate and two Newton steps (the general fp64
// division's scaling and fix-up instructions are what an entry's time went to).
__device__ __forceinline__ double reciprocal(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// The place of an entry in the order: the fp32 image of ln r = ln(q/p) less the row's centre, as a whole
// number that orders as it does (the normalisers move all entries alike and are left out, so that the places
// are known before they are; from a centre near the one they make, the image has the digits that one of the
// normalised ln r has).  Evaluated twice per entry, by the same instructions.
template <bool PROBS>
struct Placer {
  double itp, itq, center;
  __device__ __forceinline__ bool mass(float x) const {
    return x < __builtin_huge_valf() && (PROBS ? x > 0.0f : x > -__builtin_huge_valf());
  }
  __device__ __forceinline__ double log_ratio(float xp, float xq) const {
    if (!PROBS) return __builtin_fma((double)xq, itq, -((double)xp * itp));
    // ln(a/b) = 2 artanh((a - b) / (a + b)) of the mantissas, brought within a factor of 1.42 of each other (the
    // argument is below 0.172: what follows the 13th power is below 2e-12 of the sum), plus the exponents
    double a = __builtin_amdgcn_frexp_mant((double)xq), b = __builtin_amdgcn_frexp_mant((double)xp);
    int e = __builtin_amdgcn_frexp_exp((double)xq) - __builtin_amdgcn_frexp_exp((double)xp);
    if (a > 1.4143 * b) { a *= 0.5; ++e; }
    if (b > 1.4143 * a) { b *= 0.5; --e; }
    const double s = (a - b) * reciprocal(a + b), z = s * s;
    double t = 2.0 / 13.0;
    t = __builtin_fma(t, z, 2.0 / 11.0);
    t = __builtin_fma(t, z, 2.0 / 9.0);
    t = __builtin_fma(t, z, 2.0 / 7.0);
    t = __builtin_fma(t, z, 2.0 / 5.0);
    t = __builtin_fma(t, z, 2.0 / 3.0);
    t = __builtin_fma(t, z, 2.0);
    return __builtin_fma(t, s, 0.6931471805599453 * (double)e);
  }
  // (rounded to 2^-36 first: equal ratios of different entries, of which inputs of few bits have many, differ by
  // fp64's rounding, which the image of a small distance would show)
  __device__ __forceinline__ float distance(float xp, float xq) const {
    constexpr double kStep = 0x1.8p16;  // the last of its 53 bits is worth 2^-36
    return (float)(((log_ratio(xp, xq) - center) + kStep) - kStep);
  }
};
__device__ __forceinline__ int place_of(float distance) {
  const int b = __float_as_int(distance);
  return b ^ ((b >> 31) & 0x7FFFFFFF);
}
__device__ __forceinline__ float distance_of(int place) { return __int_as_float(place ^ ((place >> 31) & 0x7FFFFFFF)); }

// An entry on its way to its bucket.
struct Entry {
  float p, q;
  int place;
};

// The last bucket whose splitter is not above `place` (split[0] stands for minus infinity).
__device__ __forceinline__ int bucket_of(const int *split, int nb, int place) {
  int b = 0;
#pragma unroll
  for (int step = 128; step >= 1; step >>= 1)
    if (b + step < nb && split[b + step] <= place) b += step;
  return b;
}

// e^x for x <= 0 or so (what is below -800 comes out as 0) to about an ulp: x = n ln 2 + f, the Taylor
// series of e^f to its 13th term (|f| <= ln(2) / 2: the next one is below 2^-57), times 2^n.  No branch,
// so that an entry's two exponentials run side by side.
__device__ __forceinline__ double exp_of_negative(double x) {
  x = fmax(x, -800.0);
  const double n = __builtin_rint(x * 1.4426950408889634);
  double f = fma(n, -0x1.62e42fefa39efp-1, x);  // ln 2 to 53 bits ...
  f = fma(n, -0x1.abc9e3b39803fp-56, f);        // ... and the next 53
  double s = 1.0 / 6227020800.0;
  s = fma(s, f, 1.0 / 479001600.0);
  s = fma(s, f, 1.0 / 39916800.0);
  s = fma(s, f, 1.0 / 3628800.0);
  s = fma(s, f, 1.0 / 362880.0);
  s = fma(s, f, 1.0 / 40320.0);
  s = fma(s, f, 1.0 / 5040.0);
  s = fma(s, f, 1.0 / 720.0);
  s = fma(s, f, 1.0 / 120.0);
  s = fma(s, f, 1.0 / 24.0);
  s = fma(s, f, 1.0 / 6.0);
  s = fma(s, f, 0.5);
  s = fma(s, f, 1.0);
  s = fma(s, f, 1.0);
  return __builtin_amdgcn_ldexp(s, (int)n);
}

// acc[n] += k[n] pq / (base + (k[n] - off) slope): two quotients per reciprocal (the product of two
// denominators has to be a normal number: each is 2^-450 or more in both uses).  List sizes beyond n_k are 1.
template <int PAIRS>
__device__ __forceinline__ void add_quotients(double (&acc)[2 * PAIRS], const LmlParams &p, double pq, double base,
                                              double off, double slope) {
#pragma unroll
  for (int n = 0; n < 2 * PAIRS; n += 2) {
    const double k0 = p.kd[n], d0 = fma(k0 - off, slope, base);
    const double k1 = p.kd[n + 1], d1 = fma(k1 - off, slope, base);
    const double t = pq * reciprocal(d0 * d1);
    acc[n] = fma(k0 * t, d1, acc[n]);
    acc[n + 1] = fma(k1 * t, d0, acc[n + 1]);
  }
}

// Place and number of a group's entry as one key.
__device__ __forceinline__ unsigned long long key_of(int place, int number) {
  return ((unsigned long long)((uint32_t)place ^ 0x80000000u) << 32) | (uint32_t)number;
}

// Sorts the first n of the keys in LDS (a bitonic network; thread t holds entries t kR .. t kR + kR - 1, those
// beyond n count as the largest) and says where each came to lie: s_to[number in the key] = position.
__device__ __forceinline__ void sort_group(unsigned long long *s_key, int *s_to, const int n) {
  const int me = threadIdx.x;
  unsigned long long key[kR];
#pragma unroll
  for (int e = 0; e < kR; ++e) key[e] = me * kR + e < n ? s_key[me * kR + e] : ~0ull;
  __syncthreads();
  // (the smaller one stays where the index has no bit of `d`, the other way round in every second run of `size`)
  auto keep = [](unsigned long long &mine, const unsigned long long other, const bool smaller) {
    if ((other < mine) == smaller) mine = other;
  };
#pragma unroll 1
  for (int size = 2; size < 2 * n; size <<= 1) {
    const bool up = (me & (size / kR)) == 0;  // (of runs of kR entries and more)
#pragma unroll 1
    for (int d = size >> 1; d >= 64 * kR; d >>= 1) {  // other wavefronts' entries
      const bool smaller = ((me & (d / kR)) == 0) == up;
#pragma unroll
      for (int e = 0; e < kR; ++e) s_key[e * kThreads + me] = key[e];
      __syncthreads();
#pragma unroll
      for (int e = 0; e < kR; ++e) keep(key[e], s_key[e * kThreads + (me ^ (d / kR))], smaller);
      __syncthreads();
    }
#pragma unroll 1
    for (int d = min(size >> 1, 32 * kR); d >= kR; d >>= 1) {  // other lanes'
      const bool smaller = ((me & (d / kR)) == 0) == up;
#pragma unroll
      for (int e = 0; e < kR; ++e) keep(key[e], __shfl_xor(key[e], d / kR), smaller);
    }
#pragma unroll
    for (int d = kR / 2; d >= 1; d >>= 1)  // the thread's own
      if (d < size) {
#pragma unroll
        for (int e = 0; e < kR; ++e)
          if ((e & d) == 0) {
            const bool rising = size < kR ? (e & size) == 0 : up;
            const unsigned long long a = key[e], b = key[e | d];
            const bool swap = (b < a) == rising;
            key[e] = swap ? b : a;
            key[e | d] = swap ? a : b;
          }
      }
  }
#pragma unroll
  for (int e = 0; e < kR; ++e)
    if (me * kR + e < n) s_to[(uint32_t)key[e]] = me * kR + e;
  __syncthreads();
}

// LDS index of entry j where threads read kR neighbouring entries each (spreads them over the banks).
__device__ __forceinline__ int padded(int j) { return j + j / kR; }

// One workgroup per row, two per CU.  What bounds it: instruction issue and the latency of LDS between
// barriers, not memory: the row is read three times and a bucket byte, the masses and the place are
// written and read once (by the memory counters 56 bytes an entry of 8 input bytes, 159 in the sorting
// form).  Of the 1.6 ms that two rows of 128 256 take on a CU (four list sizes) the sample has 0.07, the first pass 0.2, the normalisers 0.13, the
// third pass 0.4 (positions 0.22, masses 0.16), the groups 0.8 (cells and their starts 0.45, the order inside
// cells 0.17, running sums 0.15, terms 0.05).  An order by the exact ratio, general divisions and a branch
// around every exponential made it 6.3 ms for 1024 rows; as it is, 3.13.
// All sums run in an order that does not depend on how the wavefronts interleave: entries keep the row's
// order within a bucket, and within a group they are ordered by their places, then as they lie in the bucket.
// PAIRS: room for that many pairs of list sizes (more than four sizes do not fit 128 registers with the
// rest, so that variant runs one workgroup per CU).
template <typename E, bool PROBS, int PAIRS>
__global__ void __launch_bounds__(kThreads, PAIRS > 2 ? 2 : 4) lml_bucket_kernel(const LmlParams p) {
  __shared__ double s_red[kWaves], s_red2[kWaves];
  __shared__ int s_redi[kWaves];
  __shared__ int s_split[kMaxBuckets + 1];  // bucket b holds the places from s_split[b] up to s_split[b + 1]
  __shared__ int s_off[kMaxBuckets + 2];    // where bucket b starts in the workspace
  __shared__ int s_next[kMaxBuckets + 1];   // how far it has been written; before that its count
  __shared__ int s_start[kMaxBuckets + 1];  // where a bucket's entries start inside the tile at hand
  __shared__ float s_scale[kMaxBuckets];    // cells of a bucket per unit of ln r
  __shared__ float2 s_mass[kGroup + kThreads];
  __shared__ int s_cell[kGroup + kThreads + 1];  // groups: entries of a cell, then where the cell starts
  __shared__ int s_info[2];
  // the cells' room also serves the sample, and the third pass: an entry's bucket in the tile's order, and
  // per wavefront and bucket the entries of the tile
  int *s_sample = s_cell;
  unsigned long long *s_key = reinterpret_cast<unsigned long long *>(s_mass);  // groups: the entries' keys
  unsigned char *s_tag = reinterpret_cast<unsigned char *>(s_cell);
  unsigned short(*s_cnt)[kMaxBuckets + 1] = reinterpret_cast<unsigned short(*)[kMaxBuckets + 1]>(s_cell + kGroup / 4);
  static_assert(kWideSamples <= kGroup && kGroup + kWaves * (kMaxBuckets + 1) * 2 <= (int)sizeof(s_cell), "sizes");

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const long long b_row = p.row0 + blockIdx.x;
  const int V = p.V;
  const E *prow = reinterpret_cast<const E *>(p.draft) + b_row * p.draft_stride_b;
  const E *qrow = reinterpret_cast<const E *>(p.target) + b_row * p.target_stride_b;
  char *work = p.work + (size_t)blockIdx.x * 24u * (size_t)V;
  Entry *bucketed = reinterpret_cast<Entry *>(work);
  unsigned char *ids = reinterpret_cast<unsigned char *>(work + 12u * (size_t)V);
  const float none = PROBS ? 0.0f : -__builtin_huge_valf();
  const float ninf = -__builtin_huge_valf();

  Placer<PROBS> pl;
  pl.itp = 1.0 / (double)p.temp_draft;
  pl.itq = 1.0 / (double)p.temp_target;

  // ---- splitters: every bucket gets about V / kQuantiles entries, at least 1024, by the sample's quantiles, and
  // places that the sample holds several times get a bucket of their own (inputs of few bits have many ties)
  static_assert(kBucketMinV > kGroup, "a row that is a single group would need none");
  int nb = 1;
  float mp, mq, left_most, right_most;  // the largest entries, the smallest and largest distance
  pl.center = 0.0;
  auto pick_splitters = [&](auto wide, const bool first) {
    constexpr int kPicks = wide.value ? kWideSamples : kSamples, kMost = wide.value ? kWideQuantiles : kQuantiles;
    constexpr int kPer = kPicks / kThreads, kMany = wide.value ? 128 : 32;
    static_assert(kMost + 2 * (kPicks / kMany) <= kMaxBuckets, "too many splitters");
    float xp[kPer], xq[kPer];
    int me = tid;
    asm volatile("" : "+v"(me));  // (or the addresses are formed before the loop, for both sizes, and spill)
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const unsigned j = (unsigned)(e * kThreads + me), jitter = j * 0x9E3779B9u;
      const int i = (int)(((unsigned long long)j * (unsigned)V + (((unsigned long long)jitter * (unsigned)V) >> 32)) / kPicks);
      xp[e] = elem<E>(prow, i);
      xq[e] = elem<E>(qrow, i);
    }
    // the centre, at first: where an entry would lie that is the sample's largest on both sides (not a median:
    // most of a row may be masked by a low value); probabilities of any size lie within 193 of 0
    if (!PROBS && first) {
      mp = mq = ninf;
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        if (pl.mass(xp[e])) mp = fmaxf(mp, xp[e]);
        if (pl.mass(xq[e])) mq = fmaxf(mq, xq[e]);
      }
      mp = (float)block_max((double)mp, s_red);
      mq = (float)block_max((double)mq, s_red);
      if (mp > ninf && mq > ninf) pl.center = uniform(pl.log_ratio(mp, mq));
    }
    int valid = 0, n_valid;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const float d = pl.mass(xp[e]) && pl.mass(xq[e]) ? pl.distance(xp[e], xq[e]) : kFar;
      s_sample[e * kThreads + tid] = fabsf(d) < kFar ? place_of(d) : 0x7FFFFFFF;
      valid += fabsf(d) < kFar ? 1 : 0;
    }
    block_prefix(valid, s_redi, &n_valid);
    for (int size = 2; size <= kPicks; size <<= 1)
      for (int stride = size >> 1; stride >= 1; stride >>= 1) {
        __syncthreads();
        for (int t = tid; t < kPicks / 2; t += kThreads) {
          const int lo = 2 * t - (t & (stride - 1)), hi = lo + stride;
          const int x = s_sample[lo], y = s_sample[hi];
          if ((x > y) == ((lo & size) == 0)) { s_sample[lo] = y; s_sample[hi] = x; }
        }
      }
    __syncthreads();
    if (n_valid == 0) return;  // uniform
    const int entries = (int)((long long)V * n_valid / kPicks);
    const int want = max(1, min(kMost, (entries + 1023) / 1024));
    // a run of `many` equal places or more in the sample is two splitters (the place is a bucket), a shorter
    // one is one, if a quantile falls into it; `many` is the least that keeps to the buckets there are
    int emit[kPer], total, before = 0;
#pragma unroll 1
    for (int many = 4; many <= kMany; many *= 2) {
      int mine = 0;
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const int j = tid * kPer + e, v = s_sample[j];
        emit[e] = 0;
        if (j < n_valid && (j == 0 || s_sample[j - 1] != v)) {
          int last = j;
          while (last + 1 < n_valid && last + 1 < j + many && s_sample[last + 1] == v) ++last;
          if (last + 1 == j + many) emit[e] = 2;
          else if (j > 0 && (long long)last * want / n_valid != (long long)(j - 1) * want / n_valid) emit[e] = 1;
        }
        mine += emit[e];
      }
      before = block_prefix(mine, s_redi, &total);
      if (total < kMaxBuckets) break;  // uniform
    }
    nb = 1 + min(total, kMaxBuckets - 1);
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const int v = s_sample[tid * kPer + e];
      for (int c = 0; c < emit[e]; ++c, ++before)
        if (1 + before < nb) s_split[1 + before] = v + c;
    }
  };
#pragma unroll 1
  for (int attempt = 0;; ++attempt) {
    nb = 1;
    if (V > kWideV) pick_splitters(std::true_type(), attempt == 0);
    else pick_splitters(std::false_type(), attempt == 0);
    for (int j = tid; j <= kMaxBuckets; j += kThreads) s_next[j] = 0;
    if (tid == 0) { s_split[0] = (int)0x80000000; s_info[0] = 0; }
    __syncthreads();

    // ---- first pass: the rows' largest entries, and every entry's bucket and the buckets' counts
    mp = mq = ninf;
    left_most = kFar;
    right_most = -kFar;
    for (int i = tid * 4; i < V; i += kThreads * 4) {
      const float4 xp4 = four<E>(prow, i, V, none), xq4 = four<E>(qrow, i, V, none);
      uint32_t packed = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float xp = at(xp4, j), xq = at(xq4, j);
        const bool hp = pl.mass(xp), hq = pl.mass(xq);
        if (hp) mp = fmaxf(mp, xp);
        if (hq) mq = fmaxf(mq, xq);
        int b = kNoBucket;
        if (hp && hq) {
          const float d = pl.distance(xp, xq);
          if (fabsf(d) < kFar) {
            left_most = fminf(left_most, d);
            right_most = fmaxf(right_most, d);
            b = nb > 1 ? bucket_of(s_split, nb, place_of(d)) : 0;
            atomicAdd(&s_next[b], 1);
          }
        }
        packed |= (uint32_t)b << (8 * j);
      }
      if (i + 3 < V) {
        *reinterpret_cast<uint32_t *>(ids + i) = packed;
      } else {
        for (int j = 0; i + j < V; ++j) ids[i + j] = (unsigned char)(packed >> (8 * j));
      }
    }
    if (PROBS) break;
    // the centre that the rows' largest entries make: if the sample's was too far from it for kReach, once more
    // from there
    mp = (float)block_max((double)mp, s_red);
    mq = (float)block_max((double)mq, s_red);
    if (!(mp > ninf && mq > ninf)) break;  // (uniform, as the next) a side without mass
    const double center = uniform(pl.log_ratio(mp, mq));
    if (attempt > 0 || fabs(center - pl.center) < (double)kFar - kReach) break;
    pl.center = center;
  }
  nb = uniform(nb);
  // (two places can be farther apart than an int reaches; one more than a place is one)
  auto of_one_place = [&](const int b) { return b >= 1 && b + 1 < nb && s_split[b + 1] <= s_split[b] + 1; };
  Side sp, sq;
  sp.probs = sq.probs = PROBS ? 1 : 0;
  sp.inv_t = pl.itp;
  sq.inv_t = pl.itq;
  // the outer buckets' outer ends: those of the row, or two e-folds from the nearest splitter (an outlier
  // must not stretch a bucket so far that its other entries share a cell)
  float left_edge = -(float)block_max(-(double)left_most, s_red), right_edge = (float)block_max((double)right_most, s_red);
  if (nb > 1) {
    left_edge = fmaxf(left_edge, distance_of(s_split[1]) - 2.0f);
    right_edge = fminf(right_edge, distance_of(s_split[nb - 1]) + 2.0f);
  }
  left_edge = uniform(left_edge);
  sp.m = PROBS ? 0.0 : uniform((double)mp);
  sq.m = PROBS ? 0.0 : uniform((double)mq);
  __syncthreads();
  {
    const int mine = tid < nb ? s_next[tid] : 0;
    int total;
    const int off = block_prefix(mine, s_redi, &total);
    if (tid < nb) {
      s_off[tid] = off;
      s_next[tid] = off;
      if (mine > kGroup && !of_one_place(tid)) s_info[0] = 1;
      // (the outer buckets have no outer splitter: the sample's end stands for it)
      const float left = tid > 0 ? distance_of(s_split[tid]) : left_edge;
      const float right = tid + 1 < nb ? distance_of(s_split[tid + 1]) : right_edge;
      s_scale[tid] = right > left ? (float)mine / (right - left) : 0.0f;
    }
    if (tid == 0) s_off[nb] = total;
  }
  __syncthreads();
  const bool leave = s_info[0] != 0;
  if (tid == 0) *flag_of(work, V) = leave ? 1 : 0;
  if (leave) return;  // (uniform) a bucket larger than a group: the row is the sorting kernel's

  // ---- second pass: the normalisers
  {
    double zp = 0.0, zq = 0.0;
    for (int i = tid * 4; i < V; i += kThreads * 4) {
      const float4 xp4 = four<E>(prow, i, V, none), xq4 = four<E>(qrow, i, V, none);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float xp = at(xp4, j), xq = at(xq4, j);
        if (PROBS) {
          zp += pl.mass(xp) ? (double)xp : 0.0;
          zq += pl.mass(xq) ? (double)xq : 0.0;
        } else {
          zp += exp_of_negative(pl.mass(xp) ? ((double)xp - sp.m) * sp.inv_t : -__builtin_huge_val());
          zq += exp_of_negative(pl.mass(xq) ? ((double)xq - sq.m) * sq.inv_t : -__builtin_huge_val());
        }
      }
    }
    sp.ln_z = log(block_sum(zp, s_red));
    sq.ln_z = log(block_sum(zq, s_red));
  }

  // ---- third pass: every tile is laid out by bucket in LDS (its entries' positions follow from the bucket
  // bytes alone), and taken from there: masses, the sums that need no order, and the masses to their
  // bucket, neighbouring threads to neighbouring addresses
  double tv = 0.0, p_first = 0.0, q_total = 0.0, sums[2 * PAIRS];
#pragma unroll
  for (int n = 0; n < 2 * PAIRS; ++n) sums[n] = 0.0;
#pragma unroll 1
  for (int t0 = 0; t0 < V; t0 += kGroup) {
    const int n_tile = min(kGroup, V - t0);
    const int base = t0 + wv * (64 * kR) + lane;  // wavefront w holds the w-th part of the tile
    float2 x[kR];
    int id[kR], where[kR];
#pragma unroll
    for (int e = 0; e < kR; ++e) {
      const int i = base + e * 64;
      id[e] = i < V ? (int)ids[i] : -1;
      x[e] = i < V ? make_float2(elem<E>(prow, i), elem<E>(qrow, i)) : make_float2(0.0f, 0.0f);
    }
    __syncthreads();  // the tile before is done with
    for (int j = tid; j < kWaves * (kMaxBuckets + 1) / 2; j += kThreads) reinterpret_cast<int *>(&s_cnt[0][0])[j] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kR; ++e) {
      // lanes of this round with the same bucket: bit by bit, keep those whose bit is like mine
      const unsigned long long live = __ballot(id[e] >= 0);
      uint32_t peers_lo = (uint32_t)live, peers_hi = (uint32_t)(live >> 32);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe(id[e], bit, 1);  // all ones if the bit is set
        const unsigned long long have = __ballot(mine != 0u);
        peers_lo &= ~((uint32_t)have ^ mine);
        peers_hi &= ~((uint32_t)(have >> 32) ^ mine);
      }
      where[e] = 0;
      if (id[e] >= 0) {
        const int rank = (int)__builtin_amdgcn_mbcnt_hi(peers_hi, __builtin_amdgcn_mbcnt_lo(peers_lo, 0u));
        const int seen = s_cnt[wv][id[e]];
        if (rank == 0) s_cnt[wv][id[e]] = (unsigned short)(seen + __popc(peers_lo) + __popc(peers_hi));
        where[e] = seen + rank;
      }
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {
      int mine = 0, all;
      if (tid <= kMaxBuckets) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          const int c = s_cnt[w][tid];
          s_cnt[w][tid] = (unsigned short)mine;
          mine += c;
        }
      }
      const int start = block_prefix(mine, s_redi, &all);
      if (tid <= kMaxBuckets) s_start[tid] = start;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kR; ++e)
      if (id[e] >= 0) {
        const int pos = s_start[id[e]] + s_cnt[wv][id[e]] + where[e];
        s_mass[pos] = x[e];
        s_tag[pos] = (unsigned char)id[e];
      }
    __syncthreads();
#pragma unroll 1
    for (int pos = tid; pos < n_tile; pos += kThreads) {
      const float2 in = s_mass[pos];
      const int b = s_tag[pos];
      const double lp = sp.log_mass(in.x), lq = sq.log_mass(in.y);
      const bool hp = lp > -__builtin_huge_val(), hq = lq > -__builtin_huge_val();
      double pm = exp_of_negative(lp), qm = exp_of_negative(lq);  // (-inf: no mass)
      const float2 m = make_float2((float)pm, (float)qm);
      tv += fabs(pm - qm);
      q_total += (double)m.y;
      // ratio 0, or near it: before all others (an entry without a bucket that has the larger ratio has no
      // p-mass in fp32)
      if (b == kNoBucket) p_first += (double)m.x;
      if (b != kNoBucket) {
        const int g = s_next[b] + (pos - s_start[b]);
        if (g < s_off[b + 1]) {  // (always; a bucket is never written past its end)
          bucketed[g] = Entry{m.x, m.y, place_of(pl.distance(in.x, in.y))};
        }
      }
      if (hp && hq && p.relaxed != nullptr) {  // q / (1 + q / (K p)) = K p q / (K p + q)
        // (where the product nears the smallest numbers, both are taken relative to the larger one: its
        // denominators, and their product, are then at least 1/4)
        int scale = 0;
        if (pm * qm < 0x1p-900) {
          scale = __builtin_amdgcn_frexp_exp(fmax(pm, qm));
          pm = __builtin_amdgcn_ldexp(pm, -scale);
          qm = __builtin_amdgcn_ldexp(qm, -scale);
        }
        const double pq = __builtin_amdgcn_ldexp(pm * qm, scale);
        if (pq > 0.0) add_quotients<PAIRS>(sums, p, pq, qm, 0.0, pm);
      }
    }
    __syncthreads();
    if (tid < nb) {
      int here = (tid < kMaxBuckets ? s_start[tid + 1] : n_tile) - s_start[tid];
      s_next[tid] += here;
    }
  }
  tv = block_sum(tv, s_red);
  if (tid == 0 && p.tv != nullptr) p.tv[b_row] = 0.5 * tv;
#pragma unroll
  for (int n = 0; n < 2 * PAIRS; ++n)
    if (n < p.n_k) {  // uniform
      if (p.relaxed != nullptr) {
        const double r = block_sum(sums[n], s_red);
        if (tid == 0) p.relaxed[b_row * p.n_k + n] = r;
      }
      sums[n] = 0.0;
    }
  q_total = uniform(block_sum(q_total, s_red));

  // ---- the groups in order, with the masses of what came before
  double p_before = uniform(block_sum(p_first, s_red)), q_before = 0.0;
  // K q / (D(r) + (K - 1) Q) of one entry, D(r) the sum of max(q_i, r p_i) over the row: the q-mass from
  // the entry on plus r times the p-mass before it (numerator and denominator times p)
  auto add_term = [&](const float2 m, const double pb, const double qb) {
    if (!(m.x > 0.0f && m.y > 0.0f)) return;
    const double pm = (double)m.x, qm = (double)m.y;
    double one = 1.0;
    asm volatile("" : "+s"(one));  // (or the list sizes less one live, and spill, across the whole loop)
    add_quotients<PAIRS>(sums, p, pm * qm, fma(q_total - qb, pm, pb * qm), one, q_total * pm);
  };
  for (int b0 = 0, b1 = 0; b0 < nb; b0 = b1) {
    b1 = b0 + 1;
    const int first = uniform(s_off[b0]);
    int n = uniform(s_off[b1]) - first;
    const bool tied = n > kGroup;  // (only a bucket of one place can be)
    if (!tied) {
      while (b1 < nb && uniform(s_off[b1 + 1]) - first <= kGroup) ++b1;
      n = uniform(s_off[b1]) - first;
    }
    if (n == 0) continue;  // uniform
    double pg = 0.0, qg = 0.0;  // the group's masses
    int me = tid;
    asm volatile("" : "+v"(me));  // (or two dozen addresses formed from it live, and spill, across the whole loop)
    if (tied) {
      // one place: any order will do, so every entry counts as the first of them
#pragma unroll 1
      for (int i = me; i < n; i += kThreads) {
        const float2 m = make_float2(bucketed[first + i].p, bucketed[first + i].q);
        pg += (double)m.x;
        qg += (double)m.y;
        add_term(m, p_before, q_before);
      }
      p_before = uniform(p_before + block_sum(pg, s_red));
      q_before = uniform(q_before + block_sum(qg, s_red));
      continue;
    }
    // cells: bucket b's entries spread over as many cells as there are, linearly in ln r between its
    // splitters (so the map is monotone, which is all the order needs; one entry per cell on average)
    float2 mass[kR];
    int cell[kR], rank[kR], place[kR], top = 1;
    while (top * 2 < b1 - b0) top *= 2;
#pragma unroll
    for (int e = 0; e < kR; ++e) {
      const int i = e * kThreads + me;
      const Entry in = bucketed[first + min(i, n - 1)];
      mass[e] = make_float2(in.p, in.q);
      place[e] = in.place;
    }
    __syncthreads();  // the group before is done with
    if (me == 0) s_info[1] = 0;
    for (int c = me; c < padded(n) + 1; c += kThreads) s_cell[c] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kR; ++e) {
      const int i = e * kThreads + me;
      int b = b0;  // the bucket it lies in
      for (int step = top; step >= 1; step >>= 1)
        if (b + step < b1 && s_off[b + step] - first <= i) b += step;
      const int low = s_split[b], high = b + 1 < nb ? s_split[b + 1] - 1 : 0x7FFFFFFE;
      const int lo = s_off[b] - first, cnt = s_off[b + 1] - s_off[b];
      const float f = (distance_of(place[e]) - (b > 0 ? distance_of(low) : left_edge)) * s_scale[b];
      const int spread = lo + (int)fminf(fmaxf(f, 0.0f), (float)(cnt - 1));
      // (in a bucket of one place the entries stay as they lie)
      cell[e] = i < n ? (high > low || b == 0 ? spread : i) : -1;
      rank[e] = i < n ? atomicAdd(&s_cell[padded(cell[e])], 1) : 0;
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    {
      // where every cell starts; thread t takes cells t kR .. t kR + kR - 1
      int c[kR], sum = 0, total;
#pragma unroll
      for (int e = 0; e < kR; ++e) {
        const int j = me * kR + e;
        c[e] = j < n ? s_cell[padded(j)] : 0;
        sum += c[e];
      }
      int start = block_prefix(sum, s_redi, &total);
#pragma unroll
      for (int e = 0; e < kR; ++e) {
        const int j = me * kR + e;
        if (j < n) s_cell[padded(j)] = start;
        start += c[e];
      }
      if (me == 0) s_cell[padded(n)] = n;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kR; ++e)
      if (cell[e] >= 0) {
        rank[e] += s_cell[padded(cell[e])];
        s_key[rank[e]] = key_of(place[e], e * kThreads + me);
      }
    if (me < 4) s_key[n + me] = ~0ull;
    int longest = 0;
#pragma unroll
    for (int e = 0; e < kR; ++e) {
      const int from = cell[e] >= 0 ? s_cell[padded(cell[e])] : n;
      const int len = cell[e] >= 0 ? s_cell[padded(cell[e] + 1)] - from : 0;
      longest = max(longest, len > 1 ? len : 0);
      cell[e] = from;
      rank[e] = from;
    }
    if (longest > kLongCell) s_info[1] = 1;
    __syncthreads();
    // entries of one cell among themselves: by place, then as they lie in the bucket
    if (s_info[1] != 0) {  // (uniform)
      sort_group(s_key, s_cell, n);
#pragma unroll
      for (int e = 0; e < kR; ++e) rank[e] = e * kThreads + me < n ? s_cell[e * kThreads + me] : n;
    } else {
      // (the thread's entries side by side, four steps at a time: what lies behind a cell has larger keys and
      // counts for nothing, so only the longest cell of the wavefront ends the loop)
      for (int t = 0; __any(t < longest); t += 4) {
#pragma unroll
        for (int e = 0; e < kR; ++e) {
          const unsigned long long mine = key_of(place[e], e * kThreads + me);
          const unsigned long long *there = s_key + min(cell[e] + t, n);
#pragma unroll
          for (int u = 0; u < 4; ++u) rank[e] += there[u] < mine ? 1 : 0;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kR; ++e)
      if (e * kThreads + me < n) s_mass[padded(rank[e])] = mass[e];
    __syncthreads();
    {
      // running sums over the entries in order; thread t takes entries t kR .. t kR + kR - 1
      const int mine = me * kR;
#pragma unroll
      for (int e = 0; e < kR; ++e) {
        mass[e] = mine + e < n ? s_mass[padded(mine + e)] : make_float2(0.0f, 0.0f);
        pg += (double)mass[e].x;
        qg += (double)mass[e].y;
      }
      double p_sum, q_sum, pb = pg, qb = qg;
      block_prefix2(pb, qb, s_red, s_red2, &p_sum, &q_sum);
      pb += p_before;
      qb += q_before;
#pragma unroll
      for (int e = 0; e < kR; ++e) {
        add_term(mass[e], pb, qb);
        pb += (double)mass[e].x;
        qb += (double)mass[e].y;
        if (e % 2 == 1) __builtin_amdgcn_sched_barrier(0);  // (all at once does not fit the registers)
      }
      p_before = uniform(p_before + p_sum);
      q_before = uniform(q_before + q_sum);
    }
  }
#pragma unroll
  for (int n = 0; n < 2 * PAIRS; ++n)
    if (n < p.n_k) {  // uniform
      const double r = block_sum(sums[n], s_red);
      if (tid == 0) p.bound[b_row * p.n_k + n] = r;
    }
}

}  // namespace

hipError_t launch_lml(hipStream_t s, const LmlParams &params) {
  LmlParams p = params;
  const bool buckets = p.V >= (p.dtype == LLC_F32 ? kBucketMinV : kBucketMinVNarrow) && p.V <= kBucketMaxV;
  p.only_flagged = buckets ? 1 : 0;
  for (p.row0 = 0; p.row0 < p.B; p.row0 += p.slots) {
    const long long left = p.B - p.row0;
    const unsigned grid = (unsigned)(left < (long long)p.slots ? left : (long long)p.slots);
    const bool f32 = p.dtype == LLC_F32;
    if (buckets) {
#define LLC_LML(E, PROBS)                                                                                  \
  if (p.n_k <= 4) hipLaunchKernelGGL((lml_bucket_kernel<E, PROBS, 2>), dim3(grid), dim3(kThreads), 0, s, p); \
  else hipLaunchKernelGGL((lml_bucket_kernel<E, PROBS, 4>), dim3(grid), dim3(kThreads), 0, s, p);
      if (f32 && p.probs) { LLC_LML(float, true) }
      else if (f32) { LLC_LML(float, false) }
      else if (p.probs) { LLC_LML(uint16_t, true) }
      else { LLC_LML(uint16_t, false) }
#undef LLC_LML
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    // (behind the bucket kernel: the rows that it left, as a rule none)
    if (f32) hipLaunchKernelGGL(lml_sort_kernel<float>, dim3(grid), dim3(kThreads), 0, s, p);
    else hipLaunchKernelGGL(lml_sort_kernel<uint16_t>, dim3(grid), dim3(kThreads), 0, s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace llc
