// The list matching lemma's lower bound on the matching probability (paper Theorem 1,
// eq. (1)), its relaxed form (the display that follows the theorem's proof sketch) and the total
// variation distance behind the two-party bound of the introduction, evaluated per row on the
// device so that a serving stack can choose the list size K from the distributions it has.
//
// Eq. (1) for K drafts drawn from p and a target q:
//   sum_j K / sum_i ( max{q_i/q_j, p_i/p_j} + (K - 1) q_i/q_j ).
// max{q_i/q_j, p_i/p_j} is q_i/q_j exactly when q_i/p_i >= q_j/p_j, so with the indices sorted by
// r = q/p the inner sum is (the q-mass from j on)/q_j + (the p-mass before j)/p_j + (K-1) Q/q_j:
// an order by r and running sums per row.  One workgroup does a whole row.  Four forms:
//
//  by cells' sums (rows of 6144 to 2.6 10^5 entries, bf16 from 8192 on): nothing is ordered or moved.  ln r is divided into some
//  7000 cells, finely where a sample of the row has many entries or much mass; one pass adds up the masses of every cell's entries
//  and how they are spread in it, as whole numbers in LDS, and a cell's terms follow from these sums (see lml_sum_kernel), but
//  for what the order inside it is worth, which is bounded.
//  by cells (a row whose cells leave too much open in all): a second pass takes the terms one by one, and entries for which the order in
//  their cell matters are resolved exactly (see lml_cell_kernel).
//  by sorting in LDS (shorter rows): four passes of a stable 8-bit radix sort on the fp32 image of ln r; masses rounded to fp32
//  (see lml_short_kernel).
//  by sorting (longer rows, and a row that the cells do not resolve either, also when they are shared out again): the same, the
//  masses travelling with their key through two buffers in the workspace.
//
// Indices whose r agree to fp32 precision may come out in either order, which together with the sorted masses' rounding
// moves a result by a relative 2^-22 at most, and so does what the cells leave open (1024 rows of 128 256 come out
// 3e-11 from the result in 64 bits by cells' sums, 1e-10 by cells, 5e-9 when sorted).
// Entries without mass on one side follow the limits: p_j = 0 or q_j = 0 gives term j = 0; as a
// summand i such an entry still counts with the mass it has on the other side.
#include "common.hpp"
#include "lml_search.hpp"

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
// What a lane gets of lane l ^ 1, l ^ 2, l ^ 3, 15 - l or 7 - l of its sixteen or eight, (l + 8) % 16, of the one N before in its sixteen, or of
// the last lane of the sixteen or thirty-two before (lanes without such a one, and rows that ROWS leaves out, get 0), without a trip through LDS.
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor3 = 0x1B, kMirror16 = 0x140, kMirror8 = 0x141, kXor8 = 0x128, kBefore = 0x110, kLast16 = 0x142,
              kLast32 = 0x143;
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int from_lane(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, true);
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ unsigned long long from_lane(unsigned long long v) {
  const uint32_t lo = (uint32_t)from_lane<CTRL, ROWS>((int)(uint32_t)v), hi = (uint32_t)from_lane<CTRL, ROWS>((int)(uint32_t)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ double from_lane(double v) {
  return __longlong_as_double((long long)from_lane<CTRL, ROWS>((unsigned long long)__double_as_longlong(v)));
}
__device__ __forceinline__ int of_lane(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ unsigned long long of_lane(unsigned long long v, int lane) {
  const uint32_t lo = (uint32_t)of_lane((int)(uint32_t)v, lane), hi = (uint32_t)of_lane((int)(uint32_t)(v >> 32), lane);
  return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ double of_lane(double v, int lane) {
  return __longlong_as_double((long long)of_lane((unsigned long long)__double_as_longlong(v), lane));
}
// The sum over every sixteen lanes of a wavefront, all of which are active; every lane gets it.
__device__ __forceinline__ double sum_of_16(double v) {
  v += from_lane<kXor1>(v);
  v += from_lane<kXor2>(v);
  v += from_lane<kMirror8>(v);
  v += from_lane<kMirror16>(v);
  return v;
}
// ... and over the wavefront: lane 63 gets it.
__device__ __forceinline__ double wave_sum(double v) {
  v = sum_of_16(v);
  v += from_lane<kLast16, 0xA>(v);
  v += from_lane<kLast32, 0xC>(v);
  return v;
}
// Inclusive prefix sums over the wavefront.
template <typename N>
__device__ __forceinline__ N prefix_of_16(N v) {
  v += from_lane<kBefore + 1>(v);
  v += from_lane<kBefore + 2>(v);
  v += from_lane<kBefore + 4>(v);
  v += from_lane<kBefore + 8>(v);
  return v;
}
template <typename N>
__device__ __forceinline__ N wave_prefix(N v) {
  v = prefix_of_16(v);
  v += from_lane<kLast16, 0xA>(v);
  v += from_lane<kLast32, 0xC>(v);
  return v;
}
// The same of several values at a time, in place; `scratch` holds as many doubles per wavefront.
template <int N>
__device__ __forceinline__ void block_sums(double (&v)[N], double *scratch) {
  const int waves = blockDim.x >> 6;
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] = wave_sum(v[n]);
  __syncthreads();
#pragma unroll
  for (int n = 0; n < N; ++n)
    if ((threadIdx.x & 63) == 63) scratch[(threadIdx.x >> 6) * N + n] = v[n];
  __syncthreads();
  const int lane = threadIdx.x & 63;  // (lane w fetches wavefront w's, of which there are sixteen at most)
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] = of_lane(sum_of_16(lane < waves ? scratch[lane * N + n] : 0.0), 0);
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

// Where the cell kernel tells the sorting one, launched behind it, that it left a row: behind the
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
          if (kp * qm > 0.0) relaxed[kk] += kp * qm / (kp + qm);
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

// ---- the form by cells

// The rows that go by cells.  Shorter ones are sorted, in LDS.  Where the line lies that is the faster way still (us a call of four list sizes, cells'
// sums against it, 1, 64 and 512 rows: fp32 6000 entries 51 : 40, 53 : 42, 108 : 82; bf16 8191: 52 : 48, 59 : 48, 120 : 97), but
// it rounds masses to fp32: a result is some 5e-9 off, by sums 3e-11, and longer rows keep that.
// Rows in doubt get a second attempt after the first from kAgainMinV entries on: what cells leave open grows with the
// entries that share one.  (Of twenty families of rows none had more than half of what is allowed at 50 257 entries, several more than
// all of it from 152 064 on.)
constexpr int kAgainMinV = 1 << 16;
constexpr int kCellMinV = 6144, kCellMinVNarrow = 8192, kCellMaxV = 1 << 18;
// The sample, and the buckets that its quantiles make.  Half of it are entries spread over the row, half the largest
// that every two threads met on either side (those near enough the row's largest to count): where a row is masked by a finite
// value, or is very sharp, what has mass would otherwise lie between two splitters.
constexpr int kSpread = 1024, kSamples = 2 * kSpread, kQuantiles = 127;
constexpr double kCounts = 0x1p-40;  // of the row's largest
constexpr int kMaxBuckets = 255;
constexpr int kCellThreads = 1024;
constexpr int kCells = 6144, kOuterCells = 384;
constexpr int kFewestCells = 8;        // of a bucket when they are shared out again
constexpr uint32_t kNoCell = 0xFFFFu;  // of an entry that lacks mass on a side
constexpr int kListed = 128;           // entries of a row whose sums are formed exactly
constexpr float kEntryError = 1e-9f;   // what cells may leave open of a result, whichever list size it is for: of one entry ...
constexpr double kRowError = 0x1.8p-23;  // ... and of all
constexpr float kFar = 512.0f;         // entries farther from the row's centre in ln r have no place
// An entry with both masses above zero in fp32 (2^-150 or more: ln >= -104) lies within 117 of the centre
// that the rows' largest entries make, in ln r: each mass is an entry's distance to its row's largest, less
// ln z, which is at most ln 2^18.  So an entry without a place, from a centre that is near that one, has no
// mass on one side, and which of such entries comes first is of no account.

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
  const N incl = wave_prefix(v);
  __syncthreads();  // scratch may still be read from the previous call
  if (lane == 63) scratch[threadIdx.x >> 6] = incl;
  __syncthreads();
  const N own = lane < waves ? scratch[lane] : N(0), upto = prefix_of_16(own);  // (sixteen wavefronts at most)
  *total = of_lane(upto, 15);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  return of_lane(upto, wave) - of_lane(own, wave) + incl - v;
}

// A value that is the same in all lanes, held in scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) { return __int_as_float(uniform(__float_as_int(v))); }
__device__ __forceinline__ double uniform(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)uniform((int)(uint32_t)b), hi = (uint32_t)uniform((int)(uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
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
__device__ __forceinline__ void add_quotients(double (&acc)[2 * PAIRS], const LmlParams &p, int n0, double pq, double base,
                                              double off, double slope) {
#pragma unroll
  for (int n = 0; n < 2 * PAIRS; n += 2) {
    const double k0 = p.kd[n0 + n], d0 = fma(k0 - off, slope, base);
    const double k1 = p.kd[n0 + n + 1], d1 = fma(k1 - off, slope, base);
    const double t = pq * reciprocal(d0 * d1);
    acc[n] = fma(k0 * t, d1, acc[n]);
    acc[n + 1] = fma(k1 * t, d0, acc[n + 1]);
  }
}

// A mass relative to its row's largest as a whole number of 2^-45ths (the sum of 2^18 of them fits 64 bits).  Whole
// numbers add up to the same sum in any order, so LDS atomics can form the cells' masses.
__device__ __forceinline__ unsigned long long fixed_mass(double e) {
  asm("" : "+v"(e));  // (the same rounding wherever it is taken)
  return (unsigned long long)__double_as_longlong(e + 128.0) - (unsigned long long)__double_as_longlong(128.0);
}

// One workgroup per row, one per CU (the cells' masses fill its LDS).  Nothing is sorted or moved.  The inner sum of term j
// over entries of other cells needs the masses before and behind j's cell only.  Over the other entries of its own cell,
// with masses P and Q in all, the sum of max(q_i p_j, p_i q_j) is P q_j times a mean of max(x_i, 1), x_i = r_i / r_j, weighed by
// p_i.  That is convex in x: no less than the maximum at the mean 1 + s = (Q p_j) / (P q_j), and no more than the chord
// over the cell there, which is (w - |s|)^2 / 4 w above it at most, wherever in the cell's width w (in x; below
// w_l (1 + w_l) of the width in ln r, up to 1.5) j lies.  It is taken as if the others lay evenly in the cell.  That
// uncertainty d is a part g = d / D of the denominator D for K = 1, where the entry's term is t, and moves its term for K
// by K f^2 t g, f = D / (D + (K - 1) p_j), which is up to K times as much: it is weighed by the largest of K f^2 / (the result
// for K) over the list sizes asked for.  D / p_j is the sum of max(q_i, r_j p_i), which depends on r_j alone and grows with it, so
// a weight belongs to a cell, taken at its right end or further right (1024 rows of 128 256, four sizes: 2.129 ms without weights,
// 2.136 so, 2.175 from a table for every entry, 2.265 by the sizes for every entry; 512 x 8 192 151 us, 154).  Where t g times that is more than kEntryError the entry's own sum is formed exactly by one more
// walk over the row's cell numbers (two large masses in one cell: a few rows in a hundred); a row whose uncertainties
// sum to more than kRowError of a result gets a second attempt, with cells shared out by where they were, and is
// left to the sorting kernel, which takes twice as long as both, if that is not enough.  (256 rows, one side flat, the other
// normal times 3, us, before, when 0.25 w stood for (w - |s|)^2 / 4 w and 2^-23 for kRowError and nearly all were sorted, and now: 128 256
// entries 2742, 1190, without a row in doubt 520; 152 064: 3362, 1389; 262 144: 5787, 2237.)
// A mass below 2^-46 of its row's largest is 0 in a cell's sum: a denominator is no less than the larger of p_j and q_j (the
// maxima are over all of a row whose masses sum to 1), so 2^18 such masses are less than 2^-28 of it.
// It takes the rows that lml_sum_kernel marked.  What bounds it: instruction issue in fp64 (two exponentials an entry and pass), the latency of LDS atomics and reads.
// The row is read three times, and two bytes an entry are written and read.  If it did every row, 1024 rows of 128 256, four sizes: 2.13 ms,
// against 3.13 with entries moved to buckets of about 1000 and those ordered in LDS; 1024 x 32 000 0.63 : 0.87,
// 512 x 152 064 bf16 1.37 : 1.94, one row 0.43 : 1.00, 64 x 262 144 0.96 : 2.11, eight sizes 512 rows 1.56 : 2.26.
// All sums run in an order that does not depend on how the wavefronts interleave.
template <typename E, bool PROBS>
__global__ void __launch_bounds__(kCellThreads, 4) lml_cell_kernel(const LmlParams p) {
  __shared__ unsigned long long s_p[kCells + 1], s_q[kCells + 1];  // a cell's masses, then what lies before it
  __shared__ float4 s_bucket[kMaxBuckets + 1];  // left end, cells per unit of ln r, first cell, last cell
  __shared__ int s_low[kCells], s_high[kCells]; // the smallest and largest place in a cell
  __shared__ int s_split[kMaxBuckets + 1];      // bucket b holds the places from s_split[b] up to s_split[b + 1]
  __shared__ double s_red[5 * (kCellThreads / 64)];
  __shared__ unsigned long long s_redu[kCellThreads / 64];
  __shared__ int s_redi[kCellThreads / 64];
  __shared__ int s_listed, s_at[kListed], s_list_cell[kListed], s_order[kListed];  // entries whose sums are formed exactly
  __shared__ unsigned long long s_above[kListed], s_below[kListed];
  __shared__ double s_ratio[kListed];
  __shared__ uint32_t s_mark[kCells / 32];
  __shared__ int s_far;
  __shared__ double s_about[kLmlMaxK];  // a list size's result, about
  __shared__ float s_scale[kLmlMaxK];   // K over that
  int *s_sample = reinterpret_cast<int *>(s_p);  // (before the cells)
  static_assert(kSamples * sizeof(int) <= sizeof(s_p) && kSamples == 2 * kCellThreads && kMaxBuckets * kFewestCells < kCells, "sizes");

  const int tid = threadIdx.x;
  const long long b_row = p.row0 + blockIdx.x;
  const int V = p.V;
  const E *prow = reinterpret_cast<const E *>(p.draft) + b_row * p.draft_stride_b;
  const E *qrow = reinterpret_cast<const E *>(p.target) + b_row * p.target_stride_b;
  char *work = p.work + (size_t)blockIdx.x * 24u * (size_t)V;
  {
    const double done = p.bound[b_row * p.n_k];
    if (done == done) {  // (uniform) the form by sums has done the row
      if (tid == 0) *flag_of(work, V) = 0;
      return;
    }
  }
  unsigned short *ids = reinterpret_cast<unsigned short *>(work);
  const float none = PROBS ? 0.0f : -__builtin_huge_valf();
  const float ninf = -__builtin_huge_valf();

  Placer<PROBS> pl;
  pl.itp = 1.0 / (double)p.temp_draft;
  pl.itq = 1.0 / (double)p.temp_target;
  pl.center = 0.0;

  // ---- first pass: the rows' largest entries, which masses are taken relative to, and the centre that they make
  float mp = ninf, mq = ninf;
  int at_p = 0, at_q = 0;  // where
  for (int i = tid * 4; i < V; i += kCellThreads * 4) {
    const float4 xp4 = four<E>(prow, i, V, none), xq4 = four<E>(qrow, i, V, none);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float xp = at(xp4, j), xq = at(xq4, j);
      if (pl.mass(xp) && xp > mp) { mp = xp; at_p = i + j; }
      if (pl.mass(xq) && xq > mq) { mq = xq; at_q = i + j; }
    }
  }
  // (every even thread stands for its neighbour too on the target's side, every odd one on the draft's)
  const bool odd = (tid & 1) != 0;
  float own = odd ? mp : mq;
  int at_own = odd ? at_p : at_q;
  {
    const float given = odd ? mq : mp, other = __shfl_xor(given, 1);
    const int at_other = __shfl_xor(odd ? at_q : at_p, 1);
    if (other > own) { own = other; at_own = at_other; }
  }
  mp = (float)block_max((double)mp, s_red);
  mq = (float)block_max((double)mq, s_red);
  const bool some = mp > ninf && mq > ninf;  // (uniform) else a side without mass: no entry has a place
  if (!PROBS && some) pl.center = uniform(pl.log_ratio(mp, mq));
  const double top_p = uniform((double)mp), top_q = uniform((double)mq);
  const double per_p = PROBS && some ? 1.0 / top_p : pl.itp, per_q = PROBS && some ? 1.0 / top_q : pl.itq;
  // the masses relative to the rows' largest (0: none)
  auto relative = [&](const float x, const double top, const double per) {
    if (PROBS) return pl.mass(x) ? (double)x * per : 0.0;
    return exp_of_negative(pl.mass(x) ? ((double)x - top) * per : -__builtin_huge_val());
  };

  // ---- splitters: the sample's quantiles, at least 16 of its entries to a bucket, and
  // places that the sample holds several times get a bucket of their own (inputs of few bits have many ties)
  int nb = 1;
  float far_left = -kFar, far_right = kFar;  // the outer buckets' outer ends: two e-folds from the sample's
  auto pick_splitters = [&]() {
    constexpr int kPicks = kSamples, kPer = kPicks / kCellThreads, kMany = 32;
    static_assert(kQuantiles + 2 * (kPicks / kMany) <= kMaxBuckets, "too many splitters");
    int valid = 0, n_valid;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      int i = at_own;
      bool counts = some;
      if (e < kPer - 1) {
        const unsigned j = (unsigned)(e * kCellThreads + tid), jitter = j * 0x9E3779B9u;
        i = (int)(((unsigned long long)j * (unsigned)V + (((unsigned long long)jitter * (unsigned)V) >> 32)) / kSpread);
      } else {
        counts = some && (odd ? relative(own, top_p, per_p) : relative(own, top_q, per_q)) >= kCounts;
      }
      const float xp = elem<E>(prow, i), xq = elem<E>(qrow, i);
      const float d = counts && pl.mass(xp) && pl.mass(xq) ? pl.distance(xp, xq) : kFar;
      s_sample[e * kCellThreads + tid] = fabsf(d) < kFar ? place_of(d) : 0x7FFFFFFF;
      valid += fabsf(d) < kFar ? 1 : 0;
    }
    block_prefix(valid, s_redi, &n_valid);
    for (int size = 2; size <= kPicks; size <<= 1)
      for (int stride = size >> 1; stride >= 1; stride >>= 1) {
        __syncthreads();
        for (int t = tid; t < kPicks / 2; t += kCellThreads) {
          const int lo = 2 * t - (t & (stride - 1)), hi = lo + stride;
          const int x = s_sample[lo], y = s_sample[hi];
          if ((x > y) == ((lo & size) == 0)) { s_sample[lo] = y; s_sample[hi] = x; }
        }
      }
    __syncthreads();
    if (n_valid == 0) return;  // uniform
    const int want = max(1, min(kQuantiles, n_valid / 16));
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
    far_left = uniform(distance_of(s_sample[0]) - 2.0f);
    far_right = uniform(distance_of(s_sample[n_valid - 1]) + 2.0f);
  };
  pick_splitters();
  nb = uniform(nb);
  __syncthreads();
  if (tid == 0) s_split[0] = (int)0x80000000;
#pragma unroll 1
  for (int attempt = 0;; ++attempt) {
    if (tid == 0) s_listed = 0;
    if (tid < kCells / 32) s_mark[tid] = 0u;
    // cells: the outer buckets, which are the longest, get kOuterCells each, the others share the rest evenly
    int my_cells = 0;  // of bucket number `tid`
    if (tid < nb) my_cells = nb <= 2 ? kCells / nb : tid == 0 || tid + 1 == nb ? kOuterCells : (kCells - 2 * kOuterCells) / (nb - 2);
    double zp, zq, first, norm_p, norm_q, unit_p, unit_q;
    constexpr int kEach = kCells / kCellThreads;
  #pragma unroll 1
    for (int round = 0;; ++round) {
      int in_all;
      const int my_first = block_prefix(my_cells, s_redi, &in_all);
      if (tid < nb) {
        const float left = tid > 0 ? distance_of(s_split[tid]) : far_left;
        const float right = tid + 1 < nb ? distance_of(s_split[tid + 1]) : far_right;
        // (two places can be farther apart than an int reaches; one more than a place is one)
        const bool one_place = tid >= 1 && tid + 1 < nb && s_split[tid + 1] <= s_split[tid] + 1;
        const float scale = one_place || !(right > left) ? 0.0f : (float)my_cells / (right - left);
        s_bucket[tid] = make_float4(left, scale, (float)my_first, (float)(my_first + my_cells - 1));
      }
      for (int c = tid; c <= kCells; c += kCellThreads) {
        s_p[c] = 0ull;
        s_q[c] = 0ull;
        if (c < kCells) { s_low[c] = 0x7FFFFFFF; s_high[c] = (int)0x80000000; }
      }
      __syncthreads();

      // ---- second pass: every entry's cell, the cells' masses, and the sums of all masses
      double p_first = 0.0;
      zp = zq = 0.0;
      for (int i = tid * 4; i < V; i += kCellThreads * 4) {
        const float4 xp4 = four<E>(prow, i, V, none), xq4 = four<E>(qrow, i, V, none);
        uint32_t packed[2] = {0u, 0u};
  #pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float xp = at(xp4, j), xq = at(xq4, j);
          const double ep = relative(xp, top_p, per_p), eq = relative(xq, top_q, per_q);
          zp += ep;
          zq += eq;
          uint32_t cell = kNoCell;
          if (some && pl.mass(xp) && pl.mass(xq)) {
            const float d = pl.distance(xp, xq);
            if (fabsf(d) < kFar) {
              const int place = place_of(d);
              const float4 bu = s_bucket[nb > 1 ? bucket_of(s_split, nb, place) : 0];
              cell = (uint32_t)(int)fminf(fmaxf((d - bu.x) * bu.y, 0.0f) + bu.z, bu.w);
              atomicAdd(&s_p[cell], fixed_mass(ep));
              atomicAdd(&s_q[cell], fixed_mass(eq));
              atomicMin(&s_low[cell], place);
              atomicMax(&s_high[cell], place);
            }
          }
          // ratio 0, or near it: before all others (an entry without a cell that has the larger ratio has no
          // p-mass to speak of)
          if (cell == kNoCell) p_first += ep;
          packed[j >> 1] |= cell << (16 * (j & 1));
        }
        if (i + 3 < V) {
          *reinterpret_cast<uint2 *>(ids + i) = make_uint2(packed[0], packed[1]);
        } else {
          for (int j = 0; i + j < V; ++j) ids[i + j] = (unsigned short)(packed[j >> 1] >> (16 * (j & 1)));
        }
      }
      zp = uniform(block_sum(zp, s_red));
      zq = uniform(block_sum(zq, s_red));
      norm_p = zp > 0.0 ? 1.0 / zp : 0.0;
      norm_q = zq > 0.0 ? 1.0 / zq : 0.0;
      first = uniform(block_sum(p_first, s_red) * norm_p);
      unit_p = 0x1p-45 * norm_p;
      unit_q = 0x1p-45 * norm_q;
      {
        unsigned long long all;
  #pragma unroll
        for (int side = 0; side < 2; ++side) {
          unsigned long long *m = side == 0 ? s_p : s_q, mine[kEach], sum = 0ull;
  #pragma unroll
          for (int e = 0; e < kEach; ++e) { mine[e] = m[tid * kEach + e]; sum += mine[e]; }
          unsigned long long before = block_prefix(sum, s_redu, &all);
  #pragma unroll
          for (int e = 0; e < kEach; ++e) { m[tid * kEach + e] = before; before += mine[e]; }
          if (tid == kCellThreads - 1) m[kCells] = before;
        }
      }
      __syncthreads();
      if (attempt == 0 || round == 1) break;
      // cells where they are wanted: a bucket's uncertainty is about the sum of t^2 w over its cells, t a cell's term and w its
      // width, and falls with the square of their number, so the sum over all buckets is least with numbers that go with
      // the cube root of t^2 w times the present number squared
      float wants = 0.0f;
      if (tid < nb) {
        for (int c = my_first; c < my_first + my_cells; ++c) {
          const double pc = (double)(s_p[c + 1] - s_p[c]) * unit_p, qc = (double)(s_q[c + 1] - s_q[c]) * unit_q;
          const double base = (1.0 - (double)s_q[c] * unit_q) * pc + ((double)s_p[c] * unit_p + first) * qc;
          const float t = pc > 0.0 && qc > 0.0 && base > 0.0 ? (float)(pc * qc * reciprocal(base)) : 0.0f;
          if (s_high[c] > s_low[c]) wants += t * t * (distance_of(s_high[c]) - distance_of(s_low[c]));
        }
        if (wants > 0.0f) wants = exp2f(log2f(wants * (float)my_cells * (float)my_cells) * (1.0f / 3.0f));
      }
      const float wanted = (float)block_sum((double)wants, s_red);
      if (tid < nb && wanted > 0.0f) my_cells = kFewestCells + (int)((float)(kCells - 1 - nb * kFewestCells) * (wants / wanted));
    }
    // about what the results will be, the thread's cells taken as one entry: uncertainties are measured against them
    const int my_cell = tid * kEach;
    const unsigned long long my_p = s_p[my_cell + kEach], my_q = s_q[my_cell];
    double about_1 = 0.0;
  #pragma unroll 1
    for (int n0 = 0; n0 < p.n_k; n0 += 4) {
      double about[4] = {0.0, 0.0, 0.0, 0.0};
      const double pc = (double)(my_p - s_p[my_cell]) * unit_p, qc = (double)(s_q[my_cell + kEach] - my_q) * unit_q;
      const double base = (1.0 - (double)my_q * unit_q) * pc + ((double)s_p[my_cell] * unit_p + first) * qc;
      const bool shared = pc > 0.0 && qc > 0.0 && base > 0.0;
      if (shared) add_quotients<2>(about, p, n0, pc * qc, base, 1.0, pc);
      double sum[5] = {about[0], about[1], about[2], about[3], shared ? pc * qc * reciprocal(base) : 0.0};
      block_sums(sum, s_red);
      about_1 = uniform(sum[4]);
  #pragma unroll
      for (int n = 0; n < 4; ++n)
        if (tid == 0 && n0 + n < p.n_k) { s_about[n0 + n] = sum[n]; s_scale[n0 + n] = (float)(p.kd[n0 + n] / sum[n]); }
    }
    // (two sides that share next to nothing: whatever is open is resolved)
    const bool some_shared = about_1 > 0x1p-90;
    const float entry_error = some_shared ? kEntryError : 0.0f;
    if (tid == 0) s_far = 0;
    __syncthreads();
    // in place of the places: a cell's width in ln r, and what its entries' uncertainties are weighed by (at the right
    // end of the thread's cells)
    {
      int right = (int)0x80000000;
  #pragma unroll
      for (int e = 0; e < kEach; ++e) {
        const int low = s_low[my_cell + e], high = s_high[my_cell + e];
        right = max(right, high);
        s_low[my_cell + e] = __float_as_int(high > low ? distance_of(high) - distance_of(low) : 0.0f);
      }
      const double r_0 = (PROBS ? top_p / top_q : 1.0) * zp * norm_q;  // q / p of an entry at distance 0
      const double before = fma((double)my_p, unit_p, first), from = fmax(1.0 - (double)my_q * unit_q, 0.0);
      const double d = fma(before, exp_of_negative((double)distance_of(right)) * r_0, from);  // D / p_j
      const float u = (float)reciprocal(fmin(fmax(d, 1.0), 0x1p900));
      float weight = some_shared ? 0.0f : 1.0f;
      for (int n = 0; some_shared && n < p.n_k; ++n) {
        const float f = __builtin_amdgcn_rcpf(fmaf((float)p.k[n] - 1.0f, u, 1.0f));
        weight = fmaxf(weight, s_scale[n] * f * f);
      }
  #pragma unroll
      for (int e = 0; e < kEach; ++e) s_high[my_cell + e] = __float_as_int(weight);
    }
    __syncthreads();

    // ---- third pass: the terms (list sizes four at a time)
    double tv = 0.0;
    float doubt = 0.0f;
  #pragma unroll 1
    for (int n0 = 0; n0 < p.n_k; n0 += 4) {
      double sums[4] = {0.0, 0.0, 0.0, 0.0}, relaxed[4] = {0.0, 0.0, 0.0, 0.0};
      // K pq / (base + (K - 1) pm) of one entry, base = D(r) p: numerator and denominator of K q / (D(r) + (K - 1) Q) times p
  #pragma unroll 1
      for (int i = tid * 4; i < V; i += kCellThreads * 4) {
        const float4 xp4 = four<E>(prow, i, V, none), xq4 = four<E>(qrow, i, V, none);
        uint32_t cells[2] = {0u, 0u};
        if (i + 3 < V) {
          const uint2 c = *reinterpret_cast<const uint2 *>(ids + i);
          cells[0] = c.x; cells[1] = c.y;
        } else {
          for (int j = 0; i + j < V; ++j) cells[j >> 1] |= (uint32_t)ids[i + j] << (16 * (j & 1));
        }
  #pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (i + j >= V) continue;
          const double ep = relative(at(xp4, j), top_p, per_p), eq = relative(at(xq4, j), top_q, per_q);
          double pm = ep * norm_p, qm = eq * norm_q;
          if (n0 == 0) tv += fabs(pm - qm);
          const uint32_t cell = (cells[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
          if (cell != kNoCell && pm >= 0x1p-150 && qm >= 0x1p-150) {
            const unsigned long long pb = s_p[cell], qb = s_q[cell + 1];
            // what else is in the cell
            const double po = fmax((double)(long long)(s_p[cell + 1] - pb - fixed_mass(ep)), 0.0) * unit_p;
            const double qo = fmax((double)(long long)(qb - s_q[cell] - fixed_mass(eq)), 0.0) * unit_q;
            const double a = qo * pm, c = po * qm;
            const float width = __int_as_float(s_low[cell]);
            const double rest = fma(fmax(1.0 - (double)qb * unit_q, 0.0), pm, fma((double)pb, unit_p, first) * qm) + pm * qm;
            double inside = fmax(a, c);
            const double base = rest + inside;
            // relative to the denominator: in fp32, as small as they are
            const double inv = reciprocal(base);
            const float cw = (float)(c * inv) * width, side = (float)((a - c) * inv), per_cw = __builtin_amdgcn_rcpf(fmaxf(cw, 1e-30f));
            const float reach = fmaxf(fmaf(cw, width, cw) - fabsf(side), 0.0f);
            const float gap = fminf((float)(fmin(a, c) * inv), width < 1.5f ? 0.25f * reach * reach * per_cw : 1.0f);
            const float open = (float)(pm * qm * inv) * gap * __int_as_float(s_high[cell]);
            if (open > entry_error) {
              if (n0 == 0) {
                const int pos = atomicAdd(&s_listed, 1);
                if (pos < kListed) { s_at[pos] = i + j; s_list_cell[pos] = (int)cell; }
              }
            } else {
              if (n0 == 0) doubt += open;
              if (width < 0.5f && 2.0f * fabsf(side) < cw) {
                const float t = 0.5f * cw + side;  // > 0
                inside = c + (double)(0.5f * t * t * per_cw) * base;
              }
              add_quotients<2>(sums, p, n0, pm * qm, rest + inside, 1.0, pm);
            }
          }
          if (ep > 0.0 && eq > 0.0 && p.relaxed != nullptr) {  // q / (1 + q / (K p)) = K p q / (K p + q)
            // (where the product nears the smallest numbers, both are taken relative to the larger one: its
            // denominators, and their product, are then at least 1/4)
            int scale = 0;
            if (pm * qm < 0x1p-900) {
              scale = __builtin_amdgcn_frexp_exp(fmax(pm, qm));
              pm = __builtin_amdgcn_ldexp(pm, -scale);
              qm = __builtin_amdgcn_ldexp(qm, -scale);
            }
            const double pq = __builtin_amdgcn_ldexp(pm * qm, scale);
            if (pq > 0.0) add_quotients<2>(relaxed, p, n0, pq, qm, 0.0, pm);
          }
        }
      }
      __syncthreads();
      const int listed = s_listed;
      if (listed > kListed) break;  // (uniform) the row is the sorting kernel's
      if (listed > 0) {
        // ---- the listed entries' cells, entry by entry: what is above each in the order, and what below
        if (n0 == 0) {
          if (tid < listed) {
            s_ratio[tid] = pl.log_ratio(elem<E>(prow, s_at[tid]), elem<E>(qrow, s_at[tid]));
            s_above[tid] = 0ull;
            s_below[tid] = 0ull;
            atomicOr(&s_mark[s_list_cell[tid] >> 5], 1u << (s_list_cell[tid] & 31));
          }
          __syncthreads();
          for (int i = tid; i < V; i += kCellThreads) {
            const uint32_t cell = ids[i];
            if (cell == kNoCell || !((s_mark[cell >> 5] >> (cell & 31u)) & 1u)) continue;
            const float xp = elem<E>(prow, i), xq = elem<E>(qrow, i);
            const double r = pl.log_ratio(xp, xq);
            for (int l = 0; l < listed; ++l) {
              if (s_list_cell[l] != (int)cell || s_at[l] == i) continue;
              if (r >= s_ratio[l])
                atomicAdd(&s_above[l], fixed_mass(relative(xq, top_q, per_q)));
              else
                atomicAdd(&s_below[l], fixed_mass(relative(xp, top_p, per_p)));
            }
          }
          if (tid < listed) {
            int before = 0;
            for (int l = 0; l < listed; ++l) before += s_at[l] < s_at[tid] ? 1 : 0;
            s_order[before] = tid;
          }
          __syncthreads();
        }
        if (tid < listed) {  // thread t takes the t-th in the row's order
          const int from = s_order[tid];
          const int i = s_at[from], cell = s_list_cell[from];
          const double pm = relative(elem<E>(prow, i), top_p, per_p) * norm_p, qm = relative(elem<E>(qrow, i), top_q, per_q) * norm_q;
          const double behind = fmax(1.0 - (double)s_q[cell + 1] * unit_q, 0.0) + (double)s_above[from] * unit_q;
          const double before = fma((double)s_p[cell] + (double)s_below[from], unit_p, first);
          add_quotients<2>(sums, p, n0, pm * qm, fma(behind, pm, before * qm) + pm * qm, 1.0, pm);
        }
      }
      double bound[5] = {sums[0], sums[1], sums[2], sums[3], (double)doubt};
      block_sums(bound, s_red);
      double others[5] = {relaxed[0], relaxed[1], relaxed[2], relaxed[3], tv};
      block_sums(others, s_red);
      if (tid == 0) {
  #pragma unroll
        for (int n = 0; n < 4; ++n)
          if (n0 + n < p.n_k) {
            // (the doubt is relative to what each result was to be about)
            if (bound[4] * s_about[n0 + n] > kRowError * bound[n]) s_far = 1;
            p.bound[b_row * p.n_k + n0 + n] = bound[n];
            if (p.relaxed != nullptr) p.relaxed[b_row * p.n_k + n0 + n] = others[n];
          }
        if (n0 == 0 && p.tv != nullptr) p.tv[b_row] = 0.5 * others[4];
      }
    }
    __syncthreads();
    const bool too_many = s_listed > kListed, in_doubt = s_far != 0;  // (uniform)
    if (attempt == 0 && !too_many && in_doubt && V >= kAgainMinV) {
      __syncthreads();  // s_listed and s_far have been read
      continue;
    }
    if (tid == 0) *flag_of(work, V) = too_many || in_doubt ? 1 : 0;
    break;
  }
}

// ---- the form by cells' sums

// A thread holds kSumEach cells.  Buckets: 127 quantiles' splitters, up to 128 of places that the sample holds often, and two
// for every heavy entry.
constexpr int kSumEach = 7, kSumCells = kSumEach * kCellThreads;
constexpr double kHeavy = 0x1p-9;     // of a side's mass: such an entry's place has a cell of its own
constexpr float kSumFar = 740.0f;     // entries farther from the row's centre in log2 r have no place (kFar in ln r)
constexpr float kBeyond = 6.0f;       // how far the outer buckets reach beyond the sample, in log2 r
// What a row's cells may leave open of a result, of kRowError: as much as those of one side flat and the other normal times 3 do
// (some 8e-13 an entry; Zipf-like rows a tenth of that or less).  More is no matter of chance but of a crowd in few cells.
constexpr double kSumErrorLeast = 0.5, kSumErrorEach = 0x1p-17;
constexpr double kShareAgain = 0x1p-18;  // what sharing the cells out again can mend
constexpr float kLaneStep = 0x1p40f;  // (a distance is a multiple of 2^-36)
constexpr double kU2Units = 0x1p35;   // of a side's mass in a cell's sum of p u (1 - u), which is no more than a quarter of the cell's, so that ...
constexpr float kU2Slip = 0x1.6a09e6p-18f;  // 1 / sqrt(kU2Units)
constexpr float kU2Most = 0x1.fp-2f;  // ... it has 32 bits in a cell with less than this (and 2^18 entries): one with more is not known
constexpr uint32_t kDitherStep = 0x9E3779B9u, kGroupStep = kDitherStep * kCellThreads;  // (2^32 over the golden ratio: its multiples are spread evenly)
constexpr float kWide = 0.5f;         // a cell this wide in ln r leaves its entries' whole terms open

// 2^y for y <= 0 or so (what is below -1074 comes out as 0, NaN too) to about an ulp: y = n + f, |f| <= 1/2, and 2^f = 1 + f P(f)
// with the P of degree 10 whose largest relative error on that range is least (1.8e-17; by Remez' exchange).
__device__ __forceinline__ double exp2_of(double y) {
  asm("v_max_f64 %0, %1, %2" : "=v"(y) : "v"(y), "s"(-1100.0));  // (fmax() takes one instruction more, to quiet a NaN that cannot be)
  const double t = y + 0x1.8p52;        // (n in the lower half)
  const double f = y - (t - 0x1.8p52);
  double s = fma(0x1.c062ee76e864cp-32, f, 0x1.e605f90accdcbp-28);
  s = fma(s, f, 0x1.b54167f262812p-24);
  s = fma(s, f, 0x1.62bfd49f13823p-20);
  s = fma(s, f, 0x1.ffcbee3aee4b9p-17);
  s = fma(s, f, 0x1.4309130960facp-13);
  s = fma(s, f, 0x1.5d87fe7bbbe3ep-10);
  s = fma(s, f, 0x1.3b2ab6fba1e1cp-7);
  s = fma(s, f, 0x1.c6b08d7048f31p-5);
  s = fma(s, f, 0x1.ebfbdff82c598p-3);
  s = fma(s, f, 0x1.62e42fefa39f3p-1);
  s = fma(s, f, 1.0);
  return __builtin_amdgcn_ldexp(s, (int)(uint32_t)__double_as_longlong(t));
}

// x >= 0 as a whole number, the largest of 32 bits if it is larger.
__device__ __forceinline__ uint32_t saturated(float x) {
  uint32_t n;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(n) : "v"(x));
  return n;
}

// A mass relative to its row's largest as a whole number of `step` 2^-52ths, a power of two and no less than the mass.
__device__ __forceinline__ unsigned long long whole_mass(double e, double step) {
  const unsigned long long sum = (unsigned long long)__double_as_longlong(e + step);
  uint32_t hi = (uint32_t)(sum >> 32);  // (the lower half of `step` is 0; written as a difference it becomes one of 64 bits again)
  asm("v_subrev_u32 %0, %1, %0" : "+v"(hi) : "s"((uint32_t)((unsigned long long)__double_as_longlong(step) >> 32)));
  return ((unsigned long long)hi << 32) | (uint32_t)sum;
}
// ... the least for masses that sum to z, which must stay below 2^63 (values of few bits are rounded alike, so that it is not chance
// alone which keeps the rounding of their sums small: with 128 throughout, as fixed_mass has it, bf16 rows came out 2e-11 off, now 3e-12).
__device__ __forceinline__ double step_for(double z) {
  return fmax(__builtin_amdgcn_ldexp(1.0, __builtin_amdgcn_frexp_exp(z) - 11), 1.0);
}

// log2(e) / t, rounded once: of twice 53 bits of either factor.
__device__ __forceinline__ double log2e_over(float t) {
  const double hi = 0x1.71547652b82fep+0, lo = 0x1.777d0ffda0d24p-56;  // log2(e)
  const double r = 1.0 / (double)t, rest = fma(-r, (double)t, 1.0) * r;  // 1 / t
  return fma(r, hi, fma(r, lo, rest * hi));
}

// A side's masses relative to a reference entry.  Logits and log-weights: 2^(x per - off); probabilities: x per.
template <bool PROBS>
struct Masses {
  double per, off;
  __device__ __forceinline__ double log2_of(float x) const { return fma((double)x, per, -off); }
  __device__ __forceinline__ double of(float x) const {
    if (PROBS) return x > 0.0f && x < __builtin_huge_valf() ? (double)x * per : 0.0;
    return exp2_of(log2_of(x));
  }
};

// acc[n] += pq / (k[n] p + q) for 2 PAIRS list sizes: the relaxed sum's quotients less their factor k[n], by one reciprocal.
// What has pq < 2^-400 (four denominators' product is far from the smallest numbers otherwise) adds less than k 2^-200 each
// and is left out: a result below kLeastRelaxed is not this form's.
constexpr double kLeastRelaxed = 0x1p-100;
template <int PAIRS>
__device__ __forceinline__ void add_relaxed(double (&acc)[4], const double *k, double pp, double q) {
  const double pq = pp * q;
  if (pq >= 0x1p-400) {
    const double d0 = fma(k[0], pp, q), d1 = fma(k[1], pp, q), d01 = d0 * d1;
    if (PAIRS == 1) {
      const double r = pq * reciprocal(d01);
      acc[0] = fma(r, d1, acc[0]);
      acc[1] = fma(r, d0, acc[1]);
    } else {
      const double d2 = fma(k[2], pp, q), d3 = fma(k[3], pp, q), d23 = d2 * d3;
      const double r = pq * reciprocal(d01 * d23), r01 = r * d23, r23 = r * d01;
      acc[0] = fma(r01, d1, acc[0]);
      acc[1] = fma(r01, d0, acc[1]);
      acc[2] = fma(r23, d3, acc[2]);
      acc[3] = fma(r23, d2, acc[3]);
    }
  }
}

// The place of a distance that is 0 or a multiple of 2^-36 below 2^11 in size takes 30 bits (the smallest such has the
// bits 0x2D800000, the largest less than 0x45000000), in the same order.
__device__ __forceinline__ int short_place(int place) {
  return place > 0 ? place - 0x2D000000 : place < 0 ? place + 0x2D000000 : 0;
}
__device__ __forceinline__ int long_place(int v) { return v > 0 ? v + 0x2D000000 : v < 0 ? v - 0x2D000000 : 0; }

// The largest of the four entries from `group` on, and where.
template <typename E>
__device__ __forceinline__ void largest_of_four(const E *row, int group, int V, float fill, float *best, int *at_best) {
  const float4 x = four<E>(row, group, V, fill);
  *best = -__builtin_huge_valf();
  *at_best = group;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (at(x, j) > *best) { *best = at(x, j); *at_best = group + j; }
}

// A SIMD serves its wavefronts oldest first, so that the last of a workgroup goes through the end of its row alone.  Whoever
// is behind one of these steps is served before those past it.
struct Steps {
  int left, at;
  __device__ __forceinline__ explicit Steps(int V) : left((V + 4 * kCellThreads - 1) / (4 * kCellThreads)), at(left >> 1) {
    __builtin_amdgcn_s_setprio(3);
    level = 3;
  }
  __device__ __forceinline__ void next() {
    if (left-- > at) return;
    at >>= 2;
    if (--level == 2) __builtin_amdgcn_s_setprio(2);
    else if (level == 1) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
  }
  __device__ __forceinline__ void done() { __builtin_amdgcn_s_setprio(0); }
  int level;
};

// The kernel's parameters, fetched once more: held from its beginning they take scalar registers that its loops have not got.
__device__ __forceinline__ const LmlParams &params_again() {
  typedef const LmlParams __attribute__((address_space(4))) *kernarg;
  uint64_t at = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(at));
  return *(const LmlParams *)(kernarg)at;
}

// One workgroup per row, one per CU (the cells fill its LDS).  A term for K is K q_j / (F(r_j) + K - 1) with
// F(r) = sum_i max(q_i, r p_i), a function of r_j = q_j / p_j alone, so what a cell of ln r adds to the result follows
// from sums over its entries, and no entry is looked at again.  With P, Q a cell's masses, r = Q / P, r_j = r (1 + s_j), v the mean of s_j^2 (weighed by p)
// and g the mean of |s_i - s_j|,
//   sum_j K q_j / (F(r_j) + K - 1) = K Q / D (1 - x ((P' + P / 2) v + P g / 2) + x^2 (P' + P / 2)^2 v + third powers of s),
// P' the p-mass and Q' the q-mass before and behind the cell, D = Q' + Q + r P' + K - 1, x = r / D.  P and Q are added up as whole numbers (whole_mass),
// v comes from a third sum, of p u (1 - u) with u an entry's place in its cell (the mean of u is known from Q / P), whose shares are rounded to 2^-35ths of the
// row's mass, up or down by the entry's place in the row: right on average, and what that may be off by in a cell counts as open.  (Rounded to the nearest of 2^-31ths the shares of
// light entries were all nothing, which looked like a cell without spread: rows whose sides share light entries only came out up to 16 x 2^-22 off, now 0.12 x 2^-22.)  And g, for which the order
// inside the cell would be needed, is taken as 4 v / w: right on average if the entries lie evenly in the cell's width w, whatever their
// number and masses are.  It is no less than 2 v / w and no more than 2 sqrt(v / 3) (the mean difference of any masses with
// that variance), so what a cell leaves open is known; an entry that is heavy on either side gets a cell without width (with others of its ratio),
// for which nothing is open.  Rows whose cells leave more open in all than kSumErrorLeast and kSumErrorEach allow get one more pass with
// cells shared out by where that was; what then still does, rows with +inf entries or without mass on a side, or whose results are so small that the rounding of
// masses may count, are marked (a NaN in the place of their first result) and left to lml_cell_kernel, behind this one.
// tv and the relaxed sums are taken in 64 bits, entry by entry, in the pass that makes the cells.
// What bounds it: issue in fp64 (0.83 of the slots; 200 instructions an entry in all).  The row is read twice.  Two exponentials an entry and pass (15 instructions each), of some 45 in the
// first pass and 110 in the second; of a row of 128 256 (220 us, four a CU in turn) those take 53 and 108 us, the sample and its order 17, the
// cells 14, sums over the workgroup and their barriers the rest.  us a call, four list sizes, entries' terms taken one by one (lml_cell_kernel for
// every row) and now: 1024 x 128 256 2135, 875; 512 x 152 064 bf16 1394, 507; 1024 x 32 000, two sizes, 645, 366; 256 x 50 257 bf16, one size, 272,
// 115; one row of 128 256 423, 170; 64 x 8192 71, 56; 256 x 128 256, one side flat and the other normal times 3, 1187, 336, target masked by -10^9 but
// for 50 297, 229, eight sizes 790, 319.  Rows whose two sides share next to nothing pay for an attempt in vain (256 x 128 256, bound 10^-4: 526, 885).
// The bound's error against 64 bits, same inputs: 1.1e-10, 3e-11; T = 1: 3.3e-10, 1.5e-10; 152 064 bf16: 7e-12, 7e-13.
template <typename E, bool PROBS>
__global__ void __launch_bounds__(kCellThreads, 4) lml_sum_kernel(const LmlParams p) {
  __shared__ unsigned long long s_p[kSumCells + 1], s_q[kSumCells + 1];  // a cell's masses, then what lies before it
  __shared__ uint32_t s_u2[kSumCells];         // sums of p u (1 - u) in 2^-35ths of the side's mass, u an entry's place in its cell
  __shared__ float4 s_bucket[kSumBuckets];     // left end, cells per unit of log2 r, first cell (its bits), largest place in the bucket in cells
  __shared__ double s_per_left[kSumBuckets];   // 2^-(left end), for whole masses
  __shared__ float s_split[2 * kSumBuckets];   // bucket b holds what lies from s_split[b] up to s_split[b + 1]
  __shared__ unsigned short s_grid[kCellThreads];  // splitters to the left of each of 1024 equal parts of the range
  __shared__ double s_red[8 * (kCellThreads / 64)];
  __shared__ unsigned long long s_redu[kCellThreads / 64];
  __shared__ int s_redi[kCellThreads / 64];
  __shared__ double s_total[2];                // the sides' masses, relative to their largest
  __shared__ double s_sizes[4];
  __shared__ int s_single, s_shared, s_most;   // buckets of a single place, and of one with several cells; splitters in one part of the range, at most
  int *s_sample = reinterpret_cast<int *>(s_p);  // (before the cells)
  static_assert(kCellMinV >= 4 * kCellThreads && kCellMinVNarrow >= 4 * kCellThreads, "every thread has four entries");
  static_assert(kSumBuckets * (kFewestCells + 1) + 2 * kOuterCells + kSumCells / 14 < kSumCells, "too few cells");

  const int tid = threadIdx.x;
  const long long b_row = p.row0 + blockIdx.x;
  const int V = p.V;
  const E *prow = reinterpret_cast<const E *>(p.draft) + b_row * p.draft_stride_b;
  const E *qrow = reinterpret_cast<const E *>(p.target) + b_row * p.target_stride_b;
  const float none = PROBS ? 0.0f : -__builtin_huge_valf();
  const float ninf = -__builtin_huge_valf(), pinf = __builtin_huge_valf();
  auto leave = [&]() {
    if (tid == 0) p.bound[b_row * p.n_k] = __builtin_nan("");
  };

  Placer<PROBS> pl;
  pl.itp = 1.0 / (double)p.temp_draft;
  pl.itq = 1.0 / (double)p.temp_target;
  pl.center = 0.0;

  // ---- first pass: the sides' sums and largest entries.  Masses are taken relative to the largest of the first
  // 64 entries, which serves unless it is so far below the row's largest that the largest's mass or the sum overflows.  (exp2_of makes any number of an
  // exponent beyond 2^31: a sum is taken if, relative to the largest, it is no less than the largest itself)
  Masses<PROBS> mp, mq;
  mp.per = PROBS ? 1.0 : log2e_over(p.temp_draft);
  mq.per = PROBS ? 1.0 : log2e_over(p.temp_target);
  double zp, zq;
  float own_p, own_q;  // the largest entry that this thread met
  int at_p, at_q;
  float top_p, top_q;
  {
    const int lane = tid & 63;
    top_p = elem<E>(prow, lane);
    top_q = elem<E>(qrow, lane);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      top_p = fmaxf(top_p, __shfl_xor(top_p, d));
      top_q = fmaxf(top_q, __shfl_xor(top_q, d));
    }
  }
#pragma unroll 1
  for (int attempt = 0;; ++attempt) {
    mp.off = uniform(fabsf(top_p) < pinf ? (double)top_p * mp.per : 0.0);
    mq.off = uniform(fabsf(top_q) < pinf ? (double)top_q * mq.per : 0.0);
    double sum_p = 0.0, sum_q = 0.0, best_p = -__builtin_huge_val(), best_q = best_p;
    at_p = at_q = tid * 4;
    Steps stage(V);
    float4 next_p = four<E>(prow, tid * 4, V, none), next_q = four<E>(qrow, tid * 4, V, none);
#pragma unroll 1
    for (int i = tid * 4; i < V; i += kCellThreads * 4) {
      stage.next();
      const float4 xp4 = next_p, xq4 = next_q;
      if (i + kCellThreads * 4 < V) {
        next_p = four<E>(prow, i + kCellThreads * 4, V, none);
        next_q = four<E>(qrow, i + kCellThreads * 4, V, none);
      }
      double yp[4], yq[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float xp = at(xp4, j), xq = at(xq4, j);
        yp[j] = PROBS ? mp.of(xp) : mp.log2_of(xp);
        yq[j] = PROBS ? mq.of(xq) : mq.log2_of(xq);
        sum_p += PROBS ? yp[j] : exp2_of(yp[j]);
        sum_q += PROBS ? yq[j] : exp2_of(yq[j]);
      }
      const double gp = fmax(fmax(yp[0], yp[1]), fmax(yp[2], yp[3])), gq = fmax(fmax(yq[0], yq[1]), fmax(yq[2], yq[3]));
      if (gp > best_p) { best_p = gp; at_p = i; }
      if (gq > best_q) { best_q = gq; at_q = i; }
    }
    stage.done();
    largest_of_four<E>(prow, at_p, V, none, &own_p, &at_p);
    largest_of_four<E>(qrow, at_q, V, none, &own_q, &at_q);
    {
      // the two sums and the two largest entries over the workgroup
      const int lane = tid & 63;
      float wave_p = own_p, wave_q = own_q;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        wave_p = fmaxf(wave_p, __shfl_xor(wave_p, d));
        wave_q = fmaxf(wave_q, __shfl_xor(wave_q, d));
      }
      sum_p = wave_sum(sum_p);
      sum_q = wave_sum(sum_q);
      __syncthreads();  // (s_red may still be read from the attempt before)
      if (lane == 63) {
        double *mine = s_red + (tid >> 6) * 4;
        mine[0] = sum_p; mine[1] = sum_q; mine[2] = (double)wave_p; mine[3] = (double)wave_q;
      }
      __syncthreads();
      const double *theirs = s_red + (lane & 15) * 4;
      zp = of_lane(sum_of_16(theirs[0]), 0);
      zq = of_lane(sum_of_16(theirs[1]), 0);
      float most_p = (float)theirs[2], most_q = (float)theirs[3];
#pragma unroll
      for (int d = 8; d >= 1; d >>= 1) {
        most_p = fmaxf(most_p, __shfl_xor(most_p, d));
        most_q = fmaxf(most_q, __shfl_xor(most_q, d));
      }
      top_p = uniform(most_p);
      top_q = uniform(most_q);
    }
    if (!(fabsf(top_p) < pinf && fabsf(top_q) < pinf) || (PROBS && !(top_p > 0.0f && top_q > 0.0f))) {  // (uniform)
      leave();
      return;
    }
    if (!PROBS) {
      const double off_p = (double)top_p * mp.per, off_q = (double)top_q * mq.per;
      zp *= exp2_of(mp.off - off_p);
      zq *= exp2_of(mq.off - off_q);
      mp.off = off_p;
      mq.off = off_q;
    }
    constexpr double kLeast = PROBS ? 0x1p-300 : 0.5;
    if (zp >= kLeast && zp < 0x1p1000 && zq >= kLeast && zq < 0x1p1000) break;
    if (attempt == 1) {  // (uniform) a NaN among the sums: an entry of +inf
      leave();
      return;
    }
  }
  if (PROBS) {
    mp.per = uniform(1.0 / (double)top_p);
    mq.per = uniform(1.0 / (double)top_q);
    zp *= mp.per;
    zq *= mq.per;
    pl.center = uniform(pl.log_ratio(top_p, top_q));
  } else {
    mp.off = uniform(mp.off);
    mq.off = uniform(mq.off);
  }
  if (tid < 4) s_sizes[tid] = p.kd[tid];
  if (tid == 0) { s_total[0] = zp; s_total[1] = zq; }  // (registers are scarce in the second pass)
  // log2 r of an entry less the row's centre, where both its masses are the largest ones' (rounded to 2^-36 first: equal
  // ratios of different entries differ by fp64's rounding)
  auto distance = [&](const float xp, const float xq, const double yp, const double yq) {
    constexpr double kStep = 0x1.8p16;
    if (!PROBS) return (float)(((yq - yp) + kStep) - kStep);
    const double d = (pl.log_ratio(xp, xq) - pl.center) * 1.4426950408889634;
    return pl.mass(xp) && pl.mass(xq) ? (float)((d + kStep) - kStep) : __builtin_nanf("");
  };

  // ---- splitters: the quantiles of a sample, half of it spread over the row, half the largest entry of every thread on one
  // side or the other (of a pair's two the even thread answers for the target; where the smaller of these is heavy
  // it takes the place of a spread entry), the places it holds several times, and those of heavy entries
  int nb = 1;
  float far_left = -kSumFar, far_right = kSumFar;
  {
    constexpr int kPer = 2, kMany = 32;
    static_assert(kSamples == kPer * kCellThreads && kSamples * sizeof(int) <= sizeof(s_p), "a sample of two entries a thread");
    const bool odd = (tid & 1) != 0;
    float own = odd ? own_p : own_q, lost = __shfl_xor(odd ? own_q : own_p, 1);
    int at_own = odd ? at_p : at_q, at_lost = __shfl_xor(odd ? at_q : at_p, 1);
    if (lost > own) {
      const float x = own; own = lost; lost = x;
      const int a = at_own; at_own = at_lost; at_lost = a;
    }
    int valid = 0, n_valid;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const float largest = e == 0 ? lost : own;
      const double m = odd ? mp.of(largest) : mq.of(largest);
      const bool heavy = m >= kHeavy * (odd ? zp : zq);
      int i = e == 0 ? at_lost : at_own;
      bool counts = true;
      if (e == 0 && !heavy) {
        const unsigned j = (unsigned)tid, jitter = j * 0x9E3779B9u;
        i = (int)(((unsigned long long)j * (unsigned)V + (((unsigned long long)jitter * (unsigned)V) >> 32)) / kSpread);
      } else {
        counts = m >= kCounts;
      }
      const float xp = elem<E>(prow, i), xq = elem<E>(qrow, i);
      const float d = distance(xp, xq, mp.log2_of(xp), mq.log2_of(xq));
      const bool has_place = counts && fabsf(d) < kSumFar;
      s_sample[e * kCellThreads + tid] = has_place ? 2 * short_place(place_of(d)) + (heavy ? 1 : 0) : 0x7FFFFFFF;
      valid += has_place ? 1 : 0;
    }
    block_prefix(valid, s_redi, &n_valid);
    // sorted: a wavefront holds 128 entries, lane l the l-th and the (64 + l)-th, and exchanges them between lanes (66 rounds
    // through LDS took 12 us of a row's 240, so 6)
    {
      const int base = (tid >> 6) * 128 + (tid & 63);
      int x[kPer];
#pragma unroll
      for (int e = 0; e < kPer; ++e) x[e] = s_sample[base + 64 * e];
#pragma unroll 1
      for (int size = 2; size <= kSamples; size <<= 1) {
        if (size >= 256) {
#pragma unroll
          for (int e = 0; e < kPer; ++e) s_sample[base + 64 * e] = x[e];
#pragma unroll 1
          for (int stride = size >> 1; stride >= 128; stride >>= 1) {
            __syncthreads();
            const int lo = 2 * tid - (tid & (stride - 1)), hi = lo + stride;
            const int a = s_sample[lo], b = s_sample[hi];
            if ((a > b) == ((lo & size) == 0)) { s_sample[lo] = b; s_sample[hi] = a; }
          }
          __syncthreads();
#pragma unroll
          for (int e = 0; e < kPer; ++e) x[e] = s_sample[base + 64 * e];
        }
        if (size >= 128) {
          const int lo = min(x[0], x[1]), hi = max(x[0], x[1]);
          const bool up = (base & size) == 0;
          x[0] = up ? lo : hi;
          x[1] = up ? hi : lo;
        }
#pragma unroll
        for (int stride = 32; stride >= 1; stride >>= 1)
          if (stride < size) {  // (uniform)
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
              int other;
              switch (stride) {
                case 1: other = from_lane<kXor1>(x[e]); break;
                case 2: other = from_lane<kXor2>(x[e]); break;
                case 4: other = from_lane<kXor3>(from_lane<kMirror8>(x[e])); break;
                case 8: other = from_lane<kXor8>(x[e]); break;
                case 16: other = __builtin_amdgcn_ds_swizzle(x[e], 0x401F); break;
                default: other = __shfl_xor(x[e], stride); break;
              }
              const bool up = ((base + 64 * e) & size) == 0, lower = (tid & stride) == 0;
              x[e] = up == lower ? min(x[e], other) : max(x[e], other);
            }
          }
      }
#pragma unroll
      for (int e = 0; e < kPer; ++e) s_sample[base + 64 * e] = x[e];
    }
    __syncthreads();
    if (n_valid > 0) {  // (uniform)
      const int want = max(1, min(kQuantiles, n_valid / 16));
      // `many` equal places or more are two splitters (the place is a bucket), and so is a heavy entry's; others
      // are one, if a quantile falls into them.  As many of them as there are buckets; heavy ones go last
      int emit[kPer], total, before = 0;
      bool tied[kPer];
#pragma unroll 1
      for (int many = 4; many <= 2 * kMany; many *= 2) {
        int mine = 0;
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
          const int j = tid * kPer + e, v = s_sample[j] >> 1, run = min(many, kMany);
          emit[e] = 0;
          tied[e] = false;
          if (j < n_valid && (j == 0 || (s_sample[j - 1] >> 1) != v)) {
            int last = j;
            while (last + 1 < n_valid && last + 1 < j + run && (s_sample[last + 1] >> 1) == v) ++last;
            tied[e] = last + 1 == j + run;
            if (tied[e] || (many <= kMany && (s_sample[last] & 1) != 0)) emit[e] = 2;
            else if (j > 0 && (unsigned)(last * want) / (unsigned)n_valid != (unsigned)((j - 1) * want) / (unsigned)n_valid) emit[e] = 1;
          }
          mine += emit[e];
        }
        before = block_prefix(mine, s_redi, &total);
        if (total < kSumBuckets) break;  // uniform
      }
      nb = 1 + min(total, kSumBuckets - 1);
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const int v = long_place(s_sample[tid * kPer + e] >> 1);
        for (int c = 0; c < emit[e]; ++c, ++before)
          if (1 + before < nb) {
            s_split[1 + before] = distance_of(v + c);
            s_per_left[1 + before] = tied[e] && c == 0 ? 1.0 : 0.0;  // (on its way to the bucket's thread)
          }
      }
      far_left = uniform(distance_of(long_place(s_sample[0] >> 1)) - kBeyond);
      far_right = uniform(distance_of(long_place(s_sample[n_valid - 1] >> 1)) + kBeyond);
    }
  }
  nb = uniform(nb);
  if (tid == 0) { s_single = 0; s_shared = 0; s_most = 0; s_per_left[0] = 0.0; }
  for (int b = tid; b < 2 * kSumBuckets; b += kCellThreads)
    if (b == 0 || b >= nb) s_split[b] = b == 0 ? ninf : kNoSplitter;
  __syncthreads();
  // an entry's bucket is looked for among the splitters that share its part of the range
  const float grid_per = uniform((float)kCellThreads / (far_right - far_left));
  auto part_of = [&](const float d) {
    return (int)__builtin_amdgcn_fmed3f((d - far_left) * grid_per, 0.0f, (float)(kCellThreads - 1));
  };
  bool one_place = false, shared_place = false;
  if (tid >= 1 && tid + 1 < nb) {
    one_place = place_of(s_split[tid + 1]) <= place_of(s_split[tid]) + 1;
    shared_place = one_place && s_per_left[tid] != 0.0;
  }
  {
    int b = 0;  // splitters in the parts before this thread's
#pragma unroll 1
    for (int step = kSumBuckets / 2; step >= 1; step >>= 1)
      if (b + step < nb && part_of(s_split[b + step]) < tid) b += step;
    s_grid[tid] = (unsigned short)b;
    const unsigned long long singles = __ballot(one_place), shared = __ballot(shared_place);
    if ((tid & 63) == 0 && singles != 0ull) {
      atomicAdd(&s_single, __popcll(singles));
      atomicAdd(&s_shared, __popcll(shared));
    }
    __syncthreads();
    const int here = (tid + 1 < kCellThreads ? (int)s_grid[tid + 1] : nb - 1) - b;
    int most = here;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) most = max(most, __shfl_xor(most, d));
    if ((tid & 63) == 0) atomicMax(&s_most, most);
    __syncthreads();
  }
  const int most = uniform(s_most), n_single = uniform(s_single), n_shared = uniform(s_shared), steps = most > 0 ? 32 - __builtin_clz(most) : 0;
  // cells: the outer buckets get kOuterCells each, a single place has one, the others share the rest evenly.  A place that the
  // sample holds often has as many as there is room for, which its entries take by their lane: additions to one address wait for each
  // other (512 x 152 064 bf16, whose bulk has some fifty ratios, 736 us with one cell a place, 518; 512 x 128 256 bf16, T = 0.7, 634, 467)
  int copies = 8;
  while (n_shared * copies > kSumCells / 14) copies >>= 1;
  copies = max(copies, 1);
  const int single_cells = n_single + n_shared * (copies - 1);
  int my_cells = 0;  // of bucket number `tid`
  if (tid < nb)
    my_cells = nb <= 2 ? kSumCells / nb : one_place ? (shared_place ? copies : 1) : tid == 0 || tid + 1 == nb ? kOuterCells :
               (kSumCells - 2 * kOuterCells - single_cells) / (nb - 2 - n_single);

#pragma unroll 1
  for (int round = 0;; ++round) {
    const double step_p = uniform(step_for(s_total[0])), step_q = uniform(step_for(s_total[1]));
    int in_all;
    const int my_first = block_prefix(my_cells, s_redi, &in_all);
    if (tid < nb) {
      const float left = tid > 0 ? s_split[tid] : far_left, right = tid + 1 < nb ? s_split[tid + 1] : far_right;
      const float per = one_place ? -kLaneStep : right > left ? (float)my_cells / (right - left) : 0.0f;
      s_per_left[tid] = exp2_of(-(double)left) * (step_q / step_p);
      s_bucket[tid] = make_float4(left, per, __int_as_float(my_first), __int_as_float(__float_as_int((float)my_cells) - 1));
    }
    for (int c = tid; c <= kSumCells; c += kCellThreads) {
      s_p[c] = 0ull;
      s_q[c] = 0ull;
      if (c < kSumCells) s_u2[c] = 0u;
    }
    __syncthreads();

    // ---- second pass: the cells' sums, tv and the relaxed sums
    const double rho = uniform(s_total[1] / s_total[0]);  // p relative to the target's largest mass (1 where the sides are alike)
    const float to_u2 = uniform((float)(kU2Units / s_total[0]));
    double tv = 0.0, p_first = 0.0, relaxed[4] = {0.0, 0.0, 0.0, 0.0};
    const float lane_step = (float)(tid & (copies - 1)) * (1.0f / kLaneStep);  // (nothing to a distance, a cell where a place has several)
    const bool first_round = round == 0, four_sizes = p.n_k > 2, want_relaxed = first_round && p.relaxed != nullptr;
    float4 next_p = four<E>(prow, tid * 4, V, none), next_q = four<E>(qrow, tid * 4, V, none);
    float up = (float)((uint32_t)tid * kDitherStep >> 8) * 0x1p-24f;
    Steps stage(V);
#pragma unroll 1
    for (int i = tid * 4; i < V; i += kCellThreads * 4) {
      stage.next();
      const float4 xp4 = next_p, xq4 = next_q;
      if (i + kCellThreads * 4 < V) {
        next_p = four<E>(prow, i + kCellThreads * 4, V, none);
        next_q = four<E>(qrow, i + kCellThreads * 4, V, none);
      }
      // (what an entry's share of the third sum is rounded up or down by, so that sums are right on average: a number from 0 to 1 that belongs
      // to its place in the row, and for its neighbour what is left to 1)
      up = __builtin_amdgcn_fractf(up + (float)(kGroupStep >> 8) * 0x1p-24f);
      double ep[4], eq[4];
      float d[4];
      int b[4];
      // (the four entries side by side: their look-ups are chains of reads from LDS)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float xp = at(xp4, j), xq = at(xq4, j);
        double yp = 0.0, yq = 0.0;
        if (PROBS) {
          ep[j] = mp.of(xp);
          eq[j] = mq.of(xq);
        } else {
          yp = mp.log2_of(xp);
          yq = mq.log2_of(xq);
          ep[j] = exp2_of(yp);
          eq[j] = exp2_of(yq);
        }
        d[j] = distance(xp, xq, yp, yq);
        b[j] = s_grid[part_of(fabsf(d[j]) < kSumFar ? d[j] : 0.0f)];
      }
      find_buckets(s_split, steps, d, b);
      float4 bu[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) bu[j] = s_bucket[b[j]];
      // (all four before the first is used, not each where it is)
#pragma unroll
      for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(bu[j].x), "+v"(bu[j].y), "+v"(bu[j].z), "+v"(bu[j].w));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (fabsf(d[j]) < kSumFar) {
          const float t = __builtin_amdgcn_fmed3f(((d[j] - bu[j].x) - lane_step) * bu[j].y, 0.0f, bu[j].w);
          const int cell = (int)t + __float_as_int(bu[j].z);
          const float u = __builtin_amdgcn_fractf(t);
          atomicAdd(&s_p[cell], whole_mass(ep[j], step_p));
          atomicAdd(&s_q[cell], whole_mass(eq[j], step_q));
          atomicAdd(&s_u2[cell], saturated(fmaf((float)ep[j] * to_u2, fmaf(-u, u, u), (j & 1) != 0 ? 1.0f - up : up)));
        } else {
          // ratio 0, or near it: before all others (an entry without a cell that has the larger ratio has no
          // p-mass to speak of)
          p_first += ep[j];
        }
      }
      if (first_round) {
        // (fetched here each time: there are no registers to hold them, of either kind)
        int from = 0;
        asm volatile("" : "+v"(from));
        const double k[4] = {s_sizes[from], s_sizes[from + 1], s_sizes[from + 2], s_sizes[from + 3]};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          ep[j] *= rho;
          tv += fabs(ep[j] - eq[j]);
        }
        if (want_relaxed && four_sizes) {
#pragma unroll
          for (int j = 0; j < 4; ++j) add_relaxed<2>(relaxed, k, ep[j], eq[j]);
        } else if (want_relaxed) {
#pragma unroll
          for (int j = 0; j < 4; ++j) add_relaxed<1>(relaxed, k, ep[j], eq[j]);
        }
      }
    }
    stage.done();
    const LmlParams &again = params_again();
    const double norm_p = 1.0 / s_total[0], norm_q = 1.0 / s_total[1], unit_p = 0x1p-52 * step_p * norm_p,
                 unit_q = 0x1p-52 * step_q * norm_q;
    bool bad = false;
    {
      double sums[6] = {p_first, tv, relaxed[0], relaxed[1], relaxed[2], relaxed[3]};
      block_sums(sums, s_red);
      p_first = uniform(sums[0]);
      if (first_round) {
        if (tid == 0 && again.tv != nullptr) again.tv[b_row] = 0.5 * sums[1] * norm_q;
#pragma unroll
        for (int n = 0; n < 4; ++n)
          if (want_relaxed && n < again.n_k) {
            const double r = again.kd[n] * sums[2 + n] * norm_q;
            if (!(r >= kLeastRelaxed)) bad = true;
            if (tid == 0) again.relaxed[b_row * again.n_k + n] = r;
          }
      }
    }
    if (bad) {  // (uniform)
      leave();
      return;
    }
    const double first = p_first * norm_p;
    {
      unsigned long long all;
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        unsigned long long *m = side == 0 ? s_p : s_q, mine[kSumEach], sum = 0ull;
#pragma unroll
        for (int e = 0; e < kSumEach; ++e) { mine[e] = m[tid * kSumEach + e]; sum += mine[e]; }
        unsigned long long before = block_prefix(sum, s_redu, &all);
#pragma unroll
        for (int e = 0; e < kSumEach; ++e) { m[tid * kSumEach + e] = before; before += mine[e]; }
        if (tid == kCellThreads - 1) m[kSumCells] = before;
      }
    }
    __syncthreads();

    // ---- the cells' terms, list sizes four at a time
    // what rounding may have done to the masses before and behind a cell (four deviations of such a sum), and in all
    const float root = sqrtf((float)V), slip_u2 = (float)(1.0 / kU2Units) * root, slip = 2.0f * root, slip_p = slip * (float)unit_p, slip_q = slip * (float)unit_q;
    const double lost_p = 0.5 * unit_p * (double)V, lost_q = 0.5 * unit_q * (double)V;
    const double may_be_open = fmin(fmax((double)V * kSumErrorEach, kSumErrorLeast), 1.0) * kRowError;
    bool open = false;
    double worst = 0.0;  // the largest doubt of a result, relative to it
#pragma unroll 1
    for (int n0 = 0; n0 < again.n_k; n0 += 4) {
      // per list size and without its factor K: terms as if nothing were spread, what spread takes from them, what is open
      double whole[4] = {0.0, 0.0, 0.0, 0.0};
      float taken[4] = {0.0f, 0.0f, 0.0f, 0.0f}, left_open[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      int c = tid * kSumEach, b = 0;  // the cell at hand and its bucket
#pragma unroll 1
      for (int step = kSumBuckets / 2; step >= 1; step >>= 1)
        if (b + step < nb && __float_as_int(s_bucket[b + step].z) <= c) b += step;
      unsigned long long here_p = s_p[c], here_q = s_q[c];
      double sum_p = (double)here_p, sum_q = (double)here_q;  // up to the cell
#pragma unroll 1
      for (const int end = c + kSumEach; c < end; ++c) {
        while (b + 1 < nb && __float_as_int(s_bucket[b + 1].z) <= c) ++b;
        const float4 bu = s_bucket[b];
        const unsigned long long next_p = s_p[c + 1], next_q = s_q[c + 1];
        const double raw_p = (double)(next_p - here_p), raw_q = (double)(next_q - here_q);
        here_p = next_p;
        here_q = next_q;
        const double P = raw_p * unit_p, Q = raw_q * unit_q, before = fma(sum_p, unit_p, first);
        sum_p += raw_p;
        sum_q += raw_q;
        const double behind = fmax(fma(-unit_q, sum_q, 1.0), 0.0);
        float doubt = 0.0f;
        if (raw_p > 0.0 && raw_q > 0.0) {
          float v = 0.0f, half_g = 0.0f, half_g_open = 0.0f, v_open = 0.0f;
          bool wide = false;
          const float fp = (float)P, per_p = __builtin_amdgcn_rcpf(fp);
          if (bu.y > 0.0f) {
            const int place = c - __float_as_int(bu.z);
            const float w = 0.69314718f * __builtin_amdgcn_rcpf(bu.y);  // (in ln r)
            wide = w > kWide || (b == 0 && place == 0) || (b + 1 == nb && place == (int)bu.w);  // (or an end: what lies beyond it is in it)
            // log2 of the mean ratio less the bucket's left end, in cells: ln(1 + t) = 2 artanh(t / (2 + t)) for small t
            const double ratio = raw_q * reciprocal(raw_p) * s_per_left[b];
            const float t = (float)(ratio - 1.0), z = t * __builtin_amdgcn_rcpf(2.0f + t), zz = z * z;
            const float small = z * fmaf(zz, fmaf(zz, fmaf(zz, 2.8853901f / 7.0f, 2.8853901f / 5.0f), 2.8853901f / 3.0f), 2.8853901f);
            const float m = (t < 0.4f ? small : __builtin_amdgcn_logf((float)ratio)) * bu.y - (float)place;
            const float within = (float)s_u2[c] * (float)(1.0 / kU2Units) * per_p;  // the mean of u (1 - u): u's variance is this below mean (1 - mean)
            // what rounding may have done to it: an entry's has a variance of no more than a quarter, nor more than what it adds.  Two deviations as if the
            // cell had all of the row's entries, which is four or more of the sum over the cells unless one of them has nearly all
            const float slip_var = fp < kU2Most ? fminf(fminf(slip_u2 * per_p, kU2Slip * __builtin_amdgcn_sqrtf(per_p)), 0.25f) : 0.25f;
            float var, mean = m;
#pragma unroll
            for (int it = 0; it < 2; ++it) {  // the logarithm of the mean ratio is half a variance above the mean place
              var = fmaxf(fmaf(-mean, mean, mean) - within, 0.0f);
              mean = __builtin_amdgcn_fmed3f(fmaf(-0.5f * w, var, m), 0.0f, 1.0f);
            }
            var = fmaxf(fmaf(-mean, mean, mean) - within, 0.0f);
            const float var_open = fmaf(0.02f * w, w, var + slip_var);  // (and a third power more)
            v = var * w * w;
            v_open = fmaf(0.25f * w, var_open, slip_var) * w * w;
            half_g = 2.0f * var * w;
            half_g_open = w * fmaxf(var_open, __builtin_amdgcn_sqrtf(var_open * (1.0f / 3.0f)) - 2.0f * var);
          }
          const double half = fma(0.5, P, before), base = fma(behind + Q, P, Q * before);
          const float half_per_p = (float)half * per_p, slips = slip_p * (__builtin_amdgcn_rcpf((float)half) + per_p);
          double den[4];
#pragma unroll
          for (int n = 0; n < 4; ++n) den[n] = fma(again.kd[n0 + n] - 1.0, P, base);
          const double d01 = den[0] * den[1], d23 = den[2] * den[3], all = P * Q * reciprocal(d01 * d23);
          const double r01 = all * d23, r23 = all * d01;
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const double term = (n < 2 ? r01 : r23) * den[n ^ 1];  // P x
            whole[n] += term;
            const float xp = (float)term, xh = xp * half_per_p;    // x times P, and times P' + P / 2
            taken[n] = fmaf(xp, fmaf(xp, half_g, xh * v * (1.0f - xh)), taken[n]);
            const float left = wide ? xp : xp * fmaf(xp, half_g_open, v_open);
            left_open[n] += fmaf(xp, fmaf(xh, slips, slip_q), left);
            doubt += left * (float)again.kd[n0 + n];
          }
        } else if (raw_q > 0.0) {
          // no p-mass that its sum would show: K q / (F + K - 1), where F is no less than 1 or than r times the p-mass before
          const float most = (float)lost_p * __builtin_amdgcn_rcpf(fmaxf((float)before, 0x1p-60f));
#pragma unroll
          for (int n = 0; n < 4; ++n) left_open[n] += fminf((float)Q * __builtin_amdgcn_rcpf((float)again.kd[n0 + n]), most);
        }
        if (n0 + 4 >= again.n_k) s_u2[c] = __float_as_uint(doubt);  // (for sharing the cells out again)
      }
      double sums[8];
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        sums[n] = (whole[n] - (double)taken[n]) * again.kd[n0 + n];
        sums[4 + n] = (double)left_open[n] * again.kd[n0 + n];
      }
      block_sums(sums, s_red);
#pragma unroll
      for (int n = 0; n < 4; ++n)
        if (n0 + n < again.n_k) {
          const double left = sums[4 + n] + lost_q;
          if (!(left <= may_be_open * sums[n])) open = true;
          worst = fmax(worst, sums[n] > 0.0 ? left / sums[n] : 1.0);
          if (tid == 0) again.bound[b_row * again.n_k + n0 + n] = sums[n];
        }
    }
    if (!open) break;  // (uniform)
    // (a shorter row with little too much is quicker left to the other form, which looks at its entries one by one)
    if (round == 1 || !(worst <= kShareAgain) || (V < kAgainMinV && worst <= kRowError)) {
      leave();
      return;
    }
    // cells where they are wanted: what a bucket leaves open falls with the square of the number of its cells, so the sum over all
    // buckets is least with numbers that go with the cube root of that times the present number squared; no fewer than keep
    // its cells narrow, up to a point
    float wants = 0.0f;
    int fewest = 0;
    if (tid < nb && !one_place) {
      const float width = (tid + 1 < nb ? s_split[tid + 1] : far_right) - (tid > 0 ? s_split[tid] : far_left);
      fewest = min(max((int)(width * (2.0f * 0.69314718f / kWide)), kFewestCells), my_cells);
      for (int c = my_first; c < my_first + my_cells; ++c) wants += __uint_as_float(s_u2[c]);
      if (wants > 0.0f) wants = exp2f(log2f(wants * (float)my_cells * (float)my_cells) * (1.0f / 3.0f));
    }
    const float wanted = (float)block_sum((double)wants, s_red);
    int all_fewest;
    block_prefix(fewest, s_redi, &all_fewest);
    if (tid < nb && !one_place && wanted > 0.0f)
      my_cells = fewest + (int)((float)(kSumCells - 1 - single_cells - all_fewest) * (wants / wanted));
  }
  // ---- the relaxed sums of the fifth list size on: one more pass
#pragma unroll 1
  for (int n0 = 4; n0 < p.n_k && p.relaxed != nullptr; n0 += 4) {
    const double rho = s_total[1] / s_total[0], norm_q = 1.0 / s_total[1];
    double relaxed[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int i = tid * 4; i < V; i += kCellThreads * 4) {
      const float4 xp4 = four<E>(prow, i, V, none), xq4 = four<E>(qrow, i, V, none);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double pp = mp.of(at(xp4, j)) * rho, eq = mq.of(at(xq4, j));
        add_relaxed<2>(relaxed, p.kd + n0, pp, eq);
      }
    }
    block_sums(relaxed, s_red);
    bool bad = false;
#pragma unroll
    for (int n = 0; n < 4; ++n)
      if (n0 + n < p.n_k) {
        const double r = p.kd[n0 + n] * relaxed[n] * norm_q;
        if (!(r >= kLeastRelaxed)) bad = true;
        if (tid == 0) p.relaxed[b_row * p.n_k + n0 + n] = r;
      }
    if (bad) leave();
  }
}

// ---- rows that fit into LDS, sorted there

constexpr int kShortThreads = 1024, kShortWaves = kShortThreads / 64;
constexpr int kCountRow = 260;  // a wavefront's 256 counters and some: four wavefronts' counters of a digit lie in different banks

// Rows too short for the forms by cells, up to ROUNDS * 1024 entries, one workgroup each; a thread holds an entry of every 1024.  The
// same sort as lml_sort_kernel's, but nothing passes through memory: an entry is its key and its index, eight bytes that go
// from LDS to registers and back in each of the four passes, and the masses stay where they are.
// What bounds it: issue (some 60 instructions an entry and pass to find the lanes with its digit, an exponential and side) and, in the
// shortest rows, the chain of four passes with four barriers each.  Two workgroups of up to 4 rounds fit on a CU (64 registers, 75 KB).
// us a call of four list sizes, through memory (lml_sort_kernel, 512 threads) and here, 1, 64, 512 and 4096 rows: fp32 1000 entries 33, 34, 47, 371 and
// 16, 16, 26, 161; 2000: 39, 40, 58, 456 and 20, 21, 34, 220; 4096: 56, 57, 90, 708 and 29, 30, 50, 338; 6000: 83, 85, 140, 1121 and
// 40, 42, 82, 634; bf16 8191: 96, 100, 158, 1261 and 48, 48, 97, 780.  Errors against 64 bits are the same.
template <typename E, int ROUNDS>
__global__ void __launch_bounds__(kShortThreads, ROUNDS <= 4 ? 8 : 4) lml_short_kernel(const LmlParams p) {
  constexpr int kEntries = ROUNDS * kShortThreads;
  __shared__ unsigned long long s_row[kEntries];  // key, index
  __shared__ float2 s_mass[kEntries];
  __shared__ unsigned short s_cnt[kShortWaves][kCountRow];  // per wavefront and digit: counts, then starts
  __shared__ double s_out[2 * kLmlMaxK + 1][kShortWaves];   // bounds, relaxed sums, tv: the wavefronts' shares
  __shared__ double s_red[2 * kShortWaves], s_seg[2][kShortWaves];
  __shared__ float s_top[2][kShortWaves];
  __shared__ int s_tot[kShortWaves];
  static_assert(kShortWaves == 16, "a lane of sixteen for every wavefront");

  const int tid = threadIdx.x, lane = tid & 63, wv = uniform(tid >> 6);
  const long long b = p.row0 + blockIdx.x;
  const int V = p.V, rounds = (V + kShortThreads - 1) / kShortThreads;
  const float finf = __builtin_huge_valf();
  const double ninf = -__builtin_huge_val();
  float x[ROUNDS], y[ROUNDS];
  {
    const E *prow = reinterpret_cast<const E *>(p.draft) + b * p.draft_stride_b;
    const E *qrow = reinterpret_cast<const E *>(p.target) + b * p.target_stride_b;
#pragma unroll
    for (int e = 0; e < ROUNDS; ++e) {
      const int i = e * kShortThreads + tid;  // (behind the row: no mass)
      x[e] = i < V ? elem<E>(prow, i) : __builtin_nanf("");
      y[e] = i < V ? elem<E>(qrow, i) : __builtin_nanf("");
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) s_cnt[wv][q * 64 + lane] = 0;

  // ---- the two sides' largest finite values and masses
  Side sp, sq;
  sp.probs = sq.probs = p.probs;
  sp.inv_t = 1.0 / (double)p.temp_draft;
  sq.inv_t = 1.0 / (double)p.temp_target;
  sp.m = sq.m = ninf;
  if (!p.probs) {
    float top_p = -finf, top_q = -finf;
#pragma unroll
    for (int e = 0; e < ROUNDS; ++e) {
      if (x[e] < finf) top_p = fmaxf(top_p, x[e]);
      if (y[e] < finf) top_q = fmaxf(top_q, y[e]);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      top_p = fmaxf(top_p, __shfl_xor(top_p, d));
      top_q = fmaxf(top_q, __shfl_xor(top_q, d));
    }
    if (lane == 0) { s_top[0][wv] = top_p; s_top[1][wv] = top_q; }
    __syncthreads();
    top_p = s_top[0][lane & 15];
    top_q = s_top[1][lane & 15];
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) {
      top_p = fmaxf(top_p, __shfl_xor(top_p, d));
      top_q = fmaxf(top_q, __shfl_xor(top_q, d));
    }
    sp.m = (double)uniform(top_p);
    sq.m = (double)uniform(top_q);
  }
  // (masses, relative to the largest at first; kept: an exponential takes longer than all else about an entry)
  double pm[ROUNDS], qm[ROUNDS], z[2] = {0.0, 0.0};
  auto mass_of = [&](const Side &side, float v) {
    if (p.probs) return v > 0.0f && v < finf ? (double)v : 0.0;
    return v < finf && v > -finf ? exp(((double)v - side.m) * side.inv_t) : 0.0;
  };
#pragma unroll
  for (int e = 0; e < ROUNDS; ++e) {
    pm[e] = qm[e] = 0.0;
    if (e < rounds) {
      pm[e] = mass_of(sp, x[e]);
      qm[e] = mass_of(sq, y[e]);
      z[0] += pm[e];
      z[1] += qm[e];
    }
  }
  block_sums(z, s_red);
  sp.ln_z = log(z[0]);
  sq.ln_z = log(z[1]);
  const double norm_p = z[0] > 0.0 ? 1.0 / z[0] : 0.0, norm_q = z[1] > 0.0 ? 1.0 / z[1] : 0.0;

  // ---- keys and masses, and the sums that need no order
  double tv = 0.0;
#pragma unroll
  for (int e = 0; e < ROUNDS; ++e)
    if (e < rounds) {
#pragma clang fp contract(off)  // (equal masses differ by 0)
      const int i = e * kShortThreads + tid;
      const double lp = sp.log_mass(x[e]), lq = sq.log_mass(y[e]);
      const bool hp = lp > ninf, hq = lq > ninf;
      float lr = -finf;             // no target mass (or none at all): sorts first
      if (hq) lr = hp ? (float)(lq - lp) : finf;
      pm[e] *= norm_p;
      qm[e] *= norm_q;
      tv += fabs(pm[e] - qm[e]);
      s_row[i] = ((unsigned long long)sort_key(lr) << 32) | (uint32_t)i;
      s_mass[i] = make_float2((float)pm[e], (float)qm[e]);
    }
  tv = wave_sum(tv);
  if (lane == 63) s_out[2 * kLmlMaxK][wv] = tv;
#pragma unroll 1
  for (int kk = 0; kk < p.n_k; ++kk) {
    const double K = p.kd[kk];
    double sum = 0.0;  // of q / (1 + q / (K p)) with one division
#pragma unroll
    for (int e = 0; e < ROUNDS; ++e)
      if (e < rounds) {
        const double kp = K * pm[e], kpq = kp * qm[e];
        if (kpq > 0.0) sum += kpq / (kp + qm[e]);
      }
    sum = wave_sum(sum);
    if (lane == 63) s_out[kLmlMaxK + kk][wv] = sum;
  }
  __syncthreads();

  // ---- stable radix sort, 8 bits a pass; wavefront w holds the w-th part of the row, `rounds` times 64 entries
  const int from = wv * 64 * rounds + lane;
#pragma unroll 1
  for (int shift = 32; shift < 64; shift += 8) {
    unsigned long long entry[ROUNDS];
    int where[ROUNDS];  // digit, and rank among the wavefront's entries of it
#pragma unroll
    for (int e = 0; e < ROUNDS; ++e)
      if (e < rounds) entry[e] = s_row[from + e * 64];
#pragma unroll
    for (int e = 0; e < ROUNDS; ++e)
      if (e < rounds) {
        const uint32_t d = (uint32_t)(entry[e] >> shift) & 255u;
        uint32_t peers_lo = ~0u, peers_hi = ~0u;  // lanes with the same digit: bit by bit, keep those whose bit is like mine
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
          const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe((int)d, bit, 1);  // all ones if the bit is set
          const unsigned long long have = __ballot(mine != 0u);
          peers_lo &= ~((uint32_t)have ^ mine);
          peers_hi &= ~((uint32_t)(have >> 32) ^ mine);
        }
        const int rank = (int)__builtin_amdgcn_mbcnt_hi(peers_hi, __builtin_amdgcn_mbcnt_lo(peers_lo, 0u));
        const int seen = s_cnt[wv][d];
        if (rank == 0) s_cnt[wv][d] = (unsigned short)(seen + __popc(peers_lo) + __popc(peers_hi));
        where[e] = seen + rank;
        __builtin_amdgcn_wave_barrier();
      }
    __syncthreads();
    {
      // four wavefronts' counters of a digit a thread, in the order of digits and wavefronts: what is before each
      const int d = tid >> 2, w0 = (tid & 3) * 4;
      int c[4], sum = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        c[j] = sum;
        sum += s_cnt[w0 + j][d];
      }
      const int incl = wave_prefix(sum);
      if (lane == 63) s_tot[wv] = incl;
      __syncthreads();
      const int before = of_lane(prefix_of_16((lane & 15) < wv ? s_tot[lane & 15] : 0), 15) + incl - sum;
#pragma unroll
      for (int j = 0; j < 4; ++j) s_cnt[w0 + j][d] = (unsigned short)(before + c[j]);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < ROUNDS; ++e)
      if (e < rounds) s_row[s_cnt[wv][(uint32_t)(entry[e] >> shift) & 255u] + where[e]] = entry[e];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 4; ++q) s_cnt[wv][q * 64 + lane] = 0;  // (this wavefront's only, until the next pass's first barrier)
    __syncthreads();
  }

  // ---- running sums over the sorted order: every wavefront's part, then each walks its own with those before it as the carry
  float2 mass[ROUNDS];
  double all_p = 0.0, all_q = 0.0;
#pragma unroll
  for (int e = 0; e < ROUNDS; ++e) {
    mass[e] = make_float2(0.0f, 0.0f);
    if (e < rounds) mass[e] = s_mass[(uint32_t)s_row[from + e * 64]];
    all_p += (double)mass[e].x;
    all_q += (double)mass[e].y;
  }
  all_p = wave_sum(all_p);
  all_q = wave_sum(all_q);
  if (lane == 63) { s_seg[0][wv] = all_p; s_seg[1][wv] = all_q; }
  __syncthreads();
  const double upto_p = prefix_of_16(s_seg[0][lane & 15]), upto_q = prefix_of_16(s_seg[1][lane & 15]);
  const double q_total = of_lane(upto_q, 15);
  double p_before = wv > 0 ? of_lane(upto_p, wv - 1) : 0.0, q_before = wv > 0 ? of_lane(upto_q, wv - 1) : 0.0;
  double common[ROUNDS];  // q_suf/q_j + p_pre/p_j, times q_j
#pragma unroll
  for (int e = 0; e < ROUNDS; ++e) {
    common[e] = 0.0;
    if (e < rounds) {
      const double pj = (double)mass[e].x, qj = (double)mass[e].y;
      const double pin = wave_prefix(pj), qin = wave_prefix(qj);  // inclusive sums over the lanes
      if (pj > 0.0 && qj > 0.0)
        common[e] = (q_total - (q_before + (qin - qj))) + (p_before + (pin - pj)) * (qj / pj);
      else
        mass[e].y = 0.0f;
      p_before += of_lane(pin, 63);
      q_before += of_lane(qin, 63);
    }
  }
#pragma unroll 1
  for (int kk = 0; kk < p.n_k; ++kk) {
    const double K = p.kd[kk];
    double sum = 0.0;
#pragma unroll
    for (int e = 0; e < ROUNDS; ++e)
      if (e < rounds && mass[e].y > 0.0f) sum += K * (double)mass[e].y / (common[e] + (K - 1.0) * q_total);
    sum = wave_sum(sum);
    if (lane == 63) s_out[kk][wv] = sum;
  }
  __syncthreads();
  // sixteen lanes a result
  const int result = tid >> 4, kk = result < kLmlMaxK ? result : result - kLmlMaxK;
  if (wv * 4 > 2 * kLmlMaxK) return;  // (whole wavefronts)
  const double sum = sum_of_16(s_out[min(result, 2 * kLmlMaxK)][tid & 15]);
  if ((tid & 15) != 0 || result > 2 * kLmlMaxK) return;
  if (result == 2 * kLmlMaxK) {
    if (p.tv != nullptr) p.tv[b] = 0.5 * sum;
  } else if (kk < p.n_k) {
    if (result < kLmlMaxK) p.bound[b * p.n_k + kk] = sum;
    else if (p.relaxed != nullptr) p.relaxed[b * p.n_k + kk] = sum;
  }
}

}  // namespace

hipError_t launch_lml(hipStream_t s, const LmlParams &params) {
  LmlParams p = params;
  const bool f32 = p.dtype == LLC_F32;
  const bool cells = p.V >= (f32 ? kCellMinV : kCellMinVNarrow) && p.V <= kCellMaxV;
  // (no workspace: as many rows as a launch may have threads for)
  constexpr long long kMostRows = 1 << 21;
  if (!cells && p.V <= 8 * kShortThreads) {
    static_assert(kCellMinV <= 8 * kShortThreads && kCellMinVNarrow <= 8 * kShortThreads, "shorter rows fit into LDS");
    for (p.row0 = 0; p.row0 < p.B; p.row0 += kMostRows) {
      const dim3 grid((unsigned)(p.B - p.row0 < kMostRows ? p.B - p.row0 : kMostRows)), block(kShortThreads);
      if (p.V <= 4 * kShortThreads) {
        if (f32) hipLaunchKernelGGL((lml_short_kernel<float, 4>), grid, block, 0, s, p);
        else hipLaunchKernelGGL((lml_short_kernel<uint16_t, 4>), grid, block, 0, s, p);
      } else {
        if (f32) hipLaunchKernelGGL((lml_short_kernel<float, 8>), grid, block, 0, s, p);
        else hipLaunchKernelGGL((lml_short_kernel<uint16_t, 8>), grid, block, 0, s, p);
      }
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  p.only_flagged = cells ? 1 : 0;
#define LLC_LML(KERNEL, ROWS)                                                                            \
  {                                                                                                      \
    if (f32 && p.probs) hipLaunchKernelGGL((KERNEL<float, true>), dim3(ROWS), dim3(kCellThreads), 0, s, p);        \
    else if (f32) hipLaunchKernelGGL((KERNEL<float, false>), dim3(ROWS), dim3(kCellThreads), 0, s, p);             \
    else if (p.probs) hipLaunchKernelGGL((KERNEL<uint16_t, true>), dim3(ROWS), dim3(kCellThreads), 0, s, p);       \
    else hipLaunchKernelGGL((KERNEL<uint16_t, false>), dim3(ROWS), dim3(kCellThreads), 0, s, p);                   \
    const hipError_t e = hipGetLastError();                                                              \
    if (e != hipSuccess) return e;                                                                       \
  }
  for (p.row0 = 0; cells && p.row0 < p.B; p.row0 += kMostRows)
    LLC_LML(lml_sum_kernel, (unsigned)(p.B - p.row0 < kMostRows ? p.B - p.row0 : kMostRows))
  for (p.row0 = 0; p.row0 < p.B; p.row0 += p.slots) {
    const long long left = p.B - p.row0;
    const unsigned grid = (unsigned)(left < (long long)p.slots ? left : (long long)p.slots);
    // (the rows that the form by sums left, as a rule none, and behind it those that this one left)
    if (cells) LLC_LML(lml_cell_kernel, grid)
    if (f32) hipLaunchKernelGGL(lml_sort_kernel<float>, dim3(grid), dim3(kThreads), 0, s, p);
    else hipLaunchKernelGGL(lml_sort_kernel<uint16_t>, dim3(grid), dim3(kThreads), 0, s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
#undef LLC_LML
  return hipSuccess;
}

}  // namespace llc
