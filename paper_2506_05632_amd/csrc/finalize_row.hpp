// The finalize step of one row: Algorithm 1's last step, accept = [Y in {X^(1..K)}] (paper Section 3),
// and the row's outputs, from its merged reductions.  Shared by the finalize kernel, which merges the
// partial results of a row that several workgroups scanned, and by the scan kernel, which finishes a
// row that is one workgroup's itself.
#pragma once

#include "common.hpp"

namespace llc {

// Smaller key wins; equal keys: smaller index, then smaller k.
__device__ __forceinline__ bool beats(double key, int idx, int k, double bkey, int bidx, int bk) {
  if (idx < 0) return false;
  if (bidx < 0) return true;
  if (key != bkey) return key < bkey;
  if (idx != bidx) return idx < bidx;
  return k < bk;
}

// A winner within this relative distance (in S/p) of the best key at another index is a near-tie.
constexpr double kNearTie = 1e-6;

// Whether the runner-up key is that close.  Log-domain keys are ln(S/p) up to a constant that both
// share, so the relative distance is expm1 of their difference.
__device__ __forceinline__ bool near_tie(double best, double second, int log_kind) {
  if (!(second < __builtin_huge_val())) return false;
  if (log_kind) return expm1(second - best) < kNearTie;
  return best > 0.0 ? (second - best) / best < kNearTie : !(second > 0.0);
}

// One reduction of a row: the smallest key, its index (-1: no entry has mass), the smallest key at
// another index, and (log kinds, where asked for) ln of the normaliser that turns keys into S/p.
struct Merged {
  double key;
  int idx;
  double sec, norm;
};

// One row, by one wavefront (all 64 lanes call it).  `pool`: the target side, the same in all lanes.
// drafts(k) gives draft k's reduction to the `width` lanes that share it (a power of two; the wavefront
// takes 64 / width drafts at a time); every lane calls it, also with k >= K.
template <typename Drafts>
__device__ __forceinline__ void finish_row(const FinalizeParams &p, const long long b, const int lane, const int width,
                                           const Merged &pool, Drafts drafts) {
  unsigned long long degenerate = 0, near = 0;
  int y = -1;
  if (p.Y != nullptr) {
    if (p.y_given) {
      // the pool's index was settled by an earlier pass (binned selection): announce its bin
      y = p.Y[b];
      if (lane == 0 && p.message != nullptr)
        p.message[b] = (y >= 0 && p.bins != nullptr) ? (int)p.bins[b * p.bins_stride_b + y] : -1;
    } else {
      y = pool.idx;
      if (lane == 0) {
        p.Y[b] = y;
        if (p.count_pool && p.stats != nullptr) {
          if (y < 0) ++degenerate;
          else if (near_tie(pool.key, pool.sec, p.log_kind)) ++near;
        }
        if (p.keyY != nullptr) {
          double out = __builtin_huge_val();
          if (y >= 0) out = p.log_kind ? exp(pool.key + pool.norm) : pool.key;
          p.keyY[b] = (float)out;
        }
      }
    }
  }
  int match = -1;
  double err = __builtin_huge_val();  // the smallest squared error among the decoders
  for (int k0 = 0; k0 < p.K; k0 += 64 / width) {
    const int k = k0 + lane / width;
    const Merged m = drafts(k);
    const bool mine = k < p.K && (lane & (width - 1)) == 0;
    if (mine) {
      p.X[b * p.K + k] = m.idx;
      if (p.count_draft && p.stats != nullptr) {
        if (m.idx < 0) ++degenerate;
        else if (near_tie(m.key, m.sec, p.log_kind)) ++near;
      }
      if (p.store_norm) p.in.lse[b * (p.K + 1) + k] = m.norm;
      if (p.log_keyX != nullptr) p.log_keyX[b * p.K + k] = m.idx >= 0 ? m.key + m.norm : __builtin_huge_val();
      if (p.log_secX != nullptr)
        p.log_secX[b * p.K + k] = (m.idx >= 0 && m.sec < __builtin_huge_val()) ? m.sec + m.norm : __builtin_huge_val();
      if (p.keyX != nullptr) {
        double out = __builtin_huge_val();
        if (m.idx >= 0) out = p.log_kind ? exp(m.key + m.norm) : m.key;
        p.keyX[b * p.K + k] = (float)out;
      }
      if (p.cand != nullptr) {
        // the decoder's output W_k = U_{X^(k)} (Appendix C) and its MMSE estimate of the source
        // (Appendix D.2), in fp64 from the fp32 inputs; NaN where the decoder found no candidate
        double w = __builtin_nan(""), est = __builtin_nan("");
        if (m.idx >= 0) {
          w = (double)p.cand[b * p.cand_stride_b + m.idx];
          if (p.side != nullptr) {
            const double t = (double)p.side[b * p.side_stride_b + k];
            est = (p.var_z * w + p.var_e * t) / (p.var_e + p.var_z + p.var_e * p.var_z);
          }
          if (p.sq_err != nullptr) {
            const double d = est - (double)p.source[b];
            const double e2 = d * d;
            if (e2 == e2) err = fmin(err, e2);
          }
        }
        if (p.W != nullptr) p.W[b * p.K + k] = (float)w;
        if (p.A_hat != nullptr) p.A_hat[b * p.K + k] = (float)est;
      }
    }
    const unsigned long long hits = __ballot(mine && y >= 0 && m.idx == y);
    if (match < 0 && hits != 0ull) match = k0 + (__ffsll((long long)hits) - 1) / width;
  }
  if (p.Y != nullptr) {
    if (p.cand != nullptr && p.sq_err != nullptr) {  // uniform
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) err = fmin(err, __shfl_xor(err, d));
      if (lane == 0) p.sq_err[b] = (float)err;
    }
    if (lane == 0) {
      p.accept[b] = match >= 0 ? 1 : 0;
      if (p.match_k != nullptr) p.match_k[b] = match;
    }
  }
  if (p.stats != nullptr && degenerate) atomicAdd(&p.stats->degenerate, degenerate);
  if (p.stats != nullptr && near && p.count_near) atomicAdd(&p.stats->near_ties, near);
}

}  // namespace llc
