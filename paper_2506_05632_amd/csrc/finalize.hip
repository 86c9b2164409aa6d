// Finalize: merge the per-chunk partial argmins of a row and take Algorithm 1's
// last step, accept = [Y in {X^(1..K)}] (paper Section 3).  Also the row
// normalisers ln sum exp(x/T) that turn log-domain keys into S/p with p
// normalised (Section 3 defines p and q as distributions; Appendix C normalises
// the importance weights the same way).
#include "finalize_row.hpp"

namespace llc {

namespace {

// Folds one more part of a draft's reduction into a running one (the parts hold different indices:
// whichever winner loses is a candidate for the runner-up).
__device__ __forceinline__ void fold_part(Merged &v, double key, int idx, double sec) {
  v.sec = fmin(v.sec, sec);
  if (beats(key, idx, 0, v.key, v.idx, 0)) {
    if (v.idx >= 0) v.sec = fmin(v.sec, v.key);
    v.key = key;
    v.idx = idx;
  } else if (idx >= 0) {
    v.sec = fmin(v.sec, key);
  }
}

// One wavefront per row.  Bound by the latency of its loads: a draft's chunk partials are fetched by
// `width` lanes at once (a power of two, at least the number of chunks if that is 64 or less) and
// merged by shuffles, 64 / width drafts at a time.  (One lane per draft walking its chunks, and one
// lane walking the pool's parts, took 5.5 us at four chunks.)
__global__ void __launch_bounds__(64) finalize_kernel(const FinalizeParams p, const int width) {
  const long long b = (long long)blockIdx.x;
  const int lane = (int)threadIdx.x, c0 = lane & (width - 1), nc = p.n_chunks;
  const bool want_sec = p.stats != nullptr || p.log_secX != nullptr;
  const double inf = __builtin_huge_val();
  // ln of a normaliser, slot k of the row: ln sum_chunks exp(share), or in place already
  auto normaliser = [&](const int k, const bool merge) {
    if (!p.need_norm || k > p.K) return 0.0;
    if (!merge) return p.in.lse[b * (p.K + 1) + k];
    const double *sh = p.in.lse_part + (b * (p.K + 1) + k) * nc;
    double m = -inf;
    for (int c = c0; c < nc; c += width) m = fmax(m, sh[c]);
    for (int d = width >> 1; d >= 1; d >>= 1) m = fmax(m, __shfl_xor(m, d));
    double sum = 0.0;
    if (m > -inf)
      for (int c = c0; c < nc; c += width) sum += exp(sh[c] - m);
    for (int d = width >> 1; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
    return m > -inf ? m + log(sum) : -inf;
  };
  Merged pool;
  pool.key = inf; pool.idx = -1; pool.sec = inf; pool.norm = 0.0;
  if (p.Y != nullptr && !p.y_given) {
    // the pool over draft groups and chunks
    const int parts = p.n_kgroups * nc;
    const long long o = b * parts;
    int bk = -1;
    for (int c = lane; c < parts; c += 64) {
      const double key = p.in.keyY[o + c];
      const int idx = p.in.idxY[o + c], k = p.in.kY[o + c];
      if (beats(key, idx, k, pool.key, pool.idx, bk)) { pool.key = key; pool.idx = idx; bk = k; }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      const double key = __shfl_xor(pool.key, d);
      const int idx = __shfl_xor(pool.idx, d), k = __shfl_xor(bk, d);
      if (beats(key, idx, k, pool.key, pool.idx, bk)) { pool.key = key; pool.idx = idx; bk = k; }
    }
    if (want_sec && p.count_pool) {
      // the runner-up at another index: a part whose winner sits at the same index (another draft
      // group met it under other race times) contributes its own runner-up instead
      for (int c = lane; c < parts; c += 64) {
        const int idx = p.in.idxY[o + c];
        if (idx >= 0) pool.sec = fmin(pool.sec, idx != pool.idx ? p.in.keyY[o + c] : p.in.secY[o + c]);
      }
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) pool.sec = fmin(pool.sec, __shfl_xor(pool.sec, d));
    }
    if (p.keyY != nullptr) pool.norm = normaliser(p.K, p.in.lse_part != nullptr && p.in.lse_part_target);
  }
  finish_row(p, b, lane, width, pool, [&](const int k) {
    Merged m;
    m.key = inf; m.idx = -1; m.sec = inf;
    const bool in = k < p.K;
    const long long o = (b * p.K + k) * nc;
    if (in)
      for (int c = c0; c < nc; c += width) fold_part(m, p.in.keyX[o + c], p.in.idxX[o + c], want_sec ? p.in.secX[o + c] : inf);
    for (int d = width >> 1; d >= 1; d >>= 1) {
      const double key = __shfl_xor(m.key, d), sec = __shfl_xor(m.sec, d);
      const int idx = __shfl_xor(m.idx, d);
      fold_part(m, key, idx, sec);
    }
    m.norm = normaliser(in ? k : p.K, p.in.lse_part != nullptr && in);
    return m;
  });
}

// ln sum_i exp(x_i / T) of one input row, in one pass over the row: every thread keeps a
// running maximum and the sum of exp relative to it (fp32 terms, four at a time, into an fp64
// running sum that is rescaled when the maximum moves).  NaN and +inf entries carry no mass.
template <typename E>
__device__ __forceinline__ void load_group(const E *row, int i0, int V, float (&v)[4]);
template <>
__device__ __forceinline__ void load_group<float>(const float *row, int i0, int V, float (&v)[4]) {
  if (i0 + 3 < V) {
    const float4 t = load_four(row + i0);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (i0 + j < V) ? row[i0 + j] : -__builtin_huge_valf();
  }
}
template <>
__device__ __forceinline__ void load_group<uint16_t>(const uint16_t *row, int i0, int V, float (&v)[4]) {
  if (i0 + 3 < V) {
    const uint2 t = load_four(row + i0);
    v[0] = __uint_as_float(t.x << 16);
    v[1] = __uint_as_float(t.x & 0xFFFF0000u);
    v[2] = __uint_as_float(t.y << 16);
    v[3] = __uint_as_float(t.y & 0xFFFF0000u);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      v[j] = (i0 + j < V) ? __uint_as_float((uint32_t)row[i0 + j] << 16) : -__builtin_huge_valf();
  }
}

template <typename E>
__global__ void __launch_bounds__(256) lse_kernel(const LseParams p) {
  __shared__ float s_max[4];
  __shared__ double s_sum[4];
  const int kd = p.per_k ? p.K : 1;  // distinct draft rows
  const int nd = p.with_drafts ? kd : 0;
  const int per_b = nd + (p.with_target ? 1 : 0);
  const long long b = blockIdx.x / (unsigned)per_b;
  int which = (int)(blockIdx.x % (unsigned)per_b);
  if (which == nd) which = kd;  // kd = the target row
  const int tid = threadIdx.x;
  const E *row;
  float T;
  long long extra = 0;
  if (p.draft_row_off != nullptr) {
    extra = p.draft_row_off[b];
    if (extra < 0) return;  // the row is not wanted
  }
  if (which == kd) {
    row = reinterpret_cast<const E *>(p.target) + p.map.target_off(b);
    T = p.temp_target;
  } else {
    row = reinterpret_cast<const E *>(p.draft) + p.map.draft_off(b) + extra + (long long)which * p.draft_stride_k;
    T = p.temp_draft != nullptr ? p.temp_draft[which] : p.temp_draft_all;
  }
  if (!p.is_logits) T = 1.0f;
  const float inf = __builtin_huge_valf();
  // log2(e)/T as a two-float sum, so that the exponent carries no systematic rounding of 1/T
  const double c64 = 1.4426950408889634 / (double)T;
  const float c_hi = (float)c64;
  const float c_lo = (float)(c64 - (double)c_hi);

  float m = -inf;     // running maximum of the entries that carry mass
  double sum = 0.0;   // sum of exp((x - m)/T) over the entries seen
  const int G = (p.V + 3) >> 2;
  // binned candidates: a draft row only lives on the announced bin (the target row is not masked)
  const bool binned = p.bins != nullptr && which != kd;
  const uint8_t *brow = binned ? p.bins + b * p.bins_stride_b : nullptr;
  int announced = -1;
  if (binned) {
    const int y = p.bin_of[b];
    if (y >= 0 && y < p.V) announced = (int)brow[y];
  }
  for (int g = tid; g < G; g += 256) {
    float v[4];
    load_group<E>(row, g * 4, p.V, v);
    if (binned) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (g * 4 + j < p.V && (int)brow[g * 4 + j] != announced) v[j] = -inf;
    }
    float gm = -inf;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (!(v[j] < inf)) v[j] = -inf;  // NaN, +inf: no mass
      gm = fmaxf(gm, v[j]);
    }
    if (gm > m) {
      if (m > -inf) {
        const float d = m - gm;
        sum *= (double)__builtin_amdgcn_exp2f(fmaf(d, c_hi, d * c_lo));
      }
      m = gm;
    }
    if (m > -inf) {
      float part = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // <= 0; entries without mass are clamped to a finite distance whose term is exactly 0
        // (an infinite one would meet c_lo's sign in the two-float product)
        const float d = fmaxf(v[j] - m, -65536.0f);
        part += __builtin_amdgcn_exp2f(fmaf(d, c_hi, d * c_lo));
      }
      sum += (double)part;
    }
  }
  float bm = m;
  for (int d = 32; d >= 1; d >>= 1) bm = fmaxf(bm, __shfl_xor(bm, d));
  if ((tid & 63) == 0) s_max[tid >> 6] = bm;
  __syncthreads();
  bm = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
  if (m > -inf && m < bm) sum *= exp2(((double)m - (double)bm) * c64);
  if (!(m > -inf)) sum = 0.0;
  for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
  if ((tid & 63) == 0) s_sum[tid >> 6] = sum;
  __syncthreads();
  if (tid == 0) {
    sum = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
    const bool ok = (bm > -inf) && (T > 0.0f) && (T < inf);
    const double lse = ok ? (double)bm / (double)T + log(sum) : -__builtin_huge_val();
    double *out = p.lse + b * (p.K + 1);
    if (which == kd) {
      out[p.K] = lse;
    } else if (kd == 1) {
      for (int k = 0; k < p.K; ++k) out[k] = lse;
    } else {
      out[which] = lse;
    }
  }
}

// Algorithm 2, the loop over positions (Section 4.2): Y_j is the candidate of the viable draft
// with the smallest key (ties: smaller index, then smaller k); drafts whose token differs from
// Y_j stop being viable; the loop ends when none is left or after the bonus position.
// One wavefront per sequence, lane k holds draft k (K <= 64); positions are fetched eight at a
// time so that the loop itself only waits for memory once per eight positions.
__global__ void __launch_bounds__(64) verify_kernel(const VerifyParams p) {
  const long long s = blockIdx.x;
  const int lane = threadIdx.x;
  const int L = p.L, K = p.K;
  const int32_t *cand = p.cand + s * (L + 1) * K;
  const double *ckey = p.cand_key + s * (L + 1) * K;
  const double *csec = p.cand_sec + s * (L + 1) * K;
  int32_t *Y = p.Y + s * (L + 1);
  float *keyY = p.keyY != nullptr ? p.keyY + s * (L + 1) : nullptr;
  bool viable = lane < K;
  bool done = false;
  int n = 0;
  unsigned long long near = 0;
  for (int j0 = 0; j0 <= L && !done; j0 += 8) {
    double key[8], sec[8];
    int idx[8], tok[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = j0 + u;
      key[u] = sec[u] = __builtin_huge_val(); idx[u] = -1; tok[u] = -2;
      if (j <= L && lane < K) {
        key[u] = ckey[(long long)j * K + lane];
        if (p.stats != nullptr) sec[u] = csec[(long long)j * K + lane];
        idx[u] = cand[(long long)j * K + lane];
        if (j < L) tok[u] = p.tokens[s * p.tok_stride_s + (long long)j * p.tok_stride_j + lane];
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = j0 + u;
      if (j > L || done) break;  // uniform
      double bkey = (viable && idx[u] >= 0) ? key[u] : __builtin_huge_val();
      int bidx = (viable && idx[u] >= 0) ? idx[u] : -1;
      int bk = lane;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        const double okey = __shfl_xor(bkey, d);
        const int oidx = __shfl_xor(bidx, d);
        const int ok = __shfl_xor(bk, d);
        if (beats(okey, oidx, ok, bkey, bidx, bk)) { bkey = okey; bidx = oidx; bk = ok; }
      }
      if (lane == 0) {
        Y[j] = bidx;
        if (keyY != nullptr) keyY[j] = bidx >= 0 ? (float)exp(bkey) : __builtin_huge_valf();
      }
      if (p.stats != nullptr && bidx >= 0) {
        // the pool's runner-up at another index: a viable draft whose own winner sits at the
        // pool's index offers its own runner-up, the others their winner
        double r = __builtin_huge_val();
        if (viable && idx[u] >= 0) r = idx[u] != bidx ? key[u] : sec[u];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) r = fmin(r, __shfl_xor(r, d));
        if (near_tie(bkey, r, 1)) ++near;
      }
      n = j + 1;
      if (j == L) { done = true; break; }
      viable = viable && tok[u] == bidx;
      if (__ballot(viable) == 0ull) done = true;
    }
  }
  if (lane == 0 && near) atomicAdd(&p.stats->near_ties, near);
  for (int j = n + lane; j <= L; j += 64) {
    Y[j] = -1;
    if (keyY != nullptr) keyY[j] = __builtin_huge_valf();
  }
  if (lane == 0) p.n_out[s] = n;
  if (p.active != nullptr && lane < K) p.active[s * K + lane] = viable ? 1 : 0;
}

// One position of the loop in its strong form (Appendix B).  One wavefront per sequence, lane k
// holds draft k.  At j == 0 the state is set up (every draft viable).
__global__ void __launch_bounds__(64) strong_step_kernel(const StrongStepParams p) {
  const long long s = blockIdx.x;
  const int lane = threadIdx.x;
  const int L = p.L, K = p.K, j = p.j;
  int32_t *Y = p.Y + s * (L + 1);
  float *keyY = p.keyY != nullptr ? p.keyY + s * (L + 1) : nullptr;
  bool viable = lane < K;
  bool running = true;
  if (j > 0) {
    viable = lane < K && p.viable[s * K + lane] != 0;
    running = p.running[s] != 0;
  }
  if (!running) {  // uniform: the loop ended at an earlier position
    if (lane == 0) {
      Y[j] = -1;
      if (keyY != nullptr) keyY[j] = __builtin_huge_valf();
      p.next_off[s] = -1;
    }
    return;
  }
  double key = __builtin_huge_val(), sec = __builtin_huge_val();
  int idx = -1;
  if (lane < K) {
    if (viable) {
      key = p.cand_key[(s * (L + 1) + j) * K + lane];
      if (p.stats != nullptr) sec = p.cand_sec[(s * (L + 1) + j) * K + lane];
      idx = p.cand[(s * (L + 1) + j) * K + lane];
    } else {
      // merge the chunks of this draft's scan (as the finalize kernel does) and normalise
      const long long o = (s * K + lane) * p.n_chunks;
      for (int c = 0; c < p.n_chunks; ++c) {
        const double ckey = p.part_key[o + c];
        const int cidx = p.part_idx[o + c];
        if (beats(ckey, cidx, 0, key, idx, 0)) {
          if (idx >= 0) sec = fmin(sec, key);
          key = ckey; idx = cidx;
        } else if (cidx >= 0) {
          sec = fmin(sec, ckey);
        }
        sec = fmin(sec, p.part_sec[o + c]);
      }
      const double norm = p.lse_sel[s * (K + 1) + lane];
      sec = (idx >= 0 && sec < __builtin_huge_val()) ? sec + norm : __builtin_huge_val();
      key = idx >= 0 ? key + norm : __builtin_huge_val();
    }
  }
  double bkey = idx >= 0 ? key : __builtin_huge_val();
  int bidx = idx, bk = lane;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const double okey = __shfl_xor(bkey, d);
    const int oidx = __shfl_xor(bidx, d);
    const int ok = __shfl_xor(bk, d);
    if (beats(okey, oidx, ok, bkey, bidx, bk)) { bkey = okey; bidx = oidx; bk = ok; }
  }
  if (lane == 0) {
    Y[j] = bidx;
    if (keyY != nullptr) keyY[j] = bidx >= 0 ? (float)exp(bkey) : __builtin_huge_valf();
  }
  if (p.stats != nullptr && bidx >= 0) {
    // the runner-up at another index, over all K drafts' race times
    double r = __builtin_huge_val();
    if (lane < K && idx >= 0) r = idx != bidx ? key : sec;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) r = fmin(r, __shfl_xor(r, d));
    if (lane == 0 && near_tie(bkey, r, 1)) atomicAdd(&p.stats->near_ties, 1ull);
  }
  bool more = j < L;
  if (more) {
    const int tok = lane < K ? p.tokens[s * p.tok_stride_s + (long long)j * p.tok_stride_j + lane] : -2;
    viable = viable && tok == bidx;
    more = __ballot(viable) != 0ull;
  }
  const unsigned long long mask = __ballot(viable);
  if (lane < K) p.viable[s * K + lane] = viable ? 1 : 0;
  if (lane == 0) {
    p.running[s] = more ? 1 : 0;
    if (!more) p.n_out[s] = j + 1;
    // the next position prices the dropped drafts with the first viable draft's row, if there are any
    const bool some_dropped = __popcll(mask) < K;
    p.next_off[s] = (more && some_dropped) ? (long long)(__ffsll((long long)mask) - 1) * p.stride_k : -1;
  }
  if (more && lane < K) {
    const int kref = __ffsll((long long)mask) - 1;
    p.lse_sel[s * (K + 1) + lane] = p.lse[(s * (L + 1) + j + 1) * (K + 1) + kref];
  }
  if (!more && p.active != nullptr && lane < K) p.active[s * K + lane] = viable ? 1 : 0;
}

// The whole loop in its strong form, one wavefront per sequence, lane k holds draft k, where every row's candidates of
// all drafts are known.  Bound by latency: a position is a trip to memory, for the row that the position before leaves, and a reduction over
// the lanes.  (See pairs_pay in api.hip for what it replaces, and where.)
__global__ void __launch_bounds__(64) strong_kernel(const StrongParams p) {
  const long long s = blockIdx.x;
  const int lane = threadIdx.x;
  const int L = p.L, K = p.K;
  int32_t *Y = p.Y + s * (L + 1);
  float *keyY = p.keyY != nullptr ? p.keyY + s * (L + 1) : nullptr;
  const bool here = lane < K;
  bool viable = here;
  int n = 0;
  for (bool more = true; more; ++n) {
    const int j = n;
    const unsigned long long mask = __ballot(viable);
    const int row = viable ? lane : __ffsll((long long)mask) - 1;  // a dropped draft is priced with the first viable one's row
    const long long at = ((s * (L + 1) + j) * K + row) * K + lane;
    const int tok = here && j < L ? p.tokens[s * p.tok_stride_s + (long long)j * p.tok_stride_j + lane] : -2;
    const int idx = here ? p.cand[at] : -1;
    double bkey = idx >= 0 ? p.cand_key[at] : __builtin_huge_val();
    int bidx = idx, bk = lane;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      const double okey = __shfl_xor(bkey, d);
      const int oidx = __shfl_xor(bidx, d), ok = __shfl_xor(bk, d);
      if (beats(okey, oidx, ok, bkey, bidx, bk)) { bkey = okey; bidx = oidx; bk = ok; }
    }
    if (lane == 0) {
      Y[j] = bidx;
      if (keyY != nullptr) keyY[j] = bidx >= 0 ? (float)exp(bkey) : __builtin_huge_valf();
    }
    more = j < L;
    if (more) {
      viable = viable && tok == bidx;
      more = __ballot(viable) != 0ull;
    }
  }
  for (int j = n + lane; j <= L; j += 64) {
    Y[j] = -1;
    if (keyY != nullptr) keyY[j] = __builtin_huge_valf();
  }
  if (lane == 0) p.n_out[s] = n;
  if (p.active != nullptr && here) p.active[s * K + lane] = viable ? 1 : 0;
}

}  // namespace

hipError_t launch_verify(hipStream_t s, const VerifyParams &p) {
  if (p.S == 0) return hipSuccess;
  hipLaunchKernelGGL(verify_kernel, dim3((unsigned)p.S), dim3(64), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_strong_step(hipStream_t s, const StrongStepParams &p) {
  if (p.S == 0) return hipSuccess;
  hipLaunchKernelGGL(strong_step_kernel, dim3((unsigned)p.S), dim3(64), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_strong(hipStream_t s, const StrongParams &p) {
  if (p.S == 0) return hipSuccess;
  hipLaunchKernelGGL(strong_kernel, dim3((unsigned)p.S), dim3(64), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_finalize(hipStream_t s, const FinalizeParams &p) {
  if (p.B == 0) return hipSuccess;
  int width = 1;
  while (width < p.n_chunks && width < 64) width *= 2;
  hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)p.B), dim3(64), 0, s, p, width);
  return hipGetLastError();
}

hipError_t launch_lse(hipStream_t s, const LseParams &p) {
  if (p.B == 0) return hipSuccess;
  const int kd = p.per_k ? p.K : 1;
  const unsigned grid = (unsigned)(p.B * ((p.with_drafts ? kd : 0) + (p.with_target ? 1 : 0)));
  if (grid == 0) return hipSuccess;
  if (p.dtype == LLC_F32)
    hipLaunchKernelGGL(lse_kernel<float>, dim3(grid), dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL(lse_kernel<uint16_t>, dim3(grid), dim3(256), 0, s, p);
  return hipGetLastError();
}

}  // namespace llc
