// How lml_sum_kernel looks for the bucket of an entry among a row's splitters.  Plain C++: a host build checks its accesses.
#pragma once

namespace llc {

constexpr int kSumBuckets = 512;
// What stands behind the last splitter of 2 kSumBuckets: nothing lies at or to the right of it, an entry at +inf (no mass on the draft's side) neither,
// so that a search ends at a bucket that there is.
constexpr float kNoSplitter = __builtin_nanf("");

// The buckets of N entries side by side (each look-up is a chain of reads): b[j] holds the number of splitters to the left of the part of the
// range that d[j] is in, and takes those in it that are not to its right; every part has fewer than 2^steps.
template <int N>
__attribute__((always_inline)) constexpr void find_buckets(const float *split, int steps, const float (&d)[N], int (&b)[N]) {
#pragma unroll 1
  for (int step = (1 << steps) >> 1; step >= 1; step >>= 1) {
#pragma unroll
    for (int j = 0; j < N; ++j) b[j] += split[b[j] + step] <= d[j] ? step : 0;
  }
}

}  // namespace llc
