// Harness for the search of lml_sum_kernel (test infrastructure): every place, those without a number among them, is looked for among
// splitters of several counts and layouts, in arrays of the kernel's sizes.  tests/test_lml_search.py builds it with -fsanitize=address and runs it.
#include "../paper_2506_05632_amd/csrc/lml_search.hpp"

#include <cmath>
#include <cstdio>
#include <limits>
#include <memory>
#include <vector>

int main() {
  using namespace llc;
  const float inf = std::numeric_limits<float>::infinity(), far = 740.0f, none = std::numeric_limits<float>::quiet_NaN();
  const float places[] = {-inf, -3e38f, -741.0f, -740.0f, -739.9f, -12.5f, -1.0f, 0.0f, 0.25f, 1.0f, 12.5f, 739.9f, 740.0f, 741.0f, 3e38f, inf, none};
  int bad = 0;
  for (const int nb : {1, 2, 3, 128, 255, 511, 512})
    for (const float spread : {0.0f, 1e-6f, 2.0f, 700.0f})  // (the first two: all splitters in one part of the range)
      for (const int parts : {1, 1024}) {
        std::unique_ptr<float[]> split(new float[2 * kSumBuckets]);
        std::unique_ptr<float[]> bucket(new float[kSumBuckets]());
        for (int b = 0; b < 2 * kSumBuckets; ++b)
          split[b] = b == 0 ? -inf : b >= nb ? kNoSplitter : nb > 2 ? spread * (2.0f * (float)(b - 1) / (float)(nb - 2) - 1.0f) : 0.0f;
        const float left = nb > 1 ? split[1] - 6.0f : -far, right = nb > 1 ? split[nb - 1] + 6.0f : far;
        auto part_of = [&](float d) { return (int)std::fmin(std::fmax((d - left) * ((float)parts / (right - left)), 0.0f), (float)(parts - 1)); };
        std::vector<int> before((size_t)parts + 1, 0);  // splitters in the parts before each
        for (int b = 1; b < nb; ++b)
          for (int i = part_of(split[b]) + 1; i <= parts; ++i) ++before[(size_t)i];
        int most = 0;
        for (int i = 0; i < parts; ++i) most = std::max(most, before[(size_t)i + 1] - before[(size_t)i]);
        const int steps = most > 0 ? 32 - __builtin_clz((unsigned)most) : 0;
        for (const float place : places)
          for (int each = -1; each < nb; ++each) {
            const float d[2] = {each < 1 ? place : split[each], place};
            int b[2];
            for (int j = 0; j < 2; ++j) b[j] = before[(size_t)part_of(std::fabs(d[j]) < far ? d[j] : 0.0f)];
            find_buckets(split.get(), steps, d, b);
            for (int j = 0; j < 2; ++j) {
              bucket[b[j]] += 1.0f;  // the kernel reads s_bucket there
              if (b[j] >= nb) ++bad;
              if (!(std::fabs(d[j]) < far)) continue;
              int want = 0;
              while (want + 1 < nb && split[want + 1] <= d[j]) ++want;
              if (b[j] != want && !(split[b[j]] == split[want])) ++bad;
            }
          }
      }
  std::printf("%d\n", bad);
  return bad != 0;
}
