// Host-side check that the words of a plan hold what one launch for any of its block columns counts in:
// both arithmetic types, one and two arrays, orders up to a million, and no fewer bytes than the
// second leaf of pivoting over the block.  Built and run by tests/test_flow_order.py; nothing here
// touches a GPU.
#include "../../paper_2503_04424_amd/csrc/kernels_flow.h"
#include "../../paper_2503_04424_amd/csrc/plan.h"

#include <cstdio>

using namespace mdet;

int main() {
  long bad = 0, cases = 0;
  for (int beta = 4; beta <= 8; beta += 4)
    for (int64_t n = 0; n <= 1100000; n += n < 300 ? 1 : n / 7 * 3 % 1000 + 61)
      for (int pivot = 0; pivot <= 1; ++pivot) {
        const SmallArea a = small_area(n, (n + 63) / 64, beta, pivot != 0);
        for (int arrays = 1; arrays <= 2; ++arrays) {
          ++cases;
          const bool ok = 4 * (uint64_t)flow_words(n, arrays) <= a.words_bytes && a.words % 256 == 0 &&
                          a.words + a.words_bytes <= a.partial && a.words_bytes >= (uint64_t)LEAF * LEAF * beta;
          if (!ok) {
            if (++bad < 20) std::printf("n %ld beta %d arrays %d\n", (long)n, beta, arrays);
          }
        }
      }
  std::printf("plans %ld bad %ld\n", cases, bad);
  return bad != 0 || cases < 1000;
}
