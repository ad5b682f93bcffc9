// Host-side check of the task order of panel_flow_kernel: every tile of a block column belongs to
// exactly one task, and everything a task waits for belongs to tasks with lower numbers.  Built
// and run by tests/test_flow_order.py; nothing here touches a GPU.
#include "../../paper_2503_04424_amd/csrc/kernels_flow.h"

#include <cstdio>
#include <vector>

using namespace mdet;

int main() {
  long bad = 0, cases = 0;
  for (int arrays = 1; arrays <= 2; ++arrays)
   for (int share = 0; share <= 2; ++share)
   for (int ntr = 1; ntr <= 140; ntr += ntr < 40 ? 1 : 9)
    for (int ntc = 1; ntc <= ntr; ntc += ntc < 20 || ntc + 7 > ntr ? 1 : 5) {
      const FlowOrder order = flow_order((int64_t)ntr * 64 - 5, (int64_t)ntc * 64 - (ntr == ntc ? 5 : 0), arrays,
                                         share * ((ntc + 1) / 2) / 2);
      const int64_t tasks = order.tasks();
      std::vector<int64_t> owner((size_t)arrays * ntr * ntc, -1);
      auto place = [&](int y, int i, int j) -> int64_t& { return owner[((size_t)y * ntr + i) * ntc + j]; };
      auto own = [&](int y, int i, int j, int64_t t) {
        if (y >= arrays || i >= ntr || j >= ntc || place(y, i, j) >= 0) ++bad;
        else place(y, i, j) = t;
      };
      for (int pass = 0; pass < 2; ++pass)
        for (int64_t t = 0; t < tasks; ++t) {
          int pair, y, j;
          const FlowKind kind = order.task((int)t, pair, y, j);
          auto before = [&](int i, int k) {              // in every array: each needs the other's rows
            for (int q = 0; q < arrays; ++q)
              if (place(q, i, k) >= t) ++bad;
          };
          if (kind == FLOW_DIAGONAL) {
            if (pass == 0) {
              for (int q = 0; q < arrays; ++q) {
                own(q, j, j, t);
                if (j > 0) own(q, j, j - 1, t);
              }
              continue;
            }
            for (int k = 0; k + 1 < j; ++k) { before(j, k); before(j - 1, k); }
            if (j > 0) before(j - 1, j - 1);
            continue;
          }
          if (kind == FLOW_NOTHING) continue;
          for (int c = j; c < j + (kind == FLOW_ROWS2 ? 2 : 1); ++c) {
            const int first = c + 1 < ntc ? c + 2 : c + 1;
            if (kind == FLOW_ROWS2 && 2 * pair < first) ++bad;       // whole pairs only
            for (int i = 2 * pair; i < 2 * pair + 2; ++i) {
              if (i < first || i >= ntr) continue;
              if (pass == 0) { own(y, i, c, t); continue; }
              before(c, c);
              if (c > j) before(c, j);
              for (int k = 0; k < j; ++k) {
                if (place(y, i, k) >= t) ++bad;
                before(c, k);
              }
            }
          }
        }
      for (int i = 0; i < ntr; ++i)
        for (int j = 0; j < ntc && j <= i; ++j)
          for (int q = 0; q < arrays; ++q)
            if (place(q, i, j) < 0) ++bad;
      if (bad && cases >= 0) std::printf("rows %d columns %d: bad %ld\n", ntr, ntc, bad);
      ++cases;
    }
  std::printf("shapes %ld bad %ld\n", cases, bad);
  return bad != 0;
}
