// How long a worker of the persistent launch polls before it gives up
// (dag.hpp, Patience): time between two polls counts up to a fixed step, so a worker
// that was held off the card for long has not waited long; one that polls all
// along gives up after the limit.  Prints "ok".
#include <cstdio>

#include "../../paper_2507_06938_amd/csrc/dag.hpp"

int main() {
  using dl::dag::Patience;
  const long long limit = 200000000, step = 10000, poll = 100;
  {  // 1000 polls, each after ten seconds off the card
    Patience p{5};
    long long now = 5;
    for (int k = 0; k < 1000; ++k)
      if (p.out(now += 1000000000LL, limit, step)) return 1;
  }
  {  // polls without a gap: gives up at the limit, not before
    Patience p{7};
    long long now = 7, k = 0;
    while (!p.out(now += poll, limit, step))
      if (++k > limit) return 2;
    if (k != limit / poll) return 3;
  }
  {  // always off the card between polls: still gives up
    Patience p{0};
    long long now = 0, k = 0;
    while (!p.out(now += 50 * step, limit, step))
      if (++k > limit) return 4;
    if (k != limit / step) return 5;
  }
  std::printf("ok\n");
  return 0;
}
