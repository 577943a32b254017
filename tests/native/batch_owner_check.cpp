// A batch's outcomes own their results: dropping the outcomes, as an error on
// the way to the caller does, frees every result.
#include <cstdio>

#include "batch.hpp"
#include "exec.hpp"

int main() {
  using gsmat::DevQueryOut;
  int freed = 0;
  const int n = 5;
  {
    std::vector<DevQueryOut> out(n);
    for (DevQueryOut& o : out) {
      o.res = decltype(o.res)(new gsmat_result);
      gsmat::Segment seg;
      seg.hold = std::shared_ptr<void>(&freed, [](void* p) { ++*(int*)p; });
      o.res->segs.push_back(seg);
    }
  }
  std::printf("freed %d of %d\n", freed, n);
  return freed == n ? 0 : 1;
}
