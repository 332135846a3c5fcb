// Host checks of the request server's choice of the next request, run by
// test_host_pick.py.
#include <cstdio>
#include <deque>

#include "../../paper_2501_03377_amd/csrc/kp_pick.h"

struct Item { int plan, passed = 0; };

static int fail(const char* what) {
  std::printf("FAILED: %s\n", what);
  return 1;
}

int main() {
  const auto holds = [](int plan) { return [plan](const Item& i) { return i.plan == plan; }; };
  {   // one worker, or nothing ready: the oldest
    std::deque<Item> q{{1}, {2}};
    if (kp::pick_request(q, true, holds(2)) != q.begin()) return fail("one worker");
    if (kp::pick_request(q, false, holds(3)) != q.begin()) return fail("nothing ready");
    if (kp::pick_request(q, false, holds(1)) != q.begin()) return fail("oldest ready");
    if (q.front().passed != 0) return fail("passed without being passed");
  }
  {   // younger ready ones go first, the oldest of them, kPassLimit times
    std::deque<Item> q{{1}};
    for (int k = 0; k < 10; ++k) q.push_back({k % 2 ? 2 : 3});
    for (int k = 0; k < kp::kPassLimit; ++k) {
      const auto it = kp::pick_request(q, false, holds(2));
      if (it->plan != 2 || it != q.begin() + 2 + k) return fail("oldest ready one");
      if (q.front().plan != 1 || q.front().passed != k + 1) return fail("count of passes");
      q.erase(it);
    }
    if (kp::pick_request(q, false, holds(2)) != q.begin()) return fail("pass limit");
    // the next oldest starts its own count
    q.pop_front();
    if (kp::pick_request(q, false, holds(2)) == q.begin() || q.front().passed != 1)
      return fail("count of the next one");
  }
  {   // the window: its last place is looked at, the one behind it is not
    std::deque<Item> q(kp::kPickWindow + 1, Item{1});
    q.back().plan = 2;
    if (kp::pick_request(q, false, holds(2)) != q.begin() || q.front().passed != 0)
      return fail("behind the window");
    q.erase(q.begin() + 1);
    if (kp::pick_request(q, false, holds(2)) != q.end() - 1) return fail("end of the window");
  }
  std::printf("pick checks ok\n");
  return 0;
}
