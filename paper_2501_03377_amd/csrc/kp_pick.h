// The queued request that a worker of the request server serves next (plain
// C++, no device code).
#pragma once

namespace kp {

// How far down the queue a worker looks for a request whose plan it holds, and
// how often the oldest request may be passed over for one.
constexpr int kPickWindow = 32;
constexpr int kPassLimit = 4;

// The oldest request, unless making its plan would delay it while a younger
// one finds its plan ready here (`ready`).  Making a plan (and binding a
// workspace, with its allocations) takes longer than a small solve, and
// another worker may hold the oldest one's plan.  The oldest request is passed
// over at most kPassLimit times (its `passed`).  alone: no other worker could
// serve it.  The queue is not empty.
template <class Queue, class Ready>
typename Queue::iterator pick_request(Queue& queue, bool alone, Ready ready) {
  const auto front = queue.begin();
  if (alone || front->passed >= kPassLimit || ready(*front)) return front;
  auto it = front + 1;
  for (int k = 1; it != queue.end() && k < kPickWindow; ++it, ++k)
    if (ready(*it)) {
      front->passed += 1;
      return it;
    }
  return front;
}

}  // namespace kp
