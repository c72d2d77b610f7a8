// The order in which a thread requests and uses its items of Step 1b (no GPU code: the host's test follows it).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace sparq {

// `items` items through two buffers: the second is requested before the first is used.  request(buffer) and use(buffer) get
// the buffer's number as a type and take the items in order.  between() runs once, behind the first requests.
// several: some thread of the wave has more than one item (the same in every lane).  A thread of such a wave that has a single
// item requests it twice (one_again() lets it start over), as there is no condition between the first two requests: the compiler
// counts requests in flight, and behind a conditional one it waits for all.
// A wave whose threads have one item at most, or none, uses the second buffer alone, which is requested and used last either
// way, so that the compiler's count holds.  When such waves requested their items twice as well, 2048 heads of 4096 positions with
// 8 channels took 79.2 us per decode, so 67.2; 512 heads 20.4 / 19.8, 4 heads at 16 384 with 32 channels (four thread groups
// per chunk) 18.9 / 18.4, 16 heads at 32 768 with 16 27.5 / 26.8.
template <class Request, class Use, class Between, class OneAgain>
__host__ __device__ __forceinline__ void two_ahead(int items, bool several, Request&& request, Use&& use, Between&& between,
                                                   OneAgain&& one_again) {
  constexpr std::integral_constant<int, 0> a{};
  constexpr std::integral_constant<int, 1> b{};
  if (items > 0) {
    if (several) {
      request(a);
      if (items == 1) one_again();
    }
    request(b);
  }
  between();                               // (outside the branch: by whole waves)
  if (items > 0) {
    int left = 2;
    if (several) {
      int i = 0;
      for (; i + 3 < items; i += 2) {      // (no conditional request inside, as above)
        use(a);
        request(a);
        use(b);
        request(b);
      }
      use(a);
      left = items - i;
      if (left == 3) request(a);
    }
    if (left >= 2) use(b);
    if (left == 3) use(a);
  }
}

}  // namespace sparq
