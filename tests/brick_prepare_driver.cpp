// brick_prepare on the CPU, one thread per GPU thread, in the order that shows a missing barrier: thread 0
// runs until it waits or is done before any other thread starts.  BRICK_PREPARE_SOURCE is the function's text
// (test_brick_prepare_order.py).
#include <condition_variable>
#include <cstdio>
#include <mutex>
#include <thread>
#include <vector>

#define __device__
#define __forceinline__ inline
#define __restrict__
struct uint4 { unsigned x, y, z, w; };
static uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return {x, y, z, w}; }
constexpr int kBrick = 16, kThreads = 256;

struct Index { int x; };
static thread_local Index threadIdx;
static std::mutex lock;
static std::condition_variable change;
static bool first_stopped = false;     // thread 0 has reached a barrier or the end
static int waiting = 0, generation = 0;

static void stop_first() {
  if (threadIdx.x == 0) { first_stopped = true; change.notify_all(); }
}
static void __syncthreads() {
  std::unique_lock<std::mutex> l(lock);
  stop_first();
  const int g = generation;
  if (++waiting == kThreads) { waiting = 0; ++generation; change.notify_all(); }
  else change.wait(l, [&] { return generation != g; });
}

#include BRICK_PREPARE_SOURCE

// Cells of brick `key` that are not 0 after a preparation in `mode` of a grid of ones; valid as given.
static long long left_over(int n, int mode, long long key, unsigned char was, unsigned touched,
                           unsigned char* now) {
  const int nbs = n / kBrick;
  std::vector<unsigned> count(nbs * nbs * nbs, 0u);
  count[key] = touched;
  std::vector<unsigned char> valid(count.size(), was);
  std::vector<unsigned long long> grid((size_t)n * n * n, 1ull);
  first_stopped = false;
  std::vector<std::thread> ts;
  for (int t = 0; t < kThreads; ++t)
    ts.emplace_back([&, t] {
      threadIdx.x = t;
      if (t) {
        std::unique_lock<std::mutex> l(lock);
        change.wait(l, [] { return first_stopped; });
      }
      brick_prepare(count.data(), n, mode, key, valid.data(), grid.data());
      std::unique_lock<std::mutex> l(lock);
      stop_first();
    });
  for (auto& t : ts) t.join();
  *now = valid[key];
  const int bx = key % nbs, by = key / nbs % nbs, bz = key / (nbs * nbs);
  long long left = 0;
  for (int z = 0; z < kBrick; ++z)
    for (int y = 0; y < kBrick; ++y)
      for (int x = 0; x < kBrick; ++x)
        left += grid[((size_t)(bz * kBrick + z) * n + by * kBrick + y) * n + bx * kBrick + x] != 0;
  return left;
}

int main() {
  const long long cells = (long long)kBrick * kBrick * kBrick;
  int bad = 0;
  for (int mode = 0; mode < 3; ++mode)
    for (int was = 0; was < 2; ++was)
      for (unsigned touched = 0; touched < 2; ++touched) {
        unsigned char now;
        const long long left = left_over(32, mode, 5, (unsigned char)was, touched, &now);
        const bool clear = mode == 0 ? touched : (mode == 1 ? touched && !was : !was);
        const int valid = mode == 0 ? touched : (mode == 1 ? was || touched : 1);
        if (left != (clear ? 0 : cells) || now != valid) {
          std::printf("mode %d valid %d touched %u: %lld cells left, valid %d\n", mode, was, touched, left, now);
          ++bad;
        }
      }
  if (!bad) std::printf("brick preparation passed\n");
  return bad != 0;
}
