// Host check of Places: threads take and give places at random. Prints how often
// more was held than is resident in any order, how many launches ran, and whether
// small ones ran side by side.
#include <atomic>
#include <cstdio>
#include <random>
#include <thread>
#include <vector>
#include "places.hpp"
using namespace pdhcg;

int main() {
  constexpr int CUS = 256, THREADS = 6, EACH = 300;
  Places places;
  std::mutex mu;
  std::vector<Places::Hold*> now;
  std::atomic<int> bad{0}, runs{0}, together{0};
  auto work = [&](int seed) {
    std::mt19937 g(seed);
    for (int i = 0; i < EACH; ++i) {
      const int per = 1 + (int)(g() % 2);
      Places::Hold h{(int)(1 + g() % (g() % 3 ? 60 : per * CUS)), per};
      places.take(h, CUS, std::chrono::seconds(60));
      {
        std::lock_guard<std::mutex> l(mu);
        now.push_back(&h);
        long total = 0;
        int p = 99;
        for (auto* q : now) {
          total += q->grid;
          p = q->per < p ? q->per : p;
        }
        if (now.size() > 1) {
          ++together;
          if (total > (long)p * CUS) ++bad;
        }
      }
      std::this_thread::sleep_for(std::chrono::microseconds(g() % 50));
      {
        std::lock_guard<std::mutex> l(mu);
        for (size_t k = 0; k < now.size(); ++k)
          if (now[k] == &h) now.erase(now.begin() + k);
      }
      places.give(h);
      ++runs;
    }
  };
  std::vector<std::thread> t;
  for (int i = 0; i < THREADS; ++i) t.emplace_back(work, i);
  for (auto& x : t) x.join();
  // a holder that never gives back: the next one goes ahead after its limit
  Places::Hold a{256, 1}, b{256, 1};
  places.take(a, CUS, std::chrono::seconds(1));
  const auto t0 = std::chrono::steady_clock::now();
  places.take(b, CUS, std::chrono::milliseconds(50));
  const auto ms = std::chrono::duration_cast<std::chrono::milliseconds>(std::chrono::steady_clock::now() - t0).count();
  places.give(b);
  places.give(a);
  printf("%d %d %d %d\n", bad.load(), runs.load(), together.load() > 0, ms >= 50);
  return 0;
}
