// A workgroup of four wavefronts as four threads: a barrier counts only those
// that have not ended.  Prints what each wavefront got from each wait.
#include <barrier>
#include <cstdio>
#include <thread>
#include <vector>

#include "lpht_wgwait.h"

namespace {

struct Workgroup {
  std::barrier<> *bar;
  int wave;
  bool leader() const { return wave == 0; }
  void sync() const { bar->arrive_and_wait(); }
};

}  // namespace

// The wavefront `leaver` ends after the first wait, the others wait once more.
int main() {
  for (int leaver = -1; leaver < 4; ++leaver) {
    std::barrier<> bar(4);
    uint32_t word = 0, got[4][2] = {};
    std::vector<std::thread> waves;
    for (int w = 0; w < 4; ++w)
      waves.emplace_back([&, w] {
        const Workgroup wg{&bar, w};
        got[w][0] = lpht::wg_wait(wg, &word, [] { return 2u; });
        if (w == leaver) {
          bar.arrive_and_drop();
          return;
        }
        got[w][1] = lpht::wg_wait(wg, &word, [&] { return leaver < 0 ? 4u : 0u; });
      });
    for (auto &t : waves) t.join();
    std::printf("%d", leaver);
    for (auto &g : got) std::printf(" %u %u", g[0], g[1]);
    std::printf("\n");
  }
}
