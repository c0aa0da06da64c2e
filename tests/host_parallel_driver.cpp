// The loops of ensemble loading (host_parallel.h), run under the thread
// sanitizer: every index once, on teams that several loops share and alone,
// with an exception, with loops inside a loop's body, and from several threads.
#include <stdio.h>
#include <stdlib.h>

#include <stdexcept>
#include <thread>
#include <vector>

#include "host_parallel.h"

using namespace ml2;

static void check(bool ok, const char *what) {
  if (ok) return;
  fprintf(stderr, "%s\n", what);
  exit(1);
}

static void loops() {
  for (int64_t n : {0, 1, 2, 7, 1000}) {
    std::vector<int> seen((size_t)n, 0);
    parallel_for(n, 1 << 20, [&](int64_t i) { ++seen[(size_t)i]; });
    for (int s : seen) check(s == 1, "an index not taken once");
  }
  bool thrown = false;
  try {
    parallel_for(1000, 1 << 20, [&](int64_t i) {
      if (i == 37) throw std::runtime_error("37");
    });
  } catch (const std::runtime_error &) {
    thrown = true;
  }
  check(thrown, "an exception lost");
  std::atomic<int> inner{0};
  parallel_for(8, 1 << 20, [&](int64_t) {
    parallel_for(8, 1 << 20, [&](int64_t) { ++inner; });
  });
  check(inner == 64, "a loop inside a loop");
}

int main() {
  std::vector<std::thread> callers;
  for (int c = 0; c < 3; ++c)
    callers.emplace_back([] {
      for (int r = 0; r < 20; ++r) {
        loops();
        Team team;
        loops();
        loops();
      }
    });
  for (std::thread &t : callers) t.join();
  printf("ok\n");
  return 0;
}
