// Checks OncePerDevice; prints "ok", or says what is wrong.
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>

#include "per_device.h"

static int fail(const char* what) {
  printf("%s\n", what);
  return 1;
}

int main() {
  {
    sptir::OncePerDevice once;
    int done[70] = {0};
    for (int turn = 0; turn < 3; ++turn)
      for (int device = 0; device < 70; ++device) once(device, [&] { ++done[device]; return true; });
    for (int device = 0; device < 64; ++device)
      if (done[device] != 1) return fail("a device was left out, or done twice");
    for (int device = 64; device < 70; ++device)
      if (done[device] != 3) return fail("a device beyond the mask is done every time");
  }
  {
    sptir::OncePerDevice once;
    int tries = 0;
    for (int turn = 0; turn < 4; ++turn) once(5, [&] { return ++tries == 3; });
    if (tries != 3) return fail("what did not succeed is done again, what did is not");
  }
  for (int turn = 0; turn < 200; ++turn) {  // nobody goes on before it is done
    sptir::OncePerDevice once;
    std::atomic<int> ready[2] = {{0}, {0}}, early{0};
    std::vector<std::thread> threads;
    for (int t = 0; t < 8; ++t)
      threads.emplace_back([&, t] {
        once(t % 2, [&] { ready[t % 2] = 1; return true; });
        if (!ready[t % 2]) ++early;
      });
    for (auto& t : threads) t.join();
    if (early) return fail("a thread went on before it was done");
  }
  printf("ok\n");
  return 0;
}
