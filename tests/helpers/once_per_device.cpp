// 8 threads make OncePerDevice's call for 3 devices at the same time, many times: each device's call is made at
// least once and, once it has succeeded, never again; a failing call is repeated; devices beyond 63 every time.
#include <cstdio>
#include <thread>
#include <vector>

#include "spin_once.h"

int main() {
  spin::OncePerDevice once;
  std::atomic<int> calls[3] = {}, plain{0};
  std::vector<std::thread> th;
  for (int t = 0; t < 8; ++t)
    th.emplace_back([&] {
      for (int i = 0; i < 20000; ++i)
        if (once.run(i % 3, 0, [&] { return ++calls[i % 3], 0; }) != 0) ++plain;
    });
  for (auto& t : th) t.join();
  const int before[3] = {calls[0], calls[1], calls[2]};
  for (int d = 0; d < 3; ++d) once.run(d, 0, [&] { return ++calls[d], 0; });
  spin::OncePerDevice other;
  int fails = 0, far = 0;
  for (int i = 0; i < 3; ++i) other.run(5, 0, [&] { return ++fails, i < 2 ? 7 : 0; });
  other.run(5, 0, [&] { return ++fails, 0; });
  for (int i = 0; i < 3; ++i) other.run(64 + 5, 0, [&] { return ++far, 0; });
  bool ok = plain == 0 && fails == 3 && far == 3;
  for (int d = 0; d < 3; ++d) ok = ok && before[d] >= 1 && before[d] <= 8 && calls[d] == before[d];
  std::printf("%d %d %d  %d %d\n", before[0], before[1], before[2], fails, far);
  return ok ? 0 : 1;
}
