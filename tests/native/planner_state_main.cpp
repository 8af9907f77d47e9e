// Host-only driver of what the planner keeps for the process, under AddressSanitizer/UBSan and ThreadSanitizer:
//   maps   each dimension and degree is fitted once, however many others come in between; concurrent callers
//          get the same entry; the sparse form holds the dense entries above the fit's rounding
//   pools  tasks that wait (for a device, here for another thread) do not hold up parallel_for, nor each other
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <string>
#include <thread>
#include <vector>

#include "planner.hpp"

static int maps() {
  std::atomic<int> fits{0};
  auto get = [&](int d, int K) -> const hdf::SparseMaps& {
    return hdf::derivative_maps(d, K, [&] {
      ++fits;
      hdf::SparseMaps m;
      m.row = {d, K};
      return m;
    });
  };
  int keys = 0;
  std::vector<const hdf::SparseMaps*> first;
  for (int d = 3; d <= 8; ++d)
    for (int K = 0; K <= 30; ++K, ++keys) first.push_back(&get(d, K));
  std::vector<std::thread> threads;
  std::atomic<int> wrong{0};
  for (int t = 0; t < 4; ++t)
    threads.emplace_back([&] {
      int i = 0;
      for (int d = 3; d <= 8; ++d)
        for (int K = 0; K <= 30; ++K, ++i) {
          const hdf::SparseMaps& m = get(d, K);
          if (&m != first[i] || m.row[0] != d || m.row[1] != K) ++wrong;
        }
    });
  for (auto& t : threads) t.join();
  if (fits != keys || wrong) {
    std::printf("%d keys fitted %d times, %d wrong entries\n", keys, fits.load(), wrong.load());
    return 1;
  }
  // d = 3, K = 1: three harmonics of degree 1 over one of degree 0, one value below the rounding bound
  std::vector<std::vector<double>> G(2);
  G[1] = {1.0, 0.0, 1e-13, 0.0, -2.0, 0.0, 3e-12, 0.0, 4.0};
  const hdf::SparseMaps m = hdf::sparse_maps(3, 1, G);
  const std::vector<int32_t> row = {0, 1, 2, 3}, h = {0, 1, 2};
  const std::vector<double> v = {1.0, -2.0, 4.0};
  if (m.row != row || m.h != h || m.v != v) {
    std::printf("sparse form differs\n");
    return 1;
  }
  return 0;
}

static int pools() {
  if (std::thread::hardware_concurrency() < 2) return 0;
  // the tasks wait until another thread's parallel_for has run and its own tasks were refused
  std::atomic<bool> done{false};
  std::atomic<int> started{0}, late{0}, nested{0};
  std::thread other([&] {
    while (!started) std::this_thread::yield();
    std::vector<int> hit(50, 0);
    hdf::parallel_for(50, [&](int i) { hit[i] += 1; });
    for (int h : hit)
      if (h != 1) ++late;
    if (hdf::try_device_tasks(4, [&](int) { ++late; })) ++late;
    done = true;
  });
  std::vector<int> ran(12, 0);
  const bool taken = hdf::try_device_tasks(12, [&](int i) {
    ++started;
    for (int ms = 0; !done && ms < 20000; ++ms) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    if (!done) ++late;
    ran[i] += 1;
    const std::thread::id self = std::this_thread::get_id();
    hdf::parallel_for(5, [&](int) { nested += std::this_thread::get_id() == self; });
  });
  other.join();
  int wrong = !taken + late + (nested != 60);
  for (int r : ran) wrong += r != 1;
  // no more tasks at once than kPoolThreads, by which callers size what each running task holds
  std::atomic<int> running{0}, most{0};
  hdf::try_device_tasks(200, [&](int) {
    const int now = ++running;
    for (int m = most; m < now && !most.compare_exchange_weak(m, now);) {
    }
    std::this_thread::sleep_for(std::chrono::milliseconds(1));
    --running;
  });
  wrong += most > hdf::kPoolThreads;
  // the pool is free again
  std::atomic<int> again{0};
  wrong += !hdf::try_device_tasks(3, [&](int) { ++again; }) + (again != 3);
  if (wrong) std::printf("pools: taken %d, late %d, nested %d, again %d\n", taken, late.load(), nested.load(), again.load());
  return wrong != 0;
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  const int rc = what == "maps" ? maps() : what == "pools" ? pools() : 2;
  if (rc == 0) std::printf("ok\n");
  return rc;
}
