// Host-only driver of what the planner keeps for the process, under AddressSanitizer/UBSan and ThreadSanitizer:
//   maps   each dimension and degree is fitted once, however many others come in between; concurrent callers
//          get the same entry; the sparse form holds the dense entries above the fit's rounding
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
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

int main(int argc, char** argv) {
  const int rc = argc > 1 && !std::strcmp(argv[1], "maps") ? maps() : 2;
  if (rc == 0) std::printf("ok\n");
  return rc;
}
