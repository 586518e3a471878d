// Which matrices of a batch share a launch of the fused block elimination
// (host only, no HIP).
#pragma once
#include <cstddef>
#include <cstdint>
#include <utility>
#include <vector>

namespace spand {

constexpr int ELIM_UNITS = 256;   // compute units of the device

// Ranges of the matrices 0 .. na-1, whose rows(i) descend, one launch each.
// One launch per 64-row size class, so that no workgroup carries waves without
// rows; *big is the range with the most rows.  Classes that follow each other
// on a stream (those before *big and those after it) and have no more matrices
// together than the device has compute units go into one launch: they would
// leave most units idle one after another.  Factorization with a launch per
// class / with joined launches, in ms: 16x16 p = 1 FP64 (four leaves in four
// classes) 10.0 / 6.8, 40x40 p = 1 FP64 15.9 / 12.6, 61x47 p = 2 FP64 23.1 /
// 21.5, 91x69 p = 3 FP64 63.8 / 62.3, 128x128 p = 2 FP32 58.6 / 56.6, 160x120
// p = 1 FP32 36.7 / 36.1, batches of 6 to 36 systems of several sizes 22-39 /
// 18-32.  A small matrix runs in a workgroup as wide as the largest of its
// launch, which has the longer chain of steps anyway.
template <typename Rows>
std::vector<std::pair<int, int>> elim_launches(int na, const Rows &rows, size_t *big) {
  std::vector<std::pair<int, int>> cls;
  *big = 0;
  if (na <= ELIM_UNITS) {
    if (na > 0) cls.push_back({0, na});
    return cls;
  }
  size_t bc = 0;
  for (int a = 0; a < na;) {
    int b = a + 1;
    while (b < na && (rows(b) + 63) / 64 == (rows(a) + 63) / 64) ++b;
    cls.push_back({a, b});
    a = b;
  }
  auto total = [&](size_t c) { return int64_t(cls[c].second - cls[c].first) * rows(cls[c].first); };
  for (size_t c = 1; c < cls.size(); ++c)
    if (total(c) > total(bc)) bc = c;
  const std::pair<int, int> m = cls[bc];
  std::vector<std::pair<int, int>> out;
  if (m.first > 0 && m.first <= ELIM_UNITS) out.push_back({0, m.first});
  else out.assign(cls.begin(), cls.begin() + std::ptrdiff_t(bc));
  *big = out.size();
  out.push_back(m);
  if (m.second < na && na - m.second <= ELIM_UNITS) out.push_back({m.second, na});
  else out.insert(out.end(), cls.begin() + std::ptrdiff_t(bc) + 1, cls.end());
  return out;
}

}  // namespace spand
