// How far a sampling product's inner dimension is split where its tiles leave
// compute units idle.  Plain C++, so that the rule can be checked on the host.
#pragma once

#include <algorithm>

namespace hss {

// Splits of a small matrix (n at least `line`): `unit` k or more each, up to
// 16, and two workgroups per compute unit.
inline long long small_splits(long long n, long long tiles, long long line, long long unit, int cus) {
  return n >= line ? std::min({16LL, n / unit, 2LL * cus / tiles}) : 1;
}

}  // namespace hss
