// Work items of a batched step: they cover its units once and in order, and
// what no item can hold is refused.
#include <cstdio>

#include "fd_internal.h"

int main() {
  int failures = 0;
  auto check = [&](bool ok, const char* what, long long units, long long per) {
    if (!ok) {
      std::printf("%s: units %lld per %lld\n", what, units, per);
      ++failures;
    }
  };
  fd::BatchItem I = {};
  I.circ = 7;
  I.RC = 3;
  I.nchunks = 5;
  for (int64_t units : {0, 1, 2, 3, 4, 5, 63, 64, 65, 1000, 4097})
    for (int64_t per : {1, 2, 3, 4, 64, 1000, 5000}) {
      std::vector<fd::BatchItem> v(1, I);   // appended to
      check(fd::batch_cut(units, per, I, &v), "refused", units, per);
      int64_t at = 0;
      for (size_t k = 1; k < v.size(); ++k) {
        const fd::BatchItem& x = v[k];
        check(x.u0 == at && x.u1 > x.u0 && x.u1 - x.u0 <= per && x.u1 <= units, "range", units, per);
        check(x.circ == 7 && x.RC == 3 && x.nchunks == 5, "members", units, per);
        at = x.u1;
      }
      check(at == units && (int64_t)v.size() - 1 == (units + per - 1) / per, "cover", units, per);
    }
  std::vector<fd::BatchItem> v;
  // the last unit numbers that an item holds
  check(fd::batch_cut(0x7fffffff, int64_t(1) << 30, I, &v) && v.back().u1 == 0x7fffffff, "largest", 0x7fffffff, 1 << 30);
  v.clear();
  for (int64_t units : {int64_t(-1), int64_t(1) << 31, int64_t(1) << 40})
    check(!fd::batch_cut(units, int64_t(1) << 30, I, &v) && v.empty(), "accepted", units, 1 << 30);
  for (int64_t per : {0, -4}) check(!fd::batch_cut(100, per, I, &v) && v.empty(), "accepted", 100, per);
  std::printf("%d failures\n", failures);
  return failures != 0;
}
