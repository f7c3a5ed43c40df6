"""CPU checks of native rules that need no device: small C++ programs compiled
against the library's own headers."""
import os
import subprocess

import paper_1503_05464_amd as P
from paper_1503_05464_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1503_05464_amd", "csrc")


def _run(tmp_path, source, compiler=("g++", "-std=c++17", "-O1", "-Wall", "-Werror"), flags=()):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(source)
    r = subprocess.run([*compiler, "-I", CSRC, "-o", str(exe), str(src), *flags], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


GEMM_OFFSETS = r"""
#include <cstdio>
#include <initializer_list>
#include "gemm_offsets.h"
using namespace hss;
int main() {
  long long fit = 0, far = 0;
  for (bool tr : {false, true})
    for (int M : {1, 2, 33, 128, 700})
      for (int K : {1, 15, 16, 17, 40, 511, 512, 513, 3000})
        for (long long base : {700LL, 1048576LL, 1050628LL, 1082402LL, 4194304LL, 8388608LL, 33554432LL, 536870911LL,
                               1LL << 31, 1LL << 40})
          for (long long d = -3; d <= 3; ++d) {
            const long long lda = base + d;
            if (lda < (tr ? M : K)) continue;
            if (!gemm_offsets_fit(tr, M, K, lda)) {
              ++far;
              continue;
            }
            ++fit;
            // every corner of the largest tile's first and last slice
            const int rows = M < kGemmMaxRows ? M : kGemmMaxRows;
            const int ns = ((K < kGemmChunk ? K : kGemmChunk) + kGemmSlice - 1) / kGemmSlice;
            for (int s : {0, ns - 1})
              for (int k : {0, kGemmSlice - 1})
                for (int r : {0, rows - 1}) {
                  const long long kk = (long long)s * kGemmSlice + k;
                  const long long want = 8 * (tr ? kk * lda + r : r * lda + kk);
                  const unsigned got = gemm_entry_offset(tr, lda, r, k) + (unsigned)s * gemm_slice_step(tr, lda);
                  if (got != want || want + 8 > 0xffffffffLL) {
                    std::printf("tr %d M %d K %d lda %lld s %d k %d r %d: %u for %lld\n", tr, M, K, lda, s, k, r, got, want);
                    return 1;
                  }
                }
          }
  // the first leading dimensions whose last slice wraps, and ordinary ones
  const bool ok = !gemm_offsets_fit(true, 64, 512, 1082402) && !gemm_offsets_fit(true, 64, 3000, 1050628) &&
                  !gemm_offsets_fit(false, 128, 64, 4300000) && !gemm_offsets_fit(false, 64, 16, 8500000) &&
                  gemm_offsets_fit(true, 64, 3000, 1048000) && gemm_offsets_fit(true, 64, 16, 30000000) &&
                  gemm_offsets_fit(false, 700, 3000, 4190000) && gemm_offsets_fit(false, 1, 64, 1 << 28);
  std::printf("%lld fit, %lld far\n", fit, far);
  return ok && fit > 100 && far > 100 ? 0 : 2;
}
"""


def test_gemm_offsets_of_a(tmp_path):
    """The batched GEMM's 32-bit offsets of A equal the 64-bit ones wherever
    its rule takes them, for leading dimensions around every place where one
    of their terms wraps; where they would wrap the rule says so."""
    _run(tmp_path, GEMM_OFFSETS)


SAMPLE_SPLITS = r"""
#include <cstdio>
#include "sample_plan.h"
using namespace hss;
int main() {
  for (int cus : {32, 64, 128, 256, 304})
    for (long long line : {512, 768})
      for (long long unit : {64, 256})
        for (long long n : {100, 511, 512, 767, 768, 1000, 2047, 4096, 8191})
          for (long long nt : {1, 2, 3, 16}) {
            const long long tiles = (n + 127) / 128 * nt, s = small_splits(n, tiles, line, unit, cus);
            const bool ok = n < line ? s == 1 : s <= 16 && s * unit <= n && s * tiles <= 2 * cus;
            if (!ok) {
              std::printf("n %lld tiles %lld on %d units: %lld splits\n", n, tiles, cus, s);
              return 1;
            }
          }
  return small_splits(1024, 8, 512, 64, 256) == 16 && small_splits(6000, 47, 512, 64, 256) == 10 ? 0 : 2;
}
"""


def test_sample_splits_follow_the_device(tmp_path):
    """The splits of a small matrix stay within two workgroups per compute
    unit of the device at hand, not of the largest."""
    _run(tmp_path, SAMPLE_SPLITS)


STAGING = r"""
#include <cstdio>
#include "hss_internal.h"
using namespace hss;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main() {
  Staging st;
  int ran[8] = {0};
  auto note = [&](int q, hipError_t e) { return st.launch([&ran, q, e] { ++ran[q]; return e; }); };
  {  // noted until the fourth, then run in order, once
    Deferred d(st);
    CHECK(note(0, hipSuccess) == hipSuccess && note(1, hipSuccess) == hipSuccess && note(2, hipSuccess) == hipSuccess);
    CHECK(ran[0] == 0 && ran[2] == 0);
    CHECK(note(3, hipSuccess) == hipSuccess && ran[0] == 1 && ran[3] == 1);
    CHECK(note(4, hipSuccess) == hipSuccess && ran[4] == 0 && d.done() == hipSuccess && ran[4] == 1);
  }
  for (int& r : ran) r = 0;
  {  // the third fails: the first two ran once, the fourth not at all, and the error stays
    Deferred d(st);
    (void)note(0, hipSuccess);
    (void)note(1, hipSuccess);
    (void)note(2, hipErrorLaunchFailure);
    (void)note(3, hipSuccess);  // its status left unread
    CHECK(note(4, hipSuccess) == hipErrorLaunchFailure);
    CHECK(st.issue() == hipErrorLaunchFailure && d.done() == hipErrorLaunchFailure);
    CHECK(ran[0] == 1 && ran[1] == 1 && ran[2] == 1 && ran[3] == 0 && ran[4] == 0);
  }
  for (int& r : ran) r = 0;
  {  // a call that ends early: what it noted is dropped
    Deferred d(st);
    (void)note(0, hipSuccess);
  }
  CHECK(ran[0] == 0 && !st.deferred && note(1, hipSuccess) == hipSuccess && ran[1] == 1);
  {  // ... and the next one starts afresh
    Deferred d(st);
    CHECK(note(2, hipSuccess) == hipSuccess && d.done() == hipSuccess && ran[2] == 1 && ran[0] == 0);
  }
  return 0;
}
"""


def test_noted_launches_run_once(tmp_path):
    """Launches that wait for their tables' copy: in order and once each, none
    after one that failed, none left over from a call that ended early, and a
    failure is reported by every later status of the call."""
    lib = os.path.dirname(P.LIB_PATH)
    _run(tmp_path, STAGING, (build._hipcc(), *build.COMMON), ("-L", lib, "-lhss", f"-Wl,-rpath,{lib}"))
