"""Host arithmetic of csrc/lds_sizes.h, compiled for the CPU: the LDS a batch allocates for a size
class holds the layout of every decode the class may run, and the default on-chip slots cost no
wave."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# A slot's on-chip slots are its class's, or fewer where its horizon (a multiple of 64 here)
# needs fewer, and its own size may be smaller than the batch's; the batch's packed rows keep
# the batch's width.
CHECK = r"""
#include <cstdio>
#include <initializer_list>
#include "lds_sizes.h"
int main() {
  int bad = 0;
  const int genes[] = {1, 2, 63, 150, 200, 1000, 4096}, widths[] = {1, 4, 5, 8, 9, 16};
  for (int n : genes)
    for (int om : widths)
      for (int cls = 64; cls <= 33600; cls += cls < 32000 ? 992 / 64 * 64 : 64)
        for (int rules = 0; rules < 2; ++rules) {
          const int omp = ffs_lds::omp_of(om);
          const size_t have = ffs_lds::batch_lds(n, omp, cls);
          for (int cap = cls; cap >= 64; cap -= cap > 32000 ? 64 : 4992)
            for (int m : {n, n > 1 ? n / 2 : 1}) {
              const size_t need = ffs_lds::lds_bytes_rules(rules, m, omp, cap);
              if (need <= have) continue;
              if (++bad <= 5)
                std::printf("genes %d row %d class %d slots %d rules %d: %zu > %zu\n", m, omp, cls,
                            cap, rules, need, have);
            }
        }
  return bad != 0;
}
"""


def _run(tmp_path, text):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(text)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I",
                    os.path.join(ROOT, "paper_1903_10741_amd", "csrc"), "-o", str(exe), str(src)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_batch_classes_hold_every_layout(tmp_path):
    _run(tmp_path, CHECK)


# Default slots: on either side of the sizes from which a population fills its waves, at several
# job counts, row widths and decode rules, a compute unit never holds fewer of its waves than at
# the 4096 slots the workspace is laid out for, and the slots stay within their bounds.
ROOMY = r"""
#include <cstdio>
#include <initializer_list>
#include "lds_sizes.h"
int main() {
  const int64_t lds = 163840, cus = 256;
  int bad = 0;
  for (int rules = 0; rules < 2; ++rules)
    for (int n : {1, 20, 50, 116, 200, 385, 1000, 4096})
      for (int omp : {4, 8, 16})
        for (int64_t horizon : {5000, 8543, 20229, 35868, 400000})
          for (int64_t pop : {1, 2, 255, 256, 257, 1024, 4070, 4096, 4097, 4300, 6000, 8192, 16384, 65536})
          for (bool groups : {false, true}) {
            const int base = 4096;
            auto bytes = [&](int cap) { return ffs_lds::lds_bytes_rules(rules, n, omp, cap); };
            const int cap = ffs_lds::roomy_slots(base, horizon, pop, groups, cus, lds, bytes);
            // waves that a unit can use: its share of the population, and one more for island
            // groups, whose launches do not spread evenly
            const int64_t use = (pop + cus - 1) / cus + groups;
            int64_t want = ffs_lds::waves_held(bytes(base), lds);
            if (want > use) want = use;
            const int64_t got = ffs_lds::waves_held(bytes(cap), lds);
            const bool ok = got >= want && cap >= base && cap % 64 == 0 &&
                            cap <= ffs_lds::kChipSlots &&
                            (cap == base || cap >= horizon || 2 * cap >= 3 * base) && cap < horizon + 64;
            if (ok) continue;
            if (++bad <= 5)
              std::printf("rules %d genes %d row %d horizon %lld pop %lld: %d slots, %lld of %lld waves\n",
                          rules, n, omp, (long long)horizon, (long long)pop, cap, (long long)got,
                          (long long)want);
          }
  return bad != 0;
}
"""


def test_default_slots_cost_no_wave(tmp_path):
    _run(tmp_path, ROOMY)
