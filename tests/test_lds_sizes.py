"""The LDS a batch allocates for a size class holds the layout of every decode the class may run
(host arithmetic of csrc/lds_sizes.h, compiled for the CPU)."""
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


def test_batch_classes_hold_every_layout(tmp_path):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(CHECK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I",
                    os.path.join(ROOT, "paper_1903_10741_amd", "csrc"), "-o", str(exe), str(src)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
