"""CPU test of the look-ahead into a unit's item list (the stream kernel's first reads): it stays
inside the list, and an empty list is not read, also where it starts at the table's first item.
The table lies between two pages that cannot be read, so a read outside ends the program."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <sys/mman.h>
#include <unistd.h>
#include <cstdio>
#include "kernels.hpp"
using namespace dmrg;
int main() {
  const long page = sysconf(_SC_PAGESIZE);
  char* m = (char*)mmap(nullptr, 3 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  if (m == MAP_FAILED) return 3;
  const int n = (int)(page / sizeof(GemmItem));
  char* end = m + 2 * page;
  GemmItem* low = (GemmItem*)(m + page);                // starts at the first readable byte
  GemmItem* high = (GemmItem*)end - n;                  // ends at the last one
  if (mprotect(m, page, PROT_NONE) || mprotect(end, page, PROT_NONE)) return 3;
  for (GemmItem* t : {low, high}) {
    for (int i = 0; i < n; ++i) t[i].K = i + 1;
    for (int lane = 0; lane < 128; ++lane) {
      if (list_depth(t, lane, 0, 0) != 0) return 1;      // a block without a product, first in the table
      if (list_depth(t, n + lane, n, n) != 0) return 1;  // and after the last item
      if (list_depth(t, n - 3 + lane, n - 3, n) != (lane < 3 ? n - 2 + lane : n)) return 2;
    }
  }
  puts("ok");
}
"""


def test_look_ahead_stays_inside_the_list(tmp_path):
    src, exe = tmp_path / "depth.cpp", tmp_path / "depth"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2609_09990_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.returncode
