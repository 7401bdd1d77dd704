"""CPU test of the device memory that is kept between calls: it is given back when an allocation
does not fit beside it, buffers in use and those of a workspace are not, and a program that never
runs out keeps them.  The program brings its own hipMalloc / hipFree with a byte budget."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2609_09990_amd")

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include "ci.hpp"
using namespace dmrg;
static size_t g_budget = 1000, g_used = 0;
static std::map<void*, size_t>& blocks() { static auto* m = new std::map<void*, size_t>; return *m; }
extern "C" hipError_t hipMalloc(void** p, size_t n) {
  if (g_used + n > g_budget * 1000) return hipErrorOutOfMemory;
  *p = std::malloc(64);  // never touched
  blocks()[*p] = n;
  g_used += n;
  return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) {
  g_used -= blocks().at(p);
  blocks().erase(p);
  std::free(p);
  return hipSuccess;
}
extern "C" hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
static bool fits(size_t kb) {
  DevMem d;
  try {
    d.reserve(kb * 1000);
  } catch (const Error& e) {
    if (e.code != ST_ENOMEM) std::exit(9);
    return false;
  }
  return true;
}
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
  {
    CiPool pool;
    auto w = pool.take();
    w->T1.reserve(600 * 1000);
    CHECK(!fits(500));  // in use: stays
    CHECK(g_used > 600 * 1000);
    pool.give(std::move(w));
    CHECK(g_used > 600 * 1000);  // kept
    CHECK(fits(300) && g_used > 600 * 1000);
    CHECK(fits(500) && g_used == 0);  // given back for an allocation that needs it
    CHECK(!fits(1200));
  }
  {
    GradWork g;
    {
      GradWork::Use use(g);
      g.P.reserve(300 * 1000);
      g.tab[1].items.reserve(300 * 1000);
      {
        GradWork::Use inner(g);
      }
      CHECK(!fits(500) && g.P.p);
    }
    CHECK(g.bytes() == 600 * 1000 && g_used > 600 * 1000);
    CHECK(fits(500) && g.bytes() == 0 && g_used == 0);
    g.ph.d_units[0].reserve(1000);
    CHECK(g.bytes() == 1000);
  }
  CHECK(g_used == 0);
  {
    static char space[1 << 20];
    Arena arena(space, sizeof(space));
    GradWork g;
    ArenaScope scope(&arena);
    {
      GradWork::Use use(g);
      g.P.reserve(1000);
    }
    const size_t before = arena.in_use();
    drop_idle_memory();
    CHECK(arena.in_use() == before && g.P.p);
    g.release();
    CHECK(arena.in_use() == 0);
  }
  CHECK(g_used == 0);
  std::puts("ok");
}
"""


def test_kept_memory_is_given_back_when_an_allocation_fails(tmp_path):
    import paper_2609_09990_amd as pk
    assert os.path.dirname(pk.LIB_PATH) == PKG
    src, exe = tmp_path / "idle.cpp", tmp_path / "idle"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(PKG, "csrc"),
                    str(src), "-o", str(exe), "-L" + PKG, "-l:libdmrg_mi355x.so", "-Wl,-rpath," + PKG,
                    "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-shlib-undefined", "-rdynamic"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stdout, r.stderr[-500:])
