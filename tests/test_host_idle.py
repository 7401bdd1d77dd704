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


THREADS = r"""
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>
#include "ci.hpp"
using namespace dmrg;
extern "C" hipError_t hipMalloc(void** p, size_t n) {
  if (n > 1000000) return hipErrorOutOfMemory;
  *p = std::malloc(64);
  return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
extern "C" hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
static std::atomic<int> g_dropped{0};
struct Early {  // runs while the object is under construction
  Early() { drop_idle_memory(); }
};
struct Probe final : IdleMemory, Early {
  Probe() { enroll(); }
  ~Probe() { retire(); }
  void drop() override { ++g_dropped; }
};
int main() {
  {
    Probe p;
    if (g_dropped != 0) return 1;
    drop_idle_memory();
    if (g_dropped != 1) return 2;
  }
  drop_idle_memory();
  if (g_dropped != 1) return 3;
  std::atomic<bool> stop{false};
  std::atomic<long> refused{0};
  std::vector<std::thread> t;
  for (int i = 0; i < 2; ++i)
    t.emplace_back([&] {  // allocations that fail
      while (!stop) {
        DevMem d;
        try {
          d.reserve(2000000);
        } catch (const Error&) {
          ++refused;
        }
      }
    });
  for (int i = 0; i < 2; ++i)
    t.emplace_back([&] {  // problems and gradients that come and go
      for (int k = 0; k < 4000; ++k) {
        CiPool pool;
        auto w = pool.take();
        w->T1.reserve(1000);
        pool.give(std::move(w));
        GradWork g;
        GradWork::Use use(g);
        g.P.reserve(1000);
        if (!g.P.p) std::abort();
      }
    });
  t[2].join();
  t[3].join();
  stop = true;
  t[0].join();
  t[1].join();
  std::puts(refused > 0 ? "ok" : "idle");
}
"""


def _run(tmp_path, source):
    import paper_2609_09990_amd as pk
    assert os.path.dirname(pk.LIB_PATH) == PKG
    src, exe = tmp_path / "idle.cpp", tmp_path / "idle"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(PKG, "csrc"), str(src), "-o", str(exe), "-L" + PKG, "-l:libdmrg_mi355x.so",
                    "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-shlib-undefined", "-rdynamic"],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stdout, r.stderr[-500:])


def test_kept_memory_is_given_back_when_an_allocation_fails(tmp_path):
    _run(tmp_path, SOURCE)


def test_objects_that_come_and_go_while_allocations_fail(tmp_path):
    """Nothing is dropped of an object that is being made or taken apart."""
    _run(tmp_path, THREADS)
