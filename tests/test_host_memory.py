"""CPU tests of the memory that the integral gradient and a product take.  The program runs the library's host code
on a HIP runtime of its own: device memory is host memory with a budget, and kernels do nothing, so
that the state's norm is zero and a gradient that came through every site ends in DMRG_ESTATE."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2609_09990_amd")

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>
#include <hip/hip_runtime.h>
#include "dmrg_mi355x.h"
#include "solver.hpp"
static size_t g_budget = size_t(1) << 60, g_used = 0, g_peak = 0;
static std::map<void*, size_t>& blocks() { static auto* m = new std::map<void*, size_t>; return *m; }
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  if (g_used + n > g_budget) return hipErrorOutOfMemory;
  *p = std::calloc(n, 1);
  blocks()[*p] = n;
  g_used += n;
  if (g_used > g_peak) g_peak = g_used;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  g_used -= blocks().at(p);
  blocks().erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 1.f; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s) {
  *g = *b = dim3(1);
  *l = 0;
  *s = nullptr;
  return hipSuccess;
}
}
// least budget of prepare + product, the peak before the product and the peak without a budget
int sigma_memory(dmrg_problem* p, dmrg_options o, int k) {
  size_t before = 0;
  auto run = [&](size_t budget) {
    dmrg_solver* s = nullptr;
    if (dmrg_solver_create(p, &o, nullptr, &s) != DMRG_OK) std::exit(1);
    g_budget = budget;
    g_peak = 0;
    int64_t len = 0;
    double fl;
    dmrg_status rc = dmrg_prepare(s, k, &len);
    before = g_peak;
    if (rc == DMRG_OK) {
      std::vector<double> psi(len), out(len);
      for (int twice = 0; twice < 2 && rc == DMRG_OK; ++twice)
        rc = dmrg_sigma(s, k, 0, len, psi.data(), out.data(), &fl);
    }
    g_budget = size_t(1) << 60;
    dmrg_solver_destroy(s);
    return rc;
  };
  if (run(size_t(1) << 60) != DMRG_OK) return 2;
  const size_t full = g_peak, prepared = before;
  size_t lo = prepared / 2, hi = full;
  while (hi - lo > full / 256) {
    const size_t mid = lo + (hi - lo) / 2;
    const dmrg_status rc = run(mid);
    if (rc != DMRG_OK && rc != DMRG_ENOMEM) return 3;
    if (rc == DMRG_OK) hi = mid;
    else lo = mid;
  }
  std::printf("%zu %zu %zu\n", prepared, hi, full);
  return 0;
}
int main(int argc, char**) {
  const int n = 10, nq = 8, M = 200;
  std::vector<double> h(n * n), B(nq * n * n), dh(n * n), dB(nq * n * n);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) h[i * n + j] = 1.0 / (1 + i + j);
  for (int q = 0; q < nq; ++q)
    for (int i = 0; i < n * n; ++i) B[q * n * n + i] = h[i] / (1 + q);
  dmrg_problem* p = nullptr;
  dmrg_options o;
  dmrg_options_default(&o);
  o.M = M;
  if (dmrg_problem_create(n, 5, 5, nq, h.data(), B.data(), 0.0, &p) != DMRG_OK) return 1;
  if (argc > 1) return sigma_memory(p, o, n / 2 - 1);
  // status of a gradient within a budget; held: what stays beside the gradient's own buffers
  size_t held = 0;
  auto run = [&](size_t budget) {
    dmrg_solver* s = nullptr;
    if (dmrg_solver_create(p, &o, nullptr, &s) != DMRG_OK) std::exit(1);
    double e;
    g_budget = budget;
    g_peak = 0;
    const dmrg_status rc = dmrg_grad(s, nullptr, dh.data(), dB.data(), &e);
    g_budget = size_t(1) << 60;
    dmrg::drop_idle_memory();
    held = g_used;
    dmrg_solver_destroy(s);
    return rc;
  };
  if (run(size_t(1) << 60) != DMRG_ESTATE) return 2;
  const size_t full = g_peak, beside = held;
  size_t lo = beside, hi = full;  // the smallest budget that is enough
  while (hi - lo > full / 256) {
    const size_t mid = lo + (hi - lo) / 2;
    const dmrg_status rc = run(mid);
    if (rc != DMRG_ESTATE && rc != DMRG_ENOMEM) return 3;
    if (rc == DMRG_ESTATE) hi = mid;
    else lo = mid;
  }
  if (g_used != 0 && (dmrg_problem_destroy(p), g_used != 0)) return 4;
  std::printf("%zu %zu %zu\n", beside, hi, full);
}
"""


def _program(tmp_path):
    import paper_2609_09990_amd as pk
    assert os.path.dirname(pk.LIB_PATH) == PKG
    src, exe = tmp_path / "grad.cpp", tmp_path / "grad"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(PKG, "csrc"), "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(exe),
                    "-L" + PKG, "-l:libdmrg_mi355x.so", "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib",
                    "-Wl,--allow-shlib-undefined", "-rdynamic"], check=True)
    return str(exe)


def _numbers(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-500:])
    print(r.stdout)
    return (int(x) for x in r.stdout.split())


def test_gradient_runs_in_less_memory_than_its_largest_batch(tmp_path):
    beside, least, full = _numbers([_program(tmp_path)])
    # the classes one by one, and rows by the piece, take less than half of what the batch takes
    assert least - beside < 0.5 * (full - beside)


def test_product_runs_without_room_for_its_partial_tiles(tmp_path):
    prepared, least, full = _numbers([_program(tmp_path), "sigma"])
    # the tables of a product's units and items remain
    assert least - prepared < 0.5 * (full - prepared)
