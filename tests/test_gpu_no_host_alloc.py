"""mg_solve_noalloc allocates no host memory either: a C program that links the library and counts
its calls of operator new (the program's own definition takes the library's calls) during the
second of two solves, over precisions, layouts and schemes and enough cycles for any growing array."""
import os
import shutil
import subprocess

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_2302_13903_amd", "_build")

PROGRAM = r"""
#include <dlfcn.h>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>
#include "mg355.h"

extern "C" {
int hipMalloc(void**, size_t);
int hipMemcpy(void*, const void*, size_t, int);
}

static bool counting = false;
static int calls = 0;

static void* counted(size_t n, void* from) {
  Dl_info where;
  if (counting && dladdr(from, &where) && where.dli_fname && std::strstr(where.dli_fname, "libmg355")) ++calls;
  void* p = std::malloc(n ? n : 1);
  if (!p) std::abort();
  return p;
}
void* operator new(size_t n) { return counted(n, __builtin_return_address(0)); }
void* operator new[](size_t n) { return counted(n, __builtin_return_address(0)); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete[](void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
void operator delete[](void* p, size_t) noexcept { std::free(p); }

int main() {
  const int n = 64;
  const size_t n3 = (size_t)n * n * n;
  std::vector<double> host(n3);
  for (size_t c = 0; c < n3; ++c) host[c] = std::sin(0.7 * (double)c);
  double *rho = nullptr, *phi = nullptr;
  if (hipMalloc((void**)&rho, n3 * 8) || hipMalloc((void**)&phi, n3 * 8) || hipMemcpy(rho, host.data(), n3 * 8, 1)) return 2;
  mg_ctx* ctx = nullptr;
  if (mg_ctx_create(&ctx, 0, 0) != MG_OK) return 3;
  const int precision[4] = {MG_PREC_FP64, MG_PREC_MIXED, MG_PREC_FP64, MG_PREC_FP64};
  int bad = 0;
  for (int q = 0; q < 4; ++q) {
    mg_params p;
    mg_default_params(&p);
    p.n = n;
    p.dx = 1.0 / n;
    p.precision = precision[q];
    p.layout = q == 2 ? MG_LAYOUT_BLOCKS : MG_LAYOUT_DENSE;
    p.scheme = q == 3 ? MG_SCHEME_FAS : MG_SCHEME_CS;
    p.fixed_cycles = 40;
    mg_bc bc;
    std::memset(&bc, 0, sizeof(bc));
    for (int f = 0; f < 6; ++f) bc.kind[f] = MG_BC_FIXED;
    double hist[64];
    int n_hist = 0;
    for (int pass = 0; pass < 2; ++pass) {
      counting = pass == 1;
      calls = 0;
      const int st = mg_solve_noalloc(ctx, &p, &bc, rho, phi, hist, &n_hist, nullptr);
      counting = false;
      if (st != MG_OK || n_hist != 41) return 4;
    }
    std::printf("case %d: %d allocations\n", q, calls);
    bad += calls;
  }
  // the counter does count the library's calls: mg_solve keeps the cycles' times
  mg_params p;
  mg_default_params(&p);
  p.n = n;
  p.dx = 1.0 / n;
  p.fixed_cycles = 40;
  mg_bc bc;
  std::memset(&bc, 0, sizeof(bc));
  double hist[64];
  int n_hist = 0;
  calls = 0;
  counting = true;
  if (mg_solve(ctx, &p, &bc, rho, phi, hist, &n_hist, nullptr) != MG_OK) return 5;
  counting = false;
  std::printf("mg_solve: %d allocations\n", calls);
  if (calls == 0) return 6;
  mg_ctx_destroy(ctx);
  return bad ? 1 : 0;
}
"""


def test_noalloc_solve_allocates_no_host_memory(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "count.cpp", tmp_path / "count"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-fno-builtin", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe),
                    "-rdynamic", os.path.join(BUILD, "libmg355.so"), f"-Wl,-rpath,{BUILD}", "-L/opt/rocm/lib",
                    "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64", "-ldl"], check=True)
    print("counting allocations", flush=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    print(r.stdout, r.stderr, flush=True)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
