"""The single-field entry points make no heap allocation of their own after a first call: none that could throw
through the C interface, none in the call for code that may not allocate.  A small program replaces operator new
and throws from it when the caller is libmsl."""
import os
import subprocess

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#define __HIP_PLATFORM_AMD__
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include "msl.h"
static bool armed = false;
__attribute__((noinline)) void* operator new(size_t n) {
  Dl_info i;
  if (armed && dladdr(__builtin_return_address(0), &i) && i.dli_fname && std::strstr(i.dli_fname, "libmsl.so")) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
template <class T> T* dev(size_t n) {
  void* p = nullptr;
  if (hipMalloc(&p, n * sizeof(T)) != hipSuccess) std::exit(9);
  hipMemset(p, 0, n * sizeof(T));
  return static_cast<T*>(p);
}
int main() {
  for (int exact = 0; exact < 2; ++exact) {
    const msl_geometry g{64, 32, 20, 1.0, 1.0, 5.0, 0.1, 0.004, exact};
    const size_t m = 64 * 32, bytes = msl_workspace_bytes(&g, 8);
    float *d = dev<float>(20 * m), *b = dev<float>(20 * m), *gd = dev<float>(20 * m), *gb = dev<float>(20 * m), *I = dev<float>(m);
    msl_c64 *f = dev<msl_c64>(m), *ck = dev<msl_c64>(3 * m), *gf = dev<msl_c64>(m);
    char* ws = dev<char>(bytes);
    for (int pass = 0; pass < 2; ++pass) {
      armed = pass == 1;
      try {
        if (msl_forward_noalloc(&g, d, b, nullptr, f, nullptr, 0, nullptr) || msl_forward(&g, d, b, nullptr, f, ck, 8, 0, ws, bytes, nullptr) ||
            msl_far_field(&g, f, I, ws, bytes, nullptr) || msl_far_field_adjoint(&g, f, I, gf, ws, bytes, nullptr) ||
            msl_adjoint(&g, d, b, nullptr, ck, 8, gf, gd, gb, nullptr, 0, ws, bytes, nullptr)) {
          armed = false;
          std::printf("error: %s\n", msl_last_error());
          return 2;
        }
      } catch (const std::bad_alloc&) {
        armed = false;
        std::printf("libmsl allocated\n");
        return 1;
      }
      armed = false;
      if (hipDeviceSynchronize() != hipSuccess) return 3;
    }
  }
  std::printf("OK\n");
  return 0;
}
"""


def test_calls_do_not_allocate(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib = os.path.join(ROOT, "paper_2212_01253_amd")
    src, exe = tmp_path / "alloc.cpp", str(tmp_path / "alloc")
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-w", "-I", os.path.join(ROOT, "include"), "-I/opt/rocm/include", "-o", exe,
                    str(src), os.path.join(lib, "libmsl.so"), "-Wl,-rpath," + lib, "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib",
                    "-lamdhip64", "-ldl"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr
