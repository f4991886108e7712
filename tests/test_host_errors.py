"""What a handle's host state says after a launch has failed (no GPU needed).

A small program links the library and defines the HIP runtime calls that it makes: launches are counted and named, none
runs, and the one with a chosen number fails.  Whatever launch of an iteration fails, A^T A has to be formed again before
anything reads it: the iteration clears it at its start and the A rule fills it at its end."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "nnrescal.h"
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

// ---- the HIP runtime as far as the library calls it: nothing runs, "device" memory is host memory
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static std::vector<std::string> trace;             // kernels launched since the last clear
static long fail_at = -1, launches = 0;
static hipError_t last = hipSuccess;
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static hipStream_t cfg_stream;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) { cfg_grid = g; cfg_block = b; cfg_lds = l; cfg_stream = s; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s) { *g = cfg_grid; *b = cfg_block; *l = cfg_lds; *s = cfg_stream; return hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
  if (launches++ == fail_at) return last = hipErrorLaunchFailure;
  trace.push_back(names()[f]);
  return hipSuccess;
}
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "the launch that was to fail"; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static void* at = calloc(1, 64u << 20); *p = at; return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
}

static void* take(size_t n, void*) { return calloc(1, n); }
static void give(void* p, void*) { free(p); }

// A^T A: the Gram kernel with its second operand equal to the first (its third template argument is true)
static bool forms_gram() {
  for (const std::string& s : trace)
    if (s.find("gram16_kernel") != std::string::npos && s.find("Lb1ELb0E") != std::string::npos) return true;
  return false;
}

static nnrescal_handle* make(nnrescal_tensor& X, nnrescal_params& p) {
  nnrescal_handle* h = nullptr;
  if (nnrescal_init(&h, &X, &p) != NNRESCAL_OK) { printf("init: %s\n", nnrescal_last_error(nullptr)); exit(2); }
  return h;
}

int main(int argc, char** argv) {
  const int k = atoi(argv[1]), n = 100, m = 2, q = 3;
  std::vector<float> x((size_t)m * n * n, 1.0f), A((size_t)q * n * k), R((size_t)q * m * k * k);
  std::vector<double> f(q);
  nnrescal_tensor X{};
  X.format = NNRESCAL_DENSE; X.n = n; X.m = m; X.dense = x.data();
  nnrescal_params p{};
  p.k = k; p.q = q; p.delta = 0.03f; p.eps_div = 1e-16f; p.alloc = take; p.dealloc = give; p.no_fused_small = 1;
  p.deterministic = atoi(argv[2]);
  int bad = 0, steps = 0;
  // a failing launch inside the first A^T A: it has to be formed again
  for (int at = 0; at < 2; ++at) {
    nnrescal_handle* h = make(X, p);
    fail_at = at; launches = 0;
    const bool failed = nnrescal_get_factors(h, A.data(), R.data(), 1) != NNRESCAL_OK;
    fail_at = -1; trace.clear();
    if (failed && (nnrescal_get_factors(h, A.data(), R.data(), 1) != NNRESCAL_OK || !forms_gram())) { printf("first A^T A, launch %d\n", at); ++bad; }
    nnrescal_destroy(h);
  }
  // every launch of an iteration with objective terms in turn, and after it every call that reads A^T A
  for (int reader = 0; reader < 3; ++reader)
    for (long at = 0;; ++at) {
      nnrescal_handle* h = make(X, p);
      if (nnrescal_mu_step(h) != NNRESCAL_OK) { printf("step\n"); return 2; }
      fail_at = at; launches = 0; trace.clear();
      int32_t done = 0;
      const nnrescal_status st = nnrescal_fit_until(h, 1, 0.0, 1, &done, nullptr);
      const bool hit = launches > at, cleared = !trace.empty();
      fail_at = -1; trace.clear();
      if (!hit) { nnrescal_destroy(h); break; }
      ++steps;
      if (st != NNRESCAL_EDEVICE) { printf("launch %ld failed, status %d\n", at, (int)st); ++bad; }
      const nnrescal_status after = reader == 0 ? nnrescal_get_factors(h, A.data(), R.data(), 1)
                                  : (reader == 1 ? nnrescal_mu_step(h) : nnrescal_objective(h, f.data(), nullptr));
      if (after != NNRESCAL_OK) { printf("launch %ld, reader %d: %s\n", at, reader, nnrescal_last_error(h)); ++bad; }
      if (cleared && !forms_gram()) { printf("launch %ld failed: reader %d takes the cleared A^T A\n", at, reader); ++bad; }
      // and once more: what has been formed is not formed again
      trace.clear();
      if (nnrescal_get_factors(h, A.data(), R.data(), 1) != NNRESCAL_OK || forms_gram()) { printf("launch %ld, reader %d: formed twice\n", at, reader); ++bad; }
      nnrescal_destroy(h);
    }
  printf("%d failing launches, %d mistakes\n", steps, bad);
  return bad || steps < 15 ? 1 : 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    import paper_2202_09512_amd as nn
    if not os.path.exists(nn.lib_path()):
        from paper_2202_09512_amd import build
        build.build(verbose=False)
    folder = tmp_path_factory.mktemp("host_errors")
    src, exe = folder / "errors.cpp", folder / "errors"
    src.write_text(SOURCE)
    # the program's own definitions come first when the library's references are bound (-rdynamic exports them)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), str(src), nn.lib_path(), "-Wl,-rpath," + os.path.dirname(nn.lib_path()),
                    "-Wl,--allow-shlib-undefined", "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("k", [8, 40])
@pytest.mark.parametrize("reproducible", [0, 1])
def test_gram_is_formed_again_after_a_failed_launch(program, k, reproducible):
    out = subprocess.run([program, str(k), str(reproducible)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr


FILL_SOURCE = r"""
#include "kernels.h"
#include <cstdio>
using namespace nnr;
int main() {
  int32_t word[FillList::kMax + 1] = {};
  FillList fl;
  for (int i = 0; i < FillList::kMax; ++i) fl.add(word + i, 4);
  fl.add(nullptr, 4);                              // no buffer: needs no place
  fl.add(word, 0);
  const bool whole = fl.count == FillList::kMax && !fl.overflow;
  fl.add(word + FillList::kMax, 4);
  const hipError_t e = launch_fill_zero_multi(fl, nullptr);
  printf("whole %d, one too many: %d\n", (int)whole, (int)e);
  return whole && e == hipErrorInvalidValue ? 0 : 1;
}
"""


def test_fill_list_refuses_what_it_cannot_hold(tmp_path):
    """A buffer that does not fit the list must not be left uncleared without a word."""
    from paper_2202_09512_amd import build
    obj = os.path.join(build.HERE, "_build", "kernels_small.o")
    if not os.path.exists(obj):
        build.build(verbose=False)
    src, exe = tmp_path / "fill.cpp", tmp_path / "fill"
    src.write_text(FILL_SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", "-std=c++17", "-O1", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(build.HERE, "csrc"),
                    str(src), "-x", "none", obj, "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
