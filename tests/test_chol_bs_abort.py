"""A wait past its bound in the back-substitution of the tile Cholesky.

The four waves of a k_chol_bs workgroup wait for the same flags, each for
itself, so one of them can reach its bound (or see the abort word of the batch)
while another finds the flag set.  Whichever wave it is, the workgroup's sums
are incomplete: the window has to be marked failed, its block left unpublished,
and a wave that reached its own bound has to set the abort word for the others.

The kernel's source is compiled for the CPU, one thread per lane, with the wave
operations on barriers; the load of a flag is where a late one is put in.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_02293_amd", "csrc")

SHIM = r"""
#pragma once
#include <cmath>
#include <cstddef>
#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
typedef void* hipStream_t;
typedef int hipError_t;
"""

HARNESS = r"""
#include <algorithm>
#include <barrier>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>
#include "vi_internal.h"
#define __shared__ static
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __builtin_amdgcn_fence(order, scope) __atomic_thread_fence(order)
#define __builtin_amdgcn_s_sleep(n) std::this_thread::yield()
#define __builtin_amdgcn_readfirstlane(v) emu_first(v)
#define __hip_atomic_load(p, order, scope) emu_load(p)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)
struct Idx { unsigned x; };
static thread_local Idx threadIdx;
static std::barrier<> block_bar(256);
static std::barrier<> wave_bar[4] = {std::barrier<>(64), std::barrier<>(64), std::barrier<>(64), std::barrier<>(64)};
static long long wave_val[4][64];
static void __syncthreads() { block_bar.arrive_and_wait(); }
static int emu_first(int v) {
  const int w = threadIdx.x / 64;
  wave_val[w][threadIdx.x % 64] = v;
  wave_bar[w].arrive_and_wait();
  const int r = (int)wave_val[w][0];
  wave_bar[w].arrive_and_wait();
  return r;
}
static unsigned long long __ballot(int v) {
  const int w = threadIdx.x / 64;
  wave_val[w][threadIdx.x % 64] = v != 0;
  wave_bar[w].arrive_and_wait();
  unsigned long long m = 0;
  for (int l = 0; l < 64; ++l) m |= (unsigned long long)wave_val[w][l] << l;
  wave_bar[w].arrive_and_wait();
  return m;
}
static int atomicAdd(int* p, int v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
static int atomicCAS(int* p, int c, int v) {
  __atomic_compare_exchange_n(p, &c, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
  return c;
}
using std::min;
static int late_waves, abort_wave = -1;                // masks, from the command line
static const int *late_flag, *abort_word;
static int emu_load(const int* f) {
  const int w = threadIdx.x / 64;
  if (f == late_flag && (late_waves >> w & 1)) return 0;
  if (f == abort_word && w == abort_wave) return 1;
  return __atomic_load_n(f, __ATOMIC_SEQ_CST);
}
namespace vi {
constexpr int NB = kCholNB, kPairTicket = kPairTicketFlag, kSpinLimit = 64;
@CODE@
}  // namespace vi
using namespace vi;
int main(int argc, char** argv) {
  late_waves = atoi(argv[1]);
  abort_wave = atoi(argv[2]);
  // one window of three dense block columns: tickets (2, 1) and 0; the flag of
  // x_1 is the late one
  const int nblk = 3, n = NB * nblk;
  std::vector<double> A((size_t)(n + NB) * n), Li((size_t)n * NB), x(n, -7.0);
  auto L = [&](int i, int j) { return i == j ? 1.0 : (i / NB == j / NB ? 0.0 : 0.01 * ((i * 7 + j * 3) % 11 - 5)); };
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < i; ++j) A[(size_t)i * n + j] = L(i, j);
  for (int i = 0; i < n; ++i) {
    A[(size_t)n * n + i] = 1.0 + i % 5;
    Li[(size_t)(i / NB) * NB * NB + (i % NB) * NB + i % NB] = 1.0;
  }
  std::vector<int> flags((nblk + 2) * nblk, 0), tab(3 * nblk + 1, 0);
  for (int i = 0; i <= nblk; ++i) tab.push_back(i == nblk ? 7 : (2 << i) - 1);
  const int tiles[] = {0, 2 | kPairTicket, 0, 0};
  int sync[4] = {0, 0, 0, 0};
  WinDev W{};
  W.n = W.npad = n;
  W.nblk = nblk;
  DevPlan D{};
  D.win = &W;
  D.chol_tiles = tiles;
  D.chol_tab = tab.data();
  DevStatus st{};
  int* xf = flags.data() + (nblk + 1) * nblk;
  late_flag = xf + 1;
  abort_word = sync + 1;
  std::vector<std::thread> th;
  for (unsigned t = 0; t < 256; ++t)
    th.emplace_back([&, t] {
      threadIdx.x = t;
      k_chol_bs(D, 0, 2, A.data(), Li.data(), x.data(), flags.data(), sync, &st);
    });
  for (auto& t : th) t.join();
  double err = 0.0;                                    // L^T x = y
  for (int j = 0; j < n; ++j) {
    double s = A[(size_t)n * n + j] - x[j];
    for (int i = j + 1; i < n; ++i) s -= L(i, j) * x[i];
    err = std::max(err, std::fabs(s));
  }
  printf("%d %d %d %d\n", st.code, xf[0], sync[1], err < 1e-12);
  return 0;
}
"""


def _function(src, head):
    """The text of the function whose declaration starts with head."""
    m = re.search(re.escape(head), src)
    assert m, head
    return src[m.start():src.index("\n}\n", m.start()) + 3]


@pytest.fixture(scope="module")
def emulated(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("chol_bs")
    src = open(os.path.join(CSRC, "k_chol.hip")).read()
    code = "".join(_function(src, h) for h in (
        "__device__ __forceinline__ void set_status(", "__device__ __forceinline__ int load_flag(",
        "__device__ __forceinline__ bool spin_flag(", "__global__ void __launch_bounds__(256) k_chol_bs("))
    (tmp / "hip").mkdir()
    (tmp / "hip" / "hip_runtime.h").write_text(SHIM)
    (tmp / "emu.cpp").write_text(HARNESS.replace("@CODE@", code))
    exe = str(tmp / "emu")
    subprocess.run(["g++", "-std=c++20", "-O1", "-w", "-pthread", "-I", str(tmp), "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), "-include", str(tmp / "hip" / "hip_runtime.h"),
                    str(tmp / "emu.cpp"), "-o", exe], check=True)

    def run(late_waves, abort_wave):
        out = subprocess.run([exe, str(late_waves), str(abort_wave)], check=True, capture_output=True, text=True,
                             timeout=60).stdout
        return [int(v) for v in out.split()]
    return run


def test_without_a_late_flag_the_block_is_solved(emulated):
    assert emulated(0, -1) == [0, 1, 0, 1]


@pytest.mark.parametrize("waves", [1, 2, 4, 8, 14, 15])
def test_any_wave_past_its_bound_fails_the_window(emulated, waves):
    code, published, abort_word, _ = emulated(waves, -1)
    assert (code, published, abort_word) == (-3, 0, 1)          # VI_EDEVICE


@pytest.mark.parametrize("wave", [0, 1, 2, 3])
def test_an_abort_seen_by_one_wave_fails_the_window(emulated, wave):
    # (with the flag late for every wave, the one that knows does not wait)
    code, published, _, _ = emulated(15, wave)
    assert (code, published) == (-3, 0)
    # the wave that knows must not publish sums of its own part either
    code, published, _, _ = emulated(1 << wave, wave)
    assert (code, published) == (-3, 0)
