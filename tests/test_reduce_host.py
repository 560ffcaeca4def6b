"""The reduction kernel's blocks on the CPU, one after the other in several orders.

Blocks of a launch run in any order and beside one another, so nothing that one
block of k_reduce writes may be read by another.  The kernel's own source is
compiled here for the host (a thread per lane, a barrier for __syncthreads) and
run with its blocks first to last, last to first and in the middle first: loss,
history, calibration gradient and the updated calibration vector must be the same
bits.  The tiles are those of the plan: 64 fields up to 32 records, 8 fields
above; an empty group has one tile."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_00250_amd", "csrc")

HARNESS = r"""
#include <hip/hip_runtime.h>
#undef __launch_bounds__
#undef __shared__
#undef __forceinline__
#define __launch_bounds__(...)
#define __shared__ static
#define __forceinline__ inline
#include <algorithm>
#include <barrier>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <thread>
#include <vector>
#include "prism_internal.h"

struct Idx { unsigned x; };
static thread_local Idx threadIdx;
static Idx blockIdx, blockDim;
static std::barrier<>* g_bar;
static void __syncthreads() { g_bar->arrive_and_wait(); }
static double g_lane[1024];
namespace prism {
static double wave_sum_f64(double x) {   // every thread of the block calls it
  g_lane[threadIdx.x] = x;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < 64; ++i) s += g_lane[(threadIdx.x & ~63u) + i];
  __syncthreads();
  return s;
}
static void atomicOr(uint32_t* p, uint32_t v) { *p |= v; }
enum { kMSE = 0, kNLL = 1, kPriorCal = 8, kStNonfiniteLoss = 1, kStNonfiniteGrad = 2 };
static float rcp(float x) { return 1.0f / x; }
static float sqrt_hw(float x) { return std::sqrt(x); }
using std::isfinite; using std::max; using std::min;
@SOURCE@
}  // namespace prism
using namespace prism;

struct State {
  std::vector<double> rec, loss, hist, calsq;
  std::vector<float> cal, gcal, m, v;
};

static State run(int mode, int items, int order) {
  const int N = 37, nb = 10, nc = nb + 2 * N + 1, stride = kRecHead + 2 * N;
  std::mt19937 rng(7 + items);
  std::uniform_real_distribution<double> u(-1.0, 1.0);
  State s;
  s.rec.resize((size_t)std::max(items, 1) * stride);
  for (double& x : s.rec) x = u(rng);
  s.cal.resize(nc); s.gcal.assign(nc, 0.0f); s.m.resize(nc); s.v.resize(nc);
  for (int i = 0; i < nc; ++i) { s.cal[i] = (float)u(rng); s.m[i] = (float)u(rng); s.v[i] = (float)std::fabs(u(rng)); }
  s.loss.assign(kLossTerms, 0.0); s.hist.assign(2 * kLossTerms, 0.0);
  // what the pass leaves per group: the sums of squares, log sigma
  s.calsq = {1.25, 0.75, 0.5, (double)s.cal[nc - 1]};
  GroupDev g{};
  g.V = 100; g.N = N; g.K = 3; g.C = 6; g.P = 17; g.mode = mode; g.bias = 1; g.n_bias = nb;
  g.priors = kPriorCal; g.nx = 10; g.ny = 10; g.nz = 1; g.rec_stride = stride; g.item_count = items;
  g.invM = items ? 0.01f : 0.0f;
  if (!items) g.V = 0;
  std::vector<TileDev> tiles;
  const int nf = items == 0 ? stride : (items <= 32 ? 64 : 8);
  for (int f0 = 0; f0 < stride; f0 += nf) tiles.push_back(TileDev{0, f0, nf, 0});
  StepInfo info{0.01f, 1.5f, 4};
  int32_t step[2] = {4, 0};
  uint32_t status = 0;
  ReduceArgs R{};
  R.groups = &g; R.tiles = tiles.data(); R.rec = s.rec.data(); R.th_cal = s.cal.data(); R.g_cal = s.gcal.data();
  R.loss = s.loss.data(); R.status = &status; R.n_tiles = (int)tiles.size(); R.n_groups = 1;
  R.model.lam_alpha = R.model.lam_beta = R.model.lam_bias = 0.01f;
  R.model.lam_sp = R.model.lam_rep = R.model.lam_sparse = R.model.lam_orphan = R.model.lam_cont = 0.1f;
  R.cal_adam = 1; R.th_cal_upd = s.cal.data(); R.m_cal = s.m.data(); R.v_cal = s.v.data();
  R.step = step; R.info = &info; R.lr = 0.01f; R.b1 = 0.9f; R.b2 = 0.999f; R.eps = 1e-8f;
  R.calsq = s.calsq.data(); R.hist = s.hist.data(); R.hist_step = step; R.hist_len = 2;
  const int n = (int)tiles.size(), nt = items > 256 ? kReduceWide : kReduceBlock;
  std::vector<int> blocks(n);
  for (int i = 0; i < n; ++i) blocks[i] = order == 0 ? i : order == 1 ? n - 1 - i : (i + n / 2) % n;
  blockDim.x = nt;
  for (int b : blocks) {
    blockIdx.x = b;
    std::barrier<> bar(nt);
    g_bar = &bar;
    std::vector<std::thread> th;
    for (int t = 0; t < nt; ++t) th.emplace_back([&, t] { threadIdx.x = t; k_reduce(R); });
    for (auto& t : th) t.join();
  }
  if (status != 0 || step[0] != 5) { printf("status %u step %d\n", status, step[0]); exit(2); }
  return s;
}

template <typename T>
static bool same(const std::vector<T>& a, const std::vector<T>& b) {
  return memcmp(a.data(), b.data(), a.size() * sizeof(T)) == 0;
}

int main(int argc, char** argv) {
  const int mode = atoi(argv[1]), items = atoi(argv[2]);
  const State a = run(mode, items, 0);
  int bad = 0;
  for (int order = 1; order < 3; ++order) {
    const State b = run(mode, items, order);
    const bool ok[] = {same(a.loss, b.loss), same(a.hist, b.hist), same(a.gcal, b.gcal), same(a.cal, b.cal)};
    for (int i = 0; i < 4; ++i)
      if (!ok[i]) { printf("order %d: output %d differs (loss %.17g, %.17g)\n", order, i, a.loss[9], b.loss[9]); bad = 1; }
  }
  return bad;
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    src = open(os.path.join(CSRC, "prism_kernels.hip")).read()
    common = open(os.path.join(CSRC, "prism_common.h")).read()
    adam = re.search(r"__device__ __forceinline__ void adam_one\(.*?\n}\n", common, flags=re.S).group(0)
    first = src.index("// a finished entry of a group's calibration gradient")
    last = src.index("// ---", src.index("void k_reduce(ReduceArgs R)"))
    d = tmp_path_factory.mktemp("reduce")
    cpp, exe = str(d / "reduce.cpp"), str(d / "reduce")
    with open(cpp, "w") as f:
        f.write(HARNESS.replace("@SOURCE@", adam + src[first:last]))
    r = subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I", CSRC, cpp, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("mode", [0, 1], ids=["mse", "nll"])
@pytest.mark.parametrize("items", [0, 1, 32, 33, 256, 257])
def test_reduction_is_the_same_in_any_order_of_its_blocks(harness, mode, items):
    r = subprocess.run([harness, str(mode), str(items)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
