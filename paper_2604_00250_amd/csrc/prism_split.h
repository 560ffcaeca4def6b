// The fused pass for problems too small to fill the device with one lane per
// voxel and measurement range (k_split): one block of four waves per 64, 32 or 16
// voxels, every lane group of a wave with its own part of the measurements.
#pragma once
#include "prism_pass.h"

namespace prism {

// A block has 64 / LS voxels; its 4 LS slots (a slot: the 64 / LS lanes of one wave that
// hold each voxel once) share the measurements evenly.  LS = 4 makes a slot a row of 16
// lanes, the unit of the per-measurement sums (RowScatter).
//
// What bounds a small problem is the chain of latencies in one block, not the work: with
// the measurements shared among four waves a 16^3 patch ran 64 blocks, 72 measurements
// one after the other on a quarter of the compute units, and the epilogue's loads,
// chain rule, optimiser and twelve wave reductions followed in one of the four waves.
// Here every slot computes the epilogue's chain rule (the same bits), but takes only its
// share of what follows: the parameters p = slot, slot + 4 LS, .. (their moments are
// loaded before the measurement loop) and the record terms of the same indices; the
// Eq. 7 gather is issued before the loop too, and nothing is loaded or transformed twice.
//
// The measurements of slot s: [N s / S, N (s + 1) / S), S = 4 LS.

// One slot's measurements, per lane (LS > 1; with LS = 1 a slot is a wave and
// measurement_loop serves): the y ring as there, the table read at the lane's own
// measurement, lanes past their range's end with validity 0.  asum: [2][N].
template <int K, int MODE, bool LD, int LS>
__device__ __forceinline__ void slot_loop(const Vox<K, LD>& x, Acc<K, LD>& acc, const float* yg, int64_t V, int vox,
                                          float valid, const float4* __restrict__ acq,
                                          const float4* __restrict__ bes, int nb, int ne, int N, float inv_s2,
                                          int lane, float* asum, double& dloss, double& dsig) {
  constexpr int S = 4 * LS;
  const int steps = (N + S - 1) / S;                 // the longest range
  const uint32_t bytes = (uint32_t)(N * V) * 4u, rowb = (uint32_t)V * 4u;   // N V 4 < 2^31 (the plan's rule)
  const int last = max(ne - 1, 0);
  auto at = [&](int n) { return load_row_f32(yg, bytes, (uint32_t)min(n, last) * rowb + (uint32_t)vox * 4u); };
  float yr[kPf];
#pragma unroll
  for (int u = 0; u < kPf; ++u) yr[u] = at(nb + u);
  const RowScatterMasks sm = row_scatter_masks(lane);
  const int bank = (lane >> 2) & 3;
  RunVox run;   // not used
  for (int t0 = 0; t0 < steps; t0 += kTile) {
    RowScatter sa, sb;
    float lacc = 0.0f, sacc = 0.0f;
    sa.acc = 0.0f;
    sb.acc = 0.0f;
    const int tn = min(kTile, steps - t0);
    for (int t = 0; t < tn; t += kPf) {
#pragma unroll
      for (int u = 0; u < kPf; ++u) {
        const int n = nb + t0 + t + u, m = min(n, last);
        const float4 a = acq[3 * m], b = acq[3 * m + 1], c = acq[3 * m + 2];
        float tl, ts, sq, sd;
        pair<K, MODE, LD, false>(x, acc, run, 0.0f, yr[u], n < ne ? valid : 0.0f, a, b, c, inv_s2, bes, tl, ts, sq, sd);
        lacc += tl;
        if (MODE == kNLL) sacc += ts;
        yr[u] = at(n + kPf);
        row_scatter_push(sa, sq, u, sm);
        row_scatter_push(sb, sd, u, sm);
      }
      const bool here = bank == (t >> 2);
      row_scatter_group(sa, here);
      row_scatter_group(sb, here);
    }
    float ra = sa.acc, rb = sb.acc;
    if (LS == 2) {  // a slot of two rows
      ra += xor16_f32(ra);
      rb += xor16_f32(rb);
    }
    const int n = nb + t0 + row_scatter_index(lane);
    if (n < ne && (LS == 4 || (lane & 16) == 0)) {
      asum[n] = ra * acq[3 * n + 2].x;
      asum[N + n] = rb;
    }
    dloss += (double)lacc;
    if (MODE == kNLL) dsig += (double)sacc;
  }
}

// The element i of a register array, i differing between lanes, by selects (through empty
// asm statements: without them the compiler turns the selects into a store of the array to
// scratch memory and a load at i, two round trips to the cache)
template <int M>
__device__ __forceinline__ float pick(const float (&x)[M], int i) {
  float r = x[0];
#pragma unroll
  for (int k = 1; k < M; ++k) {
    float t = x[k];
    asm("" : "+v"(t));
    r = i == k ? t : r;
  }
  return r;
}

// One row of 64 voxels: as many waves as the fused pass where they fit (a problem's blocks
// should all be resident at once); shorter rows run where few waves share a SIMD, and
// take the registers to keep several measurements in flight.  The Rician variants whose
// 253-259 registers come down to the 256 of two waves for at most three spilled ones are
// held to them (one iteration, 32768 voxels: K = 4, learned D, N = 96, 42.8 -> 38.8 us, K = 5, N =
// 288, 67.4 -> 65.1, 16250 voxels 50.6 -> 46.3); the larger ones (K = 5, learned D; K = 6)
// would spill 18 to 66 and run 5 to 14% slower.
constexpr int split_min_waves(int K, int MODE, bool LD, int LS) {
  if (MODE == kNLL) return K == (LD ? 4 : 5) ? 2 : 1;
  return LS == 1 ? pass_min_waves(K, MODE, LD, 1) : 1;
}

template <int K, int MODE, bool LD, int LS>
__global__ __launch_bounds__(kBlock, split_min_waves(K, MODE, LD, LS)) void k_split(PassArgs A) {
  constexpr int C = K + 3, NACC = Acc<K, LD>::N, P = 4 * K + 5 + (LD ? 2 : 0);
  constexpr int S = 4 * LS, NV = 64 / LS;                 // slots, voxels
  constexpr int MINE = (P + S - 1) / S;                   // parameters of a slot, at most
  constexpr int TERMS = 16, TMINE = (TERMS + S - 1) / S;  // record fields 2-7 and bias, of a slot
  extern __shared__ float4 smem4[];
  __shared__ double wsum[4][2];
  __shared__ float adam_sc[2];
  const ItemDev it = A.items[A.item_base + xcd_item(blockIdx.x, gridDim.x)];
  const GroupDev& g = reread(A.groups + it.group);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slot = wave * LS + (LS == 1 ? 0 : lane / NV);
  const int N = g.N, Np = padded4(N);
  const int64_t V = g.V;
  float4* bes = smem4;
  float4* acq = smem4 + (MODE == kNLL ? kBesselRows : 0);   // [3N]
  float* asum = reinterpret_cast<float*>(acq + 3 * N);      // [2][Np] (LS = 1: [4][2][Np], per wave)
  float4* comb = reinterpret_cast<float4*>(asum + (LS == 1 ? 8 : 2) * Np);  // [NACC][NV]
  const int lv = lane & (NV - 1);
  const bool ok = lv < it.nv;
  const float valid = ok ? 1.0f : 0.0f;
  const int v = it.v0 + (ok ? lv : 0);
  const uint32_t rowb = (uint32_t)V * 4u, voff = (uint32_t)v * 4u;

  // loads that nothing waits for until after the measurement loop: the slot's share of the
  // optimiser's rows
  float pp[MINE], m1[MINE], v1[MINE];
  const uint32_t blkb = (uint32_t)P * rowb;   // P V 4 < 2^31 (the plan's rule)
  if (A.adam) {
#pragma unroll
    for (int i = 0; i < MINE; ++i) {
      const uint32_t off = (uint32_t)min(slot + S * i, P - 1) * rowb + voff;
      m1[i] = load_row_f32(A.m_micro + g.micro_off, blkb, off);
      v1[i] = load_row_f32(A.v_micro + g.micro_off, blkb, off);
      pp[i] = load_row_f32(A.th_upd + g.micro_off, blkb, off);
    }
  }
  if (MODE == kNLL) stage_bessel(bes);
  stage_acquisition(A, g, acq, LS == 1);   // slot_loop takes them as they come
  if (LS == 1)
    for (int i = tid; i < 8 * Np; i += kBlock) asum[i] = 0.0f;
  if (A.adam && tid == 0) {
    adam_factors(A.step, A.lr, A.b1, A.b2, adam_sc[0], adam_sc[1]);
    if (it.first && A.info) *A.info = StepInfo{adam_sc[0], adam_sc[1], A.step[0]};
  }
  if (it.rec == 0 && wave == 3) calibration_sums(A, g, it.group, lane);
  Vox<K, LD> xs[1];
  Vox<K, LD>& x = xs[0];
  Derived D;
  bool zero_dir = false, bad_grad = false;
  load_voxel<K, LD, false>(A, g, v, x, D, zero_dir);
  const bool has_sp = (g.priors & kPriorSpatial) && g.nbh > 0;
  float sp[C];
  if (has_sp) spatial_gather<C>(A.wsp + g.w_off, A.nbr + g.nbr_off, g.nbh, V, v, sp);
  Acc<K, LD> as[1];
  Acc<K, LD>& acc = as[0];
#pragma unroll
  for (int i = 0; i < NACC; ++i) acc.r[i] = 0.0f;
  const float inv_s2 = MODE == kNLL ? expf(-2.0f * A.th_cal[g.cal_off + g.n_bias + 2 * N]) : 0.0f;
  __syncthreads();

  double dloss = 0.0, dsig = 0.0;
  if constexpr (LS == 1) {
    const int n_groups = (N + kPf - 1) / kPf;
    const int ga = n_groups * wave / 4, gb = n_groups * (wave + 1) / 4;
    const int vs[1] = {v};
    const float va[1] = {valid};
    measurement_loop<K, MODE, LD, 1, false>(A, g, xs, as, vs, va, acq, bes, ga, gb, inv_s2, lane, asum + wave * 2 * Np,
                                            dloss, dsig);
  } else {
    const int nb = (N * slot) / S, ne = (N * (slot + 1)) / S;
    slot_loop<K, MODE, LD, LS>(x, acc, A.y + g.y_off, V, v, valid, acq, bes, nb, ne, N, inv_s2, lane, asum, dloss,
                               dsig);
  }

  // the voxels' sums over the block: the slots of a wave by lane exchanges, the waves
  // through LDS, read by every slot
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    float r = acc.r[i];
    if (LS == 4) r += xor16_f32(r);
    if (LS >= 2) r += xor32_f32(r);
    if (lane < NV) reinterpret_cast<float*>(comb + i * NV + lane)[wave] = r;
  }
  dloss = wave_sum_f64(dloss);
  if (MODE == kNLL) dsig = wave_sum_f64(dsig);
  if (lane == 0) {
    wsum[wave][0] = dloss;
    wsum[wave][1] = dsig;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    const float4 t = comb[i * NV + lv];
    acc.r[i] = (t.x + t.y) + (t.z + t.w);
  }
  float gout[P];
  VoxTerms vt;
  chain_rule<K, LD>(A, g, v, D, x.d, acc, sp, gout, vt);
  double* rec = A.rec + g.rec_off + (int64_t)it.rec * g.rec_stride;
  // the slot's parameters
#pragma unroll
  for (int i = 0; i < MINE; ++i) {
    const int p = slot + S * i;
    if (ok && p < P) {
      const float gp = pick(gout, p);
      const uint32_t off = (uint32_t)p * rowb + voff;
      if (!isfinite(gp)) bad_grad = true;
      if (A.adam) {
        adam_one(pp[i], gp, m1[i], v1[i], A.b1, A.b2, A.eps, adam_sc[0], adam_sc[1]);
        store_row_f32(A.th_upd + g.micro_off, blkb, off, pp[i]);
        store_row_f32(A.m_micro + g.micro_off, blkb, off, m1[i]);
        store_row_f32(A.v_micro + g.micro_off, blkb, off, v1[i]);
      }
      if (!A.adam || A.store_grad) store_row_f32(A.g_micro + g.micro_off, blkb, off, gp);
    }
  }
  if (g.bias == 2 && ok && slot == 0) A.wsp[g.glb_off + v] = vt.glb;
  // the slot's record terms: fields 2-7 and the bias basis, summed over the voxels
  {
    const int32_t pc = A.coords[g.vox_off + v];
    const int i = pc & 1023, j = (pc >> 10) & 1023, k = (pc >> 20) & 1023;
    // the coordinates of log_bias, bit for bit
    const float xx = fmaf((float)i, g.bsc[0], g.boff[0]);
    const float yy = fmaf((float)j, g.bsc[1], g.boff[1]);
    const float zz = fmaf((float)k, g.bsc[2], g.boff[2]);
    const float on = ok ? 1.0f : 0.0f, gb = g.bias == 1 && ok ? vt.glb : 0.0f;
    const float term[TERMS] = {vt.rep * on, vt.spa * on, vt.orph * on, vt.cont * on, vt.ord * on, vt.tv * on,
                               gb, xx * gb, yy * gb, zz * gb, (xx * xx) * gb, (yy * yy) * gb, (zz * zz) * gb,
                               (xx * yy) * gb, (xx * zz) * gb, (yy * zz) * gb};
#pragma unroll
    for (int q = 0; q < TMINE; ++q) {
      const int e = slot + S * q;
      double t = (double)pick(term, min(e, TERMS - 1));
      t += dpp_f64<0xB1>(t);
      t += dpp_f64<0x4E>(t);
      t += dpp_f64<0x141>(t);
      t += dpp_f64<0x140>(t);
      if (LS <= 2) t += xor16_f64(t);
      if (LS == 1) t += xor32_f64(t);
      if (lv == 0 && e < TERMS) rec[e < 6 ? kRecRep + e : kRecBias + (e - 6)] = t;
    }
  }
  if (tid == 0) {
    rec[kRecData] = (wsum[0][0] + wsum[1][0]) + (wsum[2][0] + wsum[3][0]);
    rec[kRecSigma] = (wsum[0][1] + wsum[1][1]) + (wsum[2][1] + wsum[3][1]);
    if (!has_sp) rec[kRecSpatial] = 0.0;
  }
  if constexpr (LS == 1) {
    for (int p = tid; p < N; p += kBlock) {
      const int n = A.perm[g.perm_off + p];
      auto waves = [&](const float* s) {
        return ((double)s[0] + (double)s[2 * Np]) + ((double)s[4 * Np] + (double)s[6 * Np]);
      };
      rec[kRecAlpha + n] = waves(asum + p) * (double)acq[3 * p + 2].x;   // times exp(alpha_n)
      rec[kRecAlpha + N + n] = waves(asum + Np + p);
    }
  } else {
    for (int n = tid; n < 2 * N; n += kBlock) rec[kRecAlpha + n] = (double)asum[n];
  }
  if (bad_grad) atomicOr(A.status, (uint32_t)kStNonfiniteGrad);
  if (zero_dir) atomicOr(A.status, (uint32_t)kStZeroDir);
}

inline size_t split_lds_bytes(int N, int nacc, int ls, bool nll) {
  return (size_t)N * 3 * sizeof(float4) + (size_t)(ls == 1 ? 8 : 2) * padded4(N) * sizeof(float) +
         (size_t)nacc * (64 / ls) * sizeof(float4) + (nll ? (size_t)kBesselRows * sizeof(float4) : 0);
}

// f(kernel, LDS bytes) for the variant of one K
template <int K, int MODE, bool LD, typename F>
static auto with_split_kernel(int ls, int N, F&& f) {
  switch (ls) {
    case 4: return f(k_split<K, MODE, LD, 4>, split_lds_bytes(N, acc_count(K, LD), 4, MODE == kNLL));
    case 2: return f(k_split<K, MODE, LD, 2>, split_lds_bytes(N, acc_count(K, LD), 2, MODE == kNLL));
    default: return f(k_split<K, MODE, LD, 1>, split_lds_bytes(N, acc_count(K, LD), 1, MODE == kNLL));
  }
}
template <int K, typename F>
static auto with_split_variant(int mode, int ld, int ls, int N, F&& f) {
  if (mode == kMSE) return ld ? with_split_kernel<K, kMSE, true>(ls, N, f) : with_split_kernel<K, kMSE, false>(ls, N, f);
  return ld ? with_split_kernel<K, kNLL, true>(ls, N, f) : with_split_kernel<K, kNLL, false>(ls, N, f);
}

template <int K>
hipError_t launch_split_k(const PassArgs& a, int mode, int ld, int ls, int maxN, hipStream_t s) {
  return with_split_variant<K>(mode, ld, ls, maxN, [&](auto kernel, size_t lds) {
    if (lds > 65536) {
      hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(a.n_items), dim3(kBlock), lds, s, a);
    return hipGetLastError();
  });
}
template <int K>
int split_occupancy_k(int mode, int ld, int ls, int N) {
  if (ls == 0) {   // the fused pass with four waves on each row
    const void* fn = mode == kMSE ? (ld ? (const void*)k_pass<K, kMSE, true, 1> : (const void*)k_pass<K, kMSE, false, 1>)
                                  : (ld ? (const void*)k_pass<K, kNLL, true, 1> : (const void*)k_pass<K, kNLL, false, 1>);
    int nb = 0;
    const size_t lds = pass_lds_bytes(N, 3, acc_count(K, ld != 0), 1, mode == kNLL);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, kBlock, lds) == hipSuccess ? nb : 0;
  }
  return with_split_variant<K>(mode, ld, ls, N, [&](auto kernel, size_t lds) {
    int nb = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, kBlock, lds) == hipSuccess ? nb : 0;
  });
}

}  // namespace prism
