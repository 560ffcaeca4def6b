// HIP kernels of the PRISM analysis-by-synthesis pass for gfx950 (CDNA4, wave64)
// other than the fused pass itself (prism_pass.h, instantiated per K in
// prism_pass_k.hip, and its persistent form in prism_persistent.hip):
//
// k_spatial   Eq. 7: the residual weights rho'(r)/|N| per voxel and compartment, from
//             the logits or (26-neighbourhood) the fractions that k_fractions stored.
// k_reduce    deterministic reduction of per-item records into the calibration
//             gradient (the 8^3 trilinear log-bias grid's too) and the loss terms.
// k_stitch    blend of per-slab maps into whole-volume maps (slab fitting).
// k_adam, k_rprop  optimiser steps.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "prism_common.h"

namespace prism {

// The Eq. 7 kernels run one block per work item with up to kAuxBlock
// threads, one voxel per thread (the launch sizes the block to the largest
// item): with fewer threads each one walked several voxels and the dependent
// table-then-gather loads of each voxel in turn.
constexpr int kAuxBlock = 512;

// A launch whose groups share one C is compiled for it; where the groups differ
// (CT = 0) each block branches to the code of its own group's C, so every row of the
// Eq. 7 buffers is read and written whole either way (with C at run time, one guarded
// float at a time, 512 patches of mixed K took 42 + 116 us, now 19 + 30).
template <int CT, typename F>
__device__ __forceinline__ void with_C(int C, F&& f) {
  if constexpr (CT != 0) {
    f(std::integral_constant<int, CT>{});
  } else {
    switch (C) {
      case 4: f(std::integral_constant<int, 4>{}); break;
      case 5: f(std::integral_constant<int, 5>{}); break;
      case 6: f(std::integral_constant<int, 6>{}); break;
      case 7: f(std::integral_constant<int, 7>{}); break;
      case 8: f(std::integral_constant<int, 8>{}); break;
      default: f(std::integral_constant<int, 9>{}); break;
    }
  }
}

template <int C>
__device__ __forceinline__ void softmax_row(const float* th, int64_t V, int v, float (&r)[C]) {
  float f[kMaxC];
  softmax_at(th, V, C, v, f);
#pragma unroll
  for (int c = 0; c < C; ++c) r[c] = f[c];
}

// fractions f = softmax(logits) once per voxel, rows [V][C] (see load_row)
template <int C>
__device__ __forceinline__ void fractions_item(const PassArgs& A, const GroupDev& g, const ItemDev& it) {
  const float* th = A.th_micro + g.micro_off;
  const int64_t V = g.V;
  float* f_out = A.wsp + g.w_off + (int64_t)C * V;
  for (int lv = threadIdx.x; lv < it.nv; lv += blockDim.x) {
    const int v = it.v0 + lv;
    float r[C];
    softmax_row<C>(th, V, v, r);
    store_row<C>(f_out, v, r);
  }
}

template <int CT>
__global__ __launch_bounds__(kAuxBlock) void k_fractions(PassArgs A) {
  // the persistent launches' counters, before either starts
  if (blockIdx.x == 0 && threadIdx.x < 2) A.counters[32 * threadIdx.x] = 0;
  const ItemDev it = A.items[xcd_item(blockIdx.x, A.n_items)];
  const GroupDev g = A.groups[it.group];
  if (!((g.priors & kPriorSpatial) && g.nbh > 0)) return;
  with_C<CT>(g.C, [&](auto c) { fractions_item<decltype(c)::value>(A, g, it); });
}

// Eq. 7 residual weights w_c(x) = rho'(r_c(x)) / |N(x)| from the stored fractions.
// Neighbours are taken six at a time: all six table entries are loaded, then
// all their fraction rows (an absent neighbour reads the voxel's own row with
// weight 0), so one round trip serves six neighbours.  FROM_LOGITS: the fractions are not
// stored, each is taken from its voxel's logits again (the same bits).  The rows of the
// logits are read at consecutive voxels for every neighbour, from the cache, so with the
// 6-neighbourhood this takes less than storing the fractions first (an iteration of 16250
// voxels, K = 3: 23.8 -> 22.6 us, 262k: 58.2 -> 55.3; the volume's Eq. 7 27 -> 23 us); with
// 26 neighbours more (16250 voxels: 27.4 -> 28.3).
template <int C, bool FROM_LOGITS>
__device__ __forceinline__ double spatial_item(const PassArgs& A, const GroupDev& g, const ItemDev& it) {
  constexpr int kNb = 6;
  double lsum = 0.0;
  const int32_t* nbr = A.nbr + g.nbr_off;
  const int64_t V = g.V;
  const float* fr = A.wsp + g.w_off + (int64_t)C * V;
  const float* th = A.th_micro + g.micro_off;
  float* w_out = A.wsp + g.w_off;
  const float delta = A.model.huber_delta;
  for (int lv = threadIdx.x; lv < it.nv; lv += blockDim.x) {
    const int v = it.v0 + lv;
    float mean[C];
#pragma unroll
    for (int c = 0; c < C; ++c) mean[c] = 0.0f;
    int cnt = 0;
    for (int q0 = 0; q0 < g.nbh; q0 += kNb) {
      int u[kNb];
#pragma unroll
      for (int j = 0; j < kNb; ++j) u[j] = q0 + j < g.nbh ? nbr[(int64_t)(q0 + j) * V + v] : -1;
      float t[kNb][C];
#pragma unroll
      for (int j = 0; j < kNb; ++j) {
        if (FROM_LOGITS)
          softmax_row<C>(th, V, u[j] >= 0 ? u[j] : v, t[j]);
        else
          load_row<C>(fr, u[j] >= 0 ? u[j] : v, t[j]);
      }
#pragma unroll
      for (int j = 0; j < kNb; ++j) {
        const float on = u[j] >= 0 ? 1.0f : 0.0f;
        cnt += u[j] >= 0 ? 1 : 0;
#pragma unroll
        for (int c = 0; c < C; ++c) mean[c] = fmaf(on, t[j][c], mean[c]);
      }
    }
    float own[C];
    if (FROM_LOGITS)
      softmax_row<C>(th, V, v, own);
    else
      load_row<C>(fr, v, own);
    float ls = 0.0f;
    const float icnt = cnt > 0 ? 1.0f / (float)cnt : 0.0f;
    float w[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      w[c] = 0.0f;
      if (cnt > 0) {
        const float r = own[c] - mean[c] * icnt;
        const float ar = fabsf(r);
        ls += ar <= delta ? 0.5f * r * r : delta * (ar - 0.5f * delta);
        w[c] = (ar <= delta ? r : copysignf(delta, r)) * icnt;
      }
    }
    store_row<C>(w_out, v, w);
    lsum += (double)ls;
  }
  return lsum;
}

// A copy of the raw directions [3K][V] for the continuity prior, before the fused pass
// updates any voxel's: the pass reads its neighbours' from here.
__device__ __forceinline__ void directions_item(const PassArgs& A, const GroupDev& g, const ItemDev& it) {
  const float* th = A.th_micro + g.micro_off + (int64_t)row_v(g.C, 0, 0) * g.V;
  float* out = A.dirs + g.dir_off;
  for (int lv = threadIdx.x; lv < it.nv; lv += blockDim.x)
    for (int r = 0; r < 3 * g.K; ++r) out[(int64_t)r * g.V + it.v0 + lv] = th[(int64_t)r * g.V + it.v0 + lv];
}

template <int CT, bool FROM_LOGITS>
__global__ __launch_bounds__(kAuxBlock) void k_spatial(PassArgs A) {
  __shared__ double red[kAuxBlock / 64];
  if (FROM_LOGITS && blockIdx.x == 0 && threadIdx.x < 2) A.counters[32 * threadIdx.x] = 0;  // as k_fractions
  const ItemDev it = A.items[xcd_item(blockIdx.x, gridDim.x)];
  const GroupDev g = A.groups[it.group];
  const int tid = threadIdx.x;
  if (A.dirs && (g.priors & kPriorCont) && g.nbh > 0)
    directions_item(A, g, it);
  if (!((g.priors & kPriorSpatial) && g.nbh > 0)) return;  // the fused pass writes the record's 0
  double lsum = 0.0;
  with_C<CT>(g.C, [&](auto c) { lsum = spatial_item<decltype(c)::value, FROM_LOGITS>(A, g, it); });
  lsum = wave_sum_f64(lsum);
  if ((tid & 63) == 0) red[tid >> 6] = lsum;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int i = 0; i < (int)(blockDim.x / 64); ++i) s += red[i];
    A.rec[g.rec_off + (int64_t)it.rec * g.rec_stride + kRecSpatial] = s;
  }
}

// ---------------------------------------------------------------------------
// whole-volume slabs: blend the per-slab constrained maps (Sec. 2.5)
// ---------------------------------------------------------------------------
// constrained quantities of voxel v: S0, fractions, unit directions, f_intra [, D]
template <int K, bool LD>
__device__ __forceinline__ void maps_at(const GroupDev& g, const float* th_all, int v, float (&m)[4 * K + 5 + (LD ? 2 : 0)]) {
  constexpr int C = K + 3;
  const float* th = th_all + g.micro_off;
  const int64_t V = g.V;
  m[0] = softplus_f(th[v]);
  float f[kMaxC];
  softmax_at(th, V, C, v, f);
#pragma unroll
  for (int c = 0; c < C; ++c) m[1 + c] = f[c];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const float x = th[(int64_t)row_v(C, k, 0) * V + v];
    const float y = th[(int64_t)row_v(C, k, 1) * V + v];
    const float z = th[(int64_t)row_v(C, k, 2) * V + v];
    const float n2 = fmaf(x, x, fmaf(y, y, z * z));
    const float in = n2 > 0.0f ? 1.0f / sqrtf(n2) : 0.0f;
    m[1 + C + 3 * k] = x * in;
    m[2 + C + 3 * k] = y * in;
    m[3 + C + 3 * k] = z * in;
  }
  m[1 + C + 3 * K] = sigmoid_f(th[(int64_t)row_fin(C, K) * V + v]);
  if (LD) {
    m[2 + C + 3 * K] = softplus_f(th[(int64_t)row_dpar(C, K) * V + v]);
    m[3 + C + 3 * K] = softplus_f(th[(int64_t)(row_dpar(C, K) + 1) * V + v]);
  }
}

// One thread per output voxel: one source is copied; two are blended with the
// heavier slab as reference (the lower slab on a tie), the other slab's fibres
// matched greedily by |cos| and sign-aligned.
template <int K, bool LD>
__global__ __launch_bounds__(256) void k_stitch(StitchArgs S) {
  constexpr int C = K + 3;
  constexpr int P = 4 * K + 5 + (LD ? 2 : 0);
  const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (o >= S.n_out) return;
  const int ga = S.src_g[o], gb = S.src_g[S.n_out + o];
  const float wa = S.src_w[o], wb = S.src_w[S.n_out + o];
  float ma[P];
  maps_at<K, LD>(S.groups[ga], S.th_micro, S.src_v[o], ma);
  float out[P];
  if (gb < 0) {
#pragma unroll
    for (int p = 0; p < P; ++p) out[p] = ma[p];
  } else {
    float mb[P];
    maps_at<K, LD>(S.groups[gb], S.th_micro, S.src_v[S.n_out + o], mb);
    const bool a_ref = wa >= wb;
    const float wr = a_ref ? wa : wb, wo = a_ref ? wb : wa;
    float r[P], q[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      r[p] = a_ref ? ma[p] : mb[p];
      q[p] = a_ref ? mb[p] : ma[p];
      out[p] = wr * r[p] + wo * q[p];
    }
    int used = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const float rx = r[1 + C + 3 * k], ry = r[2 + C + 3 * k], rz = r[3 + C + 3 * k];
      float best = -1.0f, bdot = 0.0f, qf = 0.0f, qx = 0.0f, qy = 0.0f, qz = 0.0f;
      int bj = 0;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const float dot = rx * q[1 + C + 3 * j] + ry * q[2 + C + 3 * j] + rz * q[3 + C + 3 * j];
        if (!(used & (1 << j)) && fabsf(dot) > best) {
          best = fabsf(dot);
          bdot = dot;
          bj = j;
          qf = q[3 + j];
          qx = q[1 + C + 3 * j];
          qy = q[2 + C + 3 * j];
          qz = q[3 + C + 3 * j];
        }
      }
      used |= 1 << bj;
      const float sg = bdot < 0.0f ? -wo : wo;
      out[3 + k] = wr * r[3 + k] + wo * qf;
      const float dx = wr * rx + sg * qx, dy = wr * ry + sg * qy, dz = wr * rz + sg * qz;
      const float in = 1.0f / sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
      out[1 + C + 3 * k] = dx * in;
      out[2 + C + 3 * k] = dy * in;
      out[3 + C + 3 * k] = dz * in;
    }
  }
#pragma unroll
  for (int p = 0; p < P; ++p) S.maps[(int64_t)p * S.n_out + o] = out[p];
}

// a finished entry of a group's calibration gradient, and its Adam step
__device__ __forceinline__ void cal_entry(const ReduceArgs& R, const GroupDev& g, int dst, float out) {
  const int64_t i = g.cal_off + dst;
  R.g_cal[i] = out;
  if (!isfinite(out)) atomicOr(R.status, (uint32_t)kStNonfiniteGrad);
  if (R.cal_adam) {
    float p = R.th_cal_upd[i], m = R.m_cal[i], v = R.v_cal[i];
    adam_one(p, out, m, v, R.b1, R.b2, R.eps, R.info->step_size, R.info->ibc2);
    R.th_cal_upd[i] = p;
    R.m_cal[i] = m;
    R.v_cal[i] = v;
  }
}

// ---------------------------------------------------------------------------
// trilinear 8^3 log-bias gradient: dL/db(c) = sum_x w_c(x) dL/dlogB(x)
// ---------------------------------------------------------------------------
// Control point cp of one group by thread t of nt in k_reduce's launch (it reads none of
// what the tiles write: as a launch after them it took 12 us more for 30k voxels): a whole
// block, or for small boxes one wave (see prism_host.cpp).  red: one value per wave.
template <bool WAVE>
__device__ void bias_tri_point(const ReduceArgs& R, const GroupDev& g, int cp, int t, int nt, double* red) {
  const int cidx[3] = {cp >> 6, (cp >> 3) & 7, cp & 7};
  const int nn[3] = {g.nx, g.ny, g.nz};
  int lo[3], hi[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (nn[a] == 1) {
      lo[a] = 0;
      hi[a] = cidx[a] == 0 ? 0 : -1;
    } else {
      const float sc = (float)(nn[a] - 1) / 7.0f;
      lo[a] = max(0, (int)ceilf((cidx[a] - 1) * sc));
      hi[a] = min(nn[a] - 1, (int)floorf((cidx[a] + 1) * sc));
    }
  }
  double acc = 0.0;
  const int ex = hi[0] - lo[0] + 1, ey = hi[1] - lo[1] + 1, ez = hi[2] - lo[2] + 1;
  if (ex > 0 && ey > 0 && ez > 0) {
    const int tot = ex * ey * ez;   // a part of a box of at most 2^31 voxels
    const int32_t* grid = R.grid + g.grid_off;
    const float* glb = R.wsp + g.glb_off;
    // four positions per round: their voxels, then those voxels' adjoints
    for (int64_t q0 = t; q0 < tot; q0 += 4 * nt) {
      float w[4];
      int v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t qe = q0 + (int64_t)e * nt;
        const uint32_t q = (uint32_t)(qe < tot ? qe : tot - 1);
        const uint32_t ij = q / (uint32_t)ez, ia = ij / (uint32_t)ey;
        const int ii[3] = {lo[0] + (int)ia, lo[1] + (int)(ij - ia * (uint32_t)ey), lo[2] + (int)(q - ij * (uint32_t)ez)};
        v[e] = grid[((int64_t)ii[0] * g.ny + ii[1]) * g.nz + ii[2]];
        w[e] = qe < tot ? 1.0f : 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const float p = ii[a] * g.tri_sc[a];  // the coordinate of log_bias, bit for bit
          w[e] *= fmaxf(0.0f, 1.0f - fabsf(p - (float)cidx[a]));
        }
      }
      float b[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = glb[max(v[e], 0)];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (v[e] >= 0) acc += (double)w[e] * (double)b[e];
    }
  }
  acc = wave_sum_f64(acc);
  if (!WAVE) {
    if ((t & 63) == 0) red[t >> 6] = acc;
    __syncthreads();
  }
  if (t == 0) {
    double s = acc;
    if (!WAVE) {
      s = 0.0;
      for (int i = 0; i < nt / 64; ++i) s += red[i];
    }
    const float* cal = R.th_cal + g.cal_off;
    const bool cal_on = (g.priors & kPriorCal) != 0;
    cal_entry(R, g, cp, (float)(s + (cal_on ? 2.0 * (double)R.model.lam_bias * cal[cp] : 0.0)));
  }
}

// ---------------------------------------------------------------------------
// deterministic reduction of the item records
// ---------------------------------------------------------------------------
// One block per tile of nf fields: its threads in nf columns, each thread of a column
// over every (block / nf)-th record with eight loads in flight, then a tree over the
// column in LDS (a fixed order, so the result is reproducible).  The time is the loads'
// latency, so few records take wide tiles (64 fields, four threads a column) and many
// take narrow ones (8 fields: still a 64-byte piece of each record) in larger blocks.
// One launch where two stages of 64 x 64 tiles took two: 64 records of 595 fields
// 9.4 -> 4.7 us.
constexpr int kReduceBlock = 256, kReduceWide = 1024;

// From kReduceRowsFrom records up the narrow tiles are too few compute units for the
// bytes (3102 records of 595 fields: 14.9 us on 75 of them), so each run of kReduceRun
// records is first summed in place into its first record, by one block per run and 64
// fields.
__global__ __launch_bounds__(kReduceBlock) void k_reduce_rows(ReduceArgs R) {
  __shared__ double part[4][64];
  const TileDev t = R.row_tiles[blockIdx.x];
  const GroupDev g = R.groups[t.group];
  const int f = threadIdx.x & 63, s = threadIdx.x >> 6;
  const int64_t st = g.rec_stride;
  const int n = min(kReduceRun, g.item_count - t.r0);
  double* base = R.rec + g.rec_off + (int64_t)t.r0 * st + t.f0 + f;
  const bool on = t.f0 + f < g.rec_stride;
  double acc = 0.0;
  if (on) {
    double a[kReduceRun / 4];
#pragma unroll
    for (int i = 0; i < kReduceRun / 4; ++i) a[i] = base[(int64_t)min(s + 4 * i, n - 1) * st];
#pragma unroll
    for (int i = 0; i < kReduceRun / 4; ++i) acc += s + 4 * i < n ? a[i] : 0.0;
  }
  part[s][f] = acc;
  __syncthreads();
  if (s == 0 && on) base[0] = (part[0][f] + part[1][f]) + (part[2][f] + part[3][f]);
}

__global__ __launch_bounds__(kReduceWide) void k_reduce(ReduceArgs R) {
  __shared__ double part[kReduceWide];
  __shared__ double sq[3][kReduceWide / 64];
  if ((int)blockIdx.x >= R.n_tiles) {
    const int q = blockIdx.x - R.n_tiles, past = q - 512 * R.n_tri_wide;
    if (past < 0) {
      bias_tri_point<false>(R, R.groups[R.tri_groups[q / 512]], q % 512, threadIdx.x, blockDim.x, sq[0]);
    } else {
      const int per = blockDim.x >> 6, blocks = 512 / per;   // points of a block, blocks of a group
      bias_tri_point<true>(R, R.groups[R.tri_groups[R.n_tri_wide + past / blocks]],
                           past % blocks * per + (threadIdx.x >> 6), threadIdx.x & 63, 64, nullptr);
    }
    return;
  }
  const TileDev t = R.tiles[blockIdx.x];
  const GroupDev g = R.groups[t.group];
  const int tid = threadIdx.x, nt = blockDim.x;
  // the columns; an empty group has no records (and one tile, so no other block updates
  // its calibration vector while this one sums its squares)
  const bool empty = g.item_count == 0;
  const int T = empty ? 1 : nt / t.nf;
  const float* cal = R.th_cal + g.cal_off;
  const int N = g.N, nb = g.n_bias;
  const bool cal_on = (g.priors & kPriorCal) != 0;
  if (!empty) {
    const int f = tid & (t.nf - 1), s = tid / t.nf;
    double acc = 0.0;
    if (t.f0 + f < g.rec_stride) {
      const double* base = R.rec + g.rec_off + t.f0 + f;
      // (of a group that k_reduce_rows went over: the first record of each run)
      const bool rows = g.item_count > kReduceRowsFrom;
      const int64_t st = rows ? (int64_t)kReduceRun * g.rec_stride : g.rec_stride;
      const int n = rows ? (g.item_count + kReduceRun - 1) / kReduceRun : g.item_count;
      // rounds of eight loads (past the end: the last record again, times 0)
      for (int r = s; r < n; r += 8 * T) {
        double a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = base[(int64_t)min(r + i * T, n - 1) * st];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += r + i * T < n ? a[i] : 0.0;
      }
    }
    part[f * T + s] = acc;
    for (int w = T >> 1; w > 0; w >>= 1) {
      __syncthreads();
      if (s < w) part[f * T + s] += part[f * T + s + w];
    }
  } else if (cal_on) {
    double sa = 0.0, sb = 0.0, sw = 0.0;
    for (int i = tid; i < nb; i += nt) sw += (double)cal[i] * cal[i];
    for (int i = tid; i < N; i += nt) {
      sa += (double)cal[nb + i] * cal[nb + i];
      sb += (double)cal[nb + N + i] * cal[nb + N + i];
    }
    sa = wave_sum_f64(sa);
    sb = wave_sum_f64(sb);
    sw = wave_sum_f64(sw);
    if ((tid & 63) == 0) {
      sq[0][tid >> 6] = sa;
      sq[1][tid >> 6] = sb;
      sq[2][tid >> 6] = sw;
    }
  }
  // log sigma before the iteration: from the pass, since the block of another tile may
  // update theta_cal's while this one runs; an empty group's one block reads it before the
  // barrier that its own update follows
  const double sigma_log = empty ? (double)cal[nb + 2 * N] : R.calsq[kCalSums * t.group + 3];
  __syncthreads();
  auto total = [&](int f) { return empty ? 0.0 : part[f * T]; };   // field t.f0 + f
  const double M = g.V;
  const double sdata = g.mode == kMSE ? 2.0 * (double)g.invM : 1.0;
  for (int f = tid; f < t.nf && t.f0 + f < g.rec_stride; f += nt) {
    const int field = t.f0 + f;
    const double tot = total(f);
    float out = 0.0f;
    int dst = -1;
    if (field == kRecSigma) {
      dst = nb + 2 * N;
      out = g.mode == kNLL ? (float)(2.0 * N * M - tot) : 0.0f;
    } else if (field >= kRecBias && field < kRecBias + 10) {
      const int j = field - kRecBias;
      if (g.bias == 1) {
        dst = j;
        out = (float)(tot + (cal_on ? 2.0 * (double)R.model.lam_bias * cal[j] : 0.0));
      }
    } else if (field >= kRecAlpha && field < kRecAlpha + N) {
      const int n = field - kRecAlpha;
      dst = nb + n;
      out = (float)(sdata * tot + (cal_on ? 2.0 * (double)R.model.lam_alpha * cal[nb + n] : 0.0));
    } else if (field >= kRecAlpha + N) {
      const int n = field - kRecAlpha - N;
      dst = nb + N + n;
      out = (float)(sdata * tot + (cal_on ? 2.0 * (double)R.model.lam_beta * cal[nb + N + n] : 0.0));
    }
    if (dst >= 0) cal_entry(R, g, dst, out);
  }
  // an empty group's control grid has its prior alone
  if (empty && g.bias == 2)
    for (int i = tid; i < nb; i += nt)
      cal_entry(R, g, i, cal_on ? (float)(2.0 * (double)R.model.lam_bias * cal[i]) : 0.0f);
  // the step counter: no other block of this launch reads it (they read R.info)
  if (R.step && blockIdx.x == 0 && tid == 0) {
    R.step[0] = R.step[0] + 1;
    R.step[1] = 0;
  }
  if (t.f0 == 0 && tid == 0) {
    // loss terms from fields 0-7 (every tile holds at least eight fields)
    const double data = g.mode == kMSE ? total(kRecData) * (double)g.invM
                                       : total(kRecData) + 2.0 * sigma_log * (double)N * M;
    const double sp = total(kRecSpatial) * (double)R.model.lam_sp * g.invM;
    const double rp = total(kRecRep) * (double)R.model.lam_rep * g.invM;
    const double sa = total(kRecSparse) * (double)R.model.lam_sparse * g.invM;
    const double orp = total(kRecOrphan) * (double)R.model.lam_orphan * g.invM;
    const double cnt = total(kRecCont) * (double)R.model.lam_cont * g.invM;
    const double ord = total(kRecOrder) * (double)R.model.lam_order * g.invM;
    const double tv = total(kRecTV) * (double)R.model.lam_tv * g.invM;
    double cl = 0.0;
    if (cal_on) {
      double q[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        if (!empty) {
          q[i] = R.calsq[kCalSums * t.group + i];
        } else {
          q[i] = 0.0;
          for (int w = 0; w < nt / 64; ++w) q[i] += sq[i][w];
        }
      }
      cl = (double)R.model.lam_alpha * q[0] + (double)R.model.lam_beta * q[1] + (double)R.model.lam_bias * q[2];
    }
    double* L = R.loss + (int64_t)t.group * kLossTerms;
    L[0] = data;
    L[1] = sp;
    L[2] = rp;
    L[3] = sa;
    L[4] = orp;
    L[5] = cnt;
    L[6] = ord;
    L[7] = cl;
    L[8] = tv;
    L[9] = data + sp + rp + sa + orp + cnt + ord + cl + tv;
    if (!isfinite(L[9])) atomicOr(R.status, (uint32_t)kStNonfiniteLoss);
    if (R.hist) {
      int slot = (R.info ? R.info->index : R.hist_step[0]) % R.hist_len;
      if (slot < 0) slot += R.hist_len;
      double* H = R.hist + ((int64_t)slot * R.n_groups + t.group) * kLossTerms;
#pragma unroll
      for (int i = 0; i < kLossTerms; ++i) H[i] = L[i];
    }
  }
}

// ---------------------------------------------------------------------------
// optimisers
// ---------------------------------------------------------------------------
// Adam, PyTorch's form; t = step[0] + 1 is read by every block and the step
// counter is advanced afterwards by k_step_advance (stream order), so no
// block waits on another and no counter is contended.
// With advance != 0 the launch is a single block, which advances the step
// counter itself once every thread has used it.
__global__ __launch_bounds__(256) void k_adam(float* p, const float* g, float* m, float* v,
                                              int64_t n, float lr, float b1, float b2, float eps,
                                              int32_t* step, int vec4, int advance) {
  __shared__ float sc[2];
  if (threadIdx.x == 0) adam_factors(step, lr, b1, b2, sc[0], sc[1]);
  __syncthreads();
  const float step_size = sc[0], ibc2 = sc[1];
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t done = 0;
  if (vec4) {
    const int64_t n4 = n >> 2;
    float4* p4 = reinterpret_cast<float4*>(p);
    const float4* g4 = reinterpret_cast<const float4*>(g);
    float4* m4 = reinterpret_cast<float4*>(m);
    float4* v4 = reinterpret_cast<float4*>(v);
    for (int64_t i = tid; i < n4; i += stride) {
      float4 pp = p4[i], mm = m4[i], vv = v4[i];
      const float4 gg = g4[i];
      adam_one(pp.x, gg.x, mm.x, vv.x, b1, b2, eps, step_size, ibc2);
      adam_one(pp.y, gg.y, mm.y, vv.y, b1, b2, eps, step_size, ibc2);
      adam_one(pp.z, gg.z, mm.z, vv.z, b1, b2, eps, step_size, ibc2);
      adam_one(pp.w, gg.w, mm.w, vv.w, b1, b2, eps, step_size, ibc2);
      p4[i] = pp;
      m4[i] = mm;
      v4[i] = vv;
    }
    done = n4 << 2;
  }
  for (int64_t i = done + tid; i < n; i += stride) {
    float pp = p[i], mm = m[i], vv = v[i];
    adam_one(pp, g[i], mm, vv, b1, b2, eps, step_size, ibc2);
    p[i] = pp;
    m[i] = mm;
    v[i] = vv;
  }
  if (advance) {
    __syncthreads();
    if (threadIdx.x == 0) {
      step[0] = step[0] + 1;
      step[1] = 0;
    }
  }
}

__global__ void k_step_advance(int32_t* step) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    step[0] = step[0] + 1;
    step[1] = 0;
  }
}

__global__ __launch_bounds__(256) void k_rprop(float* p, const float* g, float* prev, float* st,
                                               int64_t n, float em, float ep, float smin,
                                               float smax) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    float gi = g[i];
    const float pr = gi * prev[i];
    float s = st[i];
    if (pr > 0.0f) s *= ep;
    else if (pr < 0.0f) s *= em;
    s = fminf(fmaxf(s, smin), smax);
    if (pr < 0.0f) gi = 0.0f;
    const float sg = gi > 0.0f ? 1.0f : (gi < 0.0f ? -1.0f : 0.0f);
    p[i] = p[i] - sg * s;
    prev[i] = gi;
    st[i] = s;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_pass_maxn(const PassArgs& a, int K, int mode, int learn_d, int vpl, int maxN,
                            hipStream_t s) {
  switch (K) {
    case 1: return launch_pass_k<1>(a, mode, learn_d, vpl, maxN, s);
    case 2: return launch_pass_k<2>(a, mode, learn_d, vpl, maxN, s);
    case 3: return launch_pass_k<3>(a, mode, learn_d, vpl, maxN, s);
    case 4: return launch_pass_k<4>(a, mode, learn_d, vpl, maxN, s);
    case 5: return launch_pass_k<5>(a, mode, learn_d, vpl, maxN, s);
    case 6: return launch_pass_k<6>(a, mode, learn_d, vpl, maxN, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_split_maxn(const PassArgs& a, int K, int mode, int learn_d, int ls, int maxN, hipStream_t s) {
  switch (K) {
    case 1: return launch_split_k<1>(a, mode, learn_d, ls, maxN, s);
    case 2: return launch_split_k<2>(a, mode, learn_d, ls, maxN, s);
    case 3: return launch_split_k<3>(a, mode, learn_d, ls, maxN, s);
    case 4: return launch_split_k<4>(a, mode, learn_d, ls, maxN, s);
    case 5: return launch_split_k<5>(a, mode, learn_d, ls, maxN, s);
    case 6: return launch_split_k<6>(a, mode, learn_d, ls, maxN, s);
    default: return hipErrorInvalidValue;
  }
}

int split_blocks_per_cu(int K, int mode, int learn_d, int ls, int N) {
  switch (K) {
    case 1: return split_occupancy_k<1>(mode, learn_d, ls, N);
    case 2: return split_occupancy_k<2>(mode, learn_d, ls, N);
    case 3: return split_occupancy_k<3>(mode, learn_d, ls, N);
    case 4: return split_occupancy_k<4>(mode, learn_d, ls, N);
    case 5: return split_occupancy_k<5>(mode, learn_d, ls, N);
    case 6: return split_occupancy_k<6>(mode, learn_d, ls, N);
    default: return 0;
  }
}

template <int CT>
static void launch_spatial_t(const PassArgs& a, dim3 grid, dim3 block, bool from_logits, hipStream_t s) {
  if (from_logits) {
    hipLaunchKernelGGL((k_spatial<CT, true>), grid, block, 0, s, a);
  } else {
    hipLaunchKernelGGL(k_fractions<CT>, grid, block, 0, s, a);
    hipLaunchKernelGGL((k_spatial<CT, false>), grid, block, 0, s, a);
  }
}

hipError_t launch_spatial(const PassArgs& a, int n_items, int spatial_c, int max_nv, bool from_logits,
                          hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  // whole waves, one thread per voxel of the largest item, at most kAuxBlock
  const dim3 grid(n_items), block(std::min(kAuxBlock, std::max(64, (max_nv + 63) / 64 * 64)));
  switch (spatial_c) {
    case 4: launch_spatial_t<4>(a, grid, block, from_logits, s); break;
    case 5: launch_spatial_t<5>(a, grid, block, from_logits, s); break;
    case 6: launch_spatial_t<6>(a, grid, block, from_logits, s); break;
    case 7: launch_spatial_t<7>(a, grid, block, from_logits, s); break;
    case 8: launch_spatial_t<8>(a, grid, block, from_logits, s); break;
    case 9: launch_spatial_t<9>(a, grid, block, from_logits, s); break;
    default: launch_spatial_t<0>(a, grid, block, from_logits, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_reduce(const ReduceArgs& a, int max_records, hipStream_t s) {
  if (a.n_tiles <= 0) return hipSuccess;
  if (a.n_row_tiles > 0) hipLaunchKernelGGL(k_reduce_rows, dim3(a.n_row_tiles), dim3(kReduceBlock), 0, s, a);
  // narrow tiles of up to 256 records: one round of loads with 32 threads a column; of
  // more: 128 threads a column
  const int block = max_records > 256 ? kReduceWide : kReduceBlock;
  const int tri = 512 * a.n_tri_wide + 512 / (block / 64) * (a.n_tri - a.n_tri_wide);
  hipLaunchKernelGGL(k_reduce, dim3(a.n_tiles + tri), dim3(block), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1,
                       float b2, float eps, int32_t* step, hipStream_t s, bool advance) {
  const bool vec4 = ((reinterpret_cast<uintptr_t>(p) | reinterpret_cast<uintptr_t>(g) |
                      reinterpret_cast<uintptr_t>(m) | reinterpret_cast<uintptr_t>(v)) & 15) == 0;
  int64_t blocks = (n + 2047) / 2048;
  if (blocks < 1) blocks = 1;
  if (blocks > 4096) blocks = 4096;
  // a one-block update advances the counter itself (one launch instead of two)
  const int self_advance = advance && blocks == 1 ? 1 : 0;
  if (n > 0 || self_advance)
    hipLaunchKernelGGL(k_adam, dim3((unsigned)blocks), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2,
                       eps, step, vec4 ? 1 : 0, self_advance);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !advance || self_advance) return e;
  hipLaunchKernelGGL(k_step_advance, dim3(1), dim3(64), 0, s, step);
  return hipGetLastError();
}

template <int K>
static hipError_t launch_stitch_k(const StitchArgs& a, int learn_d, hipStream_t s) {
  const unsigned blocks = (unsigned)((a.n_out + 255) / 256);
  if (learn_d)
    hipLaunchKernelGGL((k_stitch<K, true>), dim3(blocks), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_stitch<K, false>), dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_stitch(const StitchArgs& a, int K, int learn_d, hipStream_t s) {
  if (a.n_out <= 0) return hipSuccess;
  switch (K) {
    case 1: return launch_stitch_k<1>(a, learn_d, s);
    case 2: return launch_stitch_k<2>(a, learn_d, s);
    case 3: return launch_stitch_k<3>(a, learn_d, s);
    case 4: return launch_stitch_k<4>(a, learn_d, s);
    case 5: return launch_stitch_k<5>(a, learn_d, s);
    case 6: return launch_stitch_k<6>(a, learn_d, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rprop(float* p, const float* g, float* prev, float* step, int64_t n, float em,
                        float ep, float smin, float smax, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 1023) / 1024;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_rprop, dim3((unsigned)blocks), dim3(256), 0, s, p, g, prev, step, n, em, ep,
                     smin, smax);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// the Eq. 9 special functions at given arguments, as the fused pass computes them
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_rician_terms(const float* z, float* li, float* omr, float* q,
                                                      int64_t n) {
  __shared__ float4 bes[kBesselRows];
  stage_bessel(bes);
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const float zi = z[i];
    float nli, o, qi;
    rician_terms<true>(zi, bes, nli, o, &qi);
    li[i] = -nli;
    omr[i] = o;
    q[i] = qi;
  }
}

hipError_t launch_rician_terms(const float* z, float* li, float* omr, float* q, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_rician_terms, dim3((unsigned)blocks), dim3(256), 0, s, z, li, omr, q, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Static workspace of the allocation-free entry point (prism_loss_grad_noalloc)
// ---------------------------------------------------------------------------
// One array per device, held from the library's load until the process ends.
// In host code `scratch` names a host-side stand-in, not the device array:
// only the address hipGetSymbolAddress returns for the current device may be
// passed to kernels or copies.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
hipError_t g_scratch_err[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch_setup(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
  void* ptr = nullptr;
  e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e == hipSuccess && ptr == nullptr) e = hipErrorInvalidSymbol;
  if (e == hipSuccess) g_scratch_ptr[device] = ptr;
  g_scratch_err[device] = e;
  if (cur != device) (void)hipSetDevice(cur);
  return e;
}

void* static_scratch(int device, hipError_t* err) {
  if (device < 0 || device >= kMaxDevices) {
    *err = hipErrorInvalidDevice;
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  *err = g_scratch_ptr[device] ? hipSuccess
                               : (g_scratch_err[device] != hipSuccess ? g_scratch_err[device] : hipErrorNotInitialized);
  return g_scratch_ptr[device];
}

}  // namespace prism
