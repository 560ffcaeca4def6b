// Device helpers for the PRISM kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>

#include "bessel_fit.h"

namespace prism {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// hardware transcendentals: 2^x, log2(x), 1/x, 1/sqrt(x), sqrt(x) (about 1 ulp)
__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float lg2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float sqrt_hw(float x) { return __builtin_amdgcn_sqrtf(x); }

// e^x as 2^(x log2 e): two instructions, relative error a few ulp for |x| < 100
__device__ __forceinline__ float exp_hw(float x) { return ex2(x * kLog2e); }

// log(1 + e) for e >= 0 without cancellation: log2(w) ln2 * e / (w - 1), w = 1 + e
// (the second factor corrects the rounding of w; w == 1 means log1p(e) = e)
__device__ __forceinline__ float log1p_hw(float e) {
  const float w = 1.0f + e;
  return w == 1.0f ? e : lg2(w) * kLn2 * (e * rcp(w - 1.0f));
}

// numerically stable per-voxel transforms
__device__ __forceinline__ float softplus_f(float x) {
  return fmaxf(x, 0.0f) + log1p_hw(exp_hw(-fabsf(x)));
}
__device__ __forceinline__ float sigmoid_f(float x) {
  // 1 / (1 + e^-x) without overflow for large |x|
  const float e = exp_hw(-fabsf(x));
  const float s = rcp(1.0f + e);
  return x >= 0.0f ? s : e * s;
}

// One float of a row of `nbytes` bytes at byte offset `off`, through a buffer
// descriptor: the row's base stays in scalar registers and the lane supplies
// only a 32-bit offset (no per-lane 64-bit address arithmetic).  Offsets at or
// beyond nbytes read 0.  Word 3 is the gfx9-family raw 32-bit buffer format.
__device__ __forceinline__ float load_row_f32(const float* row, uint32_t nbytes, uint32_t off) {
  __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(row), (short)0, (int)nbytes, 0x00020000);
  // the builtin returns the 32 loaded bits; reinterpret them, do not convert them
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// The same for a store, and for an int32 row.  A parameter-major block [P][V]
// is P such rows of V entries (V <= 1023^3, so V * 4 < 2^32): every lane
// addresses every row with one 32-bit offset (its voxel * 4) and the row bases
// stay uniform, where 64-bit per-lane addresses take two registers per row.
__device__ __forceinline__ void store_row_f32(float* row, uint32_t nbytes, uint32_t off, float x) {
  __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(row, (short)0, (int)nbytes, 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), r, off, 0, 0);
}
__device__ __forceinline__ int32_t load_row_i32(const int32_t* row, uint32_t nbytes, uint32_t off) {
  __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int32_t*>(row), (short)0, (int)nbytes, 0x00020000);
  return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
}

// Four int32 at p + 4 i (16-byte aligned, in memory that no kernel of the call writes) by
// scalar loads; i is uniform.
__device__ __forceinline__ int4 uniform_int4(const int32_t* p, int i) {
  typedef const __attribute__((address_space(4))) int4* Cp;
  return *(const int4*)((Cp)p + i);
}

// The rows of a [rows][V] block one after the other.  The row's base stays in
// scalar registers and moves on by one addition per row; it passes through an
// empty asm statement at each row, so the compiler can neither form the bases of
// all rows early nor keep them across the measurement loop (formed as base + row V
// they were hoisted out of the loop over an item's chunks and spilled: 368 scalar
// registers of the K = 3 MSE pass, each access to one a v_readlane or v_writelane).
template <typename T>
struct RowCursor {
  T* p;
  int64_t V;
  __device__ __forceinline__ RowCursor(T* base, int64_t V_, int row = 0) : p(base + row * V_), V(V_) {}
  __device__ __forceinline__ T* next() {
    asm volatile("" : "+s"(p));
    T* r = p;
    p += V;
    return r;
  }
};

// The object at p (in memory that no kernel of the call writes) read again from here
// on, by scalar loads: its fields are needed in the prologue and in the epilogue of an
// item, and kept in scalar registers across the measurement loop they would spill.
template <typename T>
__device__ __forceinline__ const T& reread(const T* p) {
  typedef const __attribute__((address_space(4))) T* Cp;
  Cp c = (Cp)p;
  asm volatile("" : "+s"(c));
  return *(const T*)c;
}

// Work item of block b in a launch of n blocks.  The dispatcher deals blocks
// to the 8 XCDs in turn (block b to XCD b mod 8) and each XCD has its own L2;
// giving XCD x one contiguous run of items keeps the neighbours that an item
// gathers (the next row and slice of the volume) in the L2 that serves it.
// A bijection of [0, n).
__device__ __forceinline__ int xcd_item(int b, int n) {
  constexpr int kXcd = 8;
  const int q = n / kXcd, r = n % kXcd, x = b % kXcd;
  return x * q + (x < r ? x : r) + b / kXcd;
}

// ---------------------------------------------------------------------------
// wave reductions
// ---------------------------------------------------------------------------

template <int CTRL, int ROW_MASK = 0xf, int BANK_MASK = 0xf>
__device__ __forceinline__ float dpp_f32(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROW_MASK, BANK_MASK,
                                         false));
}

// Per-measurement sums over each row of 16 lanes, fed one value per lane per
// measurement in groups of four (measurement t = 4g + u of a tile of 16):
// afterwards lane l of a row holds the row's sum for measurement
// row_scatter_index(l).  Within a group the four values are reduce-scattered
// over each quad of lanes: the pair (u, u + 1) and then the two pair sums are
// combined as keep + partner(send), (keep, send) = (later, earlier) where the
// lane's level bit is set and (earlier, later) where it is clear, with the
// partner lane xor 1, then xor 2, and the level bits b0^b2, b1^b2 (b = the
// lane's bits in the row), which differ between partners, so each quad lane
// ends with the quad's sum for one of the group's measurements.  The level
// bits also agree between lanes l and l^7 and between l and l^15, so adding
// the half-row mirror and then the row mirror sums the four quads of the row
// measurement by measurement; bank g (lanes 4g..4g+3) of the row keeps the
// result of group g.  Per group of four measurements: three combines of three
// VALU operations, two adds with a mirrored operand and one select (a
// matrix-core one-hot accumulation takes one v_mfma_f32_16x16x4f32 per
// measurement, which holds the SIMD for its 32 cycles).
struct RowScatter {
  float x0, r1, q;  // within a group: pending value, pending pair sum, the quad result
  float acc;        // bank g of the row: the row sums of group g's measurements
};
struct RowScatterMasks {
  bool m[2];        // per lane: the level bits b0^b2, b1^b2
};
__device__ __forceinline__ RowScatterMasks row_scatter_masks(int lane) {
  const uint32_t l = (uint32_t)lane & 15u;
  const uint32_t b0 = l & 1u, b1 = (l >> 1) & 1u, b2 = (l >> 2) & 1u;
  return {{(b0 ^ b2) != 0, (b1 ^ b2) != 0}};
}
// the measurement of the tile (0..15) whose row sum lane l holds at the end
__device__ __forceinline__ int row_scatter_index(int lane) {
  const int l = lane & 15, b0 = l & 1, b1 = (l >> 1) & 1, b2 = (l >> 2) & 1;
  return (l & 12) | (b0 ^ b2) | (b1 ^ b2) << 1;
}
template <int CTRL>
__device__ __forceinline__ float row_scatter_combine(float x, float y, bool m) {
  return (m ? y : x) + dpp_f32<CTRL>(m ? x : y);
}
// measurement u (0..3, known at compile time) of the current group
__device__ __forceinline__ void row_scatter_push(RowScatter& s, float v, int u, const RowScatterMasks& M) {
  if ((u & 1) == 0) {
    s.x0 = v;
    return;
  }
  const float r = row_scatter_combine<0xB1>(s.x0, v, M.m[0]);   // quad_perm [1,0,3,2]
  if (u == 1)
    s.r1 = r;
  else
    s.q = row_scatter_combine<0x4E>(s.r1, r, M.m[1]);           // quad_perm [2,3,0,1]
}
// end of group g: here = (lane's bank in the row == g)
__device__ __forceinline__ void row_scatter_group(RowScatter& s, bool here) {
  float t = s.q + dpp_f32<0x141>(s.q);  // row_half_mirror: lane xor 7
  t += dpp_f32<0x140>(t);               // row_mirror: lane xor 15
  s.acc = here ? t : s.acc;
}

// Sums over the wave of two values per lane per measurement, for a group of four
// measurements (0..3): afterwards lane l holds the wave's sum of value l / 32 for
// measurement group_sums_index(l) (the same in the eight lanes of its half row).  The two
// values share a register from the first step on: v_permlane32_swap exchanges the upper half
// of one register with the lower half of the other, so one addition then leaves the first
// value's sums in the lower half and the second's in the upper half; v_permlane16_swap
// does the same for two measurements and the rows of each half, and a select with the row
// mirror for the two pairs and the halves of each row.  Four swaps, four additions; two and
// two; three; then three additions of mirrored operands: 18 operations per group for both
// values, where the reduce-scatter within rows above takes 25.  (The swaps are inline asm
// because this compiler's builtins return the first result for both outputs.  A swap needs
// two wait states after the operation that wrote its operands, which the compiler does not
// count into inline asm: the s_nop.)
struct GroupSums {
  float c, d01, d23;   // the pending measurement, the pairs (0, 1) and (2, 3)
};
__device__ __forceinline__ float swap32_sum(float x, float y) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(x), "+v"(y));
  return x + y;
}
__device__ __forceinline__ float swap16_sum(float x, float y) {
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(x), "+v"(y));
  return x + y;
}
__device__ __forceinline__ int group_sums_index(int lane) { return ((lane >> 4) & 1) | ((lane >> 3) & 1) << 1; }
// the values a, b of measurement u (known at compile time), in order
__device__ __forceinline__ void group_sums_push(GroupSums& s, float a, float b, int u) {
  const float c = swap32_sum(a, b);
  if ((u & 1) == 0)
    s.c = c;
  else if (u == 1)
    s.d01 = swap16_sum(s.c, c);
  else
    s.d23 = swap16_sum(s.c, c);
}
// hi8: the lane's bit 3
__device__ __forceinline__ float group_sums_total(const GroupSums& s, bool hi8) {
  const float kept = hi8 ? s.d23 : s.d01, sent = hi8 ? s.d01 : s.d23;
  float e = kept + dpp_f32<0x140>(sent);   // row_mirror: the lane with the other bit 3
  e += dpp_f32<0xB1>(e);                   // quad_perm xor 1
  e += dpp_f32<0x4E>(e);                   // quad_perm xor 2
  e += dpp_f32<0x141>(e);                  // row_half_mirror: the other quad
  return e;
}

// Lane exchanges across rows without per-use index arithmetic: ds_swizzle in
// bitmask mode (and-mask 0x1f, xor-mask 16: lane i reads lane i ^ 16 within
// each half-wave) and ds_bpermute from lane i ^ 32.  Full waves only.
__device__ __forceinline__ int xor16_b32(int x) { return __builtin_amdgcn_ds_swizzle(x, 0x401F); }
__device__ __forceinline__ int xor32_b32(int x) {
  return __builtin_amdgcn_ds_bpermute((int)((__lane_id() ^ 32u) << 2), x);
}
__device__ __forceinline__ float xor16_f32(float x) {
  return __builtin_bit_cast(float, xor16_b32(__builtin_bit_cast(int, x)));
}
__device__ __forceinline__ float xor32_f32(float x) {
  return __builtin_bit_cast(float, xor32_b32(__builtin_bit_cast(int, x)));
}

// A float64 through a DPP pattern (both halves; every lane of the patterns
// used here has a valid source)
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double xor16_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)xor16_b32((int)(uint32_t)u), hi = (uint32_t)xor16_b32((int)(uint32_t)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double xor32_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)xor32_b32((int)(uint32_t)u), hi = (uint32_t)xor32_b32((int)(uint32_t)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum over the 64 lanes of a full wave, the same total in every lane: within
// rows of 16 by DPP (quad_perm xor 1, xor 2, half-row mirror, row mirror, each
// leaving its group uniform), then rows 0+1 and 2+3 (xor 16), then the halves
// (xor 32).  A fixed order, so the result is reproducible bit for bit.
__device__ __forceinline__ double wave_sum_f64(double x) {
  x += dpp_f64<0xB1>(x);   // quad_perm [1,0,3,2]
  x += dpp_f64<0x4E>(x);   // quad_perm [2,3,0,1]
  x += dpp_f64<0x141>(x);  // row_half_mirror
  x += dpp_f64<0x140>(x);  // row_mirror
  x += xor16_f64(x);
  x += xor32_f64(x);
  return x;
}

// ---------------------------------------------------------------------------
// Eq. 9 special functions: -log I0e(z) and 1 - I1(z)/I0(z) for z >= 0
// ---------------------------------------------------------------------------
// The table of bessel_fit.h as the kernels read it, rows in LDS: entry i is the
// two float4 (z0, c0, c1, c2) at [i] and (c3, c4, c5, c6) at [kBesselEntries + i]
// (two arrays rather than rows of 32 bytes, so that the lanes' rows start at all
// sixteen groups of four banks).  The table is read per lane: the alternative,
// closed forms for small and for large z, runs both in nearly every wave (about
// 115 instructions, against 18 here and two LDS reads; a 16^3 patch's iteration,
// N = 288, K = 3: 66.3 -> 53.4 us, 512 mixed patches 1671 -> 1204 us).
constexpr int kBesselRows = 2 * kBesselEntries;   // float4 rows of LDS (4.9 KB)

// every thread of the block; the caller synchronises
__device__ __forceinline__ void stage_bessel(float4* tab) {
  for (int i = threadIdx.x; i < kBesselEntries; i += blockDim.x) {
    tab[i] = make_float4(kBesselZ0[i], kBesselC0[i], kBesselC1[i], kBesselC2[i]);
    tab[kBesselEntries + i] = make_float4(kBesselC3[i], kBesselC4[i], kBesselC5[i], kBesselC6[i]);
  }
}

// nli = -log I0e(z) = z - log I0(z) and omr = 1 - I1(z)/I0(z), each within 6.4e-8
// relative over [0, 65536) and 9.1e-8 above (host emulation of this algorithm; the tests
// measure the device).  omr is the derivative of nli, so one polynomial in d = z - z0 of
// the argument's interval gives both:
//   nli = c0 + d (c1 + d s),  omr = c1 + d (2 s + d s'),  s = c2 + ... + c6 d^4.
// Two kinds of argument are outside kBesselFirst <= z < kBesselSplit, in one branch that
// few waves take.  Below it (entry 0: z0 = 0, c0 = 0, c1 = 1) nli is summed as
// z + z (z s), since both roundings of z (1 + z s) would count (8.9e-8 relative against
// 6.0e-8; 512 mixed patches 789 -> 800 us with it); from kBesselSplit up (any size; z NaN
// gives NaN): the large-argument expansions.
// Q: q = 2 z omr too, from omr and what its own rounding left, so that one rounding counts.
// (The pass takes this product unrounded into a multiply-add.)
template <bool Q = false>
__device__ __forceinline__ void rician_terms(float z, const float4* tab, float& nli, float& omr, float* q = nullptr) {
  // the interval from the float's bits, clamped into the table (negative bits, a
  // negative NaN, too; below kBesselFirst to the last number of entry 0), so that one
  // comparison tells both kinds
  constexpr int kLo = __builtin_bit_cast(int, kBesselFirst) - 1;
  const int zb = __builtin_bit_cast(int, z), bits = min(max(zb, kLo), kBesselBitsHi);
  const int i = (bits - kBesselBitsLo) >> kBesselShift;
  const float4 a = tab[i], b = tab[kBesselEntries + i];
  const float d = z - a.x;
  float s = fmaf(b.w, d, b.z), ds = fmaf(b.w, d, s);
  s = fmaf(s, d, b.y);
  ds = fmaf(ds, d, s);
  s = fmaf(s, d, b.x);
  ds = fmaf(ds, d, s);
  s = fmaf(s, d, a.w);
  const float t = fmaf(d, ds, s + s);
  omr = fmaf(d, t, a.z);
  nli = fmaf(d, fmaf(d, s, a.z), a.y);
  if (Q) *q = fmaf(z + z, omr, (z + z) * fmaf(d, t, a.z - omr));
  if (bits != zb) {
    nli = fmaf(z * s, z, z);
    if (z >= kBesselSplit) {
      const float iz0 = rcp(z);
      const float iz = fmaf(fmaf(-z, iz0, 1.0f), iz0, iz0);
      const float r = 0.5f * iz;
      omr = fmaf(0.25f * iz, r, r);
      nli = fmaf(kHalfLn2, lg2(z), fmaf(-0.125f, iz, kHalfLog2Pi));
      if (Q) *q = fmaf(0.25f, iz, 1.0f);
    }
  }
}

}  // namespace prism
