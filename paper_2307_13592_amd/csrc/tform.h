// Device helpers shared by the T-form kernels (16-row tiles, one wave per
// tile; products computed transposed, so that lane (e, q) = (lane & 15,
// lane >> 4) of an accumulator tile holds output columns 16 cb + 4 q + r of
// row e): ranges of edges per wave, tile metadata, row and column sums.
#pragma once
#include "device_common.h"

namespace mgn {

constexpr int RS_GRID = 256;           // one workgroup per compute unit; a multiple of 8

// fp32 element index of (row, col) in a 16-row scratch tile of width L whose
// 16-byte chunks are XOR-swizzled by row (conflict-free both for
// accumulator-order writes and for row-order reads).
template <int L>
__device__ __forceinline__ int rs_sw32(int row, int col) {
  constexpr int M = (L / 4 < 16 ? L / 4 : 16) - 1;
  return row * L + ((((col >> 2) ^ (row & M))) << 2) + (col & 3);
}

// The wave's index in its workgroup, as a wave-uniform (scalar) value.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// A wave-uniform value held in scalar registers.
__device__ __forceinline__ int64_t rs_uniform(int64_t x) {
  const uint64_t u = (uint64_t)x;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Receiver range of this wave (one of nwv working waves per workgroup, W in
// total) within [lo_r, hi_r): receiver-aligned, about E / W edges each; the
// waves of one XCD (blockIdx % 8) get neighbouring ranges.
__device__ __forceinline__ void rs_range(const int32_t* __restrict__ row_ptr, int64_t lo_r, int64_t hi_r, int64_t& r0,
                                         int64_t& r1, int nwv) {
  const int G = gridDim.x, b = blockIdx.x, wave = wave_id();
  const int64_t W = (int64_t)G * nwv;
  const int64_t q = ((int64_t)(b & 7) * (G >> 3) + (b >> 3)) * nwv + wave;
  const int64_t e0 = row_ptr[lo_r], E = row_ptr[hi_r] - e0;
  auto find = [&](int64_t target) {  // first receiver r >= lo_r with row_ptr[r] >= target
    int64_t lo = lo_r, hi = hi_r;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (row_ptr[mid] >= target) hi = mid;
      else lo = mid + 1;
    }
    return lo;
  };
  r0 = q == 0 ? lo_r : find(e0 + E * q / W);
  r1 = q + 1 == W ? hi_r : find(e0 + E * (q + 1) / W);
}

// The same for edges [e_lo, e_lo + E) of the receivers [lo_r, hi_r), with the
// boundaries looked up through the per-edge receiver ids: two dependent loads
// where the search above takes two per halving of the receiver count (on a
// graph of 11,000 edges, half of an edge kernel's time).  A boundary inside a
// receiver's edges moves to the next receiver.  E0, E1: the range's edges.
__device__ __forceinline__ void rs_range_e(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ erecv,
                                           int64_t lo_r, int64_t hi_r, int64_t e_lo, int64_t E, int nwv, int64_t& r0,
                                           int64_t& r1, int64_t& E0, int64_t& E1) {
  const int G = gridDim.x, b = blockIdx.x, wave = wave_id();
  const int64_t W = (int64_t)G * nwv;
  const int64_t q = ((int64_t)(b & 7) * (G >> 3) + (b >> 3)) * nwv + wave;
  const int64_t t0 = E * q / W, t1 = E * (q + 1) / W;
  const bool first = q == 0, last = q + 1 == W;
  r0 = lo_r;
  r1 = last ? hi_r : lo_r;  // without edges the last wave takes all receivers
  E0 = E1 = e_lo;
  if (E > 0) {
    const int32_t a = erecv[e_lo + t0], c = erecv[e_lo + (last ? E - 1 : t1)];
    const int64_t pa = row_ptr[a], na = row_ptr[a + 1], pc = row_ptr[c], nc = row_ptr[c + 1];
    const bool ina = pa < e_lo + t0, inc = pc < e_lo + t1;
    r0 = first ? lo_r : ina ? (int64_t)a + 1 : a;
    E0 = first ? e_lo : ina ? na : pa;
    r1 = last ? hi_r : inc ? (int64_t)c + 1 : c;
    E1 = last ? e_lo + E : inc ? nc : pc;
  }
  r0 = rs_uniform(r0);
  r1 = rs_uniform(r1);
  E0 = rs_uniform(E0);
  E1 = rs_uniform(E1);
}

// Zeroes the rows (width L) of the receivers in [r0, r1) without edges (one
// wave, a lane per receiver).
__device__ __forceinline__ void rs_zero_empty(const int32_t* __restrict__ row_ptr, int64_t r0, int64_t r1, float* dst,
                                              int L) {
  const int lane = threadIdx.x & 63;
  for (int64_t r = r0 + lane; r < r1; r += 64)
    if (row_ptr[r] == row_ptr[r + 1])
      for (int c = 0; c < L; c += 4) *reinterpret_cast<float4*>(dst + r * L + c) = make_float4(0.f, 0.f, 0.f, 0.f);
}

// One 16-edge tile's metadata, every lane for its row e = lane & 15: the
// edge's receiver, sender and the next edge's receiver (-1 past the range
// end); the mask has bit j (j < 16) set where row j ends a receiver segment.
// The loads are issued one tile ahead (rt_meta_load) and turned into the
// mask when the tile starts (rt_meta_make), so no tile waits for them.
struct RsMeta {
  int32_t r, s;
  unsigned long long last;
};
struct RsMetaRaw {
  int32_t r, s, rn;
};
__device__ __forceinline__ RsMetaRaw rt_meta_load(const int32_t* __restrict__ erecv, const int32_t* __restrict__ send,
                                                  int64_t sb, int64_t e1) {
  const int e = threadIdx.x & 15;
  RsMetaRaw w{-1, 0, -1};
  if (sb + e < e1) {
    w.r = erecv[sb + e];
    w.s = send[sb + e];
    if (sb + e + 1 < e1) w.rn = erecv[sb + e + 1];
  }
  return w;
}
__device__ __forceinline__ RsMeta rt_meta_make(const RsMetaRaw& w) {
  RsMeta mt{w.r, w.s, 0};
  mt.last = __ballot(w.r >= 0 && w.rn != w.r);
  return mt;
}

// Sum over the four 16-lane groups; every lane gets the same bits.
__device__ __forceinline__ float rt_sum4(float x) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float s = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  const auto p2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return __uint_as_float(p2[0]) + __uint_as_float(p2[1]);
}

// Per-lane partial over an accumulator tile's values, four chains.
template <int NB>
__device__ __forceinline__ float rt_lane_sum(const float (&v)[NB][4]) {
  float t[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    t[r] = v[0][r];
#pragma unroll
    for (int cb = 1; cb < NB; ++cb) t[r] += v[cb][r];
  }
  return (t[0] + t[1]) + (t[2] + t[3]);
}

// One reduce-scatter step within a 16-lane group: v[0, N) -> v[0, N / 2);
// the lane keeps the half that `hi` selects, summed with the DPP partner's
// copy of it (the partner keeps the other half).  Both halves' sums are
// formed, each one add with the partner's value read through DPP (every
// lane of these patterns has a partner in its row), and one is selected:
// three instructions per pair instead of two selects, a move and an add.
template <int N, int CTRL>
__device__ __forceinline__ void rt_halve(float* v, bool hi) {
  // no contraction with a product that formed v: both partners must add the
  // same two rounded values
#pragma clang fp contract(off)
#pragma unroll
  for (int k = 0; k < N / 2; ++k) {
    const float lo = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[k]), CTRL, 0xf, 0xf, true)) + v[k];
    const float up =
        __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[k + N / 2]), CTRL, 0xf, 0xf, true)) + v[k + N / 2];
    v[k] = hi ? up : lo;
  }
}

// Column totals over a tile's 16 rows.  In: v[NV] per lane (index 4 cb + r of
// the accumulator order).  Out: lane e's v[t], t < NV / 16, is the total of
// index e * NV / 16 + t.  Partners: row mirror (e ^ 15), half-row mirror
// (e ^ 7), then e ^ 3 and e ^ 1 within quads.
template <int NV>
__device__ __forceinline__ void rt_col_totals(float (&v)[NV], int e) {
  static_assert(NV >= 16, "at least one total per lane");
  rt_halve<NV, 0x140>(v, e & 8);
  rt_halve<NV / 2, 0x141>(v, e & 4);
  rt_halve<NV / 4, 0x1B>(v, e & 2);
  rt_halve<NV / 8, 0xB1>(v, e & 1);
}

// 4 consecutive floats of a plain-order row at column 16 cb + 4 q.
__device__ __forceinline__ float4 rt_ld4(const float* __restrict__ p, int cb, int q) {
  return *reinterpret_cast<const float4*>(p + cb * 16 + q * 4);
}

// Copies n floats into LDS (all threads of the workgroup).
__device__ __forceinline__ void rt_copy_vec(float* dst, const float* __restrict__ src, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

}  // namespace mgn
