// Device helpers shared by the T-form kernels (16-row tiles, one wave per
// tile; products computed transposed, so that lane (e, q) = (lane & 15,
// lane >> 4) of an accumulator tile holds output columns 16 cb + 4 q + r of
// row e): ranges of edges per wave, tile metadata, row and column sums.
#pragma once
#include "device_common.h"

namespace mgn {

constexpr int RS_GRID = 256;           // one workgroup per compute unit; a multiple of 8

// bf16 / fp32 element index of (row, col) in a 16-row scratch tile of width
// L whose 16-byte chunks are XOR-swizzled by row (conflict-free both for
// accumulator-order writes and for fragment / row-order reads).
template <int L>
__device__ __forceinline__ int rs_sw16(int row, int col) {
  constexpr int M = (L / 8 < 16 ? L / 8 : 16) - 1;
  return row * L + ((((col >> 3) ^ (row & M))) << 3) + (col & 7);
}
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

// The edges [E0, E1) of this wave's receivers (wave `wave` of nwv per
// workgroup), of the edges [e_lo, e_lo + E) (whole receivers), with the
// boundaries looked up through the per-edge receiver ids: two dependent loads
// where the search above takes two per halving of the receiver count (on a
// graph of 11,000 edges, half of an edge kernel's time).  A boundary inside a
// receiver's edges moves past them.
__device__ __forceinline__ void rs_range_e(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ erecv,
                                           int64_t e_lo, int64_t E, int nwv, int wave, int64_t& E0, int64_t& E1) {
  const int G = gridDim.x, b = blockIdx.x;
  const int64_t W = (int64_t)G * nwv;
  const int64_t q = ((int64_t)(b & 7) * (G >> 3) + (b >> 3)) * nwv + wave;
  const int64_t t0 = E * q / W, t1 = E * (q + 1) / W;
  const bool last = q + 1 == W;
  E0 = E1 = e_lo;
  if (E > 0) {
    const int32_t a = erecv[e_lo + t0], c = erecv[e_lo + (last ? E - 1 : t1)];
    const int64_t pa = row_ptr[a], na = row_ptr[a + 1], pc = row_ptr[c], nc = row_ptr[c + 1];
    E0 = q == 0 ? e_lo : pa < e_lo + t0 ? na : pa;
    E1 = last ? e_lo + E : pc < e_lo + t1 ? nc : pc;
  }
  E0 = rs_uniform(E0);
  E1 = rs_uniform(E1);
}

// Zeroes the rows (width L) of the receivers in [lo_r, hi_r) without edges: 64
// receivers, a lane each, go to every wave in turn.  (With each wave zeroing
// between its own edges' receivers, a long run of receivers without edges fell
// to one wave: 300,000 of them at l = 128 took 6.8 ms a launch, now 0.064.)
// rs_empty_load, at the kernel's start, loads the bounds of the lane's first
// receiver, whose latency (1 us a launch on small graphs) then passes with the
// weights' on their way to LDS.
struct RsEmpty {
  int64_t r, end;
  int32_t a, b;
};
__device__ __forceinline__ RsEmpty rs_empty_load(const int32_t* __restrict__ row_ptr, int64_t lo_r, int64_t hi_r) {
  RsEmpty z{lo_r + (int64_t)blockIdx.x * blockDim.x + threadIdx.x, hi_r, 0, 0};
  if (z.r < z.end) {
    z.a = row_ptr[z.r];
    z.b = row_ptr[z.r + 1];
  }
  return z;
}
__device__ __forceinline__ void rs_zero_empty(RsEmpty z, const int32_t* __restrict__ row_ptr, float* dst, int L) {
  while (z.r < z.end) {
    if (z.a == z.b)
      for (int c = 0; c < L; c += 4) *reinterpret_cast<float4*>(dst + z.r * L + c) = make_float4(0.f, 0.f, 0.f, 0.f);
    z.r += (int64_t)gridDim.x * blockDim.x;
    if (z.r < z.end) {
      z.a = row_ptr[z.r];
      z.b = row_ptr[z.r + 1];
    }
  }
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


// ------------------------------------------------------------ bf16 T form ---
// Copies nb 16-column blocks x nkg k-groups of packed fragments (source
// block stride src_nkg k-groups, first k-group kg0) into LDS, all threads.
__device__ __forceinline__ void rs_copy_frags(uint4* dst, const uint4* __restrict__ src, int nb, int nkg, int src_nkg,
                                              int kg0) {
  const int total = nb * nkg * 64;
  for (int i = threadIdx.x; i < total; i += blockDim.x) {
    const int cb = i / (nkg * 64), kg = (i / 64) % nkg, ln = i % 64;
    dst[i] = src[((size_t)cb * src_nkg + kg0 + kg) * 64 + ln];
  }
}

// Like rs_copy_frags, with the eight k-slots of every fragment reordered so
// that slot j of lane group q pairs with k = 32 kg + 16 (j / 4) + 4 q + j % 4:
// its low half comes from lane group q / 2, its high half from 2 + q / 2,
// slots 4 (q % 2) .. of each.
__device__ __forceinline__ void rt_copy_frags(uint4* dst, const uint4* __restrict__ src, int nb, int nkg, int src_nkg,
                                              int kg0) {
  const int total = nb * nkg * 64;
  for (int i = threadIdx.x; i < total; i += blockDim.x) {
    const int cb = i / (nkg * 64), kg = (i / 64) % nkg, ln = i % 64, q = ln >> 4, c = ln & 15;
    const uint2* s = reinterpret_cast<const uint2*>(src + ((size_t)cb * src_nkg + kg0 + kg) * 64);
    const uint2 lo = s[(c + 16 * (q >> 1)) * 2 + (q & 1)];
    const uint2 hi = s[(c + 16 * (2 + (q >> 1))) * 2 + (q & 1)];
    dst[i] = make_uint4(lo.x, lo.y, hi.x, hi.y);
  }
}

// acc[cb] = sum over k-groups of W[cb][kg] (LDS, [cb][kg][lane]) x X[kg].
template <int NB, int NKG>
__device__ __forceinline__ void rt_gemm(const uint4* Wl, const uint4 (&X)[NKG], floatx4 (&acc)[NB], int lane) {
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) acc[cb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kg = 0; kg < NKG; ++kg)
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) PBF16::mma(acc[cb], Wl[(cb * NKG + kg) * 64 + lane], X[kg]);
}

// Two fp32 values -> two bf16 (round to nearest even, one conversion instruction).
__device__ __forceinline__ uint32_t bf_pack(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

// Accumulator-order values -> bf16 B operands of the next product.
template <int NB>
__device__ __forceinline__ void rt_frags(const float (&v)[NB][4], uint4 (&f)[NB / 2]) {
#pragma unroll
  for (int kg = 0; kg < NB / 2; ++kg)
    f[kg] = make_uint4(bf_pack(v[2 * kg][0], v[2 * kg][1]), bf_pack(v[2 * kg][2], v[2 * kg][3]),
                       bf_pack(v[2 * kg + 1][0], v[2 * kg + 1][1]), bf_pack(v[2 * kg + 1][2], v[2 * kg + 1][3]));
}

// T-order bf16 of one k-group -> plain order.  In: lane group q holds
// columns 32 kg + 4 q .. +3 (x, y) and 32 kg + 16 + 4 q .. +3 (z, w).  Out:
// columns 32 kg + 8 q .. +7, one 16-byte row chunk.  A lane swap between the
// group pairs (0, 1) <-> (2, 3), then one between groups 0 <-> 1 and 2 <-> 3.
__device__ __forceinline__ uint4 rt_to_plain(const uint4 f) {
  const auto s0 = __builtin_amdgcn_permlane32_swap(f.x, f.z, false, false);
  const auto s1 = __builtin_amdgcn_permlane32_swap(f.y, f.w, false, false);
  const auto t0 = __builtin_amdgcn_permlane16_swap(s0[0], s0[1], false, false);
  const auto t1 = __builtin_amdgcn_permlane16_swap(s1[0], s1[1], false, false);
  return make_uint4(t0[0], t1[0], t0[1], t1[1]);
}
// Inverse of rt_to_plain (both swaps are involutions, applied in reverse).
__device__ __forceinline__ uint4 rt_from_plain(const uint4 p) {
  const auto t0 = __builtin_amdgcn_permlane16_swap(p.x, p.z, false, false);
  const auto t1 = __builtin_amdgcn_permlane16_swap(p.y, p.w, false, false);
  const auto s0 = __builtin_amdgcn_permlane32_swap(t0[0], t0[1], false, false);
  const auto s1 = __builtin_amdgcn_permlane32_swap(t1[0], t1[1], false, false);
  return make_uint4(s0[0], s1[0], s0[1], s1[1]);
}

// The values of rt_frags -> one plain-order bf16 row, 16 bytes per lane and
// k-group.  All lanes take part in the swaps; only lanes with ok store.
// A stored bf16 ReLU output row as read (plain order: lane (e, q) holds its
// row's k-slots kg * 32 + 8 q ..) -> T-order fragments, and the ReLU mask
// their signs give: bit cb * 4 + r is set where the value is positive.
// rt_load_relu reads the row as well.
template <int NKH>
__device__ __forceinline__ void rt_relu_frags(const uint4 (&raw)[NKH], uint4 (&hf)[NKH], uint32_t& mask) {
#pragma unroll
  for (int kg = 0; kg < NKH; ++kg) {
    hf[kg] = rt_from_plain(raw[kg]);
    const uint32_t w[4] = {hf[kg].x, hf[kg].y, hf[kg].z, hf[kg].w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // dword i: block 2 kg + i / 2, rows r = 2 (i % 2) .. + 1
      const int cb = 2 * kg + i / 2, r = 2 * (i % 2);
      mask |= ((w[i] & 0x7fffu) != 0u && !(w[i] & 0x8000u) ? 1u : 0u) << (cb * 4 + r);
      mask |= (((w[i] >> 16) & 0x7fffu) != 0u && !(w[i] & 0x80000000u) ? 1u : 0u) << (cb * 4 + r + 1);
    }
  }
}
// Whether the value of T-order fragments hf at accumulator position
// (cb, r) is positive: bf16 bits with the sign clear and a nonzero
// magnitude, the test rt_relu_frags makes for its mask bit cb * 4 + r.
template <int NKH>
__device__ __forceinline__ bool rt_relu_on(const uint4 (&hf)[NKH], int cb, int r) {
  const uint4 f = hf[cb / 2];
  const int i = 2 * (cb % 2) + r / 2;
  const uint32_t w = i == 0 ? f.x : i == 1 ? f.y : i == 2 ? f.z : f.w;
  return (int32_t)(r % 2 ? (w & 0xffff0000u) : (w << 16)) > 0;
}
template <int NKH>
__device__ __forceinline__ void rt_load_relu(const uint16_t* __restrict__ hp, int q, uint4 (&hf)[NKH],
                                             uint32_t& mask) {
  uint4 raw[NKH];
#pragma unroll
  for (int kg = 0; kg < NKH; ++kg) raw[kg] = *reinterpret_cast<const uint4*>(hp + kg * 32 + q * 8);
  rt_relu_frags<NKH>(raw, hf, mask);
}

template <int NKH>
__device__ __forceinline__ void rt_store_frags(uint16_t* __restrict__ row, int q, const uint4 (&f)[NKH], bool ok) {
  uint4 p[NKH];
#pragma unroll
  for (int kg = 0; kg < NKH; ++kg) p[kg] = rt_to_plain(f[kg]);
  if (ok) {
#pragma unroll
    for (int kg = 0; kg < NKH; ++kg) *reinterpret_cast<uint4*>(row + kg * 32 + q * 8) = p[kg];
  }
}

// bf16 plain-order 16-byte chunk (8 columns) -> its T-order values: cb 2 kg
// gets .x/.y, cb 2 kg + 1 gets .z/.w (columns 4 q + r of each block).
__device__ __forceinline__ void rw_unpack(const uint4 p, float (&lo)[4], float (&hi)[4]) {
  const uint4 t = rt_from_plain(p);
  lo[0] = __uint_as_float(t.x << 16);
  lo[1] = __uint_as_float(t.x & 0xffff0000u);
  lo[2] = __uint_as_float(t.y << 16);
  lo[3] = __uint_as_float(t.y & 0xffff0000u);
  hi[0] = __uint_as_float(t.z << 16);
  hi[1] = __uint_as_float(t.z & 0xffff0000u);
  hi[2] = __uint_as_float(t.w << 16);
  hi[3] = __uint_as_float(t.w & 0xffff0000u);
}

}  // namespace mgn
