// fp32 T-form kernels (gfx950): the edge half of a block with its first
// Linear split by rows, and the node projections that go with it.
//
// The first Linear acts on [e | v_s | v_r]; its sender and receiver column
// blocks are applied once per node (node_proj_f32_kernel), so per edge
// z_1 = W_e e + P_s[s] + P_r[r] takes L x L products instead of 3L x L.  All
// products are computed transposed (Y^T = W X^T): a weight fragment is the
// MFMA A operand, a 16-row tile of activations the B operand.  With
// v_mfma_f32_16x16x4_f32 lane (e, q) supplies one k value of row e per
// instruction; taking the four values 16 kg + 4 q + r (r = 0..3) of a 16-byte
// chunk in four instructions makes one layout serve everywhere: the packed
// weights (lane (i, q): W[16 cb + i][16 kg + 4 q ..]), rows in memory in plain
// column order (16 bytes per lane and 16-column block), and the accumulators,
// which hold columns 16 cb + 4 q + r of row e and so are the next product's B
// operand as they stand.  One wave works alone on 16-edge tiles of its own
// receiver-aligned range (a very large receiver: of its share of a workgroup's,
// tf_range); the per-edge weights sit in LDS.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "tform.h"

namespace mgn {

namespace {

// Waves per workgroup: two per SIMD.  The fp32 MFMA and the vector ALU take
// turns (counters at l = 128: matrix pipe busy 70 % of the SIMD cycles, vector
// instructions 20 % forward and 24 % backward, which add up to 90 and 94 %), so
// more waves hide nothing more: at l = 128 they spill (12 waves: forward 1.03 ms,
// backward 1.84 ms on 1.35M edges against 0.84 and 1.22), at l = 64 they cut the
// ranges finer (16 waves: backward 113 us on 270,000 edges against 101).
constexpr int TF_NWV = 8, TF_NTH = 64 * TF_NWV;

// Fragment slot of lane (i, q) in a packed 16 x 16 weight block held in LDS:
// the q-th run of 16 slots, its order XORed with q.  A 16-byte read by all
// lanes (product with W) is a permutation of each 256-byte run; a 4-byte read
// of the transposed element order (product with W^T, tf_gemm_t) then touches
// every bank once.
__device__ __forceinline__ int tf_slot(int i, int q) { return 16 * q + (i ^ q); }

// Copies NB 16-column blocks x NK k-groups of packed fragments (source block
// stride SRC k-groups, first k-group kg0) into LDS in tf_slot order, NTH
// threads, the loads of up to eight fragments per thread in flight.
template <int NB, int SRC, int NTH, int NK = NB>
__device__ __forceinline__ void tf_copy_frags(void* dst, const uint4* __restrict__ src, int kg0) {
  constexpr int TOTAL = NB * NK * 64, IT = (TOTAL + NTH - 1) / NTH, U = IT < 8 ? IT : 8;
  uint4* d = reinterpret_cast<uint4*>(dst);
  for (int j0 = 0; j0 < IT; j0 += U) {
    uint4 v[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int i = threadIdx.x + (j0 + j) * NTH, blk = i >> 6;
      if (TOTAL % (NTH * U) == 0 || i < TOTAL) v[j] = src[((blk / NK) * SRC + kg0 + blk % NK) * 64 + (i & 63)];
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int i = threadIdx.x + (j0 + j) * NTH;
      if (TOTAL % (NTH * U) == 0 || i < TOTAL) d[(i & ~63) + tf_slot(i & 15, (i >> 4) & 3)] = v[j];
    }
  }
}

// acc[cb] = sum over k-groups of W[cb][kg] (LDS) x X[kg].
template <int NB, int NK = NB>
__device__ __forceinline__ void tf_gemm(const float4* Wl, const float4 (&X)[NK], floatx4 (&acc)[NB], int slot) {
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) acc[cb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kg = 0; kg < NK; ++kg) {
    float4 w[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) w[cb] = Wl[(cb * NK + kg) * 64 + slot];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[cb].x, X[kg].x, acc[cb], 0, 0, 0);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[cb].y, X[kg].y, acc[cb], 0, 0, 0);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[cb].z, X[kg].z, acc[cb], 0, 0, 0);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[cb].w, X[kg].w, acc[cb], 0, 0, 0);
  }
}

// The same from the packed weights in memory (SRC k-groups per block, first
// kg0): the same sums in the same order.
template <int NB, int SRC>
__device__ __forceinline__ void tf_gemm_mem(const uint4* __restrict__ W, int kg0, const float4 (&X)[NB],
                                            floatx4 (&acc)[NB], int lane) {
  const float4* Wl = reinterpret_cast<const float4*>(W) + kg0 * 64 + lane;
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) acc[cb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kg = 0; kg < NB; ++kg) {
    float4 w[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) w[cb] = Wl[(cb * SRC + kg) * 64];
    const float x[4] = {X[kg].x, X[kg].y, X[kg].z, X[kg].w};
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        const float wr[4] = {w[cb].x, w[cb].y, w[cb].z, w[cb].w};
        acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr[r], x[r], acc[cb], 0, 0, 0);
      }
  }
}

// The same with W^T, from the same LDS copy of W: output block cb takes
// W[16 kg + 4 q + r][16 cb + i], element i % 4 of the slot of lane
// (4 q + r, i / 4) in block (kg, cb).  tb[r] is that element's index in a block.
__device__ __forceinline__ void tf_t_index(int i, int q, int (&tb)[4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) tb[r] = tf_slot(4 * q + r, i >> 2) * 4 + (i & 3);
}
template <int NB>
__device__ __forceinline__ void tf_gemm_t(const float* Wl, const float4 (&X)[NB], floatx4 (&acc)[NB],
                                          const int (&tb)[4]) {
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) acc[cb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kg = 0; kg < NB; ++kg) {
    const float x[4] = {X[kg].x, X[kg].y, X[kg].z, X[kg].w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float w[NB];
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) w[cb] = Wl[(kg * NB + cb) * 256 + tb[r]];
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[cb], x[r], acc[cb], 0, 0, 0);
    }
  }
}

// A tile's metadata as rt_meta_load, rows past the range end repeating the
// range's last edge (their results are never used).  past: what follows the
// range's last edge.
__device__ __forceinline__ RsMetaRaw tf_meta_load(const int32_t* __restrict__ erecv, const int32_t* __restrict__ send,
                                                  int64_t sb, int64_t e1, int32_t past) {
  const int64_t e = sb + (threadIdx.x & 15);
  const int64_t i = e < e1 ? e : e1 - 1;
  RsMetaRaw w;
  w.r = erecv[i];
  w.s = send[i];
  w.rn = e + 1 < e1 ? erecv[e + 1] : past;
  return w;
}
__device__ __forceinline__ RsMeta tf_meta_make(const RsMetaRaw& w, int n) {
  RsMeta mt{w.r, w.s, 0};
  mt.last = __ballot((int)(threadIdx.x & 15) < n && w.rn != w.r);
  return mt;
}

// A wave's edges [E0, E1).  SPLIT, for graphs with very large receivers: the
// workgroup takes whole receivers, its waves an even share of the 16-edge
// tiles each, so a receiver's edges may go on from one wave to the next.
// Otherwise each of the nact working waves takes whole receivers.
struct TfRange {
  int64_t E0, E1;
  int32_t past;     // receiver id after the last edge that does not end a sum: the last edge's own, if it goes on; else -1
  bool open;        // the first receiver's edges began in an earlier wave, and their end has not been reached
};
template <bool SPLIT>
__device__ __forceinline__ TfRange tf_range(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ erecv,
                                            int64_t e_lo, int64_t E, int nact) {
  const int wave = wave_id();
  TfRange r{0, 0, -1, false};
  if constexpr (SPLIT) {
    int64_t B0, B1;
    rs_range_e(row_ptr, erecv, e_lo, E, 1, 0, B0, B1);
    const int64_t T = (B1 - B0 + 15) / 16;
    r.E0 = B0 + 16 * (T * wave / TF_NWV);
    r.E1 = wave + 1 == TF_NWV ? B1 : B0 + 16 * (T * (wave + 1) / TF_NWV);
    if (r.E0 < r.E1) {
      const int32_t last = erecv[r.E1 - 1];
      if (r.E1 < B1 && erecv[r.E1] == last) r.past = last;
      r.open = r.E0 > B0 && erecv[r.E0 - 1] == erecv[r.E0];
    }
    r.past = __builtin_amdgcn_readfirstlane(r.past);
    r.open = __builtin_amdgcn_readfirstlane(r.open) != 0;
  } else if (wave < nact) {
    rs_range_e(row_ptr, erecv, e_lo, E, nact, wave, r.E0, r.E1);
  }
  return r;
}

// Ordered receiver sums of a tile's values v (columns 16 cb + 4 q + r of row
// e): 64 columns at a time through the wave's 2 KiB scratch, 32 of them per
// half (lanes 0..31, then 32..63), so that two L x L weight matrices leave
// room for eight waves' scratch at L = 128.  Each lane carries the running sum
// of column ln + 64 j; a segment's total is stored at its last row.  SPLIT: the
// end of a segment that an earlier wave began (open) goes to head instead.
template <int L, bool SPLIT>
__device__ __forceinline__ void tf_segment_sums(const float4 (&v)[L / 16], float* scr, const RsMeta& mt, int n, int ln,
                                                float (&run)[L / 64], float* dst, float (&head)[L / 64], bool& open) {
  const int e = ln & 15, q = ln >> 4;
  const int first = SPLIT && open && mt.last ? __builtin_ctzll(mt.last) : -1;
#pragma unroll
  for (int j = 0; j < L / 64; ++j) {
    float x[16];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
        *reinterpret_cast<float4*>(scr + rs_sw32<32>(e, c * 16 + q * 4)) = v[4 * j + 2 * half + c];
      if ((ln >> 5) == half) {
#pragma unroll
        for (int row = 0; row < 16; ++row) x[row] = scr[rs_sw32<32>(row, ln & 31)];
      }
    }
#pragma unroll
    for (int row = 0; row < 16; ++row) {
      if (row < n) {
        run[j] += x[row];
        if ((mt.last >> row) & 1ull) {
          if (SPLIT && row == first) head[j] = run[j];
          else dst[(int64_t)__builtin_amdgcn_readlane(mt.r, row) * L + ln + 64 * j] = run[j];
          run[j] = 0.f;
        }
      }
    }
  }
  if (SPLIT && first >= 0) open = false;
}

// SPLIT, after a workgroup's last tile: the sums of the receivers whose edges
// went on from one wave to the next, in wave order, by the wave in which they
// began.  run: what the wave's last, unended segment came to.  lds:
// 2 * TF_NWV * L floats and TF_NWV words, free to overwrite.
template <int L>
__device__ __forceinline__ void tf_join(const TfRange& r, bool open, const float (&head)[L / 64],
                                        const float (&run)[L / 64], unsigned char* lds, float* dst) {
  const int wave = wave_id(), lane = threadIdx.x & 63;
  float* H = reinterpret_cast<float*>(lds);
  float* T = H + TF_NWV * L;
  int* on = reinterpret_cast<int*>(T + TF_NWV * L);
  // no segment ended in the wave (or it had no edges): its run is the middle of a sum
  const bool through = open || r.E0 >= r.E1;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < L / 64; ++j) {
    H[wave * L + lane + 64 * j] = head[j];
    T[wave * L + lane + 64 * j] = run[j];
  }
  if (lane == 0) on[wave] = through;
  __syncthreads();
  if (through || r.past < 0) return;
  // the receiver ends in a later wave of the workgroup, so the loop meets its head
#pragma unroll
  for (int j = 0; j < L / 64; ++j) {
    float s = run[j];
    for (int u = wave + 1; u < TF_NWV; ++u) {
      s += (on[u] ? T : H)[u * L + lane + 64 * j];
      if (!on[u]) break;
    }
    dst[(int64_t)r.past * L + lane + 64 * j] = s;
  }
}

template <int NB>
__device__ __forceinline__ float tf_lane_sum(const float4 (&v)[NB]) {
  float4 t = v[0];
#pragma unroll
  for (int cb = 1; cb < NB; ++cb) {
    t.x += v[cb].x;
    t.y += v[cb].y;
    t.z += v[cb].z;
    t.w += v[cb].w;
  }
  return (t.x + t.y) + (t.z + t.w);
}

// 1 / std of a row whose lane values are y, given its mean.
template <int NB, int L>
__device__ __forceinline__ float tf_rstd(const float4 (&y)[NB], float mu, float eps) {
  float4 d[NB];
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) {
    const float a = y[cb].x - mu, b = y[cb].y - mu, c = y[cb].z - mu, e = y[cb].w - mu;
    d[cb] = make_float4(a * a, b * b, c * c, e * e);
  }
  return 1.0f / sqrtf(rt_sum4(tf_lane_sum<NB>(d)) / L + eps);
}

__device__ __forceinline__ float4 tf_add(const floatx4& a, const float4& b) {
  return make_float4(a[0] + b.x, a[1] + b.y, a[2] + b.z, a[3] + b.w);
}
__device__ __forceinline__ float4 tf_relu(const float4& v) {
  return make_float4(v.x > 0.f ? v.x : 0.f, v.y > 0.f ? v.y : 0.f, v.z > 0.f ? v.z : 0.f, v.w > 0.f ? v.w : 0.f);
}
template <int NB>
__device__ __forceinline__ void tf_load(const float* __restrict__ p, int q, float4 (&v)[NB]) {
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) v[cb] = rt_ld4(p, cb, q);
}
template <int NB>
__device__ __forceinline__ void tf_store(float* p, int q, const float4 (&v)[NB]) {
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) *reinterpret_cast<float4*>(p + cb * 16 + q * 4) = v[cb];
}

// ------------------------------------------------------------ edge forward ---
template <int L, int D>
struct TfFwdLay {
  static constexpr int NB = L / 16, W = L * L * 4;
  static constexpr int OFF_VEC = D * W;                 // last bias, gamma, beta[, hidden bias]
  static constexpr int OFF_SCR = OFF_VEC + (D == 3 ? 4 : 3) * L * 4;
  static constexpr int SCR = 16 * 32 * 4;
  static constexpr int END = OFF_SCR + TF_NWV * SCR;
  static_assert(END <= 160 * 1024, "LDS");
};

// Forward of one block's edge half.  Bound by the matrix pipe: 4 L^2 flops per
// edge at 157 TFLOP/s (L = 128, 1.35M edges: 0.56 ms; measured 0.84 ms with
// the vector instructions between the products, 1.99 ms for the streaming
// kernel, which applies the whole 3L x L first Linear per edge).  P_r may share its rows with a.agg: a
// receiver's row is read with its edges' tiles and its sum stored after them,
// by the same wave.  HS: there are no P_s rows of the halo (ps_halo null, a
// workspace without room for them); a tile with halo senders forms its own, the
// same bits, with W_s from L2 (270,000 owned and 30,000 halo nodes, 3.7M edges,
// two blocks at l = 128: 9.25 ms against 6.55 with the rows).
template <int L, int D, bool SPLIT, bool HS>
__global__ __launch_bounds__(TF_NTH) void edge_fwd_f32_kernel(EdgeFwdArgs a, int64_t n_edges, int nact) {
  using Lay = TfFwdLay<L, D>;
  constexpr int NB = Lay::NB;
  extern __shared__ __align__(16) unsigned char lds[];
  float4* W1 = reinterpret_cast<float4*>(lds);
  float4* WH = reinterpret_cast<float4*>(lds + Lay::W);
  float4* WL = reinterpret_cast<float4*>(lds + (D - 1) * Lay::W);
  float* vbl = reinterpret_cast<float*>(lds + Lay::OFF_VEC);
  float* vg = vbl + L;
  float* vbt = vbl + 2 * L;
  float* vbh = vbl + 3 * L;
  const int wave = wave_id(), lane = threadIdx.x & 63;
  float* scr = reinterpret_cast<float*>(lds + Lay::OFF_SCR + wave * Lay::SCR);
  const RsEmpty empty = rs_empty_load(a.row_ptr, 0, a.n_owned);
  const TfRange rg = tf_range<SPLIT>(a.row_ptr, a.erecv, 0, n_edges, nact);
  const int64_t E0 = rg.E0, E1 = rg.E1;
  bool open = rg.open;
  tf_copy_frags<NB, 3 * NB, TF_NTH>(W1, a.mlp.lin[0].wf, 0);
  if constexpr (D == 3) tf_copy_frags<NB, NB, TF_NTH>(WH, a.mlp.lin[1].wf, 0);
  tf_copy_frags<NB, NB, TF_NTH>(WL, a.mlp.lin[D - 1].wf, 0);
  rt_copy_vec(vbl, a.mlp.lin[D - 1].b, L);
  rt_copy_vec(vg, a.mlp.gamma, L);
  rt_copy_vec(vbt, a.mlp.beta, L);
  if constexpr (D == 3) rt_copy_vec(vbh, a.mlp.lin[1].b, L);
  __syncthreads();
  rs_zero_empty(empty, a.row_ptr, a.agg, L);
  if (!SPLIT && E0 >= E1) return;
  const float* Ein = reinterpret_cast<const float*>(a.Ein);
  float* Eout = reinterpret_cast<float*>(a.Eout);
  float* hid = reinterpret_cast<float*>(a.hid_out);
  float run[L / 64] = {}, head[L / 64] = {};
  // e^k rows of a tile are loaded while the tile before runs its last
  // product, the P rows at the tile's start: they are added after its first
  // product, which hides them.  So no product waits for a load, nor, through
  // the in-order memory counter, for the stores issued before it.  Past the
  // range's end its last edge is read again.
  float4 ef[NB];
  auto load_e = [&](int64_t sb, int ln) {
    tf_load<NB>(Ein + (sb + (ln & 15) < E1 ? sb + (ln & 15) : E1 - 1) * L, ln >> 4, ef);
  };
  RsMetaRaw cur{};
  if (!SPLIT || E0 < E1) {
    cur = tf_meta_load(a.erecv, a.send, E0, E1, rg.past);
    load_e(E0, lane);
  }
  for (int64_t sb = E0; sb < E1; sb += 16) {
    int ln = lane;  // an opaque copy: lane-dependent addresses are formed per tile, not kept in registers
    asm volatile("" : "+v"(ln));
    const int e = ln & 15, q = ln >> 4, slot = tf_slot(e, q);
    const int n = (int)(E1 - sb < 16 ? E1 - sb : 16);
    const bool ok = e < n;
    const RsMeta mt = tf_meta_make(cur, n);
    float4 ps[NB], pr[NB];
    const bool far = mt.s >= a.n_owned;
    const int64_t hrow = ((int64_t)mt.s - a.n_owned) * L;
    // HS: a halo sender's latents in the place of its P_s (other rows of the
    // product are not used)
    tf_load<NB>(far ? (HS ? a.H : a.ps_halo) + hrow : a.ps + (int64_t)mt.s * L, q, ps);
    tf_load<NB>(a.pr + (int64_t)mt.r * L, q, pr);
    cur = tf_meta_load(a.erecv, a.send, sb + 16, E1, rg.past);
    __builtin_amdgcn_sched_barrier(0);
    floatx4 acc[NB];
    if constexpr (HS) {
      if (__ballot(far)) {
        tf_gemm_mem<NB, 3 * NB>(a.mlp.lin[0].wf, NB, ps, acc, ln);
#pragma unroll
        for (int cb = 0; cb < NB; ++cb)
          if (far) ps[cb] = make_float4(acc[cb][0], acc[cb][1], acc[cb][2], acc[cb][3]);
      }
    }
    tf_gemm<NB>(W1, ef, acc, slot);
    float4 h[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      const float4 z = tf_add(acc[cb], ps[cb]);
      h[cb] = tf_relu(make_float4(z.x + pr[cb].x, z.y + pr[cb].y, z.z + pr[cb].z, z.w + pr[cb].w));
    }
    if (hid && ok) tf_store<NB>(hid + (sb + e) * L, q, h);
    if constexpr (D == 3) {
      tf_gemm<NB>(WH, h, acc, slot);
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) h[cb] = tf_relu(tf_add(acc[cb], rt_ld4(vbh, cb, q)));
    }
    float4 ek[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) ek[cb] = ef[cb];
    load_e(sb + 16, ln);
    __builtin_amdgcn_sched_barrier(0);
    tf_gemm<NB>(WL, h, acc, slot);
    float4 y[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) y[cb] = tf_add(acc[cb], rt_ld4(vbl, cb, q));
    const float mu = rt_sum4(tf_lane_sum<NB>(y)) / L;
    const float rs = tf_rstd<NB, L>(y, mu, a.eps);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {  // y becomes m
      const float4 g = rt_ld4(vg, cb, q), bt = rt_ld4(vbt, cb, q);
      y[cb].x = g.x * ((y[cb].x - mu) * rs) + bt.x;
      y[cb].y = g.y * ((y[cb].y - mu) * rs) + bt.y;
      y[cb].z = g.z * ((y[cb].z - mu) * rs) + bt.z;
      y[cb].w = g.w * ((y[cb].w - mu) * rs) + bt.w;
    }
    if (Eout && ok) {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb)
        ek[cb] = make_float4(ek[cb].x + y[cb].x, ek[cb].y + y[cb].y, ek[cb].z + y[cb].z, ek[cb].w + y[cb].w);
      tf_store<NB>(Eout + (sb + e) * L, q, ek);
    }
    tf_segment_sums<L, SPLIT>(y, scr, mt, n, ln, run, a.agg, head, open);
  }
  if constexpr (SPLIT) tf_join<L>(rg, open, head, run, lds, a.agg);
}

// ----------------------------------------------------------- edge backward ---
template <int L, int D>
struct TfBwdLay {
  static constexpr int NB = L / 16, W = L * L * 4;
  // the last [and hidden] Linear once each (product and transposed product
  // read the same copy), then W_e in the backward packing
  static constexpr int OFF_WH = W, OFF_W1 = (D - 1) * W;
  static constexpr int OFF_VEC = D * W;                 // last bias, gamma[, hidden bias]
  static constexpr int OFF_SCR = OFF_VEC + (D == 3 ? 3 : 2) * L * 4;
  static constexpr int SCR = 16 * 32 * 4;
  static constexpr int END = OFF_SCR + TF_NWV * SCR;
  static constexpr int NVEC = (D + 2) * L;              // bias / gamma / beta partials per wave
  static_assert(END <= 160 * 1024 && TF_NWV * NVEC * 4 <= OFF_SCR, "LDS");
};

// Backward of one block's edge half, bound by the matrix pipe as the forward
// (6 L^2 flops per edge; L = 128, 1.35M edges: floor 0.84 ms, measured 1.22 ms,
// the streaming kernel 3.15 ms with every weight fragment read from L2 for
// each tile).  It starts from the forward's h_1 (a.hid_in): the
// layers after the first recomputed, LayerNorm backward, the data gradients
// down to dz_0, de^k = de^{k+1} + dz_0 W_e, receiver sums of dz_0 over the
// consumed dagg rows, per-workgroup bias / LayerNorm partials.
template <int L, int D, bool SPLIT>
__global__ __launch_bounds__(TF_NTH) void edge_bwd_f32_kernel(EdgeBwdArgs a, int64_t n_edges, int nact) {
  using Lay = TfBwdLay<L, D>;
  constexpr int NB = Lay::NB, NV = 4 * NB, NR = NV / 16;
  extern __shared__ __align__(16) unsigned char lds[];
  float* WL = reinterpret_cast<float*>(lds);
  float* WH = reinterpret_cast<float*>(lds + Lay::OFF_WH);
  float4* W1 = reinterpret_cast<float4*>(lds + Lay::OFF_W1);
  float* vbl = reinterpret_cast<float*>(lds + Lay::OFF_VEC);
  float* vg = vbl + L;
  float* vbh = vbl + 2 * L;
  const int wave = wave_id(), lane = threadIdx.x & 63;
  float* scr = reinterpret_cast<float*>(lds + Lay::OFF_SCR + wave * Lay::SCR);
  const RsEmpty empty = rs_empty_load(a.row_ptr, a.r_lo, a.r_hi);
  const TfRange rg = tf_range<SPLIT>(a.row_ptr, a.erecv, a.e_base, n_edges, nact);
  const int64_t E0 = rg.E0, E1 = rg.E1;
  bool open = rg.open;
  tf_copy_frags<NB, NB, TF_NTH>(WL, a.mlp.lin[D - 1].wf, 0);
  if constexpr (D == 3) tf_copy_frags<NB, NB, TF_NTH>(WH, a.mlp.lin[1].wf, 0);
  tf_copy_frags<NB, NB, TF_NTH>(W1, a.mlp.lin[0].wb, 0);  // e block: the first NB column blocks
  rt_copy_vec(vbl, a.mlp.lin[D - 1].b, L);
  rt_copy_vec(vg, a.mlp.gamma, L);
  if constexpr (D == 3) rt_copy_vec(vbh, a.mlp.lin[1].b, L);
  __syncthreads();
  rs_zero_empty(empty, a.row_ptr, a.dagg, L);
  // column totals of the bias / LayerNorm gradients (rt_col_totals' share of
  // each lane): gamma, beta, last bias, hidden biases
  constexpr int NQ = 2 + D;
  float qacc[NQ][NR];
#pragma unroll
  for (int k = 0; k < NQ; ++k)
#pragma unroll
    for (int t = 0; t < NR; ++t) qacc[k][t] = 0.f;
  auto coltot = [&](const float4 (&x)[NB], int k, int e) {
    float f[NV];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      f[4 * cb] = x[cb].x;
      f[4 * cb + 1] = x[cb].y;
      f[4 * cb + 2] = x[cb].z;
      f[4 * cb + 3] = x[cb].w;
    }
    rt_col_totals<NV>(f, e);
#pragma unroll
    for (int t = 0; t < NR; ++t) qacc[k][t] += f[t];
  };
  const float* hin = reinterpret_cast<const float*>(a.hid_in);
  const float* dnx = reinterpret_cast<const float*>(a.de_next);
  float* deo = reinterpret_cast<float*>(a.de_out);
  float run[L / 64] = {}, head[L / 64] = {};
  // h_1 rows of a tile are loaded while the tile before runs its last
  // product, de^{k+1} (the last block has none: its loads re-read the h_1 rows
  // and are replaced by zeros) and dagg at the tile's start, used after its
  // first product (cf. edge_fwd_f32_kernel)
  float4 h1[NB];
  auto load_h1 = [&](int64_t sb, int ln) {
    tf_load<NB>(hin + (sb + (ln & 15) < E1 ? sb + (ln & 15) : E1 - 1) * L, ln >> 4, h1);
  };
  RsMetaRaw cur{};
  if (E0 < E1) {
    cur = tf_meta_load(a.erecv, a.send, E0, E1, rg.past);
    load_h1(E0, lane);
  }
  for (int64_t sb = E0; sb < E1; sb += 16) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int e = ln & 15, q = ln >> 4, slot = tf_slot(e, q);
    const int n = (int)(E1 - sb < 16 ? E1 - sb : 16);
    const bool ok = e < n;
    const RsMeta mt = tf_meta_make(cur, n);
    const int64_t srow = (sb - a.e_base + e) * L;
    float4 de[NB], dm[NB];
    tf_load<NB>((dnx ? dnx : hin) + (sb + (ok ? e : n - 1)) * L, q, de);
    tf_load<NB>(a.dagg + (int64_t)mt.r * L, q, dm);
    cur = tf_meta_load(a.erecv, a.send, sb + 16, E1, rg.past);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t mask[2] = {0u, 0u};  // ReLU derivative of the hidden layers, bit cb * 4 + r
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      mask[0] |= (h1[cb].x > 0.f ? 1u : 0u) << (4 * cb);
      mask[0] |= (h1[cb].y > 0.f ? 1u : 0u) << (4 * cb + 1);
      mask[0] |= (h1[cb].z > 0.f ? 1u : 0u) << (4 * cb + 2);
      mask[0] |= (h1[cb].w > 0.f ? 1u : 0u) << (4 * cb + 3);
    }
    floatx4 acc[NB];
    if constexpr (D == 3) {
      tf_gemm<NB>(reinterpret_cast<const float4*>(WH), h1, acc, slot);
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        h1[cb] = tf_relu(tf_add(acc[cb], rt_ld4(vbh, cb, q)));
        mask[1] |= (h1[cb].x > 0.f ? 1u : 0u) << (4 * cb);
        mask[1] |= (h1[cb].y > 0.f ? 1u : 0u) << (4 * cb + 1);
        mask[1] |= (h1[cb].z > 0.f ? 1u : 0u) << (4 * cb + 2);
        mask[1] |= (h1[cb].w > 0.f ? 1u : 0u) << (4 * cb + 3);
      }
      if (ok) tf_store<NB>(reinterpret_cast<float*>(a.hid[1]) + srow, q, h1);
    }
    tf_gemm<NB>(reinterpret_cast<const float4*>(WL), h1, acc, slot);
    float4 y[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) y[cb] = tf_add(acc[cb], rt_ld4(vbl, cb, q));
    const bool has_de = dnx != nullptr;
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      if (!has_de) de[cb] = make_float4(0.f, 0.f, 0.f, 0.f);
      dm[cb].x = ok ? dm[cb].x + de[cb].x : 0.f;
      dm[cb].y = ok ? dm[cb].y + de[cb].y : 0.f;
      dm[cb].z = ok ? dm[cb].z + de[cb].z : 0.f;
      dm[cb].w = ok ? dm[cb].w + de[cb].w : 0.f;
    }
    const float mu = rt_sum4(tf_lane_sum<NB>(y)) / L;
    const float rs = tf_rstd<NB, L>(y, mu, a.eps);
    // LayerNorm backward: dy = rstd (dm g - mean(dm g) - xhat mean(dm g xhat))
    float t1, t2;
    {
      float4 d1[NB], d2[NB];
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        const float4 g = rt_ld4(vg, cb, q);
        y[cb] = make_float4((y[cb].x - mu) * rs, (y[cb].y - mu) * rs, (y[cb].z - mu) * rs, (y[cb].w - mu) * rs);
        d1[cb] = make_float4(dm[cb].x * g.x, dm[cb].y * g.y, dm[cb].z * g.z, dm[cb].w * g.w);
        d2[cb] = make_float4(d1[cb].x * y[cb].x, d1[cb].y * y[cb].y, d1[cb].z * y[cb].z, d1[cb].w * y[cb].w);
      }
      t1 = rt_sum4(tf_lane_sum<NB>(d1)) / L;
      t2 = rt_sum4(tf_lane_sum<NB>(d2)) / L;
    }
    coltot(dm, 1, e);
    float4 v[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      const float4 g = rt_ld4(vg, cb, q);
      v[cb].x = rs * (dm[cb].x * g.x - t1 - y[cb].x * t2);
      v[cb].y = rs * (dm[cb].y * g.y - t1 - y[cb].y * t2);
      v[cb].z = rs * (dm[cb].z * g.z - t1 - y[cb].z * t2);
      v[cb].w = rs * (dm[cb].w * g.w - t1 - y[cb].w * t2);
      // gamma's column terms
      dm[cb] = make_float4(dm[cb].x * y[cb].x, dm[cb].y * y[cb].y, dm[cb].z * y[cb].z, dm[cb].w * y[cb].w);
    }
    if (ok) tf_store<NB>(reinterpret_cast<float*>(a.delta[D - 1]) + srow, q, v);
    coltot(dm, 0, e);
    coltot(v, 2, e);
    // hidden layers: dz_{j-1} = (dz_j W_j) * [z_{j-1} > 0]
    int tb[4];
    tf_t_index(e, q, tb);
#pragma unroll
    for (int j = D - 1; j >= 1; --j) {
      tf_gemm_t<NB>(j == D - 1 ? WL : WH, v, acc, tb);
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        const uint32_t mk = mask[j - 1] >> (4 * cb);
        v[cb] = make_float4(mk & 1u ? acc[cb][0] : 0.f, mk & 2u ? acc[cb][1] : 0.f, mk & 4u ? acc[cb][2] : 0.f,
                            mk & 8u ? acc[cb][3] : 0.f);
      }
      if (ok) tf_store<NB>(reinterpret_cast<float*>(a.delta[j - 1]) + srow, q, v);
      coltot(v, 2 + j, e);
    }
    load_h1(sb + 16, ln);
    __builtin_amdgcn_sched_barrier(0);
    // edge-stream gradient: de^k = de^{k+1} + dz_0 W_1[:, e-block]
    tf_gemm<NB>(W1, v, acc, slot);
    if (ok) {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) de[cb] = tf_add(acc[cb], de[cb]);
      tf_store<NB>(deo + (sb + e) * L, q, de);
    }
    tf_segment_sums<L, SPLIT>(v, scr, mt, n, ln, run, a.dagg, head, open);
  }
  if constexpr (SPLIT) tf_join<L>(rg, open, head, run, lds, a.dagg);
  // column partials: lane (e, q)'s totals are columns 16 cb + 4 q + r for
  // index e * NR + t = 4 cb + r; then the waves in order through LDS (the
  // weight area is free now)
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds);
  {
    float* rw = red + wave * Lay::NVEC;
#pragma unroll
    for (int t = 0; t < NR; ++t) {
      const int i = (lane & 15) * NR + t;
      const int col = (i >> 2) * 16 + (lane >> 4) * 4 + (i & 3);
#pragma unroll
      for (int h = 0; h < D - 1; ++h) rw[h * L + col] = qacc[3 + h][t];
      rw[(D - 1) * L + col] = qacc[2][t];
      rw[D * L + col] = qacc[0][t];
      rw[(D + 1) * L + col] = qacc[1][t];
    }
  }
  __syncthreads();
  float* vp = a.vpart + (int64_t)blockIdx.x * a.nvec;
  for (int i = threadIdx.x; i < Lay::NVEC; i += TF_NTH) {
    float t = 0.f;
    for (int w = 0; w < TF_NWV; ++w) t += red[w * Lay::NVEC + i];
    vp[i] = t;
  }
}

// --------------------------------------------------------- node projections ---
// P_s[n] = W_s v_n for the local nodes (owned rows to ps, halo rows to
// ps_halo) and P_r[n] = W_r v_n + b_1 for the owned ones.  Each workgroup
// takes one side, so two share a CU's LDS.
template <int L>
__global__ __launch_bounds__(TF_NTH) void node_proj_f32_kernel(const float* V, const float* H, int64_t n_owned,
                                                               int64_t n_halo, Lin w1, float* ps, float* ps_halo,
                                                               float* pr) {
  constexpr int NB = L / 16;
  extern __shared__ __align__(16) unsigned char lds[];
  float4* W = reinterpret_cast<float4*>(lds);
  const int side = (blockIdx.x >> 3) & 1;
  tf_copy_frags<NB, 3 * NB, TF_NTH>(W, w1.wf, (1 + side) * NB);
  __syncthreads();
  const int wave = wave_id(), lane = threadIdx.x & 63;
  const int64_t to = (n_owned + 15) / 16, nt = side ? to : to + (n_halo + 15) / 16;
  const int64_t nblk = gridDim.x >> 1, blk = (blockIdx.x & 7) + 8 * (blockIdx.x >> 4);
  for (int64_t t = blk + nblk * wave; t < nt; t += nblk * TF_NWV) {
    int ln = lane;  // opaque: the weight fragments are read per tile, not kept in registers
    asm volatile("" : "+v"(ln));
    const int e = ln & 15, q = ln >> 4, slot = tf_slot(e, q);
    const bool halo = t >= to;
    const int64_t row0 = (halo ? t - to : t) * 16, rows = halo ? n_halo : n_owned;
    const int64_t row = row0 + e;
    const bool ok = row < rows;
    float4 x[NB];
    tf_load<NB>((halo ? H : V) + (ok ? row : row0) * L, q, x);
    floatx4 acc[NB];
    tf_gemm<NB>(W, x, acc, slot);
    if (ok) {
      float* o = (side ? pr : halo ? ps_halo : ps) + row * L;
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        float4 v = make_float4(acc[cb][0], acc[cb][1], acc[cb][2], acc[cb][3]);
        if (side) v = tf_add(acc[cb], rt_ld4(w1.b, cb, q));
        *reinterpret_cast<float4*>(o + cb * 16 + q * 4) = v;
      }
    }
  }
}

// --------------------------------------------------------------- row MLPs ---
// Encoders and the node half of a block.  Their backward has three phases:
//   A  the first Linear's ReLU output h_1 (from the features, or [v | agg]);
//   B  the layers after it recomputed, LayerNorm backward, the data gradients
//      down to dz_0;
//   C  (node half) dv = dm + dz_0 W_1[:, v-block], dagg = dz_0 W_1[:, agg-block].
// Phases share a kernel when their weights fit the LDS together (L = 64, and
// the encoders); the node half at L = 128 (128, 64 and 128 KiB) runs one launch
// per phase, and what passes between them (h_1, dz_0) is stored for the weight
// gradients anyway.  NKF: k-groups of an encoder's features (one: at
// most 16).
template <int L, int D, int KIND, int NKF, bool A, bool B, bool C>
struct TfRowsLay {
  static constexpr int NB = L / 16, W = L * L * 4;
  static constexpr bool NODE = KIND == NODE_BLOCK;
  static constexpr int NK1 = NODE ? 2 * NB : NKF;                   // k-groups of the first Linear
  static constexpr int OFF_WH = A ? NB * NK1 * 1024 : 0;            // D - 1 matrices, the last Linear first
  static constexpr int OFF_WC = OFF_WH + (B ? (D - 1) * W : 0);
  static constexpr int OFF_VEC = OFF_WC + (C ? 2 * W : 0);          // b_1, last bias, gamma[, hidden bias]
  static constexpr int OFF_SCR = OFF_VEC + (D == 3 ? 4 : 3) * L * 4;
  // ENC_EDGE: dz_0 scratch (16 rows x 32 columns) and the tile's features (4 columns)
  static constexpr int SCR = 16 * 32 * 4 + 16 * 16;
  static constexpr int END = OFF_SCR + (KIND == ENC_EDGE ? TF_NWV * SCR : 0);
  static constexpr int NVEC = (D + 2) * L;
  static_assert(END <= 160 * 1024 && (!B || TF_NWV * NVEC * 4 <= OFF_VEC), "LDS");
};

// Features 16 kg + 4 q .. + 3 of a row of fin columns (zero past them).
template <int NKF>
__device__ __forceinline__ void tf_features(const float* __restrict__ x, int fin, int q, float4 (&v)[NKF]) {
#pragma unroll
  for (int kg = 0; kg < NKF; ++kg) {
    const int c = 16 * kg + 4 * q;
    v[kg].x = c < fin ? x[c] : 0.f;
    v[kg].y = c + 1 < fin ? x[c + 1] : 0.f;
    v[kg].z = c + 2 < fin ? x[c + 2] : 0.f;
    v[kg].w = c + 3 < fin ? x[c + 3] : 0.f;
  }
}

template <int NB>
__device__ __forceinline__ uint32_t tf_positive(const float4 (&h)[NB]) {
  uint32_t m = 0;
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) {
    m |= (h[cb].x > 0.f ? 1u : 0u) << (4 * cb);
    m |= (h[cb].y > 0.f ? 1u : 0u) << (4 * cb + 1);
    m |= (h[cb].z > 0.f ? 1u : 0u) << (4 * cb + 2);
    m |= (h[cb].w > 0.f ? 1u : 0u) << (4 * cb + 3);
  }
  return m;
}

// Encoder forward: LN(MLP(features)).
template <int L, int D, int NKF>
struct TfEncLay {
  static constexpr int NB = L / 16, W = L * L * 4;
  static constexpr int OFF_WH = NB * NKF * 1024, OFF_VEC = OFF_WH + (D - 1) * W;
  static constexpr int END = OFF_VEC + (D == 3 ? 5 : 4) * L * 4;  // b_1, last bias, gamma, beta[, hidden bias]
  static_assert(END <= 160 * 1024, "LDS");
};
template <int L, int D, int NKF>
__global__ __launch_bounds__(TF_NTH) void enc_fwd_f32_kernel(RowsFwdArgs a) {
  using Lay = TfEncLay<L, D, NKF>;
  constexpr int NB = Lay::NB;
  extern __shared__ __align__(16) unsigned char lds[];
  float4* W1 = reinterpret_cast<float4*>(lds);
  float4* WL = reinterpret_cast<float4*>(lds + Lay::OFF_WH);
  float4* WH = reinterpret_cast<float4*>(lds + Lay::OFF_WH + Lay::W);
  float* vb1 = reinterpret_cast<float*>(lds + Lay::OFF_VEC);
  float *vbl = vb1 + L, *vg = vb1 + 2 * L, *vbt = vb1 + 3 * L, *vbh = vb1 + 4 * L;
  tf_copy_frags<NB, NKF, TF_NTH, NKF>(W1, a.mlp.lin[0].wf, 0);
  tf_copy_frags<NB, NB, TF_NTH>(WL, a.mlp.lin[D - 1].wf, 0);
  if constexpr (D == 3) tf_copy_frags<NB, NB, TF_NTH>(WH, a.mlp.lin[1].wf, 0);
  rt_copy_vec(vb1, a.mlp.lin[0].b, L);
  rt_copy_vec(vbl, a.mlp.lin[D - 1].b, L);
  rt_copy_vec(vg, a.mlp.gamma, L);
  rt_copy_vec(vbt, a.mlp.beta, L);
  if constexpr (D == 3) rt_copy_vec(vbh, a.mlp.lin[1].b, L);
  __syncthreads();
  const int wave = wave_id(), lane = threadIdx.x & 63;
  const int64_t nt = (a.rows + 15) / 16;
  // tiles go round the workgroups first: few rows still use every CU
  for (int64_t t = blockIdx.x + (int64_t)gridDim.x * wave; t < nt; t += (int64_t)gridDim.x * TF_NWV) {
    int ln = lane;  // opaque: the weight fragments are read per tile, not kept in registers
    asm volatile("" : "+v"(ln));
    const int e = ln & 15, q = ln >> 4, slot = tf_slot(e, q);
    const int64_t row = t * 16 + e;
    const bool ok = row < a.rows;
    float4 x[NKF];
    tf_features<NKF>(a.in0 + (ok ? row : t * 16) * a.fin, a.fin, q, x);
    floatx4 acc[NB];
    tf_gemm<NB, NKF>(W1, x, acc, slot);
    float4 h[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) h[cb] = tf_relu(tf_add(acc[cb], rt_ld4(vb1, cb, q)));
    if constexpr (D == 3) {
      tf_gemm<NB>(WH, h, acc, slot);
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) h[cb] = tf_relu(tf_add(acc[cb], rt_ld4(vbh, cb, q)));
    }
    tf_gemm<NB>(WL, h, acc, slot);
    float4 y[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) y[cb] = tf_add(acc[cb], rt_ld4(vbl, cb, q));
    const float mu = rt_sum4(tf_lane_sum<NB>(y)) / L;
    const float rs = tf_rstd<NB, L>(y, mu, a.eps);
    if (ok) {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        const float4 g = rt_ld4(vg, cb, q), bt = rt_ld4(vbt, cb, q);
        y[cb].x = g.x * ((y[cb].x - mu) * rs) + bt.x;
        y[cb].y = g.y * ((y[cb].y - mu) * rs) + bt.y;
        y[cb].z = g.z * ((y[cb].z - mu) * rs) + bt.z;
        y[cb].w = g.w * ((y[cb].w - mu) * rs) + bt.w;
      }
      tf_store<NB>(reinterpret_cast<float*>(a.out) + row * L, q, y);
    }
  }
}

template <int L, int D, int KIND, int NKF, bool A, bool B, bool C>
__global__ __launch_bounds__(TF_NTH) __attribute__((amdgpu_waves_per_eu(2, 2))) void rows_bwd_f32_kernel(RowsBwdArgs a) {
  using Lay = TfRowsLay<L, D, KIND, NKF, A, B, C>;
  constexpr int NB = Lay::NB, NV = 4 * NB, NR = NV / 16, NK1 = Lay::NK1;
  constexpr bool NODE = Lay::NODE;
  extern __shared__ __align__(16) unsigned char lds[];
  float4* W1 = reinterpret_cast<float4*>(lds);
  float* WL = reinterpret_cast<float*>(lds + Lay::OFF_WH);
  float* WH = reinterpret_cast<float*>(lds + Lay::OFF_WH + Lay::W);
  float4* WC = reinterpret_cast<float4*>(lds + Lay::OFF_WC);
  float* vb1 = reinterpret_cast<float*>(lds + Lay::OFF_VEC);
  float *vbl = vb1 + L, *vg = vb1 + 2 * L, *vbh = vb1 + 3 * L;
  const int wave = wave_id(), lane = threadIdx.x & 63;
  if constexpr (A) {
    tf_copy_frags<NB, NK1, TF_NTH, NK1>(W1, a.mlp.lin[0].wf, 0);
    rt_copy_vec(vb1, a.mlp.lin[0].b, L);
  }
  if constexpr (B) {
    tf_copy_frags<NB, NB, TF_NTH>(WL, a.mlp.lin[D - 1].wf, 0);
    if constexpr (D == 3) tf_copy_frags<NB, NB, TF_NTH>(WH, a.mlp.lin[1].wf, 0);
    rt_copy_vec(vbl, a.mlp.lin[D - 1].b, L);
    rt_copy_vec(vg, a.mlp.gamma, L);
    if constexpr (D == 3) rt_copy_vec(vbh, a.mlp.lin[1].b, L);
  }
  if constexpr (C) tf_copy_frags<2 * NB, NB, TF_NTH, NB>(WC, a.mlp.lin[0].wb, 0);
  __syncthreads();
  // column totals: gamma, beta, last bias, hidden biases
  constexpr int NQ = 2 + D;
  float qacc[NQ][NR];
#pragma unroll
  for (int k = 0; k < NQ; ++k)
#pragma unroll
    for (int t = 0; t < NR; ++t) qacc[k][t] = 0.f;
  auto coltot = [&](const float4 (&x)[NB], int k, int e) {
    float f[NV];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      f[4 * cb] = x[cb].x;
      f[4 * cb + 1] = x[cb].y;
      f[4 * cb + 2] = x[cb].z;
      f[4 * cb + 3] = x[cb].w;
    }
    rt_col_totals<NV>(f, e);
#pragma unroll
    for (int t = 0; t < NR; ++t) qacc[k][t] += f[t];
  };
  // ENC_EDGE with w1_part: the first Linear's weight gradient, columns
  // lane + 64 j, features 0 .. 3
  float w1acc[L / 64][4] = {};
  float* scr = reinterpret_cast<float*>(lds + Lay::OFF_SCR + wave * Lay::SCR);
  float4* xs = reinterpret_cast<float4*>(scr + 16 * 32);
  const int64_t nt = (a.rows + 15) / 16;
  for (int64_t t = blockIdx.x + (int64_t)gridDim.x * wave; t < nt; t += (int64_t)gridDim.x * TF_NWV) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int e = ln & 15, q = ln >> 4, slot = tf_slot(e, q);
    const int64_t row = t * 16 + e;
    const bool ok = row < a.rows;
    const int64_t src = ok ? row : t * 16;  // rows past the end repeat the tile's first (dm = 0, nothing stored)
    floatx4 acc[NB];
    float4 h[NB], dm[NB];
    if constexpr (A) {
      float4 x[NK1];
      if constexpr (NODE) {
        tf_load<NB>(a.in0 + src * L, q, reinterpret_cast<float4(&)[NB]>(x[0]));
        tf_load<NB>(a.in1 + src * L, q, reinterpret_cast<float4(&)[NB]>(x[NB]));
      } else {
        tf_features<NKF>(a.in0 + src * a.fin, a.fin, q, x);
        if constexpr (KIND == ENC_EDGE) {
          if (q == 0) xs[e] = x[0];
        }
      }
      if constexpr (B) tf_load<NB>(a.dm + src * L, q, dm);
      tf_gemm<NB, NK1>(W1, x, acc, slot);
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) h[cb] = tf_relu(tf_add(acc[cb], rt_ld4(vb1, cb, q)));
      if (ok) tf_store<NB>(reinterpret_cast<float*>(a.hid[0]) + row * L, q, h);
    } else if constexpr (B) {
      tf_load<NB>(reinterpret_cast<const float*>(a.hid[0]) + src * L, q, h);
      tf_load<NB>(a.dm + src * L, q, dm);
    }
    float4 v[NB];
    if constexpr (B) {
      uint32_t mask[2] = {tf_positive<NB>(h), 0u};
      if constexpr (D == 3) {
        tf_gemm<NB>(reinterpret_cast<const float4*>(WH), h, acc, slot);
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) h[cb] = tf_relu(tf_add(acc[cb], rt_ld4(vbh, cb, q)));
        mask[1] = tf_positive<NB>(h);
        if (ok) tf_store<NB>(reinterpret_cast<float*>(a.hid[1]) + row * L, q, h);
      }
      tf_gemm<NB>(reinterpret_cast<const float4*>(WL), h, acc, slot);
      float4 y[NB];
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) y[cb] = tf_add(acc[cb], rt_ld4(vbl, cb, q));
      if (!ok) {
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) dm[cb] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      const float mu = rt_sum4(tf_lane_sum<NB>(y)) / L;
      const float rs = tf_rstd<NB, L>(y, mu, a.eps);
      // LayerNorm backward: dy = rstd (dm g - mean(dm g) - xhat mean(dm g xhat))
      float t1, t2;
      {
        float4 d1[NB], d2[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
          const float4 g = rt_ld4(vg, cb, q);
          y[cb] = make_float4((y[cb].x - mu) * rs, (y[cb].y - mu) * rs, (y[cb].z - mu) * rs, (y[cb].w - mu) * rs);
          d1[cb] = make_float4(dm[cb].x * g.x, dm[cb].y * g.y, dm[cb].z * g.z, dm[cb].w * g.w);
          d2[cb] = make_float4(d1[cb].x * y[cb].x, d1[cb].y * y[cb].y, d1[cb].z * y[cb].z, d1[cb].w * y[cb].w);
        }
        t1 = rt_sum4(tf_lane_sum<NB>(d1)) / L;
        t2 = rt_sum4(tf_lane_sum<NB>(d2)) / L;
      }
      coltot(dm, 1, e);
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        const float4 g = rt_ld4(vg, cb, q);
        v[cb].x = rs * (dm[cb].x * g.x - t1 - y[cb].x * t2);
        v[cb].y = rs * (dm[cb].y * g.y - t1 - y[cb].y * t2);
        v[cb].z = rs * (dm[cb].z * g.z - t1 - y[cb].z * t2);
        v[cb].w = rs * (dm[cb].w * g.w - t1 - y[cb].w * t2);
        // gamma's column terms
        y[cb] = make_float4(dm[cb].x * y[cb].x, dm[cb].y * y[cb].y, dm[cb].z * y[cb].z, dm[cb].w * y[cb].w);
      }
      if (ok) tf_store<NB>(reinterpret_cast<float*>(a.delta[D - 1]) + row * L, q, v);
      coltot(y, 0, e);
      coltot(v, 2, e);
      int tb[4];
      tf_t_index(e, q, tb);
#pragma unroll
      for (int j = D - 1; j >= 1; --j) {
        tf_gemm_t<NB>(j == D - 1 ? WL : WH, v, acc, tb);
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
          const uint32_t mk = mask[j - 1] >> (4 * cb);
          v[cb] = make_float4(mk & 1u ? acc[cb][0] : 0.f, mk & 2u ? acc[cb][1] : 0.f, mk & 4u ? acc[cb][2] : 0.f,
                              mk & 8u ? acc[cb][3] : 0.f);
        }
        if ((KIND != ENC_EDGE || j > 1 || !a.w1_part) && ok)
          tf_store<NB>(reinterpret_cast<float*>(a.delta[j - 1]) + row * L, q, v);
        coltot(v, 2 + j, e);
      }
      if constexpr (KIND == ENC_EDGE) {
        if (a.w1_part) {
          // dW_1 += dz_0^T x over the tile's rows (zero past its end), in row
          // order; the scratch passes 32 columns at a time (tf_segment_sums)
#pragma unroll
          for (int j = 0; j < L / 64; ++j) {
            float z[16];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
              for (int c = 0; c < 2; ++c)
                *reinterpret_cast<float4*>(scr + rs_sw32<32>(e, c * 16 + q * 4)) = v[4 * j + 2 * half + c];
              if ((ln >> 5) == half) {
#pragma unroll
                for (int r = 0; r < 16; ++r) z[r] = scr[rs_sw32<32>(r, ln & 31)];
              }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const float4 x = xs[r];
              w1acc[j][0] = fmaf(z[r], x.x, w1acc[j][0]);
              w1acc[j][1] = fmaf(z[r], x.y, w1acc[j][1]);
              w1acc[j][2] = fmaf(z[r], x.z, w1acc[j][2]);
              w1acc[j][3] = fmaf(z[r], x.w, w1acc[j][3]);
            }
          }
        }
      }
    }
    if constexpr (C) {
      if constexpr (!B) {
        tf_load<NB>(reinterpret_cast<const float*>(a.delta[0]) + src * L, q, v);
        tf_load<NB>(a.dm + src * L, q, dm);
      }
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {
        tf_gemm<NB>(WC + pass * NB * NB * 64, v, acc, slot);
        if (ok) {
          float* o = (pass == 0 ? a.dx0 : a.dx1) + row * L;
#pragma unroll
          for (int cb = 0; cb < NB; ++cb)
            *reinterpret_cast<float4*>(o + cb * 16 + q * 4) =
                pass == 0 ? tf_add(acc[cb], dm[cb]) : make_float4(acc[cb][0], acc[cb][1], acc[cb][2], acc[cb][3]);
        }
      }
    }
  }
  if constexpr (B) {
    // column partials (edge_bwd_f32_kernel), then the fused weight gradient,
    // summed over the waves in order
    __syncthreads();
    float* red = reinterpret_cast<float*>(lds);
    {
      float* rw = red + wave * Lay::NVEC;
#pragma unroll
      for (int t = 0; t < NR; ++t) {
        const int i = (lane & 15) * NR + t;
        const int col = (i >> 2) * 16 + (lane >> 4) * 4 + (i & 3);
#pragma unroll
        for (int h = 0; h < D - 1; ++h) rw[h * L + col] = qacc[3 + h][t];
        rw[(D - 1) * L + col] = qacc[2][t];
        rw[D * L + col] = qacc[0][t];
        rw[(D + 1) * L + col] = qacc[1][t];
      }
    }
    __syncthreads();
    float* vp = a.vpart + (int64_t)blockIdx.x * a.nvec;
    for (int i = threadIdx.x; i < Lay::NVEC; i += TF_NTH) {
      float s = 0.f;
      for (int w = 0; w < TF_NWV; ++w) s += red[w * Lay::NVEC + i];
      vp[i] = s;
    }
    if constexpr (KIND == ENC_EDGE) {
      if (a.w1_part) {
        static_assert(TF_NWV * L * 16 <= Lay::OFF_VEC, "LDS");
        __syncthreads();
        float4* rw = reinterpret_cast<float4*>(lds);
#pragma unroll
        for (int j = 0; j < L / 64; ++j)
          rw[wave * L + lane + 64 * j] = make_float4(w1acc[j][0], w1acc[j][1], w1acc[j][2], w1acc[j][3]);
        __syncthreads();
        for (int i = threadIdx.x; i < 4 * L; i += TF_NTH) {
          float s = 0.f;
          for (int w = 0; w < TF_NWV; ++w) s += red[w * 4 * L + i];
          if ((i & 3) < a.fin) a.w1_part[(int64_t)blockIdx.x * L * a.fin + (i >> 2) * a.fin + (i & 3)] = s;
        }
      }
    }
  }
}

// Few rows: a wave per (16-row tile, group of CB output column blocks), its
// weights read straight from the packed copy.  A tile's whole product keeps
// one SIMD's matrix pipe busy for 7.8 us at 3 L x L (L = 128), and with under
// TF_COLS_TILES tiles most SIMDs have none; this way neighbouring waves share
// a tile, and no workgroup waits for 64 - 128 KiB of weights to reach its LDS.
constexpr int TF_COLS_TILES = 512;

// acc[c] = sum over k-groups of W[cb0 + c][kg0 + kg] x X[kg]; W: packed, SRC
// k-groups per block.
template <int CB, int NK, int SRC>
__device__ __forceinline__ void tf_gemm_cols(const uint4* __restrict__ W, int cb0, int kg0, const float4 (&X)[NK],
                                             floatx4 (&acc)[CB], int lane) {
  const float4* Wl = reinterpret_cast<const float4*>(W) + lane;
  float4 w[CB][NK];
#pragma unroll
  for (int kg = 0; kg < NK; ++kg)
#pragma unroll
    for (int c = 0; c < CB; ++c) w[c][kg] = Wl[((cb0 + c) * SRC + kg0 + kg) * 64];
#pragma unroll
  for (int c = 0; c < CB; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kg = 0; kg < NK; ++kg) {
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[c][kg].x, X[kg].x, acc[c], 0, 0, 0);
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[c][kg].y, X[kg].y, acc[c], 0, 0, 0);
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[c][kg].z, X[kg].z, acc[c], 0, 0, 0);
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[c][kg].w, X[kg].w, acc[c], 0, 0, 0);
  }
}

// node_proj_f32_kernel for few rows: units (tile, side, column group); halo
// tiles after the owned ones, sender side only.
template <int L>
__global__ __launch_bounds__(256) void node_proj_cols_kernel(const float* V, const float* H, int64_t n_owned,
                                                             int64_t n_halo, Lin w1, float* ps, float* ps_halo,
                                                             float* pr) {
  constexpr int NB = L / 16, CB = 2, G = NB / CB;
  const int lane = threadIdx.x & 63, e = lane & 15, q = lane >> 4;
  const int to = (int)((n_owned + 15) / 16), th = (int)((n_halo + 15) / 16);
  const int u = blockIdx.x * 4 + wave_id();
  if (u >= (2 * to + th) * G) return;
  const int cb0 = u % G * CB, ts = u / G;
  const bool halo = ts >= 2 * to;
  const int side = halo ? 0 : ts & 1;
  const int64_t row0 = (int64_t)(halo ? ts - 2 * to : ts >> 1) * 16, row = row0 + e;
  const bool ok = row < (halo ? n_halo : n_owned);
  float4 x[NB];
  tf_load<NB>((halo ? H : V) + (ok ? row : row0) * L, q, x);
  floatx4 acc[CB];
  tf_gemm_cols<CB, NB, 3 * NB>(w1.wf, cb0, (1 + side) * NB, x, acc, lane);
  if (ok) {
    float* o = (side ? pr : halo ? ps_halo : ps) + row * L;
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      float4 v = make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
      if (side) v = tf_add(acc[c], rt_ld4(w1.b, cb0 + c, q));
      *reinterpret_cast<float4*>(o + (cb0 + c) * 16 + q * 4) = v;
    }
  }
}

// Phases A and C of the node half's backward (rows_bwd_f32_kernel) for few rows.
template <int L, bool PHASE_C>
__global__ __launch_bounds__(256) void node_bwd_cols_kernel(RowsBwdArgs a) {
  constexpr int NB = L / 16, CB = 2, G = (PHASE_C ? 2 * NB : NB) / CB;
  const int lane = threadIdx.x & 63, e = lane & 15, q = lane >> 4;
  const int u = blockIdx.x * 4 + wave_id(), cb0 = u % G * CB;
  const int64_t row0 = (int64_t)(u / G) * 16, row = row0 + e;
  if (row0 >= a.rows) return;
  const bool ok = row < a.rows;
  const int64_t src = ok ? row : row0;
  floatx4 acc[CB];
  if constexpr (!PHASE_C) {
    float4 x[2 * NB];
    tf_load<NB>(a.in0 + src * L, q, reinterpret_cast<float4(&)[NB]>(x[0]));
    tf_load<NB>(a.in1 + src * L, q, reinterpret_cast<float4(&)[NB]>(x[NB]));
    tf_gemm_cols<CB, 2 * NB, 2 * NB>(a.mlp.lin[0].wf, cb0, 0, x, acc, lane);
    if (ok) {
#pragma unroll
      for (int c = 0; c < CB; ++c)
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.hid[0]) + row * L + (cb0 + c) * 16 + q * 4) =
            tf_relu(tf_add(acc[c], rt_ld4(a.mlp.lin[0].b, cb0 + c, q)));
    }
  } else {
    float4 z[NB];
    tf_load<NB>(reinterpret_cast<const float*>(a.delta[0]) + src * L, q, z);
    tf_gemm_cols<CB, NB, NB>(a.mlp.lin[0].wb, cb0, 0, z, acc, lane);
    const bool agg = cb0 >= NB;
    if (ok) {
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        const int cb = cb0 + c - (agg ? NB : 0);
        float4 v = make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
        if (!agg) v = tf_add(acc[c], rt_ld4(a.dm + row * L, cb, q));
        *reinterpret_cast<float4*>((agg ? a.dx1 : a.dx0) + row * L + cb * 16 + q * 4) = v;
      }
    }
  }
}

// Node half forward, v + LN(MLP([v | agg])).  Phase A: h_1 = relu(W_1 [v | agg]
// + b_1); phase B: the rest.  L = 64 runs both in one launch; at L = 128 (128
// and 64 KiB of weights) phase A leaves h_1 in the output rows, which phase B's
// wave reads before it writes them.
template <int L, int D, bool A, bool B>
struct TfNodeFwdLay {
  static constexpr int NB = L / 16, W = L * L * 4;
  static constexpr int OFF_WH = A ? 2 * W : 0, OFF_VEC = OFF_WH + (B ? (D - 1) * W : 0);
  static constexpr int END = OFF_VEC + 5 * L * 4;  // b_1, last bias, gamma, beta, hidden bias
  static_assert(END <= 160 * 1024, "LDS");
};
template <int L, int D, bool A, bool B>
__global__ __launch_bounds__(TF_NTH) void node_fwd_f32_kernel(RowsFwdArgs a) {
  using Lay = TfNodeFwdLay<L, D, A, B>;
  constexpr int NB = Lay::NB;
  extern __shared__ __align__(16) unsigned char lds[];
  float4* W1 = reinterpret_cast<float4*>(lds);
  float4* WL = reinterpret_cast<float4*>(lds + Lay::OFF_WH);
  float4* WH = reinterpret_cast<float4*>(lds + Lay::OFF_WH + Lay::W);
  float* vb1 = reinterpret_cast<float*>(lds + Lay::OFF_VEC);
  float *vbl = vb1 + L, *vg = vb1 + 2 * L, *vbt = vb1 + 3 * L, *vbh = vb1 + 4 * L;
  if constexpr (A) {
    tf_copy_frags<NB, 2 * NB, TF_NTH, 2 * NB>(W1, a.mlp.lin[0].wf, 0);
    rt_copy_vec(vb1, a.mlp.lin[0].b, L);
  }
  if constexpr (B) {
    tf_copy_frags<NB, NB, TF_NTH>(WL, a.mlp.lin[D - 1].wf, 0);
    if constexpr (D == 3) tf_copy_frags<NB, NB, TF_NTH>(WH, a.mlp.lin[1].wf, 0);
    rt_copy_vec(vbl, a.mlp.lin[D - 1].b, L);
    rt_copy_vec(vg, a.mlp.gamma, L);
    rt_copy_vec(vbt, a.mlp.beta, L);
    if constexpr (D == 3) rt_copy_vec(vbh, a.mlp.lin[1].b, L);
  }
  __syncthreads();
  const int wave = wave_id(), lane = threadIdx.x & 63;
  float* out = reinterpret_cast<float*>(a.out);
  const int64_t nt = (a.rows + 15) / 16;
  for (int64_t t = blockIdx.x + (int64_t)gridDim.x * wave; t < nt; t += (int64_t)gridDim.x * TF_NWV) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int e = ln & 15, q = ln >> 4, slot = tf_slot(e, q);
    const int64_t row = t * 16 + e;
    const bool ok = row < a.rows;
    const int64_t src = ok ? row : t * 16;
    floatx4 acc[NB];
    float4 h[NB], v[NB];
    if constexpr (A) {
      float4 x[2 * NB];
      tf_load<NB>(a.in0 + src * L, q, v);
      tf_load<NB>(a.in1 + src * L, q, reinterpret_cast<float4(&)[NB]>(x[NB]));
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) x[cb] = v[cb];
      tf_gemm<NB, 2 * NB>(W1, x, acc, slot);
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) h[cb] = tf_relu(tf_add(acc[cb], rt_ld4(vb1, cb, q)));
      if constexpr (!B) {
        if (ok) tf_store<NB>(out + row * L, q, h);
      }
    } else {
      tf_load<NB>(out + src * L, q, h);
      tf_load<NB>(a.in0 + src * L, q, v);
    }
    if constexpr (B) {
      if constexpr (D == 3) {
        tf_gemm<NB>(WH, h, acc, slot);
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) h[cb] = tf_relu(tf_add(acc[cb], rt_ld4(vbh, cb, q)));
      }
      tf_gemm<NB>(WL, h, acc, slot);
      float4 y[NB];
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) y[cb] = tf_add(acc[cb], rt_ld4(vbl, cb, q));
      const float mu = rt_sum4(tf_lane_sum<NB>(y)) / L;
      const float rs = tf_rstd<NB, L>(y, mu, a.eps);
      if (ok) {
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
          const float4 g = rt_ld4(vg, cb, q), bt = rt_ld4(vbt, cb, q);
          y[cb].x = (g.x * ((y[cb].x - mu) * rs) + bt.x) + v[cb].x;
          y[cb].y = (g.y * ((y[cb].y - mu) * rs) + bt.y) + v[cb].y;
          y[cb].z = (g.z * ((y[cb].z - mu) * rs) + bt.z) + v[cb].z;
          y[cb].w = (g.w * ((y[cb].w - mu) * rs) + bt.w) + v[cb].w;
        }
        tf_store<NB>(out + row * L, q, y);
      }
    }
  }
}

// The same for few rows (L = 128, depth 2): a workgroup of four waves per
// 16-row tile, two output column blocks per wave and product, the weights read
// straight from the packed copies; h_1 and the row sums pass through LDS.
// 1,885 rows: 9 us a launch, against 17 for four waves on 64-row tiles.
__global__ __launch_bounds__(256) void node_fwd_cols_kernel(RowsFwdArgs a) {
  constexpr int L = 128, NB = 8, CB = 2, LDH = L + 4;
  __shared__ __align__(16) float H[16 * LDH];
  __shared__ float S[2][4][16];
  const int wave = wave_id(), lane = threadIdx.x & 63, e = lane & 15, q = lane >> 4, cb0 = wave * CB;
  const int64_t row0 = (int64_t)blockIdx.x * 16, row = row0 + e;
  const bool ok = row < a.rows;
  const int64_t src = ok ? row : row0;
  float4 x[2 * NB], v[CB];
  tf_load<NB>(a.in0 + src * L, q, reinterpret_cast<float4(&)[NB]>(x[0]));
  tf_load<NB>(a.in1 + src * L, q, reinterpret_cast<float4(&)[NB]>(x[NB]));
  floatx4 acc[CB];
  tf_gemm_cols<CB, 2 * NB, 2 * NB>(a.mlp.lin[0].wf, cb0, 0, x, acc, lane);
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    *reinterpret_cast<float4*>(H + e * LDH + (cb0 + c) * 16 + q * 4) =
        tf_relu(tf_add(acc[c], rt_ld4(a.mlp.lin[0].b, cb0 + c, q)));
    v[c] = rt_ld4(a.in0 + src * L, cb0 + c, q);
  }
  __syncthreads();
  float4 h[NB];
#pragma unroll
  for (int kg = 0; kg < NB; ++kg) h[kg] = *reinterpret_cast<const float4*>(H + e * LDH + kg * 16 + q * 4);
  tf_gemm_cols<CB, NB, NB>(a.mlp.lin[1].wf, cb0, 0, h, acc, lane);
  float4 y[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) y[c] = tf_add(acc[c], rt_ld4(a.mlp.lin[1].b, cb0 + c, q));
  const float s1 = rt_sum4(tf_lane_sum<CB>(y));
  if (q == 0) S[0][wave][e] = s1;
  __syncthreads();
  const float mu = (((S[0][0][e] + S[0][1][e]) + S[0][2][e]) + S[0][3][e]) / L;
  float4 d[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    const float4 u = make_float4(y[c].x - mu, y[c].y - mu, y[c].z - mu, y[c].w - mu);
    d[c] = make_float4(u.x * u.x, u.y * u.y, u.z * u.z, u.w * u.w);
  }
  const float s2 = rt_sum4(tf_lane_sum<CB>(d));
  if (q == 0) S[1][wave][e] = s2;
  __syncthreads();
  const float rs = 1.0f / sqrtf((((S[1][0][e] + S[1][1][e]) + S[1][2][e]) + S[1][3][e]) / L + a.eps);
  if (ok) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const float4 g = rt_ld4(a.mlp.gamma, cb0 + c, q), bt = rt_ld4(a.mlp.beta, cb0 + c, q);
      float4 o;
      o.x = (g.x * ((y[c].x - mu) * rs) + bt.x) + v[c].x;
      o.y = (g.y * ((y[c].y - mu) * rs) + bt.y) + v[c].y;
      o.z = (g.z * ((y[c].z - mu) * rs) + bt.z) + v[c].z;
      o.w = (g.w * ((y[c].w - mu) * rs) + bt.w) + v[c].w;
      *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.out) + row * L + (cb0 + c) * 16 + q * 4) = o;
    }
  }
}

template <class F>
void allow_lds(F* fn, int bytes) {
  if (bytes > 65536) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// Working waves per workgroup for `edges` edges: one per SIMD while that gives
// every wave a single 16-edge tile (ranges are receiver-aligned, so 11 edges a
// wave on average), else all.  On 10,900 edges a wave per full tile (three a
// workgroup) left some waves two tiles: forward 27.8 us.
int tf_waves(int64_t edges) { return edges <= (int64_t)4 * RS_GRID * 11 ? 4 : TF_NWV; }

template <int L, int D, bool SPLIT, bool HS>
hipError_t edge_fwd_f32_t(const EdgeFwdArgs& a, int64_t n_edges, hipStream_t st) {
  using Lay = TfFwdLay<L, D>;
  allow_lds(edge_fwd_f32_kernel<L, D, SPLIT, HS>, Lay::END);
  hipLaunchKernelGGL((edge_fwd_f32_kernel<L, D, SPLIT, HS>), dim3(RS_GRID), dim3(TF_NTH), Lay::END, st, a,
                     n_edges, tf_waves(n_edges));
  return hipGetLastError();
}
template <int L, int D, bool SPLIT>
hipError_t edge_bwd_f32_t(const EdgeBwdArgs& a, int64_t n_edges, hipStream_t st) {
  using Lay = TfBwdLay<L, D>;
  allow_lds(edge_bwd_f32_kernel<L, D, SPLIT>, Lay::END);
  hipLaunchKernelGGL((edge_bwd_f32_kernel<L, D, SPLIT>), dim3(RS_GRID), dim3(TF_NTH), Lay::END, st, a,
                     n_edges, tf_waves(n_edges));
  return hipGetLastError();
}

// Whether one receiver's edges are more than a wave should take alone: over
// twice the share of each, and four tiles.  At l = 128, two blocks forward and
// backward on 259,000 edges (share 126): largest receiver 300 edges 3.00 ms
// with a wave alone on it, 2.34 split; 10,000 edges 34.3 and 9.1.  On 2.7M
// edges (share 1,340): 1,000 edges 20.0 ms alone, 18.4 without that receiver;
// 3,000 edges 29.9 and 19.6.
bool tf_split(int64_t edges, int64_t max_degree) {
  const int64_t share = edges / (RS_GRID * TF_NWV);
  return max_degree > (share > 32 ? 2 * share : 64);
}

template <int L>
hipError_t node_proj_f32_t(const float* V, const float* H, int64_t n_owned, int64_t n_halo, const Lin& w1, float* ps,
                           float* ps_halo, float* pr, hipStream_t st) {
  const int64_t tiles = (n_owned + 15) / 16 + (n_halo + 15) / 16;
  if (tiles <= TF_COLS_TILES) {
    const int64_t units = (2 * ((n_owned + 15) / 16) + (n_halo + 15) / 16) * (L / 32);
    hipLaunchKernelGGL((node_proj_cols_kernel<L>), dim3((unsigned)((units + 3) / 4)), dim3(256), 0, st, V, H, n_owned,
                       n_halo, w1, ps, ps_halo, pr);
    return hipGetLastError();
  }
  // both sides: 256 workgroups each, two to a CU
  hipLaunchKernelGGL((node_proj_f32_kernel<L>), dim3(2 * RS_GRID), dim3(TF_NTH), L * L * 4, st, V, H, n_owned, n_halo,
                     w1, ps, ps_halo, pr);
  return hipGetLastError();
}

int tf_rows_grid(int64_t rows) {
  const int64_t t = (rows + 15) / 16;
  return (int)(t < 1 ? 1 : t < RS_GRID ? t : RS_GRID);
}

template <int L, int D, int NKF>
hipError_t enc_fwd_f32_t(const RowsFwdArgs& a, hipStream_t st) {
  using Lay = TfEncLay<L, D, NKF>;
  allow_lds(enc_fwd_f32_kernel<L, D, NKF>, Lay::END);
  hipLaunchKernelGGL((enc_fwd_f32_kernel<L, D, NKF>), dim3(tf_rows_grid(a.rows)), dim3(TF_NTH), Lay::END, st, a);
  return hipGetLastError();
}

template <int L, int D, bool A, bool B>
hipError_t node_fwd_f32_t(const RowsFwdArgs& a, hipStream_t st) {
  using Lay = TfNodeFwdLay<L, D, A, B>;
  allow_lds(node_fwd_f32_kernel<L, D, A, B>, Lay::END);
  hipLaunchKernelGGL((node_fwd_f32_kernel<L, D, A, B>), dim3(tf_rows_grid(a.rows)), dim3(TF_NTH), Lay::END, st, a);
  return hipGetLastError();
}

template <int L, int D, int KIND, int NKF, bool A, bool B, bool C>
hipError_t rows_bwd_f32_t(const RowsBwdArgs& a, hipStream_t st) {
  using Lay = TfRowsLay<L, D, KIND, NKF, A, B, C>;
  allow_lds(rows_bwd_f32_kernel<L, D, KIND, NKF, A, B, C>, Lay::END);
  hipLaunchKernelGGL((rows_bwd_f32_kernel<L, D, KIND, NKF, A, B, C>), dim3(tf_rows_grid(a.rows)), dim3(TF_NTH), Lay::END,
                     st, a);
  return hipGetLastError();
}

template <int L, int D>
hipError_t rows_bwd_f32_d(int kind, const RowsBwdArgs& a, hipStream_t st) {
  if (kind == NODE_BLOCK) {
    if constexpr (L == 64) {
      return rows_bwd_f32_t<L, D, NODE_BLOCK, 1, true, true, true>(a, st);
    } else {
      const int64_t tiles = (a.rows + 15) / 16;
      const bool cols = tiles > 0 && tiles <= TF_COLS_TILES;
      if (cols)  // (phase A: L / 32 column groups of a tile, phase C: L / 16)
        hipLaunchKernelGGL((node_bwd_cols_kernel<L, false>), dim3((unsigned)(tiles * (L / 32) / 4)), dim3(256), 0, st, a);
      hipError_t e = cols ? hipGetLastError() : rows_bwd_f32_t<L, D, NODE_BLOCK, 1, true, false, false>(a, st);
      if (e == hipSuccess) e = rows_bwd_f32_t<L, D, NODE_BLOCK, 1, false, true, false>(a, st);
      if (e != hipSuccess) return e;
      if (cols) {
        hipLaunchKernelGGL((node_bwd_cols_kernel<L, true>), dim3((unsigned)(tiles * (L / 16) / 4)), dim3(256), 0, st, a);
        return hipGetLastError();
      }
      if (e == hipSuccess) e = rows_bwd_f32_t<L, D, NODE_BLOCK, 1, false, false, true>(a, st);
      return e;
    }
  }
  if (kind == ENC_EDGE)
    return a.fin <= 16 ? rows_bwd_f32_t<L, D, ENC_EDGE, 1, true, true, false>(a, st) : hipErrorInvalidValue;
  return a.fin <= 16 ? rows_bwd_f32_t<L, D, ENC_NODE, 1, true, true, false>(a, st) : hipErrorInvalidValue;
}

}  // namespace

bool rows_f32(int prec, int L, int D, int kind, int fin) {
  if (prec != F32 || (L != 64 && L != 128)) return false;
  return kind == NODE_BLOCK || ((kind == ENC_NODE || kind == ENC_EDGE) && fin <= 16);
}
// (128, 3) keeps the other forward kernels, as its edge half does, which takes
// many times their work.
bool rows_fwd_f32(int prec, int L, int D, int kind, int fin) {
  return rows_f32(prec, L, D, kind, fin) && edge_f32(prec, L, D);
}
int rows_f32_grid(int64_t rows) { return tf_rows_grid(rows); }
int rows_f32_w1_parts(int64_t rows, int kind, int fin) { return kind == ENC_EDGE && fin <= 4 ? tf_rows_grid(rows) : 0; }

hipError_t launch_rows_fwd_f32(int L, int D, int kind, const RowsFwdArgs& a, hipStream_t st) {
  if (a.rows == 0) return hipSuccess;
  if (kind == NODE_BLOCK) {
    if (L == 64) return D == 2 ? node_fwd_f32_t<64, 2, true, true>(a, st) : node_fwd_f32_t<64, 3, true, true>(a, st);
    if (L != 128 || D != 2) return hipErrorInvalidValue;
    const int64_t tiles = (a.rows + 15) / 16;
    if (tiles <= TF_COLS_TILES) {
      hipLaunchKernelGGL(node_fwd_cols_kernel, dim3((unsigned)tiles), dim3(256), 0, st, a);
      return hipGetLastError();
    }
    const hipError_t e = node_fwd_f32_t<128, 2, true, false>(a, st);
    return e == hipSuccess ? node_fwd_f32_t<128, 2, false, true>(a, st) : e;
  }
  if (L == 64) return D == 2 ? enc_fwd_f32_t<64, 2, 1>(a, st) : enc_fwd_f32_t<64, 3, 1>(a, st);
  if (L == 128 && D == 2) return enc_fwd_f32_t<128, 2, 1>(a, st);
  return hipErrorInvalidValue;
}
hipError_t launch_rows_bwd_f32(int L, int D, int kind, const RowsBwdArgs& a, hipStream_t st) {
  if (L == 64) return D == 2 ? rows_bwd_f32_d<64, 2>(kind, a, st) : rows_bwd_f32_d<64, 3>(kind, a, st);
  if (L == 128) return D == 2 ? rows_bwd_f32_d<128, 2>(kind, a, st) : rows_bwd_f32_d<128, 3>(kind, a, st);
  return hipErrorInvalidValue;
}

bool edge_f32(int prec, int L, int D) { return prec == F32 && (L == 64 || (L == 128 && D == 2)); }

hipError_t launch_edge_fwd_f32(int L, int D, const EdgeFwdArgs& a, int64_t n_edges, int64_t max_degree,
                               hipStream_t st) {
  const bool split = tf_split(n_edges, max_degree), hs = !a.ps_halo && a.H;
#define EF(LL, DD)                                                            \
  if (L == LL && D == DD) {                                                   \
    if (hs) return split ? edge_fwd_f32_t<LL, DD, true, true>(a, n_edges, st) \
                         : edge_fwd_f32_t<LL, DD, false, true>(a, n_edges, st); \
    return split ? edge_fwd_f32_t<LL, DD, true, false>(a, n_edges, st)        \
                 : edge_fwd_f32_t<LL, DD, false, false>(a, n_edges, st);      \
  }
  EF(64, 2) EF(64, 3) EF(128, 2)
#undef EF
  return hipErrorInvalidValue;
}
hipError_t launch_edge_bwd_f32(int L, int D, const EdgeBwdArgs& a, int64_t n_edges, int64_t max_degree,
                               hipStream_t st) {
  if (!a.hid_in) return hipErrorInvalidValue;
  const bool split = tf_split(n_edges, max_degree);
#define EB(LL, DD) \
  if (L == LL && D == DD) \
    return split ? edge_bwd_f32_t<LL, DD, true>(a, n_edges, st) : edge_bwd_f32_t<LL, DD, false>(a, n_edges, st);
  EB(64, 2) EB(64, 3) EB(128, 2)
#undef EB
  return hipErrorInvalidValue;
}
hipError_t launch_node_proj_f32(int L, const float* V, const float* H, int64_t n_owned, int64_t n_halo, const Lin& w1,
                                float* ps, float* ps_halo, float* pr, hipStream_t st) {
  if (n_owned + n_halo == 0) return hipSuccess;
  if (L == 64) return node_proj_f32_t<64>(V, H, n_owned, n_halo, w1, ps, ps_halo, pr, st);
  if (L == 128) return node_proj_f32_t<128>(V, H, n_owned, n_halo, w1, ps, ps_halo, pr, st);
  return hipErrorInvalidValue;
}

}  // namespace mgn
