// Layer passes at l = 256 in bf16 (gfx950): the backward of the edge half, the
// node half and the encoders over many rows, one launch per Linear.
//
// One l x l bf16 layer is 128 KiB, a workgroup's LDS less one scratch area.
// The fused kernels (edge_bwd_rw, rows_rw_bwd, rows_rw_enc_bwd) stream every
// layer through LDS in chunks, for every 64 rows anew, with a barrier per
// chunk; at one wave per SIMD each step waits for its chunk, its gathers and
// the tile's stores (edge backward of 1.39M edges at depth 3: 4.1 ms, the
// matrix pipe busy 7 % of it; as passes 2.4 ms, at 5 TB/s).  The forward, whose
// hidden rows nothing else reads, is the other way round (three passes 1.35
// ms, the fused kernel 1.13) and stays fused.  Here a layer stays in LDS for the whole
// launch and eight waves work alone on 16-row tiles of their own ranges (T
// form); rows travel between the launches through HBM, most of them in the
// buffers that the weight gradients read anyway.  What bounds a pass is that
// traffic: 1 to 3 KB a row.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "tform.h"

namespace mgn {

namespace {

constexpr int WL = 256, WNB = WL / 16, WNK = WL / 32, WNV = 4 * WNB, WNR = WNV / 16;
constexpr int W_NWV = 8, W_NTH = 64 * W_NWV;
constexpr int W_OFF_VEC = WNB * WNK * 64 * 16;          // after the layer: up to 3 vectors
constexpr int W_OFF_SCR = W_OFF_VEC + 3 * WL * 4;       // per wave: 2 KiB
constexpr int W_END = W_OFF_SCR + W_NWV * 2048;
static_assert(W_END <= 160 * 1024, "LDS");

struct WideArgs {
  const uint4* w;      // packed layer
  int src_nkg;         // its k-groups per block
  const float *b, *gamma;
  float eps;
  int64_t rows;
  const uint16_t* x;   // operand rows [rows][l]
  uint16_t* out;       // result rows
  const uint16_t* h;   // MASK: the ReLU output whose sign masks the result
  const float* feat;   // ENC: features [rows][fin]
  int fin;
  const float* proj;   // EDGE1: node projections [n_local][2l]
  const int32_t *send, *recv;  // per row
  const float* dagg;   // LNB, OUT: fp32 gradient rows, by recv (edges) or, recv null, by row; or null
  const uint16_t* de;  // LNB: gradient rows added to dagg's (or alone); DE: de^{k+1}; or null
  float* vpart;        // LNB, MASK: [grid][nvec], columns from voff
  int nvec, voff;
  // DE: receivers [r_lo, r_hi), their edges [e_lo, e_lo + rows); x, out, de are
  // indexed from e_lo on, recv / send from edge 0
  const int32_t* row_ptr;
  int64_t r_lo, r_hi, e_lo;
  float* sum;          // DE: dagg, overwritten by the receiver sums of x
  float* out32;        // OUT: fp32 result rows
};

// The layer's fragments into LDS: PERM for operands in T order (rt_copy_frags).
template <bool PERM>
__device__ __forceinline__ void wide_copy(uint4* dst, const uint4* __restrict__ src, int src_nkg) {
  constexpr int IT = WNB * WNK * 64 / W_NTH;
#pragma unroll
  for (int j0 = 0; j0 < IT; j0 += 8) {
    uint4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = threadIdx.x + (j0 + j) * W_NTH, blk = i >> 6, ln = i & 63;
      const uint4* s = src + (size_t)((blk / WNK) * src_nkg + blk % WNK) * 64;
      if constexpr (PERM) {
        const int q = ln >> 4, c = ln & 15;
        const uint2* s2 = reinterpret_cast<const uint2*>(s);
        const uint2 lo = s2[(c + 16 * (q >> 1)) * 2 + (q & 1)], hi = s2[(c + 16 * (2 + (q >> 1))) * 2 + (q & 1)];
        v[j] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      } else {
        v[j] = s[ln];
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) dst[threadIdx.x + (j0 + j) * W_NTH] = v[j];
  }
}

__device__ __forceinline__ void wide_load(const uint16_t* __restrict__ row, int q, uint4 (&v)[WNK]) {
#pragma unroll
  for (int kg = 0; kg < WNK; ++kg) v[kg] = *reinterpret_cast<const uint4*>(row + kg * 32 + q * 8);
}

// Column totals of a tile added to this lane's share (index 4 e + t).
__device__ __forceinline__ void wide_coltot(const float (&x)[WNB][4], float (&acc)[WNR], int e) {
  float f[WNV];
#pragma unroll
  for (int cb = 0; cb < WNB; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r) f[4 * cb + r] = x[cb][r];
  rt_col_totals<WNV>(f, e);
#pragma unroll
  for (int t = 0; t < WNR; ++t) acc[t] += f[t];
}

// The waves' column totals (NQ vectors) in wave order -> vpart.
template <int NQ>
__device__ __forceinline__ void wide_vec(const float (&acc)[NQ][WNR], unsigned char* lds, const WideArgs& a) {
  const int wave = wave_id(), lane = threadIdx.x & 63;
  __syncthreads();  // the layer is not read any more
  float* red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int t = 0; t < WNR; ++t) {
    const int i = (lane & 15) * WNR + t, col = (i >> 2) * 16 + (lane >> 4) * 4 + (i & 3);
#pragma unroll
    for (int k = 0; k < NQ; ++k) red[(wave * NQ + k) * WL + col] = acc[k][t];
  }
  __syncthreads();
  float* vp = a.vpart + (int64_t)blockIdx.x * a.nvec + a.voff;
  for (int i = threadIdx.x; i < NQ * WL; i += W_NTH) {
    float s = 0.f;
    for (int w = 0; w < W_NWV; ++w) s += red[w * NQ * WL + i];
    vp[i] = s;
  }
}

// ----------------------------------------------------------- rows in any order ---
// EDGE1: relu(W_e x + P_s[send] + P_r[recv]); ENC: relu(W_1 features + b);
// HID: relu(W x + b); LNB: y = W x + b, LayerNorm backward of dm = dagg + de
// (either may be absent), column totals [last bias, gamma, beta]; MASK: (W^T x)
// where h > 0, column totals; OUT: W^T x + dagg, fp32.
enum { W_EDGE1, W_ENC, W_HID, W_LNB, W_MASK, W_OUT };

template <int KIND>
__global__ __launch_bounds__(W_NTH) __attribute__((amdgpu_waves_per_eu(2, 2))) void wide_rows_kernel(WideArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  uint4* W = reinterpret_cast<uint4*>(lds);
  float* vb = reinterpret_cast<float*>(lds + W_OFF_VEC);
  float* vg = vb + WL;
  const int wave = wave_id(), lane = threadIdx.x & 63;
  if constexpr (KIND == W_ENC) rs_copy_frags(W, a.w, WNB, 1, a.src_nkg, 0);
  else wide_copy<KIND != W_EDGE1>(W, a.w, a.src_nkg);
  if constexpr (KIND == W_ENC || KIND == W_HID || KIND == W_LNB) rt_copy_vec(vb, a.b, WL);
  if constexpr (KIND == W_LNB) rt_copy_vec(vg, a.gamma, WL);
  __syncthreads();
  constexpr int NQ = KIND == W_LNB ? 3 : 1;
  float qacc[NQ][WNR] = {};
  // contiguous tiles per wave, neighbouring ranges on one XCD (shared node rows)
  const int64_t T = (a.rows + 15) / 16, NWAVES = (int64_t)gridDim.x * W_NWV;
  const int64_t w = ((int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * W_NWV + wave;
  const int64_t t1 = T * (w + 1) / NWAVES;
  for (int64_t t = T * w / NWAVES; t < t1; ++t) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int e = ln & 15, q = ln >> 4;
    const int64_t row = t * 16 + e;
    const bool ok = row < a.rows;
    const int64_t src = ok ? row : t * 16;  // rows past the end repeat the tile's first (never stored; dm = 0)
    floatx4 acc[WNB];
    float v[WNB][4];
    if constexpr (KIND == W_ENC) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = q * 8 + j < a.fin ? a.feat[src * a.fin + q * 8 + j] : 0.f;
      const uint4 xf[1] = {
          make_uint4(bf_pack(x[0], x[1]), bf_pack(x[2], x[3]), bf_pack(x[4], x[5]), bf_pack(x[6], x[7]))};
      rt_gemm<WNB, 1>(W, xf, acc, ln);
    } else {
      uint4 raw[WNK];
      wide_load(a.x + src * WL, q, raw);
      if constexpr (KIND == W_EDGE1) {
        const float* sp = a.proj + (int64_t)a.send[src] * (2 * WL);
        const float* rp = a.proj + (int64_t)a.recv[src] * (2 * WL) + WL;
        float4 ps[WNB], pr[WNB];
#pragma unroll
        for (int cb = 0; cb < WNB; ++cb) {
          ps[cb] = rt_ld4(sp, cb, q);
          pr[cb] = rt_ld4(rp, cb, q);
        }
        __builtin_amdgcn_sched_barrier(0);
        rt_gemm<WNB, WNK>(W, raw, acc, ln);
#pragma unroll
        for (int cb = 0; cb < WNB; ++cb) {
          v[cb][0] = fmaxf((acc[cb][0] + ps[cb].x) + pr[cb].x, 0.f);
          v[cb][1] = fmaxf((acc[cb][1] + ps[cb].y) + pr[cb].y, 0.f);
          v[cb][2] = fmaxf((acc[cb][2] + ps[cb].z) + pr[cb].z, 0.f);
          v[cb][3] = fmaxf((acc[cb][3] + ps[cb].w) + pr[cb].w, 0.f);
        }
      } else if constexpr (KIND == W_LNB) {
        uint4 dr[WNK];
        float4 dm[WNB];
        const bool has_de = a.de != nullptr, has_agg = a.dagg != nullptr;
        wide_load((has_de ? a.de : a.x) + src * WL, q, dr);  // (no de: re-reads x, replaced by zeros)
        if (has_agg) {
          const float* gp = a.dagg + (a.recv ? (int64_t)a.recv[src] : src) * WL;
#pragma unroll
          for (int cb = 0; cb < WNB; ++cb) dm[cb] = rt_ld4(gp, cb, q);
        } else {
#pragma unroll
          for (int cb = 0; cb < WNB; ++cb) dm[cb] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kg = 0; kg < WNK; ++kg) raw[kg] = rt_from_plain(raw[kg]);
        rt_gemm<WNB, WNK>(W, raw, acc, ln);
        float g[WNB][4];  // dm
#pragma unroll
        for (int kg = 0; kg < WNK; ++kg) {
          float lo[4] = {0.f, 0.f, 0.f, 0.f}, hi[4] = {0.f, 0.f, 0.f, 0.f};
          rw_unpack(has_de ? dr[kg] : make_uint4(0u, 0u, 0u, 0u), lo, hi);
          const float4 d0 = dm[2 * kg], d1 = dm[2 * kg + 1];
          const float a0[4] = {d0.x, d0.y, d0.z, d0.w}, a1[4] = {d1.x, d1.y, d1.z, d1.w};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            g[2 * kg][r] = ok ? a0[r] + lo[r] : 0.f;
            g[2 * kg + 1][r] = ok ? a1[r] + hi[r] : 0.f;
          }
        }
#pragma unroll
        for (int cb = 0; cb < WNB; ++cb) {
          const float4 b4 = rt_ld4(vb, cb, q);
          v[cb][0] = acc[cb][0] + b4.x;
          v[cb][1] = acc[cb][1] + b4.y;
          v[cb][2] = acc[cb][2] + b4.z;
          v[cb][3] = acc[cb][3] + b4.w;
        }
        // LayerNorm (v becomes xhat), then its backward
        const float mu = rt_sum4(rt_lane_sum<WNB>(v)) / WL;
        float s2 = 0.f;
#pragma unroll
        for (int cb = 0; cb < WNB; ++cb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float d = v[cb][r] - mu;
            s2 += d * d;
          }
        const float rs = 1.0f / sqrtf(rt_sum4(s2) / WL + a.eps);
        float u1 = 0.f, u2 = 0.f;
#pragma unroll
        for (int cb = 0; cb < WNB; ++cb) {
          const float4 g4 = rt_ld4(vg, cb, q);
          const float gm[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v[cb][r] = (v[cb][r] - mu) * rs;
            const float d = g[cb][r] * gm[r];
            u1 += d;
            u2 += d * v[cb][r];
          }
        }
        u1 = rt_sum4(u1) / WL;
        u2 = rt_sum4(u2) / WL;
        wide_coltot(g, qacc[2], e);  // beta
#pragma unroll
        for (int cb = 0; cb < WNB; ++cb) {
          const float4 g4 = rt_ld4(vg, cb, q);
          const float gm[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float xh = v[cb][r];
            v[cb][r] = rs * (g[cb][r] * gm[r] - u1 - xh * u2);
            g[cb][r] *= xh;
          }
        }
        wide_coltot(g, qacc[1], e);  // gamma
        wide_coltot(v, qacc[0], e);  // last bias
      } else {
        uint4 hr[WNK];
        if constexpr (KIND == W_MASK) wide_load(a.h + src * WL, q, hr);
#pragma unroll
        for (int kg = 0; kg < WNK; ++kg) raw[kg] = rt_from_plain(raw[kg]);
        rt_gemm<WNB, WNK>(W, raw, acc, ln);
        if constexpr (KIND == W_MASK) {
#pragma unroll
          for (int kg = 0; kg < WNK; ++kg) hr[kg] = rt_from_plain(hr[kg]);
#pragma unroll
          for (int cb = 0; cb < WNB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[cb][r] = ok && rt_relu_on<WNK>(hr, cb, r) ? acc[cb][r] : 0.f;
          wide_coltot(v, qacc[0], e);
        }
      }
    }
    if constexpr (KIND == W_ENC || KIND == W_HID) {
#pragma unroll
      for (int cb = 0; cb < WNB; ++cb) {
        const float4 b4 = rt_ld4(vb, cb, q);
        v[cb][0] = fmaxf(acc[cb][0] + b4.x, 0.f);
        v[cb][1] = fmaxf(acc[cb][1] + b4.y, 0.f);
        v[cb][2] = fmaxf(acc[cb][2] + b4.z, 0.f);
        v[cb][3] = fmaxf(acc[cb][3] + b4.w, 0.f);
      }
    }
    if constexpr (KIND == W_OUT) {
      if (ok) {
#pragma unroll
        for (int cb = 0; cb < WNB; ++cb) {
          float4 d = make_float4(0.f, 0.f, 0.f, 0.f);
          if (a.dagg) d = rt_ld4(a.dagg + row * WL, cb, q);
          *reinterpret_cast<float4*>(a.out32 + row * WL + cb * 16 + q * 4) =
              make_float4(acc[cb][0] + d.x, acc[cb][1] + d.y, acc[cb][2] + d.z, acc[cb][3] + d.w);
        }
      }
    } else {
      uint4 o[WNK];
      rt_frags<WNB>(v, o);
      rt_store_frags<WNK>(a.out + row * WL, q, o, ok);
    }
  }
  if constexpr (KIND == W_LNB || KIND == W_MASK) wide_vec<NQ>(qacc, lds, a);
}

// ------------------------------------------------------ rows in receiver order ---
// de^k = de + W^T x (fp32 sum, stored as bf16), receiver sums of x over the
// consumed dagg rows.
__global__ __launch_bounds__(W_NTH) __attribute__((amdgpu_waves_per_eu(2, 2))) void wide_de_kernel(WideArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  uint4* W = reinterpret_cast<uint4*>(lds);
  const int wave = wave_id(), lane = threadIdx.x & 63;
  uint16_t* scr = reinterpret_cast<uint16_t*>(lds + W_OFF_SCR + wave * 2048);
  const RsEmpty empty = rs_empty_load(a.row_ptr, a.r_lo, a.r_hi);
  int64_t E0, E1;
  rs_range_e(a.row_ptr, a.recv, a.e_lo, a.rows, W_NWV, wave, E0, E1);
  wide_copy<true>(W, a.w, a.src_nkg);
  __syncthreads();
  rs_zero_empty(empty, a.row_ptr, a.sum, WL);
  if (E0 >= E1) return;
  float run[WL / 64] = {};
  RsMeta mt_next = rt_meta_make(rt_meta_load(a.recv, a.send, E0, E1));
  const uint32_t keep = a.de ? 0xffffffffu : 0u;  // without de^{k+1} (last block) x is read again and replaced by zeros
  for (int64_t sb = E0; sb < E1; sb += 16) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int e = ln & 15, q = ln >> 4;
    const int n = (int)(E1 - sb < 16 ? E1 - sb : 16);
    const bool ok = e < n;
    const RsMeta mt = mt_next;
    const RsMetaRaw nxt = rt_meta_load(a.recv, a.send, sb + 16, E1);
    const int64_t row = sb - a.e_lo + e, src = sb - a.e_lo + (ok ? e : 0);
    uint4 raw[WNK], er[WNK];
    wide_load(a.x + src * WL, q, raw);
    wide_load((a.de ? a.de : a.x) + src * WL, q, er);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kg = 0; kg < WNK; ++kg) raw[kg] = rt_from_plain(raw[kg]);
    floatx4 acc[WNB];
    rt_gemm<WNB, WNK>(W, raw, acc, ln);
    mt_next = rt_meta_make(nxt);
    uint4 o[WNK];
#pragma unroll
    for (int kg = 0; kg < WNK; ++kg) {
      float lo[4], hi[4];
      rw_unpack(make_uint4(er[kg].x & keep, er[kg].y & keep, er[kg].z & keep, er[kg].w & keep), lo, hi);
      const floatx4 m0 = acc[2 * kg], m1 = acc[2 * kg + 1];
      o[kg] = rt_to_plain(make_uint4(bf_pack(lo[0] + m0[0], lo[1] + m0[1]), bf_pack(lo[2] + m0[2], lo[3] + m0[3]),
                                     bf_pack(hi[0] + m1[0], hi[1] + m1[1]), bf_pack(hi[2] + m1[2], hi[3] + m1[3])));
    }
    if (ok) {
      uint16_t* op = a.out + row * WL;
#pragma unroll
      for (int kg = 0; kg < WNK; ++kg) *reinterpret_cast<uint4*>(op + kg * 32 + q * 8) = o[kg];
    }
    // ordered receiver sums of x, 64 columns at a time through the wave's
    // scratch tile; a segment's total goes out at its last row
#pragma unroll
    for (int j = 0; j < WL / 64; ++j) {
#pragma unroll
      for (int kg = 2 * j; kg < 2 * j + 2; ++kg) {
        const int c0 = (kg - 2 * j) * 32 + q * 4;
        *reinterpret_cast<uint2*>(scr + rs_sw16<64>(e, c0)) = make_uint2(raw[kg].x, raw[kg].y);
        *reinterpret_cast<uint2*>(scr + rs_sw16<64>(e, c0 + 16)) = make_uint2(raw[kg].z, raw[kg].w);
      }
      float x[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = bf2f(scr[rs_sw16<64>(r, ln)]);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (r < n) {
          run[j] += x[r];
          if ((mt.last >> r) & 1ull) {
            a.sum[(int64_t)__builtin_amdgcn_readlane(mt.r, r) * WL + ln + 64 * j] = run[j];
            run[j] = 0.f;
          }
        }
      }
    }
  }
}

template <class F>
hipError_t wide_launch(F* fn, const WideArgs& a, hipStream_t st) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, W_END);
  hipLaunchKernelGGL(fn, dim3(RS_GRID), dim3(W_NTH), W_END, st, a);
  return hipGetLastError();
}

}  // namespace

bool edge_wide(int prec, int L, int D, int64_t edges) {
  return prec == BF16 && L == WL && (D == 2 || D == 3) && edges >= WIDE_ROWS;
}

namespace {

// From h_1 (h[0]) and, at depth 3, room for h_2 (h[1]): the layers after the
// first recomputed and differentiated, dz_0 into d[0].  a: rows, de, dagg,
// recv, eps, vpart, nvec set.
hipError_t wide_mlp_bwd(int D, const Mlp& m, WideArgs a, uint16_t* const (&h)[2], void* const (&d)[3],
                        hipStream_t st) {
  hipError_t e = hipSuccess;
  a.src_nkg = WNK;
  if (D == 3) {
    a.w = m.lin[1].wf;
    a.b = m.lin[1].b;
    a.x = h[0];
    a.out = h[1];
    e = wide_launch(wide_rows_kernel<W_HID>, a, st);
  }
  a.w = m.lin[D - 1].wf;
  a.b = m.lin[D - 1].b;
  a.gamma = m.gamma;
  a.x = h[D - 2];
  a.out = reinterpret_cast<uint16_t*>(d[D - 1]);
  a.voff = (D - 1) * WL;
  if (e == hipSuccess) e = wide_launch(wide_rows_kernel<W_LNB>, a, st);
  for (int j = D - 1; j >= 1 && e == hipSuccess; --j) {
    a.w = m.lin[j].wb;
    a.x = reinterpret_cast<const uint16_t*>(d[j]);
    a.out = reinterpret_cast<uint16_t*>(d[j - 1]);
    a.h = h[j - 1];
    a.voff = (j - 1) * WL;
    e = wide_launch(wide_rows_kernel<W_MASK>, a, st);
  }
  return e;
}

}  // namespace

hipError_t launch_edge_bwd_wide(int D, const EdgeBwdArgs& b, int64_t rows, hipStream_t st) {
  const int64_t e0 = b.e_base;
  WideArgs a{};
  a.rows = rows;
  a.eps = b.eps;
  a.send = b.send + e0;
  a.recv = b.erecv + e0;
  a.vpart = b.vpart;
  a.nvec = b.nvec;
  uint16_t* h1 = reinterpret_cast<uint16_t*>(b.hid[0]);
  hipError_t e = hipSuccess;
  if (b.hid_in) {
    h1 = const_cast<uint16_t*>(reinterpret_cast<const uint16_t*>(b.hid_in)) + e0 * WL;
  } else {
    if (!b.proj) return hipErrorInvalidValue;
    a.w = b.mlp.lin[0].wf;
    a.src_nkg = 3 * WNK;
    a.x = reinterpret_cast<const uint16_t*>(b.Ein) + e0 * WL;
    a.out = h1;
    a.proj = b.proj;
    e = wide_launch(wide_rows_kernel<W_EDGE1>, a, st);
    if (e != hipSuccess) return e;
  }
  a.dagg = b.dagg;
  a.de = b.de_next ? reinterpret_cast<const uint16_t*>(b.de_next) + e0 * WL : nullptr;
  uint16_t* const h[2] = {h1, reinterpret_cast<uint16_t*>(b.hid[1])};
  e = wide_mlp_bwd(D, b.mlp, a, h, b.delta, st);
  if (e != hipSuccess) return e;
  a.w = b.mlp.lin[0].wb;
  a.src_nkg = WNK;
  a.x = reinterpret_cast<const uint16_t*>(b.delta[0]);
  a.out = reinterpret_cast<uint16_t*>(b.de_out) + e0 * WL;
  a.send = b.send;
  a.recv = b.erecv;
  a.row_ptr = b.row_ptr;
  a.r_lo = b.r_lo;
  a.r_hi = b.r_hi;
  a.e_lo = e0;
  a.sum = b.dagg;
  return wide_launch(wide_de_kernel, a, st);
}

bool rows_wide(int prec, int L, int D, int kind, int64_t rows) {
  return kind != DECODER && edge_wide(prec, L, D, rows);
}

hipError_t launch_rows_bwd_wide(int D, int kind, const RowsBwdArgs& b, hipStream_t st) {
  WideArgs a{};
  a.rows = b.rows;
  a.eps = b.eps;
  a.vpart = b.vpart;
  a.nvec = b.nvec;
  uint16_t* h1 = reinterpret_cast<uint16_t*>(b.hid[0]);
  hipError_t e = hipSuccess;
  if (kind == NODE_BLOCK) {
    if (!b.hid_in) return hipErrorInvalidValue;
    h1 = const_cast<uint16_t*>(reinterpret_cast<const uint16_t*>(b.hid_in));
  } else {
    a.w = b.mlp.lin[0].wf;
    a.src_nkg = b.mlp.lin[0].nkgf;
    a.b = b.mlp.lin[0].b;
    a.feat = b.in0;
    a.fin = b.fin;
    a.out = h1;
    e = wide_launch(wide_rows_kernel<W_ENC>, a, st);
    if (e != hipSuccess) return e;
  }
  if (b.dm16) a.de = b.dm16;
  else a.dagg = b.dm;
  uint16_t* const h[2] = {h1, reinterpret_cast<uint16_t*>(b.hid[1])};
  e = wide_mlp_bwd(D, b.mlp, a, h, b.delta, st);
  for (int pass = 0; pass < 2 && kind == NODE_BLOCK && e == hipSuccess; ++pass) {
    // dv = dm + dz_0 W_1[:, v-block], dagg = dz_0 W_1[:, agg-block]
    a.w = b.mlp.lin[0].wb + (size_t)pass * WNB * WNK * 64;
    a.src_nkg = WNK;
    a.x = reinterpret_cast<const uint16_t*>(b.delta[0]);
    a.dagg = pass == 0 ? b.dm : nullptr;
    a.out32 = pass == 0 ? b.dx0 : b.dx1;
    e = wide_launch(wide_rows_kernel<W_OUT>, a, st);
  }
  return e;
}

}  // namespace mgn
