// Weight gradients in groups (gfx950): dW = D^T A over rows for a list of
// jobs in one launch, then one launch that adds the partials of all of them
// and the bias / LayerNorm partials of the group's row kernels.
//
// A job's output is cut into 64 x 64 tiles; a wave (a unit) reduces one tile
// over a contiguous range of rows in its accumulator registers, without LDS
// or barriers, and the units of all jobs share one grid of about two waves
// per SIMD.  Small graphs are what this shape is for: a block has seven to
// nine such products of a few thousand rows, and one launch each (42 us, a
// few workgroups that wait for their loads) plus one per reduction was a third
// of a training step; see dw_plan for the split.
//
// fp32: the 16x16x4 MFMA takes one value per lane, so row-major loads need no
// transpose: lane (q, m) = (lane >> 4, lane & 15) loads columns 4 m .. + 3 of
// row q of both operands, and accumulator block (c, c') holds
// dW[4 i + c][4 j + c'] at (i, j) of its 16 x 16 tile.  bf16: lane (q, m) loads
// the same four columns of rows 8 q .. + 7 and transposes them in registers
// (v_perm) into 16x16x32 k-fragments; the block layout is the same.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "tform.h"

namespace mgn {

namespace {

constexpr int DG_NT = 256;

__device__ __forceinline__ float4 dg_zero4() { return make_float4(0.f, 0.f, 0.f, 0.f); }

// ------------------------------------------------------------------- fp32 ---
// One 16-row step: D and A values of rows row0 + 4 g + q (zero past R).
// AVEC: A's rows are 16-byte aligned; otherwise (node features, 11 wide) its
// columns are read one by one.
template <bool AVEC>
__device__ __forceinline__ void dg_load_f32(const DwJob& j, int64_t row0, int q, int oc, int ic, float4 (&d)[4],
                                            float4 (&a)[4]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int64_t row = row0 + 4 * g + q;
    const bool ok = row < j.R;
    const int64_t r = ok ? row : j.R - 1;
    d[g] = dg_zero4();
    a[g] = dg_zero4();
    if (ok && oc < j.ldd) d[g] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(j.D) + r * j.ldd + oc);
    const float* ap = r < j.n_first ? reinterpret_cast<const float*>(j.A) + r * j.lda
                                    : reinterpret_cast<const float*>(j.A2) + (r - j.n_first) * j.lda;
    if constexpr (AVEC) {
      if (ok && ic < j.I) a[g] = *reinterpret_cast<const float4*>(ap + ic);
    } else {
      if (ok && ic < j.I) a[g].x = ap[ic];
      if (ok && ic + 1 < j.I) a[g].y = ap[ic + 1];
      if (ok && ic + 2 < j.I) a[g].z = ap[ic + 2];
      if (ok && ic + 3 < j.I) a[g].w = ap[ic + 3];
    }
  }
}

__device__ __forceinline__ float dg_c(const float4& v, int c) { return c == 0 ? v.x : c == 1 ? v.y : c == 2 ? v.z : v.w; }

template <bool AVEC>
__device__ __forceinline__ void dg_run_f32(const DwJob& j, int64_t s0, int64_t s1, int q, int oc, int ic,
                                           floatx4 (&acc)[4][4]) {
  float4 d[4], a[4], dn[4], an[4];
  if (s0 < s1) dg_load_f32<AVEC>(j, s0 * 16, q, oc, ic, dn, an);
  for (int64_t st = s0; st < s1; ++st) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      d[g] = dn[g];
      a[g] = an[g];
    }
    if (st + 1 < s1) dg_load_f32<AVEC>(j, (st + 1) * 16, q, oc, ic, dn, an);
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int cc = 0; cc < 4; ++cc)
          acc[c][cc] = __builtin_amdgcn_mfma_f32_16x16x4f32(dg_c(d[g], c), dg_c(a[g], cc), acc[c][cc], 0, 0, 0);
  }
}

// ------------------------------------------------------------------- bf16 ---
// Rows 8 q .. 8 q + 7 of a 32-row step, four columns, as bf16 pairs v[r][k]
// (columns 2 k, 2 k + 1); fp32 sources stay fp32 in x.
template <bool F32, bool VEC>
__device__ __forceinline__ void dg_load_bf16(const void* p, int ld, int64_t row, int64_t R, int col, int cols,
                                             uint2 (&v)[8], float4 (&x)[8]) {
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const bool ok = row + r < R;
    const int64_t rr = ok ? row + r : R - 1;
    if constexpr (F32) {
      const float* s = reinterpret_cast<const float*>(p) + rr * ld;
      x[r] = dg_zero4();
      if constexpr (VEC) {
        if (ok && col < cols) x[r] = *reinterpret_cast<const float4*>(s + col);
      } else {
        if (ok && col < cols) x[r].x = s[col];
        if (ok && col + 1 < cols) x[r].y = s[col + 1];
        if (ok && col + 2 < cols) x[r].z = s[col + 2];
        if (ok && col + 3 < cols) x[r].w = s[col + 3];
      }
    } else {
      v[r] = make_uint2(0u, 0u);
      if (ok && col < cols) v[r] = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(p) + rr * ld + col);
    }
  }
}

__device__ __forceinline__ uint32_t dg_pack(float a, float b) { return (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16); }

__device__ __forceinline__ void dg_round(const float4 (&x)[8], uint2 (&v)[8]) {
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = make_uint2(dg_pack(x[r].x, x[r].y), dg_pack(x[r].z, x[r].w));
}
// x = hi + lo within 2^-17 of it (relative), both bf16
__device__ __forceinline__ void dg_split(const float4 (&x)[8], uint2 (&hi)[8], uint2 (&lo)[8]) {
  dg_round(x, hi);
#pragma unroll
  for (int r = 0; r < 8; ++r)
    lo[r] = make_uint2(
        dg_pack(x[r].x - __uint_as_float(hi[r].x << 16), x[r].y - __uint_as_float(hi[r].x & 0xffff0000u)),
        dg_pack(x[r].z - __uint_as_float(hi[r].y << 16), x[r].w - __uint_as_float(hi[r].y & 0xffff0000u)));
}

// v[r] (row r, columns 2 k low / 2 k + 1 high of dword k) -> k-fragments f[c]
// of column c: dword p holds rows 2 p (low) and 2 p + 1.
__device__ __forceinline__ void dg_transpose(const uint2 (&v)[8], uint4 (&f)[4]) {
  uint32_t t[4][4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    t[0][p] = __builtin_amdgcn_perm(v[2 * p + 1].x, v[2 * p].x, 0x05040100u);
    t[1][p] = __builtin_amdgcn_perm(v[2 * p + 1].x, v[2 * p].x, 0x07060302u);
    t[2][p] = __builtin_amdgcn_perm(v[2 * p + 1].y, v[2 * p].y, 0x05040100u);
    t[3][p] = __builtin_amdgcn_perm(v[2 * p + 1].y, v[2 * p].y, 0x07060302u);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) f[c] = make_uint4(t[c][0], t[c][1], t[c][2], t[c][3]);
}

__device__ __forceinline__ void dg_mma(const uint4 (&fd)[4], const uint4 (&fa)[4], floatx4 (&acc)[4][4]) {
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) PBF16::mma(acc[c][cc], fd[c], fa[cc]);
}

template <bool D32, bool A32, bool AVEC>
__device__ __forceinline__ void dg_run_bf16(const DwJob& j, int64_t s0, int64_t s1, int q, int oc, int ic,
                                            floatx4 (&acc)[4][4]) {
  uint2 dv[8], av[8];
  float4 dx[8], ax[8];
  auto load = [&](int64_t st) {
    dg_load_bf16<D32, true>(j.D, j.ldd, st * 32 + 8 * q, j.R, oc, j.ldd, dv, dx);
    dg_load_bf16<A32, AVEC>(j.A, j.lda, st * 32 + 8 * q, j.R, ic, j.I, av, ax);
  };
  if (s0 < s1) load(s0);
  for (int64_t st = s0; st < s1; ++st) {
    uint4 fd[4], fl[4], fa[4];
    if constexpr (D32) {
      uint2 hi[8], lo[8];
      dg_split(dx, hi, lo);
      dg_transpose(hi, fd);
      dg_transpose(lo, fl);
    } else {
      dg_transpose(dv, fd);
    }
    if constexpr (A32) dg_round(ax, av);
    dg_transpose(av, fa);
    if (st + 1 < s1) load(st + 1);
    dg_mma(fd, fa, acc);
    if constexpr (D32) dg_mma(fl, fa, acc);
  }
}

// ---------------------------------------------------------------- kernels ---
// Unit u of the group: job by first unit, then row split s and tile t (tiles
// fastest: a workgroup's waves share their rows in the cache).
template <int P_>
__global__ __launch_bounds__(DG_NT) __attribute__((amdgpu_waves_per_eu(2))) void dw_group_kernel(DwGroup g) {
  // blocks are dealt round-robin to the 8 XCDs: neighbouring units stay on one
  const int per = (gridDim.x + 7) >> 3;
  const int vb = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  const int u = vb * (DG_NT / 64) + wave_id();
  if (u >= g.units) return;
  int ji = 0;
  while (ji + 1 < g.n && u >= g.job[ji + 1].unit0) ++ji;
  const DwJob j = g.job[ji];
  const int s = (u - j.unit0) / j.tiles, t = (u - j.unit0) % j.tiles;
  const int lane = threadIdx.x & 63, q = lane >> 4, m = lane & 15;
  const int oc = (t / j.ti) * 64 + 4 * m, ic = (t % j.ti) * 64 + 4 * m;
  floatx4 acc[4][4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) acc[c][cc] = floatx4{0.f, 0.f, 0.f, 0.f};
  constexpr int STEP = P_ == F32 ? 16 : 32;
  const int64_t steps = (j.R + STEP - 1) / STEP;
  const int64_t s0 = steps * s / j.S, s1 = steps * (s + 1) / j.S;
  if constexpr (P_ == F32) {
    if (j.avec) dg_run_f32<true>(j, s0, s1, q, oc, ic, acc);
    else dg_run_f32<false>(j, s0, s1, q, oc, ic, acc);
  } else {
    if (j.d32) dg_run_bf16<true, false, true>(j, s0, s1, q, oc, ic, acc);
    else if (!j.a32) dg_run_bf16<false, false, true>(j, s0, s1, q, oc, ic, acc);
    else if (j.avec) dg_run_bf16<false, true, true>(j, s0, s1, q, oc, ic, acc);
    else dg_run_bf16<false, true, false>(j, s0, s1, q, oc, ic, acc);
  }
  float4* out = reinterpret_cast<float4*>(g.part) + (int64_t)u * 1024 + lane;
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int cc = 0; cc < 4; ++cc)
      out[(c * 4 + cc) * 64] = make_float4(acc[c][cc][0], acc[c][cc][1], acc[c][cc][2], acc[c][cc][3]);
}

// dst (+)= sum of the partials, in a fixed order: block (job, tile,
// accumulator block), four threads per 16 bytes each summing the splits
// k = set (mod 4) in ascending k, combined in set order.  Then the vector
// partials: 16 outputs per block, 16 sets of slots.
__global__ __launch_bounds__(DG_NT) void dw_group_reduce_kernel(DwGroup g) {
  __shared__ float4 sh[DG_NT];
  const int tid = threadIdx.x;
  int b = blockIdx.x;
  for (int ji = 0; ji < g.n; ++ji) {
    const DwJob& j = g.job[ji];
    const int nb = j.tiles * 16;
    if (b >= nb) {
      b -= nb;
      continue;
    }
    const int t = b >> 4, blk = b & 15, lane = tid & 63, set = tid >> 6;
    const float4* p = reinterpret_cast<const float4*>(g.part) + ((int64_t)(j.unit0 + t) * 16 + blk) * 64 + lane;
    float4 x = dg_zero4();
#pragma unroll 8
    for (int k = set; k < j.S; k += 4) {
      const float4 y = p[(int64_t)k * j.tiles * 1024];
      x.x += y.x;
      x.y += y.y;
      x.z += y.z;
      x.w += y.w;
    }
    sh[tid] = x;
    __syncthreads();
    if (set == 0) {
      const float4 a = sh[lane], c = sh[64 + lane], d = sh[128 + lane], e = sh[192 + lane];
      const float v[4] = {((a.x + c.x) + d.x) + e.x, ((a.y + c.y) + d.y) + e.y, ((a.z + c.z) + d.z) + e.z,
                          ((a.w + c.w) + d.w) + e.w};
      const int i = (t % j.ti) * 64 + 4 * (lane & 15) + (blk & 3);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = (t / j.ti) * 64 + 4 * (4 * (lane >> 4) + r) + (blk >> 2);
        if (o < j.O && i < j.I) {
          float* d1 = j.dst + (int64_t)o * j.ldw + i;
          *d1 = (j.accumulate ? *d1 : 0.f) + v[r];
        }
      }
    }
    return;
  }
  float* shf = reinterpret_cast<float*>(sh);
  for (int vi = 0; vi < g.nv; ++vi) {
    const DwVec& w = g.vec[vi];
    const int nb = (w.nvec + 15) / 16;
    if (b >= nb) {
      b -= nb;
      continue;
    }
    const int c = tid & 15, set = tid >> 4, i = b * 16 + c;
    float x = 0.f;
    if (i < w.nvec) {
#pragma unroll 8
      for (int k = set; k < w.slots; k += 16) x += w.part[(int64_t)k * w.nvec + i];
    }
    shf[tid] = x;
    __syncthreads();
    if (set == 0 && i < w.nvec) {
      float v = shf[c];
#pragma unroll
      for (int k = 1; k < 16; ++k) v += shf[16 * k + c];
      for (int k = 0; k < w.nseg; ++k) {
        const VecSeg& sg = w.seg[k];
        if (i >= sg.vec_off && i < sg.vec_off + sg.len) {
          float* d1 = w.dst + sg.param_off + (i - sg.vec_off);
          *d1 = (w.accumulate ? *d1 : 0.f) + v;
        }
      }
    }
    return;
  }
}

// Row splits of every job.  About 2,048 units in all (two waves per SIMD),
// shared among the jobs by rows x tiles; at least 64 rows each, since a unit's
// 16 KiB of partials, written and read back, cost what about 30 rows of its
// products do.  At most DW_MAX_UNITS units (the partials' workspace).
void dw_plan(DwGroup& g) {
  double cost = 0;
  for (int i = 0; i < g.n; ++i) cost += (double)g.job[i].tiles * g.job[i].R;
  int u = 0;
  for (int i = 0; i < g.n; ++i) {
    DwJob& j = g.job[i];
    int64_t s = cost > 0 ? (int64_t)(2048.0 * j.R / cost) : 0;
    const int64_t most = (j.R + 63) / 64;
    if (s > most) s = most;
    if (s < 1) s = j.R > 0 ? 1 : 0;
    j.S = (int)s;
    j.unit0 = u;
    u += j.S * j.tiles;
  }
  g.units = u;
}

}  // namespace

hipError_t launch_dw_group(int prec, DwGroup& g, hipStream_t st) {
  if (g.n == 0 && g.nv == 0) return hipSuccess;
  dw_plan(g);
  if (g.units > DW_MAX_UNITS) return hipErrorInvalidValue;
  if (g.units > 0) {
    const unsigned blocks = (unsigned)((g.units + DG_NT / 64 - 1) / (DG_NT / 64));
    const dim3 grid((blocks + 7) / 8 * 8);
    if (prec == F32) hipLaunchKernelGGL((dw_group_kernel<F32>), grid, dim3(DG_NT), 0, st, g);
    else hipLaunchKernelGGL((dw_group_kernel<BF16>), grid, dim3(DG_NT), 0, st, g);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  int blocks = 0;
  for (int i = 0; i < g.n; ++i) blocks += g.job[i].tiles * 16;
  for (int i = 0; i < g.nv; ++i) blocks += (g.vec[i].nvec + 15) / 16;
  hipLaunchKernelGGL(dw_group_reduce_kernel, dim3(blocks), dim3(DG_NT), 0, st, g);
  return hipGetLastError();
}

}  // namespace mgn
