// Initialisation path of the reconstruction (Sec. 3.1): an FDK
// reconstruction of the projections, then Gaussian means sampled with
// probability proportional to the gradient magnitude of the
// background-thresholded FDK volume, densities k times the FDK intensity at
// the sample, zero rotation, scale equal to the nearest-neighbour distance.
//
// FDK (Feldkamp, Davis and Kress) for a full circular scan on a flat
// detector, discretised on the detector rescaled to the rotation axis
// (pitch p' = pitch * sod / sdd, coordinates a', b'):
//   weight    pw = p * sod / sqrt(sod^2 + a'^2 + b'^2)
//   filter    q[n] = p' sum_k h[n - k] pw[k],  h[0] = 1 / (4 p'^2),
//             h[m odd] = -1 / (pi^2 m^2 p'^2), h[m even] = 0  (Ram-Lak)
//   backproject f(x) = 1/2 * (2 pi / V) * sum_views (sod / t2)^2 q(u(x), v(x))
// with t2 the depth of x along the central ray, (u, v) the detector pixel
// coordinates of x's projection (the rasterizer's camera model), bilinear
// interpolation between pixel centres and zero outside the detector.
//
// Sampling is exact in integers: per-voxel weights are the FP32 gradient
// magnitude (or, for intensity sampling, the thresholded value) quantised to
// 24 bits of its maximum, their 64-bit prefix sum is
// the CDF, and draw i takes the voxel whose CDF interval holds
// floor(u_i * total) (u_i given, FP64).
#include <algorithm>
#include <cmath>

#include "fgs_internal.h"

namespace fgs {
namespace {

constexpr int kMaxFilterRow = 8192;

// The ramp filter as a product of matrices. The Ram-Lak taps are zero at even
// distances, so apart from the centre tap an even sample is filtered from the
// odd ones and an odd sample from the even ones: two half-size Toeplitz
// products, out[r][2a + p] = sum_b pw[r][2b + 1 - p] G[a - b + p], with
// G[d] = h[2d - 1]. They run on v_mfma_f32_32x32x2_f32 (FP32 operands, FP32
// accumulation). A workgroup of 8 waves takes 32 rows and kFilterSeg output
// samples; per input segment it stages the weighted samples by parity
// (stride 258: the 32 rows and the two reduction slots of an operand read fall
// in 64 different banks) and the 512 taps that the segment pair needs, so the
// tap's division is made once per 32 rows instead of once per product. Wave w
// owns two 32 x 32 result tiles of one parity. Bound by the matrix cores' FP32
// rate (64 cycles per instruction, W^2 / 2 products per row: 65 us for 75
// views of 512^2). Measured there: 2.39 ms with a thread per sample, a
// division and two LDS reads per tap; 0.130 ms now.
constexpr int kFilterRows = 32;
constexpr int kFilterSeg = 512;
constexpr int kFilterHalf = kFilterSeg / 2;
constexpr int kFilterPiece = 32;
constexpr int kFilterStride = kFilterHalf + 2;
typedef float f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(512) void fdk_filter_kernel(const float *__restrict__ img, int W, int H, int64_t n_rows,
                                                         float sod, float pu, float pv, float cu, float cv,
                                                         float *__restrict__ q) {
  __shared__ float s_pw[2][kFilterRows][kFilterStride];
  __shared__ float s_tap[2 * kFilterHalf];
  const int64_t r0 = int64_t(blockIdx.x) * kFilterRows;
  const int nr = int(min(int64_t(kFilterRows), n_rows - r0));
  const int h0 = int(r0 % H);
  const int A0 = int(blockIdx.y) * kFilterHalf;  // first output pair of the segment
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int par = wid & 1;                       // parity of this wave's outputs
  const int at = (wid >> 1) * 64;                // its tiles: pairs A0 + at .. + 31 and + 32 .. + 63
  const int l32 = lane & 31, lh = lane >> 5;
  const float pi2 = 9.8696044010893586f;
  const float inv = 1.f / (pu * pu);
  f32x16 acc0 = {0.f}, acc1 = {0.f};
  const int n_seg = (W + kFilterSeg - 1) / kFilterSeg;
  for (int sg = 0; sg < n_seg; ++sg) {
    const int j0 = sg * kFilterSeg;
    const int d0 = A0 - sg * kFilterHalf - (kFilterHalf - 1);  // G index of s_tap[0]
    __syncthreads();
    {
      const int d = d0 + int(threadIdx.x);
      const float m = float(2 * d - 1);
      // The neighbours' taps come below; not zero here, so that an infinite
      // sample adds its infinity to the neighbours and not a NaN (a finite one
      // adds nothing that its own tap's 1e-38th part would show).
      s_tap[threadIdx.x] = fabsf(m) > 1.f ? -inv / (pi2 * m * m) : -1e-37f;
    }
    const int j = j0 + int(threadIdx.x);
    const float a = (float(j) + 0.5f - cu) * pu;
    const float wa = sod * sod + a * a;
    for (int r = 0; r < kFilterRows; ++r) {
      float v = 0.f;
      if (r < nr && j < W) {
        const float b = (float((h0 + r) % H) + 0.5f - cv) * pv;
        v = img[(r0 + r) * int64_t(W) + j] * sod / sqrtf(wa + b * b);
      }
      s_pw[threadIdx.x & 1][r][threadIdx.x >> 1] = v;
    }
    // the samples just before and just after the segment, one row per thread
    if (threadIdx.x < 2 * kFilterRows) {
      const int r = threadIdx.x >> 1, jn = (threadIdx.x & 1) ? j0 - 1 : j0 + kFilterSeg;
      float v = 0.f;
      if (r < nr && jn >= 0 && jn < W) {
        const float an = (float(jn) + 0.5f - cu) * pu, b = (float((h0 + r) % H) + 0.5f - cv) * pv;
        v = img[(r0 + r) * int64_t(W) + jn] * sod / sqrtf(sod * sod + an * an + b * b);
      }
      s_pw[threadIdx.x & 1][r][kFilterHalf] = v;
    }
    __syncthreads();
    const float *ain = &s_pw[1 - par][l32][lh];
    const float *tap = &s_tap[at + l32 - lh + par + kFilterHalf - 1];
    if (2 * (A0 + at) + par < W) {
      // pieces of kFilterPiece products, each summed by itself and then added:
      // shorter chains of roundings than one running sum; those past the row's
      // end hold zeros (75 views of 32^2: 19.6 us with them)
      const int b_end = min(kFilterHalf, (W - j0 + 1) / 2);
      for (int b0 = 0; b0 < b_end; b0 += kFilterPiece) {
        f32x16 p0 = {0.f}, p1 = {0.f};
#pragma unroll
        for (int b = b0; b < b0 + kFilterPiece; b += 2) {
          const float x = ain[b];
          p0 = __builtin_amdgcn_mfma_f32_32x32x2f32(x, tap[-b], p0, 0, 0, 0);
          p1 = __builtin_amdgcn_mfma_f32_32x32x2f32(x, tap[32 - b], p1, 0, 0, 0);
        }
        acc0 += p0;
        acc1 += p1;
      }
      // The centre tap and its two neighbours, which cancel four fifths of it,
      // are added to each other first: no long sum is carried at the centre
      // tap's size. Result register r of lane l: row 8 (r / 4) + 4 (l / 32) +
      // r % 4, column l % 32.
      if (sg == int(blockIdx.y)) {
        const float t0 = 0.25f * inv, t1 = -inv / pi2;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = 8 * (r >> 2) + 4 * lh + (r & 3);
          const float *same = s_pw[par][row], *other = s_pw[1 - par][row];
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const int a = at + 32 * t + l32;
            const float l = other[par ? a : (a ? a - 1 : kFilterHalf)], g = other[a + par];
            const float near = fmaf(t1, l + g, t0 * same[a]);
            (t ? acc1 : acc0)[r] += near;
          }
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r >> 2) + 4 * lh + (r & 3);
    s_pw[par][row][at + l32] = pu * acc0[r];
    s_pw[par][row][at + 32 + l32] = pu * acc1[r];
  }
  __syncthreads();
  const int n = 2 * A0 + int(threadIdx.x);
  if (n < W)
    for (int r = 0; r < nr; ++r)
      q[(r0 + r) * int64_t(W) + n] = s_pw[threadIdx.x & 1][r][threadIdx.x >> 1];
}

struct FdkGeom {
  float sod, fu, fv, cu, cv;
  int W, H, views, view_begin;
  float scale;  // 1/2 * 2 pi / V
  const float *angles;
  float origin[3], h[3];
  int dims[3];
  int blocks_x;  // 16 x 16 patches of columns per row of patches
};

// Voxels from which a run is 16 long: there 16-voxel runs still give every CU 16
// waves (below, runs of 4, whose per-column work is shared by fewer samples).
constexpr uint64_t kFdkLongVoxels = uint64_t(4) << 20;

// The piece of a view that a workgroup's voxels project to: the detector
// samples from (u, w) on, cols x rows of them. cols = 0: not staged.
struct FdkPatch {
  int u, w, cols, rows;
};
constexpr int kPatchCols = 48, kPatchRows = 40, kPatchStride = 49;
constexpr int kPatchWaveRows = kPatchRows / 4;  // rows that each of the four waves stages

// A workgroup takes 16 x 16 columns of voxels (a wave 8 x 8 of them) and a run
// of RUN voxels along z. Per view the depth, its reciprocal, u and the weight
// are those of a column, and only v changes along the run. The detector piece
// that the workgroup projects to is staged in LDS, zero outside the detector
// (so no sample tests its bounds), two buffers in turn: the next view's piece
// is in flight while the current one is sampled. Read from global memory, the
// two pair gathers of a sample cost about 22 cycles each whatever their
// locality; from LDS they are two short reads. Bound by VALU issue, about 15
// instructions per sample. Measured at 75 views of 512^2 and 256^3 voxels:
// 2.79 ms with a thread per voxel, 1.48 ms with the run but global gathers,
// 0.80 ms now. A view whose piece is too large for the buffer (a
// coarse grid on a fine detector) or that holds voxels at or behind the
// source is sampled from global memory, with bounds tests.
template <int RUN>
__global__ __launch_bounds__(256) void fdk_backproject_kernel(FdkGeom G, const float *__restrict__ q,
                                                              float *__restrict__ vol) {
  __shared__ float s_cs[1024][2];
  __shared__ FdkPatch s_patch[1024];
  __shared__ float s_q[2][kPatchRows * kPatchStride];
  const int bx = int(blockIdx.x) % G.blocks_x, by = int(blockIdx.x) / G.blocks_x;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ix = bx * 16 + (wid & 1) * 8 + (lane & 7);
  const int iy = by * 16 + (wid >> 1) * 8 + (lane >> 3);
  const bool inside = ix < G.dims[0] && iy < G.dims[1];
  const int64_t nxy = int64_t(G.dims[0]) * G.dims[1];
  const int64_t idx = int64_t(iy) * G.dims[0] + ix;
  auto centre = [&](int a, int i) { return G.origin[a] + (float(i) + 0.5f) * G.h[a]; };
  const float x = centre(0, ix), y = centre(1, iy);
  const uint64_t HW = uint64_t(G.H) * uint64_t(G.W);
  const float cuh = G.cu - 0.5f, cvh = G.cv - 0.5f;
  // v of a voxel at height z, with the reciprocal depth of its column
  auto row = [&](float z, float it) { return fmaf(-G.fv * z, it, cvh); };
  // blocks step over the runs: the grid holds at most 65535 of them
  for (int iz0 = int(blockIdx.y) * RUN; iz0 < G.dims[2]; iz0 += int(gridDim.y) * RUN) {
    __syncthreads();
    // every view's piece: u and v are extreme at corners of the workgroup's
    // box; a pixel is added all round for their rounding
    for (int v = threadIdx.x; v < G.views; v += 256) {
      float sn, cs;
      sincosf(G.angles[G.view_begin + v], &sn, &cs);
      s_cs[v][0] = cs;
      s_cs[v][1] = sn;
      float u0 = INFINITY, u1 = -INFINITY, i0 = INFINITY, i1 = 0.f;
      bool ok = true;
      for (int c = 0; c < 4; ++c) {
        const float dx = centre(0, bx * 16 + (c & 1) * 15) - G.sod * cs;
        const float dy = centre(1, by * 16 + (c >> 1) * 15) - G.sod * sn;
        const float t0 = -sn * dx + cs * dy, t2 = -cs * dx - sn * dy;
        ok = ok && t2 > 0.01f * G.sod;
        const float it = 1.f / t2, u = fmaf(G.fu * t0, it, cuh);
        u0 = fminf(u0, u);
        u1 = fmaxf(u1, u);
        i0 = fminf(i0, it);
        i1 = fmaxf(i1, it);
      }
      const float za = centre(2, iz0), zb = centre(2, iz0 + RUN - 1);
      const float wa = row(za, i0), wb = row(za, i1), wc = row(zb, i0), wd = row(zb, i1);
      const float w0 = fminf(fminf(wa, wb), fminf(wc, wd)), w1 = fmaxf(fmaxf(wa, wb), fmaxf(wc, wd));
      FdkPatch P = {0, 0, 0, 0};
      if (ok && u0 > -1.0e6f && u1 < 1.0e6f && w0 > -1.0e6f && w1 < 1.0e6f) {
        P.u = int(floorf(u0)) - 1;
        P.w = int(floorf(w0)) - 1;
        const int cols = int(floorf(u1)) + 3 - P.u, rows = int(floorf(w1)) + 3 - P.w;
        if (cols <= kPatchCols && rows <= kPatchRows) {
          P.cols = cols;
          P.rows = rows;
        }
      }
      s_patch[v] = P;
    }
    __syncthreads();
    // rows wid, wid + 4, ... of a view's piece, lane = column
    float pre[kPatchWaveRows];
    auto fetch = [&](int v) {
      const FdkPatch P = s_patch[v];
      const float *qv = q + uint64_t(v) * HW;
      const int uu = P.u + lane;
#pragma unroll
      for (int j = 0; j < kPatchWaveRows; ++j) {
        const int r = wid + 4 * j, ww = P.w + r;
        pre[j] = 0.f;
        if (r < P.rows && ww >= 0 && ww < G.H && lane < P.cols && uu >= 0 && uu < G.W)
          pre[j] = qv[uint64_t(ww) * G.W + uu];
      }
    };
    auto store = [&](int v) {
      const FdkPatch P = s_patch[v];
      float *dst = s_q[v & 1];
#pragma unroll
      for (int j = 0; j < kPatchWaveRows; ++j)
        if (wid + 4 * j < P.rows && lane < P.cols) dst[(wid + 4 * j) * kPatchStride + lane] = pre[j];
    };
    float z[RUN], acc[RUN];
#pragma unroll
    for (int k = 0; k < RUN; ++k) {
      z[k] = centre(2, iz0 + k);
      acc[k] = 0.f;
    }
    fetch(0);
    store(0);
    __syncthreads();
    for (int v = 0; v < G.views; ++v) {
      if (v + 1 < G.views) fetch(v + 1);
      const float c = s_cs[v][0], s = s_cs[v][1];
      const FdkPatch P = s_patch[v];
      // t = W (x - src), rows e0 = (-s, c, 0), e1 = (0, 0, -1), e2 = (-c, -s, 0)
      const float dx = x - G.sod * c, dy = y - G.sod * s;
      const float t0 = -s * dx + c * dy;
      const float t2 = -c * dx - s * dy;
      if (inside && t2 > 0.f) {
        const float it = 1.f / t2;
        const float u = fmaf(G.fu * t0, it, cuh);
        const float u0f = floorf(u);
        const int u0 = int(u0f);
        const float fu = u - u0f, gu = 1.f - fu;
        const float wt = G.sod * it, wt2 = wt * wt;
        if (P.cols) {
          const float *base = s_q[v & 1] + (u0 - P.u) - P.w * kPatchStride;
#pragma unroll
          for (int k = 0; k < RUN; ++k) {
            const float w = row(z[k], it);
            const float w0f = floorf(w);
            const float fw = w - w0f;
            const float *p = base + __mul24(int(w0f), kPatchStride);
            const float top = fmaf(fu, p[1], gu * p[0]);
            const float bot = fmaf(fu, p[kPatchStride + 1], gu * p[kPatchStride]);
            acc[k] = fmaf(wt2, fmaf(fw, bot, (1.f - fw) * top), acc[k]);
          }
        } else {
          const float *qv = q + uint64_t(v) * HW;
          auto at = [&](uint32_t du, int w0, uint32_t dw) -> float {
            return index_inside(u0, du, G.W) && index_inside(w0, dw, G.H)
                       ? qv[uint64_t(uint32_t(w0) + dw) * G.W + (uint32_t(u0) + du)]
                       : 0.f;
          };
#pragma unroll 1
          for (int k = 0; k < RUN; ++k) {
            const float w = row(centre(2, iz0 + k), it);
            const float w0f = floorf(w);
            const int w0 = int(w0f);
            const float fw = w - w0f;
            const float top = fmaf(fu, at(1, w0, 0), gu * at(0, w0, 0));
            const float bot = fmaf(fu, at(1, w0, 1), gu * at(0, w0, 1));
            const float val = fmaf(fw, bot, (1.f - fw) * top);
#pragma unroll
            for (int j = 0; j < RUN; ++j) acc[j] = j == k ? fmaf(wt2, val, acc[j]) : acc[j];
          }
        }
      }
      if (v + 1 < G.views) store(v + 1);
      __syncthreads();
    }
    if (inside) {
#pragma unroll
      for (int k = 0; k < RUN; ++k)
        if (iz0 + k < G.dims[2]) vol[int64_t(iz0 + k) * nxy + idx] = G.scale * acc[k];
    }
  }
}

// A voxel per thread, sampled from global memory, with the arithmetic of the
// kernel above.
__global__ __launch_bounds__(256) void fdk_voxel_kernel(FdkGeom G, const float *__restrict__ q,
                                                        float *__restrict__ vol) {
  __shared__ float s_cs[1024][2];
  for (int v = threadIdx.x; v < G.views; v += 256) {
    float sn, cs;
    sincosf(G.angles[G.view_begin + v], &sn, &cs);
    s_cs[v][0] = cs;
    s_cs[v][1] = sn;
  }
  __syncthreads();
  const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t nxy = int64_t(G.dims[0]) * G.dims[1];
  if (idx >= nxy * G.dims[2]) return;
  const int iz = int(idx / nxy), ixy = int(idx - iz * nxy), iy = ixy / G.dims[0], ix = ixy - iy * G.dims[0];
  auto centre = [&](int a, int i) { return G.origin[a] + (float(i) + 0.5f) * G.h[a]; };
  const float x = centre(0, ix), y = centre(1, iy), z = centre(2, iz);
  const float cuh = G.cu - 0.5f, cvh = G.cv - 0.5f;
  float acc = 0.f;
  for (int v = 0; v < G.views; ++v) {
    const float c = s_cs[v][0], s = s_cs[v][1];
    const float dx = x - G.sod * c, dy = y - G.sod * s;
    const float t0 = -s * dx + c * dy;
    const float t2 = -c * dx - s * dy;
    if (!(t2 > 0.f)) continue;
    const float it = 1.f / t2;
    const float u = fmaf(G.fu * t0, it, cuh), w = fmaf(-G.fv * z, it, cvh);
    const float u0f = floorf(u), w0f = floorf(w);
    const int u0 = int(u0f), w0 = int(w0f);
    const float fu = u - u0f, gu = 1.f - fu, fw = w - w0f;
    const float wt = G.sod * it, wt2 = wt * wt;
    const float *qv = q + uint64_t(v) * (uint64_t(G.H) * uint64_t(G.W));
    auto at = [&](uint32_t du, uint32_t dw) -> float {
      return index_inside(u0, du, G.W) && index_inside(w0, dw, G.H)
                 ? qv[uint64_t(uint32_t(w0) + dw) * G.W + (uint32_t(u0) + du)]
                 : 0.f;
    };
    const float top = fmaf(fu, at(1, 0), gu * at(0, 0));
    const float bot = fmaf(fu, at(1, 1), gu * at(0, 1));
    acc = fmaf(wt2, fmaf(fw, bot, (1.f - fw) * top), acc);
  }
  vol[idx] = G.scale * acc;
}

// ------------------------------------------------------------ init sampling

constexpr int kRedThreads = 256;
constexpr int kRedBlocks = 1024;

__global__ __launch_bounds__(kRedThreads) void max_partial_kernel(const float *__restrict__ a, uint64_t n,
                                                                  float *__restrict__ partial) {
  __shared__ float sh[kRedThreads / 64];
  float m = -INFINITY;
  for (uint64_t i = uint64_t(blockIdx.x) * kRedThreads + threadIdx.x; i < n; i += uint64_t(gridDim.x) * kRedThreads)
    m = fmaxf(m, a[i]);
  for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = sh[0];
    for (int w = 1; w < kRedThreads / 64; ++w) t = fmaxf(t, sh[w]);
    partial[blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(kRedThreads) void max_final_kernel(const float *__restrict__ partial, int nb,
                                                                float *__restrict__ dst) {
  __shared__ float sh[kRedThreads / 64];
  float m = -INFINITY;
  for (int i = threadIdx.x; i < nb; i += kRedThreads) m = fmaxf(m, partial[i]);
  for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = sh[0];
    for (int w = 1; w < kRedThreads / 64; ++w) t = fmaxf(t, sh[w]);
    dst[0] = t;
  }
}

// Gradient magnitude (central differences, zero outside the grid) of the
// volume with voxels below background_fraction * max set to zero, and its
// maximum per workgroup. A workgroup of 64 x 4 columns walks kGradRun slices:
// the neighbours along z stay in registers and no index is divided out. Bound
// by memory: 256^3, 100 us with a thread per voxel (and 22 us for the maximum
// in a pass of its own), 59 us now.
constexpr int kGradRun = 16;

__global__ __launch_bounds__(256) void grad_mag_kernel(const float *__restrict__ vol, int nx, int ny, int nz,
                                                       float background_fraction,
                                                       const float *__restrict__ vmax,
                                                       float *__restrict__ gmag, float *__restrict__ partial) {
#pragma clang fp contract(off)
  __shared__ float sh[4];
  const float thr = background_fraction * vmax[0];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int ix = int(blockIdx.x) * 64 + lane;
  const int64_t slice = int64_t(nx) * ny;
  float m = 0.f;
  // (steps over y and z: a grid axis holds at most 65535 blocks)
  for (int iy = int(blockIdx.y) * 4 + wid; ix < nx && iy < ny; iy += int(gridDim.y) * 4) {
    const float *col = vol + int64_t(iy) * nx + ix;
    auto cut = [&](float v) { return v >= thr ? v : 0.f; };
    for (int z0 = int(blockIdx.z) * kGradRun; z0 < nz; z0 += int(gridDim.z) * kGradRun) {
      const int z1 = min(nz, z0 + kGradRun);
      float below = z0 > 0 ? cut(col[(z0 - 1) * slice]) : 0.f, here = cut(col[z0 * slice]);
      for (int z = z0; z < z1; ++z) {
        const float *p = col + z * slice;
        const float above = z + 1 < nz ? cut(p[slice]) : 0.f;
        const float xr = ix + 1 < nx ? cut(p[1]) : 0.f, xl = ix > 0 ? cut(p[-1]) : 0.f;
        const float yr = iy + 1 < ny ? cut(p[nx]) : 0.f, yl = iy > 0 ? cut(p[-nx]) : 0.f;
        const float gx = 0.5f * (xr - xl);
        const float gy = 0.5f * (yr - yl);
        const float gz = 0.5f * (above - below);
        const float sq = gx * gx + gy * gy;
        const float g = sqrtf(sq + gz * gz);
        gmag[z * slice + int64_t(iy) * nx + ix] = g;
        m = fmaxf(m, g);
        below = here;
        here = above;
      }
    }
  }
  for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
  if (lane == 0) sh[wid] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    partial[(uint64_t(blockIdx.z) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] =
        fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

// Intensity weighting: the volume itself with voxels below
// background_fraction * max (and negative values) set to zero.
__global__ __launch_bounds__(256) void intensity_kernel(const float *__restrict__ vol, uint64_t nv,
                                                        float background_fraction,
                                                        const float *__restrict__ vmax,
                                                        float *__restrict__ wgt) {
  const uint64_t idx = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= nv) return;
  const float thr = background_fraction * vmax[0];
  const float v = vol[idx];
  wgt[idx] = (v >= thr && v > 0.f) ? v : 0.f;
}

__device__ __forceinline__ float trilinear(const float *__restrict__ vol, const int dims[3], const float c[3]) {
  const float f0 = floorf(c[0]), f1 = floorf(c[1]), f2 = floorf(c[2]);
  const int i0 = int(f0), j0 = int(f1), k0 = int(f2);
  const float a = c[0] - f0, b = c[1] - f1, g = c[2] - f2;
  float acc = 0.f;
  for (int dz = 0; dz < 2; ++dz)
    for (int dy = 0; dy < 2; ++dy)
      for (int dx = 0; dx < 2; ++dx) {
        if (!index_inside(i0, dx, dims[0]) || !index_inside(j0, dy, dims[1]) || !index_inside(k0, dz, dims[2])) continue;
        const int x = i0 + dx, y = j0 + dy, z = k0 + dz;
        const float wgt = (dx ? a : 1.f - a) * (dy ? b : 1.f - b) * (dz ? g : 1.f - g);
        acc = fmaf(wgt, vol[(int64_t(z) * dims[1] + y) * dims[0] + x], acc);
      }
  return acc;
}

struct InitGrid {
  float origin[3], h[3];
  int dims[3];
};

__global__ __launch_bounds__(256) void sample_kernel(const uint64_t *__restrict__ cdf, uint64_t nvox,
                                                     const float *__restrict__ vol, InitGrid G,
                                                     const double *__restrict__ uni, int64_t n,
                                                     float density_scale, fgs_gaussian_grads out) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint64_t total = cdf[nvox];
  uint64_t target = static_cast<uint64_t>(floor(uni[i] * double(total)));
  if (target >= total) target = total - 1;
  // largest k with cdf[k] <= target (cdf is non-decreasing, cdf[0] = 0)
  uint64_t lo = 0, hi = nvox;  // invariant: cdf[lo] <= target < cdf[hi] (cdf[nvox] = total > target)
  while (hi - lo > 1) {
    const uint64_t mid = (lo + hi) >> 1;
    if (cdf[mid] <= target)
      lo = mid;
    else
      hi = mid;
  }
  const int64_t k = int64_t(lo);
  const int ix = int(k % G.dims[0]), iy = int((k / G.dims[0]) % G.dims[1]),
            iz = int(k / (int64_t(G.dims[0]) * G.dims[1]));
  const int idx3[3] = {ix, iy, iz};
  float p[3], c[3];
  for (int a = 0; a < 3; ++a) {
    const double j = uni[(a + 1) * n + i];
    p[a] = float(double(G.origin[a]) + (double(idx3[a]) + j) * double(G.h[a]));
    c[a] = float(double(idx3[a]) + j - 0.5);
  }
  const float rho = density_scale * trilinear(vol, G.dims, c);
  for (int a = 0; a < 3; ++a) out.mean[a * n + i] = p[a];
  out.quat[i] = 1.f;
  out.quat[n + i] = 0.f;
  out.quat[2 * n + i] = 0.f;
  out.quat[3 * n + i] = 0.f;
  out.density[i] = rho;
}

// Isotropic log-scale = log of the distance to the nearest other mean,
// floored at min_dist: the smallest FP32 squared distance over all others.
__device__ __forceinline__ float dist2(float dx, float dy, float dz) { return fmaf(dx, dx, fmaf(dy, dy, dz * dz)); }

__device__ __forceinline__ void write_scale(float best, float min_dist, int64_t i, int64_t n,
                                            float *__restrict__ log_scale) {
  const float d = fmaxf(sqrtf(best), min_dist);
  const float l = logf(d);
  log_scale[i] = l;
  log_scale[n + i] = l;
  log_scale[2 * n + i] = l;
}

// Brute force over LDS tiles: for a few points (1,000: 33 us, 53 by cells, most of
// it launches) and for the few calls whose cell arrays do not fit the
// workspace (many Gaussians drawn from a small grid).
constexpr int64_t kFewPoints = 1024;

__global__ __launch_bounds__(256) void nn_scale_kernel(const float *__restrict__ mean, int64_t n,
                                                       float min_dist, float *__restrict__ log_scale) {
  __shared__ float s_p[3][256];
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  float px = 0.f, py = 0.f, pz = 0.f;
  if (i < n) {
    px = mean[i];
    py = mean[n + i];
    pz = mean[2 * n + i];
  }
  float best = INFINITY;
  for (int64_t base = 0; base < n; base += 256) {
    __syncthreads();
    const int64_t j = base + threadIdx.x;
    if (j < n) {
      s_p[0][threadIdx.x] = mean[j];
      s_p[1][threadIdx.x] = mean[n + j];
      s_p[2][threadIdx.x] = mean[2 * n + j];
    }
    __syncthreads();
    const int m = int(min(int64_t(256), n - base));
    for (int t = 0; t < m; ++t) {
      const float d2 = dist2(s_p[0][t] - px, s_p[1][t] - py, s_p[2][t] - pz);
      best = (base + t != i) ? fminf(best, d2) : best;
    }
  }
  if (i < n) write_scale(best, min_dist, i, n, log_scale);
}

// Nearest neighbour over a grid of cubic cells. Points are counted into
// cells (count, scan, fill), then a thread searches the cells around its
// point, ring by ring, until no cell left can hold a nearer one. The order of
// the points inside a cell is not fixed, their minimum is: the result is the
// brute force's, bit for bit. Cells are chosen for four per point: the
// samples lie on surfaces and fill few of them (a cube of 2 per point holds
// twice the candidates). Bound by the latency of the candidates' loads,
// some 85 ns each: a point that is not decided by the cells up to kMaxRings away
// (an isolated one), or that would look at more than max_look points (a small
// object in a wide grid: most points in a few cells), is left to the pass
// over all points below, whose work does not depend on where the points are.
// Measured at 50,000 points: 1.58 ms by brute force (196 workgroups, n^2
// distances), 0.07 ms for the seven launches where they lie on surfaces; the
// whole placement with all of them around one voxel 1.88 ms by brute force,
// 7.3 by cells alone, 1.42 now; 5,000, some of them isolated, 0.45, 0.90 and 0.41.
struct Cells {
  float o[3], edge, inv;
  int d[3];
};
constexpr int kCellsPerPoint = 4;
constexpr int kMaxRings = 3;

__device__ __forceinline__ int cell_of(const Cells &C, int a, float p) {
  return min(max(int((p - C.o[a]) * C.inv), 0), C.d[a] - 1);
}

__device__ __forceinline__ uint32_t cell_index(const Cells &C, float x, float y, float z) {
  return (uint32_t(cell_of(C, 2, z)) * uint32_t(C.d[1]) + uint32_t(cell_of(C, 1, y))) * uint32_t(C.d[0]) +
         uint32_t(cell_of(C, 0, x));
}

__global__ __launch_bounds__(256) void cell_zero_kernel(uint32_t *__restrict__ count, uint32_t n) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < n) count[i] = 0u;
}

__global__ __launch_bounds__(256) void cell_count_kernel(const float *__restrict__ mean, int64_t n, Cells C,
                                                         uint32_t *__restrict__ count, uint32_t *__restrict__ rank) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) rank[i] = atomicAdd(&count[cell_index(C, mean[i], mean[n + i], mean[2 * n + i])], 1u);
}

__global__ __launch_bounds__(256) void cell_fill_kernel(const float *__restrict__ mean, int64_t n, Cells C,
                                                        const uint32_t *__restrict__ start,
                                                        const uint32_t *__restrict__ rank,
                                                        float4 *__restrict__ pts) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  const float x = mean[i], y = mean[n + i], z = mean[2 * n + i];
  pts[start[cell_index(C, x, y, z)] + rank[i]] = make_float4(x, y, z, __uint_as_float(uint32_t(i)));
}

// rest[0 .. rest_n[0]): the points left over; their log_scale holds +infinity,
// where the pass over all points gathers the squared distance.
__global__ __launch_bounds__(64) void nn_cells_kernel(const float4 *__restrict__ pts, int64_t n, Cells C,
                                                      const uint32_t *__restrict__ start, float min_dist,
                                                      int max_look, uint32_t *__restrict__ rest_n,
                                                      uint32_t *__restrict__ rest, float *__restrict__ log_scale) {
  const int64_t q = int64_t(blockIdx.x) * 64 + threadIdx.x;
  if (q >= n) return;
  const float4 p = pts[q];
  const int cx = cell_of(C, 0, p.x), cy = cell_of(C, 1, p.y), cz = cell_of(C, 2, p.z);
  const int c[3] = {cx, cy, cz};
  const float pc[3] = {p.x, p.y, p.z};
  float best = INFINITY;
  // cells [x0, x1] of row (y, z): one contiguous piece of pts, [a, e)
  auto row_of = [&](int x0, int x1, int y, int z, uint32_t &a, uint32_t &e) {
    x0 = max(x0, 0);
    x1 = min(x1, C.d[0] - 1);
    a = e = 0u;
    if (x0 > x1 || y < 0 || y >= C.d[1] || z < 0 || z >= C.d[2]) return;
    const uint32_t row = (uint32_t(z) * uint32_t(C.d[1]) + uint32_t(y)) * uint32_t(C.d[0]);
    a = start[row + uint32_t(x0)];
    e = start[row + uint32_t(x1) + 1u];
  };
  int left = max_look;
  auto look = [&](uint32_t a, uint32_t e) {
    if (int(e - a) > left) {
      left = -1;
      return;
    }
    left -= int(e - a);
    for (uint32_t k = a; k < e; ++k) {
      const float4 o = pts[k];
      const float d2 = dist2(o.x - p.x, o.y - p.y, o.z - p.z);
      if (k != uint32_t(q)) best = fminf(best, d2);
    }
  };
  auto scan = [&](int x0, int x1, int y, int z) {
    uint32_t a, e;
    row_of(x0, x1, y, z, a, e);
    look(a, e);
  };
  // the nine rows around the point's cell, their ends loaded together
  uint32_t a9[9], e9[9], sum9 = 0;
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    row_of(cx - 1, cx + 1, cy + j % 3 - 1, cz + j / 3 - 1, a9[j], e9[j]);
    sum9 += e9[j] - a9[j];
  }
  if (sum9 > uint32_t(max_look)) left = -1;
#pragma unroll
  for (int j = 0; j < 9; ++j) look(a9[j], e9[j]);
  bool found = false;
  for (int r = 1;;) {
    // distance to the nearest face of the searched cube that has cells beyond
    // it, less the rounding of a face and of a point's cell
    float face = INFINITY;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float slack = 1e-3f * C.edge + 4e-6f * fabsf(pc[a]) + 4e-6f * fabsf(C.o[a]);
      if (c[a] - r > 0) face = fminf(face, pc[a] - (C.o[a] + float(c[a] - r) * C.edge) - slack);
      if (c[a] + r < C.d[a] - 1) face = fminf(face, C.o[a] + float(c[a] + r + 1) * C.edge - pc[a] - slack);
    }
    found = left >= 0 && (face == INFINITY || (face > 0.f && best <= face * face * 0.9999f));
    if (found || left < 0 || r == kMaxRings) break;
    ++r;
    for (int z = -r; z <= r; ++z)
      for (int y = -r; y <= r; ++y) {
        if (z == -r || z == r || y == -r || y == r) {
          scan(cx - r, cx + r, cy + y, cz + z);
        } else {
          scan(cx - r, cx - r, cy + y, cz + z);
          scan(cx + r, cx + r, cy + y, cz + z);
        }
      }
  }
  const int64_t i = int64_t(__float_as_uint(p.w));
  if (found) write_scale(best, min_dist, i, n, log_scale);
  const uint64_t more = __ballot(!found);
  if (!found) {
    const int lane = threadIdx.x, first = __ffsll(static_cast<unsigned long long>(more)) - 1;
    uint32_t at = 0;
    if (lane == first) at = atomicAdd(rest_n, uint32_t(__popcll(more)));
    at = __shfl(at, first, 64);
    rest[at + uint32_t(__popcll(more & ((1ull << lane) - 1ull)))] = uint32_t(q);
    log_scale[i] = INFINITY;
  }
}

// The points left over against all n: an item is 256 of them and kRestSeg
// others, staged in LDS, so that a few points' work is spread too; the pieces
// meet in log_scale by an atomic minimum over the bits (squares are not
// negative), which no order changes. 50,000 points all left over: 2.5 G
// distances.
constexpr int kRestSeg = 2048;

__global__ __launch_bounds__(256) void nn_rest_kernel(const float4 *__restrict__ pts, int64_t n,
                                                      const uint32_t *__restrict__ rest_n,
                                                      const uint32_t *__restrict__ rest,
                                                      float *__restrict__ log_scale) {
  __shared__ float4 s_p[256];
  const uint32_t m = rest_n[0], groups = (m + 255u) / 256u;
  const uint32_t segs = uint32_t((n + kRestSeg - 1) / kRestSeg);
  for (uint64_t item = blockIdx.x; item < uint64_t(groups) * segs; item += gridDim.x) {
    const uint32_t g = uint32_t(item / segs), sg = uint32_t(item - uint64_t(g) * segs);
    const uint32_t j = g * 256u + threadIdx.x;
    const bool mine = j < m;
    const uint32_t q = mine ? rest[j] : 0u;
    const float4 p = pts[q];
    float best = INFINITY;
    const int64_t k0 = int64_t(sg) * kRestSeg, k1 = min(n, k0 + kRestSeg);
    for (int64_t base = k0; base < k1; base += 256) {
      __syncthreads();
      if (base + threadIdx.x < k1) s_p[threadIdx.x] = pts[base + threadIdx.x];
      __syncthreads();
      const int cnt = int(min(int64_t(256), k1 - base));
      const int own = int(int64_t(q) - base);  // the point itself, if it is in this tile
#pragma unroll 4
      for (int t = 0; t < cnt; ++t) {
        const float4 o = s_p[t];
        const float d2 = dist2(o.x - p.x, o.y - p.y, o.z - p.z);
        best = t != own ? fminf(best, d2) : best;
      }
    }
    if (mine) atomicMin(reinterpret_cast<unsigned int *>(log_scale) + __float_as_uint(p.w), __float_as_uint(best));
  }
}

__global__ __launch_bounds__(256) void nn_rest_scale_kernel(const float4 *__restrict__ pts, int64_t n,
                                                            const uint32_t *__restrict__ rest_n,
                                                            const uint32_t *__restrict__ rest, float min_dist,
                                                            float *__restrict__ log_scale) {
  for (uint32_t j = blockIdx.x * 256u + threadIdx.x; j < rest_n[0]; j += gridDim.x * 256u) {
    const int64_t i = int64_t(__float_as_uint(pts[rest[j]].w));
    write_scale(log_scale[i], min_dist, i, n, log_scale);
  }
}

// Cells of a box of the given extents holding about kCellsPerPoint n of them.
Cells make_cells(const float o[3], const double extent[3], int64_t n) {
  Cells C{};
  double edge = std::cbrt(extent[0] * extent[1] * extent[2] / (double(kCellsPerPoint) * double(n)));
  double widest = std::max(extent[0], std::max(extent[1], extent[2]));
  edge = std::max(edge, widest / 1024.0);
  for (int a = 0; a < 3; ++a) {
    C.o[a] = o[a];
    C.d[a] = std::max(1, int(std::ceil(extent[a] / edge)));
  }
  C.edge = float(edge);
  C.inv = 1.f / C.edge;
  return C;
}

// Whether a grid is backprojected from staged pieces: enough voxels for the
// chip, and not too many lost to the padding of its columns and runs. 75 views,
// backprojection by a voxel per thread and from pieces: 256^2 to 64^3 67 and 154 us, 160^2 to
// 80^3 100 and 96, 192^2 to 96^3 162 and 134; 512^2 to slices of 512 x 512: one 47 and 126,
// three 106 and 124, eight 250 and 227; 512^2 to 256^3 (runs of 16) 2,605 and 801.
constexpr uint64_t kFdkStagedVoxels = uint64_t(1) << 19;
bool fdk_staged(const FdkGeom &G, int run) {
  const uint64_t nxy = uint64_t(G.dims[0]) * G.dims[1], n = nxy * G.dims[2];
  auto up = [](uint64_t d, uint64_t m) { return (d + m - 1) / m * m; };
  const uint64_t padded = up(G.dims[0], 16) * up(G.dims[1], 16) * up(G.dims[2], run);
  return n >= kFdkStagedVoxels && 4 * padded <= (run == 16 ? 12 : 5) * n;
}

}  // namespace
}  // namespace fgs

using namespace fgs;

extern "C" int fgs_fdk(const float *img, const fgs_geom *geom, int32_t view_begin, int32_t view_count,
                       const fgs_grid *grid, float *vol, fgs_workspace *ws, void *stream) {
  if (!img || !geom || !grid || !vol || !ws || !geom->angles) return fail(FGS_E_INVALID, "null argument");
  if (geom->mode != FGS_CONE) return fail(FGS_E_UNSUPPORTED, "FDK is implemented for cone beam only");
  if (view_count <= 0 || view_count > 1024 || view_begin < 0 || int64_t(view_begin) + view_count > geom->n_views)
    return fail(FGS_E_INVALID, "view range (at most 1024 views)");
  if (geom->det_w <= 0 || geom->det_w > kMaxFilterRow || geom->det_h <= 0)
    return fail(FGS_E_INVALID, "detector size (rows up to 8192 pixels)");
  for (int a = 0; a < 3; ++a)
    if (grid->dims[a] <= 0 || !(grid->spacing[a] > 0.f)) return fail(FGS_E_INVALID, "grid");
  const uint64_t qn = uint64_t(view_count) * geom->det_h * geom->det_w;
  ws->needed = align_up(qn * sizeof(float));
  if (!ws->ptr || ws->bytes < ws->needed) return fail(FGS_E_CAPACITY, "workspace too small");
  ws->kind = 0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  float *q = static_cast<float *>(ws->ptr);
  const float ratio = geom->sod / geom->sdd;
  const float cu = 0.5f * float(geom->det_w) + geom->off_u, cv = 0.5f * float(geom->det_h) + geom->off_v;
  const int64_t n_rows = int64_t(view_count) * geom->det_h;
  dim3 fgrid(grid_for(uint64_t(n_rows), kFilterRows), grid_for(uint64_t(geom->det_w), kFilterSeg));
  fdk_filter_kernel<<<fgrid, 512, 0, s>>>(img, geom->det_w, geom->det_h, n_rows, geom->sod, geom->pitch_u * ratio,
                                          geom->pitch_v * ratio, cu, cv, q);
  FGS_LAUNCH_CHECK("fdk_filter_kernel");
  FdkGeom G{};
  G.sod = geom->sod;
  G.fu = geom->sdd / geom->pitch_u;
  G.fv = geom->sdd / geom->pitch_v;
  G.cu = cu;
  G.cv = cv;
  G.W = geom->det_w;
  G.H = geom->det_h;
  G.views = view_count;
  G.view_begin = view_begin;
  G.scale = float(M_PI / double(view_count));
  G.angles = geom->angles;
  for (int a = 0; a < 3; ++a) {
    G.origin[a] = grid->origin[a];
    G.h[a] = grid->spacing[a];
    G.dims[a] = grid->dims[a];
  }
  const uint64_t nxy = uint64_t(grid->dims[0]) * grid->dims[1];
  const bool lng = nxy * uint64_t(grid->dims[2]) >= kFdkLongVoxels;
  G.blocks_x = (grid->dims[0] + 15) / 16;
  const dim3 bgrid(unsigned(G.blocks_x) * unsigned((grid->dims[1] + 15) / 16),
                   std::min(65535u, grid_for(uint64_t(grid->dims[2]), lng ? 16 : 4)));
  if (!fdk_staged(G, lng ? 16 : 4))
    fdk_voxel_kernel<<<grid_for(nxy * uint64_t(grid->dims[2]), 256), 256, 0, s>>>(G, q, vol);
  else if (lng)
    fdk_backproject_kernel<16><<<bgrid, 256, 0, s>>>(G, q, vol);
  else
    fdk_backproject_kernel<4><<<bgrid, 256, 0, s>>>(G, q, vol);
  FGS_LAUNCH_CHECK("fdk_backproject_kernel / fdk_voxel_kernel");
  return FGS_OK;
}

enum class Weighting { kGradient, kIntensity };

static int sampling_init(Weighting mode, const float *vol, const fgs_grid *grid, float background_fraction,
                         float density_scale, float min_scale, int64_t n, const double *uniforms,
                         fgs_gaussians_out *out, fgs_workspace *ws, void *stream) {
  if (!vol || !grid || !uniforms || !out || !ws || !out->mean || !out->log_scale || !out->quat || !out->density)
    return fail(FGS_E_INVALID, "null argument");
  if (n <= 0) return fail(FGS_E_INVALID, "n must be positive");
  for (int a = 0; a < 3; ++a)
    if (grid->dims[a] <= 0 || !(grid->spacing[a] > 0.f)) return fail(FGS_E_INVALID, "grid");
  const uint64_t nv = uint64_t(grid->dims[0]) * grid->dims[1] * grid->dims[2];
  Carver c(nullptr);
  uint64_t o_part, o_g, o_w, o_scan;
  c.take<float>(kRedBlocks + 2, &o_part);
  c.take<float>(nv, &o_g);
  c.take<uint64_t>(nv + 1, &o_w);
  c.take<uint32_t>(scan_scratch_words(nv), &o_scan);
  ws->needed = c.used;
  if (!ws->ptr || ws->bytes < ws->needed) return fail(FGS_E_CAPACITY, "workspace too small");
  ws->kind = 0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  char *b = static_cast<char *>(ws->ptr);
  float *part = reinterpret_cast<float *>(b + o_part);
  float *vmax = part + kRedBlocks;       // holds max(vol)
  float *gmax = part + kRedBlocks + 1;   // holds max(gradient magnitude)
  float *gmag = reinterpret_cast<float *>(b + o_g);
  uint64_t *w = reinterpret_cast<uint64_t *>(b + o_w);
  const int nb = int(std::min<uint64_t>(kRedBlocks, (nv + kRedThreads - 1) / kRedThreads));
  max_partial_kernel<<<nb, kRedThreads, 0, s>>>(vol, nv, part);
  max_final_kernel<<<1, kRedThreads, 0, s>>>(part, nb, vmax);
  FGS_LAUNCH_CHECK("max_final_kernel");
  if (mode == Weighting::kGradient) {
    // the workgroups' maxima go where the prefix sum will be (8 bytes a voxel: room for one per voxel)
    const dim3 gg(grid_for(uint64_t(grid->dims[0]), 64), std::min(65535u, grid_for(uint64_t(grid->dims[1]), 4)),
                  std::min(65535u, grid_for(uint64_t(grid->dims[2]), kGradRun)));
    grad_mag_kernel<<<gg, 256, 0, s>>>(vol, grid->dims[0], grid->dims[1], grid->dims[2], background_fraction, vmax,
                                       gmag, reinterpret_cast<float *>(w));
    FGS_LAUNCH_CHECK("grad_mag_kernel");
    max_final_kernel<<<1, kRedThreads, 0, s>>>(reinterpret_cast<float *>(w), int(gg.x * gg.y * gg.z), gmax);
  } else {
    intensity_kernel<<<grid_for(nv, 256), 256, 0, s>>>(vol, nv, background_fraction, vmax, gmag);
    FGS_LAUNCH_CHECK("intensity_kernel");
    max_partial_kernel<<<nb, kRedThreads, 0, s>>>(gmag, nv, part);
    max_final_kernel<<<1, kRedThreads, 0, s>>>(part, nb, gmax);
  }
  FGS_LAUNCH_CHECK("max_final_kernel");
  float gm_host = 0.f;
  FGS_HIP(hipMemcpyAsync(&gm_host, gmax, sizeof(float), hipMemcpyDeviceToHost, s));
  FGS_HIP(hipStreamSynchronize(s));
  if (!(gm_host > 0.f))
    return fail(FGS_E_INVALID, mode == Weighting::kGradient ? "the thresholded volume has no gradient to sample"
                                                            : "the thresholded volume has no mass to sample");
  int st = exclusive_scan_quantized(gmag, gmax, w, nv, reinterpret_cast<uint32_t *>(b + o_scan), s);
  if (st != FGS_OK) return st;
  InitGrid G{};
  for (int a = 0; a < 3; ++a) {
    G.origin[a] = grid->origin[a];
    G.h[a] = grid->spacing[a];
    G.dims[a] = grid->dims[a];
  }
  sample_kernel<<<grid_for(uint64_t(n), 256), 256, 0, s>>>(w, nv, vol, G, uniforms, n, density_scale, *out);
  FGS_LAUNCH_CHECK("sample_kernel");
  // the weights and their prefix sum are done with: their room holds the cells
  double extent[3];
  for (int a = 0; a < 3; ++a) extent[a] = double(G.h[a]) * G.dims[a];
  const Cells C = make_cells(G.origin, extent, n);
  const uint64_t nc = uint64_t(C.d[0]) * C.d[1] * C.d[2];
  Carver cc(nullptr);
  uint64_t o_cell, o_rank, o_pts, o_cscan;
  cc.take<uint32_t>(nc + 2, &o_cell);  // the last word: the number of points left over
  cc.take<uint32_t>(uint64_t(n), &o_rank);
  cc.take<float4>(uint64_t(n), &o_pts);
  cc.take<uint32_t>(scan_scratch_words(nc), &o_cscan);
  if (n <= kFewPoints || o_g + cc.used > c.used || n > 0x7fffffff || nc > 0x7fffffff) {
    nn_scale_kernel<<<grid_for(uint64_t(n), 256), 256, 0, s>>>(out->mean, n, min_scale, out->log_scale);
    FGS_LAUNCH_CHECK("nn_scale_kernel");
    return FGS_OK;
  }
  char *r = b + o_g;
  uint32_t *cell = reinterpret_cast<uint32_t *>(r + o_cell), *rank = reinterpret_cast<uint32_t *>(r + o_rank);
  float4 *pts = reinterpret_cast<float4 *>(r + o_pts);
  const unsigned nb_n = grid_for(uint64_t(n), 256);
  cell_zero_kernel<<<grid_for(nc + 2, 256), 256, 0, s>>>(cell, uint32_t(nc + 2));
  cell_count_kernel<<<nb_n, 256, 0, s>>>(out->mean, n, C, cell, rank);
  FGS_LAUNCH_CHECK("cell_count_kernel");
  st = exclusive_scan_u32(cell, nc, reinterpret_cast<uint32_t *>(r + o_cscan), s);
  if (st != FGS_OK) return st;
  cell_fill_kernel<<<nb_n, 256, 0, s>>>(out->mean, n, C, cell, rank, pts);
  FGS_LAUNCH_CHECK("cell_fill_kernel");
  // the ranks are done with: their room holds the points left over
  uint32_t *rest = rank, *rest_n = cell + nc + 1;
  const int max_look = int(std::max<int64_t>(256, n / 16));
  nn_cells_kernel<<<grid_for(uint64_t(n), 64), 64, 0, s>>>(pts, n, C, cell, min_scale, max_look, rest_n, rest,
                                                           out->log_scale);
  FGS_LAUNCH_CHECK("nn_cells_kernel");
  const uint64_t items = uint64_t(nb_n) * grid_for(uint64_t(n), kRestSeg);
  nn_rest_kernel<<<unsigned(std::min<uint64_t>(2048, items)), 256, 0, s>>>(pts, n, rest_n, rest, out->log_scale);
  FGS_LAUNCH_CHECK("nn_rest_kernel");
  nn_rest_scale_kernel<<<std::min(256u, nb_n), 256, 0, s>>>(pts, n, rest_n, rest, min_scale, out->log_scale);
  FGS_LAUNCH_CHECK("nn_rest_scale_kernel");
  return FGS_OK;
}

extern "C" int fgs_gradient_init(const float *vol, const fgs_grid *grid, float background_fraction,
                                 float density_scale, float min_scale, int64_t n, const double *uniforms,
                                 fgs_gaussians_out *out, fgs_workspace *ws, void *stream) {
  return sampling_init(Weighting::kGradient, vol, grid, background_fraction, density_scale, min_scale, n,
                       uniforms, out, ws, stream);
}

extern "C" int fgs_intensity_init(const float *vol, const fgs_grid *grid, float background_fraction,
                                  float density_scale, float min_scale, int64_t n, const double *uniforms,
                                  fgs_gaussians_out *out, fgs_workspace *ws, void *stream) {
  return sampling_init(Weighting::kIntensity, vol, grid, background_fraction, density_scale, min_scale, n,
                       uniforms, out, ws, stream);
}

extern "C" int fgs_reduce_max(const float *x, int64_t n, float *out, fgs_workspace *ws, void *stream) {
  if (!x || !out || !ws || n <= 0) return fail(FGS_E_INVALID, "invalid argument");
  ws->needed = uint64_t(kRedBlocks) * sizeof(float);
  if (!ws->ptr || ws->bytes < ws->needed) return fail(FGS_E_CAPACITY, "workspace too small");
  ws->kind = 0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  float *part = static_cast<float *>(ws->ptr);
  const int nb = int(std::min<uint64_t>(kRedBlocks, (uint64_t(n) + kRedThreads - 1) / kRedThreads));
  max_partial_kernel<<<nb, kRedThreads, 0, s>>>(x, uint64_t(n), part);
  max_final_kernel<<<1, kRedThreads, 0, s>>>(part, nb, out);
  FGS_LAUNCH_CHECK("max_final_kernel");
  return FGS_OK;
}
