// Voxelizer (Eq. 2, Sec. 3.3) for gfx950: the density field sampled at the
// voxel centres of a regular grid, each Gaussian limited to its kappa-sigma
// ellipsoid, and its backward.
//
// Same structure as the rasterizer, one dimension up:
//   record kernel   per Gaussian: centre in voxel-index coordinates and rho
//                   (float4, the position+radius packing of Sec. 3.5), the
//                   voxel-unit inverse covariance pre-scaled by -log2(e)/2,
//                   half-extents in voxels and the 3D rectangle of 8^3-voxel
//                   tiles its box touches;
//   count kernel    a wave per Gaussian with a large rectangle, for four of
//                   them with small ones (a wave each where they are few): of the rectangle's tiles, those the
//                   support ellipsoid actually reaches (bounds at the tile's
//                   centre decide most, the exact box test the rest; about 57%
//                   of the box's tiles for the standard scan);
//   scan / emit     keys of the reached tiles; the sort's value is the
//                   emission slot, whose Gaussian is gid[slot];
//   stable radix sort / ranges as in the rasterizer;
//   forward         one wave per 8^3 tile (grids with few tiles: several, with
//                   partial volumes); 16 lanes walk a quarter's list, each one
//                   x-row of 8 voxels (short lists: 64 lanes the tile's); records staged in LDS in batches of 64;
//                   where Gaussians span many tiles, interior quarters by
//                   products along the row;
//   backward        one or four waves per tile; each lane owns one (tile,
//                   Gaussian) pair and sums the ten moments sum g e {1, d, d d^T}
//                   over the tile's 512 voxels into the pair's emission slot; per
//                   Gaussian, its contiguous slots are reduced in a fixed
//                   order and the chain rule applied.
#include <algorithm>

#include "fgs_internal.h"

namespace fgs {
namespace {

constexpr int kVT = 8;     // voxel tile side
constexpr int kWave = 64;

struct __align__(16) Rect3 {
  unsigned short v[8];     // x0, y0, z0, x1, y1, z1, 0, 0
};

struct GridDev {
  float origin[3];
  const float *origin_dev;  // device copy of the origin read instead of origin[] (null: off)
  float h[3];
  int dims[3];
  int nt[3];               // tiles per axis
  float kappa;
  float tau;               // density-aware support threshold (0 = off)
};

// Voxel-unit quantities of one Gaussian: W = diag(h) R diag(1/s) is such
// that A_vox = W W^T is the inverse covariance in voxel-index units.
struct VoxGauss {
  float pv[3];             // centre in voxel-index coordinates
  float W[3][3];
  float A[3][3];
  float r[3];              // kap-sigma half-extents in voxels
};

__device__ __forceinline__ void vox_gauss(const GaussParams &P, const GridDev &G, float kap, VoxGauss &V) {
  for (int a = 0; a < 3; ++a) {
    const float o = G.origin_dev ? G.origin_dev[a] : G.origin[a];
    V.pv[a] = (P.p[a] - o) / G.h[a] - 0.5f;
    float var = 0.f;
    for (int j = 0; j < 3; ++j) {
      V.W[a][j] = G.h[a] * P.R[3 * a + j] / P.s[j];
      const float rs = P.R[3 * a + j] * P.s[j];
      var += rs * rs;
    }
    V.r[a] = kap * sqrtf(var) / G.h[a];
  }
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b)
      V.A[a][b] = V.W[a][0] * V.W[b][0] + V.W[a][1] * V.W[b][1] + V.W[a][2] * V.W[b][2];
}

__device__ __forceinline__ void vox_span(float c, float r, int n_tiles, int &t0, int &t1) {
#pragma clang fp contract(off)
  const float lim = 16777216.f;
  float lo = fminf(fmaxf(c - r, -lim), lim);
  float hi = fminf(fmaxf(c + r, -lim), lim);
  t0 = max(static_cast<int>(floorf(lo)) >> 3, 0);
  t1 = min(static_cast<int>(floorf(hi)) >> 3, n_tiles - 1);
}

// The tile culling test keeps tiles whose best voxel centre has
// d^2 <= k2 + kappa^2 (kCullSlack - 1), k2 the Gaussian's support bound (a
// Mahalanobis radius about 0.05% beyond the kappa support): a superset of the
// per-voxel test. On the pre-scaled exponent: arg >= thr_g + thr_widen, with
// thr_g the Gaussian's threshold (a1.z) and thr_widen = thr (kCullSlack - 1).
constexpr float kCullSlack = 1.001f;
constexpr float kLn2 = 0.6931471805599453f;

__global__ void zero_u64_kernel(unsigned long long *p, int n) {
  if (int(threadIdx.x) < n) p[threadIdx.x] = 0ull;
}

__global__ __launch_bounds__(256) void vox_record_kernel(fgs_gaussians g, GridDev G,
                                                         float4 *__restrict__ prho,
                                                         float4 *__restrict__ a0,
                                                         float4 *__restrict__ a1,
                                                         float4 *__restrict__ radii,
                                                         Rect3 *__restrict__ rect) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < g.n) {
    GaussParams P;
    load_gauss(g, i, P);
    // support on the pre-scaled exponent arg = -log2(e)/2 d^2: arg >= thr_g,
    // thr_g = -log2(e)/2 kappa^2, raised to log2(tau / rho) by the
    // density-aware support (d^2 <= min(kappa^2, 2 ln(rho / tau)), Sec. 3.5
    // boxes that also take the density into account); a Gaussian with
    // rho <= tau is left out
    const float k = -0.5f * kLog2e;
    float kap = G.kappa, thr_g = k * G.kappa * G.kappa;
    bool dropped = false;
    if (G.tau > 0.f) {
      if (P.rho > G.tau) {
        const float l2 = log2f(P.rho) - log2f(G.tau);
        thr_g = fmaxf(thr_g, -l2);
        const float k2t = 2.f * kLn2 * l2;
        if (k2t < kap * kap) kap = sqrtf(k2t);
      } else {
        dropped = true;
      }
    }
    VoxGauss V;
    vox_gauss(P, G, kap, V);
    prho[i] = make_float4(V.pv[0], V.pv[1], V.pv[2], P.rho);
    a0[i] = make_float4(k * V.A[0][0], 2.f * k * V.A[0][1], 2.f * k * V.A[0][2], k * V.A[1][1]);
    a1[i] = make_float4(2.f * k * V.A[1][2], k * V.A[2][2], thr_g, 0.f);
    radii[i] = make_float4(V.r[0], V.r[1], V.r[2], 0.f);
    int t0[3], t1[3];
    bool empty = dropped;
    for (int a = 0; a < 3; ++a) {
      vox_span(V.pv[a], V.r[a], G.nt[a], t0[a], t1[a]);
      empty |= t0[a] > t1[a];
    }
    Rect3 rc;
    if (empty || !isfinite(V.pv[0] + V.pv[1] + V.pv[2])) {
      for (int a = 0; a < 8; ++a) rc.v[a] = 0;
      rc.v[0] = rc.v[1] = rc.v[2] = 1;
    } else {
      for (int a = 0; a < 3; ++a) {
        rc.v[a] = static_cast<unsigned short>(t0[a]);
        rc.v[3 + a] = static_cast<unsigned short>(t1[a]);
      }
      rc.v[6] = rc.v[7] = 0;
    }
    rect[i] = rc;
  }
}

// Largest value of the pre-scaled (negative definite) form
// arg(d) = c0.x dx^2 + dx (c0.y dy + c0.z dz) + c0.w dy^2 + c1.x dy dz + c1.y dz^2
// over the box lo <= p + d <= hi. Its maximiser lies on one of the three
// planes x_a = clamp(p_a); on each, the restricted 2D form is maximised over
// the face rectangle along its two clamped lines (the same construction as
// the rasterizer's quadrant test, one dimension up). The quotients that do not
// depend on the box are taken once per Gaussian.
struct BoxTest {
  float M[3][3];
  float kb[3], kc[3];  // maximiser of plane a's 2D form per unit of D, negated
  float inv[3];        // 1 / M[a][a]
  bool degenerate;     // a 2 x 2 minor is not positive: every box counts as reached

  __device__ __forceinline__ BoxTest(const float4 &c0, const float4 &c1)
      : M{{c0.x, 0.5f * c0.y, 0.5f * c0.z}, {0.5f * c0.y, c0.w, 0.5f * c1.x}, {0.5f * c0.z, 0.5f * c1.x, c1.y}} {
    degenerate = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int b = (a + 1) % 3, c = (a + 2) % 3;
      const float det = M[b][b] * M[c][c] - M[b][c] * M[b][c];
      degenerate |= !(det > 0.f);
      const float id = 1.f / det;
      kb[a] = (M[c][c] * M[a][b] - M[b][c] * M[a][c]) * id;
      kc[a] = (M[b][b] * M[a][c] - M[b][c] * M[a][b]) * id;
      inv[a] = 1.f / M[a][a];
    }
  }

  // d0: the box's lower corner less the Gaussian's centre; side: its side
  __device__ __forceinline__ float qmax(const float (&d0)[3], float side) const {
    float best = -INFINITY;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int b = (a + 1) % 3, c = (a + 2) % 3;
      const float D = fminf(fmaxf(0.f, d0[a]), d0[a] + side);
      const float lb = d0[b], hb = d0[b] + side, lc = d0[c], hc = d0[c] + side;
      const float yb1 = fminf(fmaxf(-D * kb[a], lb), hb);
      const float yc1 = fminf(fmaxf(-fmaf(M[b][c], yb1, D * M[a][c]) * inv[c], lc), hc);
      const float yc2 = fminf(fmaxf(-D * kc[a], lc), hc);
      const float yb2 = fminf(fmaxf(-fmaf(M[b][c], yc2, D * M[a][b]) * inv[b], lb), hb);
      const float f1 = fmaf(M[a][a] * D, D, fmaf(2.f * D, fmaf(M[a][b], yb1, M[a][c] * yc1),
                            fmaf(yb1, fmaf(M[b][b], yb1, 2.f * M[b][c] * yc1), M[c][c] * yc1 * yc1)));
      const float f2 = fmaf(M[a][a] * D, D, fmaf(2.f * D, fmaf(M[a][b], yb2, M[a][c] * yc2),
                            fmaf(yb2, fmaf(M[b][b], yb2, 2.f * M[b][c] * yc2), M[c][c] * yc2 * yc2)));
      best = fmaxf(best, fmaxf(f1, f2));
    }
    return best;
  }

  // Whether the support reaches one of the voxel centres of tile (tx, ty, tz),
  // as far as the culling threshold says (a superset test).
  __device__ __forceinline__ bool hit(const float4 &p, uint32_t tx, uint32_t ty, uint32_t tz, float thr_cull) const {
    const float d0[3] = {float(tx * kVT) - p.x, float(ty * kVT) - p.y, float(tz * kVT) - p.z};
    return degenerate || qmax(d0, float(kVT - 1)) >= thr_cull;
  }
};

// Tile j of the rectangle, row-major (x fastest).
__device__ __forceinline__ void tile_coords(const Rect3 &rc, uint32_t j, uint32_t &tx, uint32_t &ty, uint32_t &tz) {
  const uint32_t nx = uint32_t(rc.v[3]) - rc.v[0] + 1u, ny = uint32_t(rc.v[4]) - rc.v[1] + 1u;
  const uint32_t jz = j / (nx * ny);
  const uint32_t jxy = j - jz * nx * ny;
  const uint32_t jy = jxy / nx;
  tx = rc.v[0] + (jxy - jy * nx);
  ty = rc.v[1] + jy;
  tz = rc.v[2] + jz;
}

__device__ __forceinline__ uint32_t rect_tiles(const Rect3 &rc) {
  if (rc.v[0] > rc.v[3] || rc.v[1] > rc.v[4] || rc.v[2] > rc.v[5]) return 0u;
  return (uint32_t(rc.v[3]) - rc.v[0] + 1u) * (uint32_t(rc.v[4]) - rc.v[1] + 1u) * (uint32_t(rc.v[5]) - rc.v[2] + 1u);
}

// The hit ballots of the first kHitWords rounds are kept by the count, so the
// emission reads them instead of repeating the test (rectangles of at most
// kHitTiles tiles).
constexpr int kHitWords = 8;
constexpr int kHitTiles = 64 * kHitWords;

// A lane's tile of a rectangle walked 64 tiles at a time, row-major: the
// coordinates advance by additions (one division per rectangle, not per tile).
struct TileWalk {
  uint32_t x, y, z;      // relative to the rectangle's first tile
  uint32_t nx, ny;
  uint32_t sx, sy, sz;   // 64 tiles on
  __device__ __forceinline__ TileWalk(const Rect3 &rc, uint32_t j) {
    nx = uint32_t(rc.v[3]) - rc.v[0] + 1u;
    ny = uint32_t(rc.v[4]) - rc.v[1] + 1u;
    const uint32_t q = j / nx, p = 64u / nx;
    x = j - q * nx;
    z = q / ny;
    y = q - z * ny;
    sx = 64u - p * nx;
    sz = p / ny;
    sy = p - sz * ny;
  }
  __device__ __forceinline__ void next() {
    x += sx;
    const uint32_t cx = x >= nx ? 1u : 0u;
    x -= cx ? nx : 0u;
    y += sy + cx;
    const uint32_t cy = y >= ny ? 1u : 0u;
    y -= cy ? ny : 0u;
    z += sz + cy;
  }
};

// Hits among tiles [j0, j0 + n) of the rectangle, n <= kHitTiles, as ballots
// words[] in LDS (bit i of words[g]: tile j0 + 64 g + i): BoxTest's decisions.
// Most tiles need no exact test: the tangent at the tile's centre bounds the
// form over the tile from above (missed), its value at the tile's point
// nearest the centre of the Gaussian from below (hit); both with a margin of
// 4e-6 of the terms' sizes, above their rounding and the exact test's. Only
// the tiles in between, about one in six, are collected and tested exactly,
// 64 at a time. A form whose 2 x 2 minors are not positive keeps every tile,
// as the exact test does. 500,000 Gaussians at 512^3 (1,900 tiles per
// rectangle): count and emission 8.9 + 8.5 ms with an exact test per tile,
// 2.1 + 3.3 ms now (the keys written are 6.6 GB).
__device__ __forceinline__ void chunk_hits(const Rect3 &rc, uint32_t j0, uint32_t n, const float4 &p, const float4 &c0,
                                           const float4 &c1, float thr_cull, int lane,
                                           unsigned long long *__restrict__ words,
                                           unsigned short *__restrict__ unsure) {
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const float h = 0.5f * (kVT - 1);
  const BoxTest box(c0, c1);
  const float size = fabsf(c0.x) + fabsf(c0.y) + fabsf(c0.z) + fabsf(c0.w) + fabsf(c1.x) + fabsf(c1.y);
  TileWalk w(rc, j0 + uint32_t(lane));
  uint32_t n_unsure = 0;
  for (uint32_t g = 0; g * 64u < n; ++g) {
    const uint32_t i = g * 64u + uint32_t(lane);
    bool hit = false, open = false;
    if (i < n) {
      const float lx = float((w.x + rc.v[0]) * kVT), ly = float((w.y + rc.v[1]) * kVT),
                  lz = float((w.z + rc.v[2]) * kVT);
      const float dx = lx + h - p.x, dy = ly + h - p.y, dz = lz + h - p.z;
      const float hx = fmaf(c0.y, dy, c0.z * dz), hy = fmaf(c1.x, dz, c0.w * dy);
      const float q = fmaf(dx, fmaf(c0.x, dx, hx), fmaf(dy, hy, c1.y * dz * dz));
      const float gx = fmaf(2.f * c0.x, dx, hx), gy = fmaf(c0.y, dx, fmaf(c0.w, dy, hy)),
                  gz = fmaf(c0.z, dx, fmaf(c1.x, dy, 2.f * c1.y * dz));
      const float far = fmaxf(fmaxf(fabsf(dx), fabsf(dy)), fabsf(dz)) + h;
      const float margin = 4e-6f * fmaf(size * far, far, fabsf(thr_cull));
      // the tile's point nearest the Gaussian's centre, from the tile's centre
      const float nx = fminf(fmaxf(-dx, -h), h), ny = fminf(fmaxf(-dy, -h), h), nz = fminf(fmaxf(-dz, -h), h);
      const float ex = dx + nx, ey = dy + ny, ez = dz + nz;
      const float near = fmaf(ex, fmaf(c0.x, ex, fmaf(c0.y, ey, c0.z * ez)),
                              fmaf(ey, fmaf(c0.w, ey, c1.x * ez), c1.y * ez * ez));
      hit = box.degenerate || near >= thr_cull + margin;
      open = !hit && !(fmaf(h, fabsf(gx) + fabsf(gy) + fabsf(gz), q) < thr_cull - margin);
    }
    const uint64_t bal = __ballot(hit), amb = __ballot(open);
    if (open) unsure[n_unsure + __popcll(amb & lt)] = static_cast<unsigned short>(i);
    n_unsure += uint32_t(__popcll(amb));
    if (lane == 0) words[g] = bal;
    w.next();
  }
  wave_lds_sync();
  for (uint32_t r = 0; r < n_unsure; r += 64) {
    if (r + uint32_t(lane) < n_unsure) {
      const uint32_t i = unsure[r + lane];
      uint32_t tx, ty, tz;
      tile_coords(rc, j0 + i, tx, ty, tz);
      if (box.hit(p, tx, ty, tz, thr_cull)) atomicOr(&words[i >> 6], 1ull << (i & 63u));
    }
  }
  wave_lds_sync();
}

// A wave takes four Gaussians. Rectangles of at most 64 tiles are walked by 16
// lanes each, all four at once; larger ones by the whole wave, one after the
// other (200,000 Gaussians of 30-odd tiles at 256^3: 140 us with a wave per
// Gaussian, 75 us now).
constexpr int kWaveGauss = 4;
constexpr uint32_t kSmallTiles = 64;
// Below this many Gaussians a wave takes one, by the code for large
// rectangles: four, one after the other, leave SIMDs without a wave. Count and
// emission at 256^3, four and one per wave: 2,000 Gaussians of sigma 15 voxels 121 + 181
// and 89 + 129 us, 700 of 25 voxels 208 + 320 and 108 + 167; 16,000 of 5 voxels 19.6 + 15.5
// and 15.5 + 13.2, of 1.5 voxels 6.4 + 6.3 and 11.6 + 7.7.
constexpr uint64_t kFewGauss = 16384;

// Calls f(std::integral_constant<int, Gaussians per wave>).
template <typename F>
void with_wave_gauss(uint64_t n, F &&f) {
  if (n < kFewGauss)
    f(std::integral_constant<int, 1>());
  else
    f(std::integral_constant<int, kWaveGauss>());
}

// The number of tiles of each Gaussian's rectangle that its support reaches
// (the key count).
template <int PER>
__global__ __launch_bounds__(256) void vox_count_kernel(int64_t n, const float4 *__restrict__ prho,
                                                        const float4 *__restrict__ a0,
                                                        const float4 *__restrict__ a1,
                                                        const Rect3 *__restrict__ rect, float thr_widen,
                                                        uint32_t *__restrict__ count,
                                                        unsigned long long *__restrict__ hits) {
  __shared__ unsigned long long s_words[4][kHitWords];
  __shared__ unsigned short s_unsure[4][kHitTiles];
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = (int64_t(blockIdx.x) * 4 + wid) * PER;
  if (i0 >= n) return;
  const int grp = lane >> 4, l16 = lane & 15;
  if (PER > 1) {
    const int64_t i = i0 + grp;
    Rect3 rc{};
    uint32_t nt = 0;
    if (i < n) {
      rc = rect[i];
      nt = rect_tiles(rc);
    }
    const uint32_t small = nt <= kSmallTiles ? nt : 0u;
    unsigned long long word = 0;
    if (__ballot(small != 0u)) {
      float4 p = make_float4(0.f, 0.f, 0.f, 0.f), c0 = p, c1 = p;
      if (small) {
        p = prho[i];
        c0 = a0[i];
        c1 = a1[i];
      }
      const BoxTest box(c0, c1);
      const float thr_cull = c1.z + thr_widen;
      for (uint32_t r = 0; __ballot(r < small); r += 16) {
        bool hit = false;
        if (r + uint32_t(l16) < small) {
          uint32_t tx, ty, tz;
          tile_coords(rc, r + uint32_t(l16), tx, ty, tz);
          hit = box.hit(p, tx, ty, tz, thr_cull);
        }
        word |= ((__ballot(hit) >> (16 * grp)) & 0xffffull) << r;
      }
    }
    if (i < n && l16 == 0 && nt <= kSmallTiles) {
      if (nt) hits[uint64_t(i) * kHitWords] = word;
      count[i] = uint32_t(__popcll(word));
    }
  }
  for (int g = 0; g < PER; ++g) {
    const int64_t i = i0 + g;
    if (i >= n) break;
    const Rect3 rc = rect[i];
    const uint32_t nt = rect_tiles(rc);
    if (PER > 1 && nt <= kSmallTiles) continue;
    uint32_t cnt = 0;
    const float4 p = prho[i], c0 = a0[i], c1 = a1[i];
    for (uint32_t j0 = 0; j0 < nt; j0 += kHitTiles) {
      const uint32_t m = min(uint32_t(kHitTiles), nt - j0);
      chunk_hits(rc, j0, m, p, c0, c1, c1.z + thr_widen, lane, s_words[wid], s_unsure[wid]);
      const unsigned long long wd = uint32_t(lane) * 64u < m ? s_words[wid][lane & (kHitWords - 1)] : 0ull;
      if (nt <= uint32_t(kHitTiles) && uint32_t(lane) * 64u < m) hits[uint64_t(i) * kHitWords + lane] = wd;
      uint32_t c = uint32_t(__popcll(wd));
#pragma unroll
      for (int d = 1; d < kHitWords; d <<= 1) c += __shfl_xor(c, d, 64);
      cnt += uint32_t(__builtin_amdgcn_readfirstlane(int(c)));
      wave_lds_sync();
    }
    if (lane == 0) count[i] = cnt;
  }
}

// The keys of the tiles that each Gaussian's support reaches, in row-major
// order, at its offset. The sort's value is the emission slot q (a Gaussian's
// slots are contiguous, which is where the backward writes its partial sums);
// gid[q] is the Gaussian.
template <int PER>
__global__ __launch_bounds__(256) void vox_emit_kernel(int64_t n, int ntx, int nty, const float4 *__restrict__ prho,
                                                       const float4 *__restrict__ a0,
                                                       const float4 *__restrict__ a1,
                                                       const Rect3 *__restrict__ rect, float thr_widen,
                                                       const uint32_t *__restrict__ offset,
                                                       const unsigned long long *__restrict__ hits,
                                                       uint32_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                                       uint32_t *__restrict__ gid, const uint32_t *__restrict__ kdev) {
  // nothing to emit: no pairs, or more than the lists were laid out for
  if (kdev[0] == 0u) return;
  __shared__ unsigned long long s_words[4][kHitWords];
  __shared__ unsigned short s_unsure[4][kHitTiles];
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = (int64_t(blockIdx.x) * 4 + wid) * PER;
  if (i0 >= n) return;
  const int grp = lane >> 4, l16 = lane & 15;
  auto put = [&](uint32_t q, uint32_t tx, uint32_t ty, uint32_t tz, int64_t i) {
    keys[q] = (tz * uint32_t(nty) + ty) * uint32_t(ntx) + tx;
    vals[q] = q;
    gid[q] = uint32_t(i);
  };
  if (PER > 1) {
    const int64_t i = i0 + grp;
    unsigned long long word = 0;
    uint32_t o = 0;
    Rect3 rc{};
    if (i < n) {
      o = offset[i];
      if (offset[i + 1] != o) {
        rc = rect[i];
        if (rect_tiles(rc) <= kSmallTiles) word = hits[uint64_t(i) * kHitWords];
      }
    }
    for (uint32_t r = 0; __ballot(word >> r != 0ull); r += 16) {
      const uint32_t j = r + uint32_t(l16);
      if ((word >> j) & 1ull) {
        uint32_t tx, ty, tz;
        tile_coords(rc, j, tx, ty, tz);
        put(o + uint32_t(__popcll(word & ((1ull << j) - 1ull))), tx, ty, tz, i);
      }
      if (r == 48) break;
    }
  }
  for (int g = 0; g < PER; ++g) {
    const int64_t i = i0 + g;
    if (i >= n) break;
    uint32_t o = offset[i];
    if (o == offset[i + 1]) continue;
    const Rect3 rc = rect[i];
    const uint32_t nt = rect_tiles(rc);
    if (PER > 1 && nt <= kSmallTiles) continue;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const bool stored = nt <= uint32_t(kHitTiles);  // the count kept this rectangle's ballots
    TileWalk w(rc, uint32_t(lane));
    for (uint32_t j0 = 0; j0 < nt; j0 += kHitTiles) {
      const uint32_t m = min(uint32_t(kHitTiles), nt - j0);
      if (!stored) {
        const float4 p = prho[i], c0 = a0[i], c1 = a1[i];
        chunk_hits(rc, j0, m, p, c0, c1, c1.z + thr_widen, lane, s_words[wid], s_unsure[wid]);
      }
      for (uint32_t gw = 0; gw * 64u < m; ++gw) {
        const uint64_t bal = stored ? hits[uint64_t(i) * kHitWords + gw] : s_words[wid][gw];
        if ((bal >> lane) & 1ull)
          put(o + uint32_t(__popcll(bal & lt)), w.x + rc.v[0], w.y + rc.v[1], w.z + rc.v[2], i);
        o += uint32_t(__popcll(bal));
        w.next();
      }
      wave_lds_sync();
    }
  }
}

__global__ __launch_bounds__(256) void vox_ranges_kernel(const uint32_t *__restrict__ skeys, uint64_t K_cap,
                                                         const uint32_t *__restrict__ kdev, uint32_t T,
                                                         uint32_t *__restrict__ start) {
  const uint64_t K = min(K_cap, uint64_t(kdev[0]));
  const uint64_t k = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  // A thread writes the starts of the tiles between its key's and the previous
  // one's; a long run of empty tiles (the margins of a grid) is filled by the
  // whole wave (200,000 Gaussians in the middle of 256^3: 145 us with a thread
  // per run, 10 us now).
  int64_t prev = 0, cur = 0;
  if (k <= K) {
    prev = (k == 0) ? -1 : int64_t(skeys[k - 1]);
    cur = (k == K) ? int64_t(T) : int64_t(skeys[k]);
  }
  const bool wide = cur - prev > 8;
  if (!wide)
    for (int64_t t = prev + 1; t <= cur; ++t) start[t] = uint32_t(k);
  const int lane = threadIdx.x & 63;
  for (uint64_t todo = __ballot(wide); todo; todo &= todo - 1) {
    const int src = __ffsll(static_cast<unsigned long long>(todo)) - 1;
    const int64_t a = __shfl(prev, src, 64), c = __shfl(cur, src, 64);
    const uint32_t v = uint32_t(k - uint64_t(lane) + uint64_t(src));
    for (int64_t t = a + 1 + lane; t <= c; t += 64) start[t] = v;
  }
}

// kCount = true: count the (voxel, Gaussian) pairs in the support whose voxel
// lies in the grid (the algorithmic work) instead of writing the volume.
template <bool kCount, int TPB>
__global__ __launch_bounds__(kWave * TPB) void vox_fwd_kernel(const uint32_t *__restrict__ start,
                                                         const uint32_t *__restrict__ svals,
                                                         const float4 *__restrict__ prho,
                                                         const float4 *__restrict__ a0,
                                                         const float4 *__restrict__ a1,
                                                         const uint32_t *__restrict__ gid, GridDev G,
                                                         uint32_t n_tiles, int n_chunks,
                                                         float *__restrict__ vol,
                                                         unsigned long long *__restrict__ counter) {
  __shared__ float4 s_all[TPB][3][kWave];
  const int wid = threadIdx.x / kWave;
  float4 *s_p = s_all[wid][0], *s_a0 = s_all[wid][1], *s_a1 = s_all[wid][2];
  // work unit = (tile, chunk): chunk c takes batches c, c + n_chunks, ... of
  // the tile's list and writes its own partial volume (n_chunks > 1)
  // (whole tiles: runs on a narrow grid, an empty 256^3 76 us against 80; turned on
  // a wide one, 512^3 with 15 pairs per tile in a body 0.74 ms against 0.99)
  uint32_t blk;
  if (n_chunks > 1)
    blk = xcd_block(blockIdx.x, gridDim.x);
  else
    blk = G.nt[0] <= int(kXcds) * 4 ? xcd_run_block(blockIdx.x, gridDim.x) : turned_block(blockIdx.x, gridDim.x);
  const uint32_t unit = blk * TPB + wid;
  if (unit >= n_tiles * uint32_t(n_chunks)) return;
  const uint32_t tile = unit / uint32_t(n_chunks);
  const uint32_t chunk = unit - tile * uint32_t(n_chunks);
  const int tx = int(tile % uint32_t(G.nt[0]));
  const int tyz = int(tile / uint32_t(G.nt[0]));
  const int ty = tyz % G.nt[1];
  const int tz = tyz / G.nt[1];
  const int lane = threadIdx.x & (kWave - 1);
  const int y = ty * kVT + (lane & 7);
  const int z = tz * kVT + (lane >> 3);
  const float fx0 = float(tx * kVT), fy = float(y), fz = float(z);
  float acc[kVT];
#pragma unroll
  for (int k = 0; k < kVT; ++k) acc[k] = 0.f;
  const uint32_t b0 = start[tile], e = start[tile + 1];
  for (uint32_t b = b0 + chunk * kWave; b < e; b += kWave * uint32_t(n_chunks)) {
    const uint32_t m = min(uint32_t(kWave), e - b);
    if (uint32_t(lane) < m) {
      const uint32_t r = gid[svals[b + lane]];
      s_p[lane] = prho[r];
      s_a0[lane] = a0[r];
      s_a1[lane] = a1[r];
    }
    wave_lds_sync();
    for (uint32_t j = 0; j < m; ++j) {
      const float4 p = s_p[j];
      const float4 c0 = s_a0[j];
      const float4 c1 = s_a1[j];
      const float dy = fy - p.y, dz = fz - p.z;
      const float B = fmaf(c0.y, dy, c0.z * dz);
      const float Cc = fmaf(dy, fmaf(c0.w, dy, c1.x * dz), c1.y * dz * dz);
      const float dx0 = fx0 - p.x;
      // exponent along the row, expanded about the first voxel:
      // arg(dx0 + k) = arg0 + k (2 a dx0 + B) + a k^2
      const float arg0 = fmaf(dx0, fmaf(c0.x, dx0, B), Cc);
      const float E = fmaf(2.f * c0.x, dx0, B);
#pragma unroll
      for (int k = 0; k < kVT; ++k) {
        const float fk = float(k);
        const float arg = (k == 0) ? arg0 : fmaf(fk, fmaf(c0.x, fk, E), arg0);
        if (kCount) {
          acc[k] += (arg >= c1.z) ? 1.f : 0.f;
        } else {
          const float ex = __builtin_amdgcn_exp2f(arg);
          acc[k] = fmaf(p.w, (arg >= c1.z) ? ex : 0.f, acc[k]);
        }
      }
    }
    wave_lds_sync();
  }
  if (kCount) {
    unsigned long long n = 0;
    if (y < G.dims[1] && z < G.dims[2]) {
#pragma unroll
      for (int k = 0; k < kVT; ++k)
        if (tx * kVT + k < G.dims[0]) n += static_cast<unsigned long long>(acc[k]);
    }
    for (int d = 32; d > 0; d >>= 1) n += __shfl_xor(n, d, 64);
    if (lane == 0 && n) atomicAdd(counter, n);
    return;
  }
  if (y < G.dims[1] && z < G.dims[2]) {
    const uint64_t n_vox = uint64_t(G.dims[0]) * uint64_t(G.dims[1]) * uint64_t(G.dims[2]);
    float *row = vol + uint64_t(chunk) * n_vox + (uint64_t(z) * G.dims[1] + y) * uint64_t(G.dims[0]);
#pragma unroll
    for (int k = 0; k < kVT; ++k) {
      const int x = tx * kVT + k;
      if (x < G.dims[0]) row[x] = acc[k];
    }
  }
}

// ---------------------------------------------------------- large grids
//
// On grids with a wave per tile (no chunks) the forward sorts a tile's pairs
// by quarter of the tile (8 x 4 x 4 voxels, whole x-rows) before evaluating
// them: a quarter that the support does not reach is skipped, one that lies
// inside the support altogether ("interior") needs no cutoff test, and only
// the rest ("boundary") is evaluated as vox_fwd_kernel does. Both decisions
// come from the value and the gradient of the exponent at the quarter's
// centre: the form is concave, so its tangent plane bounds it from above
// (skip), and its value less every term's largest drop bounds it from below
// (interior). Both keep a margin of 0.1% of the kappa cutoff and of 4e-6 of the
// terms' sizes, which is above the rounding of these bounds and of the exponents
// that the per-voxel test compares (in needles the terms cancel, and the first
// margin alone is not), so every voxel keeps the decision of that test.

// Tiles per Gaussian and pairs per tile from which interior quarters (forward)
// and pairs (backward) are evaluated by products along the row. They change the
// order of the sums. Products pay where many quarters are interior: Gaussians
// all over 512^3, some 260 pairs per tile, forward and backward in list order and by
// products: 24 tiles per Gaussian (sigma 3 voxels) 5.97 + 10.2 and 5.64 + 10.7 ms, 87
// tiles 5.79 + 9.53 and 4.90 + 9.13, 130 tiles 5.67 + 9.44 and 4.63 + 8.63, 1,030 tiles
// 5.01 + 8.45 and 3.49 + 7.41. And they pay where a list fills the backward's rounds of
// 64, of which it makes two kinds: 130 tiles per Gaussian, 86 pairs per tile
// 1.71 + 4.04 and 1.55 + 4.09 ms, 26 pairs 0.77 + 1.75 and 0.81 + 2.57, 9 pairs
// 0.68 + 1.74 and 0.72 + 2.42.
constexpr uint64_t kProductKeysPerRecord = 96, kProductKeysPerTile = kWave;

// Which of the two kinds of kernel a call without chunks takes: the host knows
// where it read the pair count back; at a fixed key capacity it launches both
// (unless the capacity itself is below the line), and the blocks of one return
// at once. Every kernel of the product kind runs where the count reaches
// `from`, the others elsewhere, so a call's bits do not depend on how its
// lists were laid out.
struct VoxPick {
  const uint32_t *kdev;  // null: picked on the host
  uint64_t from;
};
__device__ __forceinline__ bool picked(const VoxPick &pick, bool product) {
  return !pick.kdev || (uint64_t(pick.kdev[0]) >= pick.from) == product;
}

// A pair's exponent over the tile, arg(k, Y, Z) = a00 + a10 Y + a01 Z + a20 Y^2
// + a11 Y Z + a02 Z^2 + k (e0 + e1 Y + e2 Z) + c k^2 for voxel k of the x-row
// (Y, Z), half-integers from the tile's centre.
struct TilePoly {
  float a00, a10, a01, e0;
  float g[3];  // gradient at the centre
  float q;     // value at the centre
  float err;   // bound on the rounding of the form's values over the tile
};

__device__ __forceinline__ TilePoly tile_poly(const float4 &p, const float4 &c0, const float4 &c1, float ox, float oy,
                                              float oz) {
  TilePoly T;
  const float dx = ox - p.x, dy = oy - p.y, dz = oz - p.z;
  const float hx = fmaf(c0.y, dy, c0.z * dz), hy = fmaf(c1.x, dz, c0.w * dy);
  T.q = fmaf(dx, fmaf(c0.x, dx, hx), fmaf(dy, hy, c1.y * dz * dz));
  T.g[0] = fmaf(2.f * c0.x, dx, hx);
  T.g[1] = fmaf(c0.y, dx, fmaf(2.f * c0.w, dy, c1.x * dz));
  T.g[2] = fmaf(c0.z, dx, fmaf(c1.x, dy, 2.f * c1.y * dz));
  const float h = 0.5f * (kVT - 1);
  const float size = fabsf(c0.x) + fabsf(c0.y) + fabsf(c0.z) + fabsf(c0.w) + fabsf(c1.x) + fabsf(c1.y);
  const float far = fmaxf(fmaxf(fabsf(dx), fabsf(dy)), fabsf(dz)) + h;
  T.err = 4e-6f * size * far * far;
  T.a00 = fmaf(h * h, c0.x, fmaf(-h, T.g[0], T.q));
  T.a10 = fmaf(-h, c0.y, T.g[1]);
  T.a01 = fmaf(-h, c0.z, T.g[2]);
  T.e0 = fmaf(-2.f * h, c0.x, T.g[0]);
  return T;
}

// Bits Q: quarter Q = (y half) + 2 (z half) reached by the support; interior.
__device__ __forceinline__ void quarter_masks(const TilePoly &T, const float4 &c0, const float4 &c1, float thr_cull,
                                              float thr_int, uint32_t &reach, uint32_t &inner) {
  // half-extents of a quarter's voxel centres: 3.5, 1.5, 1.5; its centre is at Y, Z = +-2
  const float drop = fmaf(12.25f, fabsf(c0.x), fmaf(2.25f, fabsf(c0.w) + fabsf(c1.y),
                          fmaf(5.25f, fabsf(c0.y) + fabsf(c0.z), 2.25f * fabsf(c1.x))));
  reach = inner = 0;
#pragma unroll
  for (int Q = 0; Q < 4; ++Q) {
    const float Y = (Q & 1) ? 2.f : -2.f, Z = (Q >> 1) ? 2.f : -2.f;
    const float gx = fmaf(c0.y, Y, fmaf(c0.z, Z, T.g[0]));
    const float gy = fmaf(2.f * c0.w, Y, fmaf(c1.x, Z, T.g[1]));
    const float gz = fmaf(c1.x, Y, fmaf(2.f * c1.y, Z, T.g[2]));
    const float q = fmaf(Y, fmaf(c0.w, Y, fmaf(c1.x, Z, T.g[1])), fmaf(Z, fmaf(c1.y, Z, T.g[2]), T.q));
    const float slope = fmaf(3.5f, fabsf(gx), 1.5f * (fabsf(gy) + fabsf(gz)));
    if (!(q + slope < thr_cull - T.err)) reach |= 1u << Q;
    if (q - slope - drop >= thr_int + T.err) inner |= 1u << Q;
  }
  // the products along a row stay far from the ends of FP32's range: their
  // exponent is at most |threshold| + 49 |c|
  inner &= (thr_int > -64.f && c0.x > -0.75f) ? reach : 0u;
}

// The quarters' lists of a batch of 64 pairs: slots whose bit Q of mask is
// set, in slot order, padded with the null slot to an even common length,
// which is returned. s_list: [4][kWave].
__device__ __forceinline__ int quarter_lists(uint32_t mask, int lane, uint8_t *s_list) {
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  int n[4], most = 0;
#pragma unroll
  for (int Q = 0; Q < 4; ++Q) {
    const bool bit = (mask >> Q) & 1u;
    const uint64_t bal = __ballot(bit);
    if (bit) s_list[Q * kWave + __popcll(bal & lt)] = uint8_t(lane);
    n[Q] = __popcll(bal);
    most = max(most, n[Q]);
  }
  most = (most + 1) & ~1;
#pragma unroll
  for (int Q = 0; Q < 4; ++Q)
    if (lane >= n[Q] && lane < most) s_list[Q * kWave + lane] = uint8_t(kWave);
  return most;
}

// Tiles in descending order of the lengths of their lists, by classes of a
// quarter of the mean length (all from eight times the mean on are one), in
// grid order within a class. counts: [blocks][kLengthClasses].
constexpr int kLengthClasses = 32;
__device__ __forceinline__ uint32_t length_class(const uint32_t *start, uint32_t n_tiles, uint32_t t) {
  const uint32_t mean = start[n_tiles] / n_tiles + 1u;
  return uint32_t(kLengthClasses - 1) - min(4u * (start[t + 1] - start[t]) / mean, uint32_t(kLengthClasses - 1));
}

__global__ __launch_bounds__(1024) void tile_classes_kernel(const uint32_t *__restrict__ start, uint32_t n_tiles,
                                                            uint32_t *__restrict__ counts) {
  __shared__ uint32_t s_n[kLengthClasses];
  if (threadIdx.x < kLengthClasses) s_n[threadIdx.x] = 0u;
  __syncthreads();
  const uint32_t t = blockIdx.x * 1024u + threadIdx.x;
  if (t < n_tiles) atomicAdd(&s_n[length_class(start, n_tiles, t)], 1u);
  __syncthreads();
  if (threadIdx.x < kLengthClasses) counts[blockIdx.x * kLengthClasses + threadIdx.x] = s_n[threadIdx.x];
}

__global__ __launch_bounds__(1024) void tile_order_kernel(const uint32_t *__restrict__ start, uint32_t n_tiles,
                                                          const uint32_t *__restrict__ counts,
                                                          uint32_t *__restrict__ order) {
  constexpr int kWaves = 1024 / kWave;
  __shared__ uint32_t s_total[kLengthClasses], s_before[kLengthClasses], s_wave[kWaves][kLengthClasses];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  // each class: its tiles in the grid, and in the blocks before this one
  if (threadIdx.x < kLengthClasses) s_total[threadIdx.x] = s_before[threadIdx.x] = 0u;
  __syncthreads();
  const uint32_t c0 = threadIdx.x % kLengthClasses;
  uint32_t total = 0, before = 0;
  for (uint32_t b = threadIdx.x / kLengthClasses; b < gridDim.x; b += 1024 / kLengthClasses) {
    const uint32_t n = counts[b * kLengthClasses + c0];
    total += n;
    before += b < blockIdx.x ? n : 0u;
  }
  atomicAdd(&s_total[c0], total);
  atomicAdd(&s_before[c0], before);
  const uint32_t t = blockIdx.x * 1024u + threadIdx.x;
  const bool ok = t < n_tiles;
  const uint32_t c = ok ? length_class(start, n_tiles, t) : 0u;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t rank = 0;
#pragma unroll
  for (int k = 0; k < kLengthClasses; ++k) {
    const uint64_t bal = __ballot(ok && c == uint32_t(k));
    if (lane == 0) s_wave[wid][k] = uint32_t(__popcll(bal));
    if (c == uint32_t(k)) rank = uint32_t(__popcll(bal & lt));
  }
  __syncthreads();
  if (!ok) return;
  uint32_t at = s_before[c] + rank;
  for (uint32_t k = 0; k < c; ++k) at += s_total[k];
  for (int w = 0; w < wid; ++w) at += s_wave[w][c];
  order[at] = t;
}

// One wave per 8^3 tile; 16-lane group Q owns quarter Q, each lane one x-row
// of 8 voxels, and walks its list of reached pairs in list order: the sums
// are vox_fwd_kernel's, bit for bit. Bound by VALU issue. Measured with
// 200,000 Gaussians at 256^3 in a body (sigma 3 voxels): 1.35 ms with whole
// tiles, compare and select, and a contiguous eighth of the grid per XCD; 0.65
// ms in runs of blocks per XCD, 0.46 by the order of tile_order_kernel.
template <int TPB>
__global__ __launch_bounds__(kWave * TPB) void vox_fwd_ordered_kernel(const uint32_t *__restrict__ start,
                                                                      const uint32_t *__restrict__ svals,
                                                                      const float4 *__restrict__ prho,
                                                                      const float4 *__restrict__ a0,
                                                                      const float4 *__restrict__ a1,
                                                                      const uint32_t *__restrict__ gid, GridDev G,
                                                                      uint32_t n_tiles, const uint32_t *__restrict__ order, float thr_widen,
                                                                      VoxPick pick, float *__restrict__ vol) {
  if (!picked(pick, false)) return;
  // slot kWave: a pair that adds nothing
  __shared__ float4 s_all[TPB][3][kWave + 1];
  __shared__ uint8_t s_list_all[TPB][4 * kWave];
  const int wid = threadIdx.x / kWave;
  float4 *s_p = s_all[wid][0], *s_a0 = s_all[wid][1], *s_a1 = s_all[wid][2];
  const uint32_t place = (order ? blockIdx.x : xcd_run_block(blockIdx.x, gridDim.x)) * TPB + wid;
  if (place >= n_tiles) return;
  const uint32_t tile = order ? uint32_t(__builtin_amdgcn_readfirstlane(int(order[place]))) : place;
  const int tx = int(tile % uint32_t(G.nt[0]));
  const int tyz = int(tile / uint32_t(G.nt[0]));
  const int ty = tyz % G.nt[1];
  const int tz = tyz / G.nt[1];
  const int lane = threadIdx.x & (kWave - 1);
  const int grp = lane >> 4;
  const int y = ty * kVT + (grp & 1) * 4 + (lane & 3), z = tz * kVT + (grp >> 1) * 4 + ((lane >> 2) & 3);
  const float fx0 = float(tx * kVT), fy = float(y), fz = float(z);
  const float h = 0.5f * (kVT - 1);
  if (lane == 0) {
    s_p[kWave] = s_a0[kWave] = make_float4(0.f, 0.f, 0.f, 0.f);
    s_a1[kWave] = make_float4(0.f, 0.f, INFINITY, 0.f);  // threshold above every exponent
  }
  float acc[kVT];
#pragma unroll
  for (int k = 0; k < kVT; ++k) acc[k] = 0.f;
  const uint32_t e = start[tile + 1];
  for (uint32_t b = start[tile]; b < e; b += kWave) {
    uint32_t reach = 0, inner = 0;
    if (b + lane < e) {
      const uint32_t r = gid[svals[b + lane]];
      const float4 p = prho[r], c0 = a0[r], c1 = a1[r];
      const TilePoly T = tile_poly(p, c0, c1, fx0 + h, float(ty * kVT) + h, float(tz * kVT) + h);
      quarter_masks(T, c0, c1, c1.z + thr_widen, c1.z - thr_widen, reach, inner);
      s_p[lane] = p;
      s_a0[lane] = c0;
      s_a1[lane] = c1;
    }
    const int n = quarter_lists(reach, lane, s_list_all[wid]);
    wave_lds_sync();
    const uint8_t *list = s_list_all[wid] + grp * kWave;
    for (int i = 0; i < n; ++i) {
      const int j = int(list[i]);
      const float4 p = s_p[j], c0 = s_a0[j], c1 = s_a1[j];
      const float dy = fy - p.y, dz = fz - p.z;
      const float B = fmaf(c0.y, dy, c0.z * dz);
      const float Cc = fmaf(dy, fmaf(c0.w, dy, c1.x * dz), c1.y * dz * dz);
      const float dx0 = fx0 - p.x;
      const float arg0 = fmaf(dx0, fmaf(c0.x, dx0, B), Cc);
      const float E = fmaf(2.f * c0.x, dx0, B);
      float arg[kVT], ex[kVT];
#pragma unroll
      for (int k = 0; k < kVT; ++k) {
        const float fk = float(k);
        arg[k] = (k == 0) ? arg0 : fmaf(fk, fmaf(c0.x, fk, E), arg0);
        ex[k] = __builtin_amdgcn_exp2f(arg[k]);
      }
      masked_fma8(acc, p.w, arg, ex, c1.z);
    }
    wave_lds_sync();
  }
  if (y < G.dims[1] && z < G.dims[2]) {
    float *row = vol + (uint64_t(z) * G.dims[1] + y) * uint64_t(G.dims[0]);
#pragma unroll
    for (int k = 0; k < kVT; ++k) {
      const int x = tx * kVT + k;
      if (x < G.dims[0]) row[x] = acc[k];
    }
  }
}

// One wave per 8^3 tile; 16-lane group Q owns quarter Q and walks its lists,
// its two 8-lane halves taking two entries at a time, each lane two x-rows
// (one y, two z) of 8 voxels; the halves' sums of the same voxels are added
// once at the end. Interior entries: exp2 of the row's first exponent and of
// its first step, then a voxel costs a product, p_{k+1} = p_k R, and an FMA
// with the pair's rho exp2(c k^2) (its eight values computed once per pair by
// the lane that stages it), 3.4 instructions per voxel with the row's share
// against 8.4 for the boundary path (v_exp_f32 takes two issue slots), whose
// arithmetic is vox_fwd_kernel's. Bound by VALU issue. Measured with
// 500,000 Gaussians at 512^3 (sigma 15 voxels): 54.3 ms with a whole tile per
// pair and compare and select, 32.4 ms now.
template <int TPB>
__global__ __launch_bounds__(kWave * TPB) void vox_fwd_product_kernel(const uint32_t *__restrict__ start,
                                                                      const uint32_t *__restrict__ svals,
                                                                      const float4 *__restrict__ prho,
                                                                      const float4 *__restrict__ a0,
                                                                      const float4 *__restrict__ a1,
                                                                      const uint32_t *__restrict__ gid, GridDev G,
                                                                      uint32_t n_tiles, float thr_widen, VoxPick pick,
                                                                      float *__restrict__ vol) {
  if (!picked(pick, true)) return;
  // per batch slot (slot kWave: a pair that adds nothing): the form's
  // coefficients, the tile polynomial, rho exp2(c k^2), and (p, rho)
  __shared__ float4 s_all[TPB][6][kWave + 1];
  __shared__ uint8_t s_list_all[TPB][2][4 * kWave];
  const int wid = threadIdx.x / kWave;
  float4 *s_c = s_all[wid][0], *s_d = s_all[wid][1], *s_t = s_all[wid][2], *s_e = s_all[wid][3],
         *s_f = s_all[wid][4], *s_p = s_all[wid][5];
  const uint32_t tile = xcd_run_block(blockIdx.x, gridDim.x) * TPB + wid;
  if (tile >= n_tiles) return;
  const int tx = int(tile % uint32_t(G.nt[0]));
  const int tyz = int(tile / uint32_t(G.nt[0]));
  const int ty = tyz % G.nt[1];
  const int tz = tyz / G.nt[1];
  const int lane = threadIdx.x & (kWave - 1);
  const int grp = lane >> 4, half = (lane >> 3) & 1;
  const int ly = (grp & 1) * 4 + (lane & 3), lz = (grp >> 1) * 4 + ((lane >> 2) & 1) * 2;
  const int y = ty * kVT + ly, z = tz * kVT + lz;
  const float fx0 = float(tx * kVT), fy = float(y), fz = float(z);
  const float h = 0.5f * (kVT - 1);
  const float Y = float(ly) - h, Z = float(lz) - h;
  const float ox = fx0 + h, oy = float(ty * kVT) + h, oz = float(tz * kVT) + h;
  if (lane == 0) {
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    s_c[kWave] = s_t[kWave] = s_e[kWave] = s_f[kWave] = s_p[kWave] = zero;
    s_d[kWave] = make_float4(0.f, 0.f, INFINITY, 0.f);  // threshold above every exponent
  }
  float acc[2][kVT];
#pragma unroll
  for (int k = 0; k < kVT; ++k) acc[0][k] = acc[1][k] = 0.f;
  const uint32_t e = start[tile + 1];
  for (uint32_t b = start[tile]; b < e; b += kWave) {
    uint32_t reach = 0, inner = 0;
    if (b + lane < e) {
      const uint32_t r = gid[svals[b + lane]];
      const float4 p = prho[r], c0 = a0[r], c1 = a1[r];
      const TilePoly T = tile_poly(p, c0, c1, ox, oy, oz);
      quarter_masks(T, c0, c1, c1.z + thr_widen, c1.z - thr_widen, reach, inner);
      s_c[lane] = make_float4(c0.y, c0.z, c0.w, c1.x);
      s_d[lane] = make_float4(c1.y, c0.x, c1.z, 0.f);
      s_p[lane] = p;
      if (inner) {
        s_t[lane] = make_float4(T.a00, T.a10, T.a01, T.e0);
        s_e[lane] = make_float4(p.w, p.w * __builtin_amdgcn_exp2f(c0.x), p.w * __builtin_amdgcn_exp2f(4.f * c0.x),
                                p.w * __builtin_amdgcn_exp2f(9.f * c0.x));
        s_f[lane] = make_float4(p.w * __builtin_amdgcn_exp2f(16.f * c0.x), p.w * __builtin_amdgcn_exp2f(25.f * c0.x),
                                p.w * __builtin_amdgcn_exp2f(36.f * c0.x), p.w * __builtin_amdgcn_exp2f(49.f * c0.x));
      }
    }
    const int n_in = quarter_lists(inner, lane, s_list_all[wid][0]);
    const int n_bd = quarter_lists(reach & ~inner, lane, s_list_all[wid][1]);
    wave_lds_sync();
    const uint8_t *l_in = s_list_all[wid][0] + grp * kWave + half, *l_bd = s_list_all[wid][1] + grp * kWave + half;
    for (int i = 0; i < n_in; i += 2) {
      const int j = int(l_in[i]);
      const float4 c = s_c[j], d = s_d[j], t = s_t[j], u = s_e[j], v = s_f[j];
      const float C[kVT] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
      const float ay = fmaf(Y, fmaf(c.z, Y, t.y), t.x);  // a00 + a10 Y + a20 Y^2
      const float az = fmaf(c.w, Y, t.z);                // a01 + a11 Y
      const float ey = fmaf(c.x, Y, t.w);                // e0 + e1 Y
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const float Zw = Z + float(w);
        float pk = __builtin_amdgcn_exp2f(fmaf(Zw, fmaf(d.x, Zw, az), ay));
        const float R = __builtin_amdgcn_exp2f(fmaf(c.y, Zw, ey));
        acc[w][0] = fmaf(pk, C[0], acc[w][0]);
#pragma unroll
        for (int k = 1; k < kVT; ++k) {
          pk *= R;
          acc[w][k] = fmaf(pk, C[k], acc[w][k]);
        }
      }
    }
    for (int i = 0; i < n_bd; i += 2) {
      const int j = int(l_bd[i]);
      const float4 c = s_c[j], d = s_d[j], p = s_p[j];
      const float dy = fy - p.y, dx0 = fx0 - p.x;
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const float dz = (fz + float(w)) - p.z;
        const float B = fmaf(c.x, dy, c.y * dz);
        const float Cc = fmaf(dy, fmaf(c.z, dy, c.w * dz), d.x * dz * dz);
        const float arg0 = fmaf(dx0, fmaf(d.y, dx0, B), Cc);
        const float E = fmaf(2.f * d.y, dx0, B);
        float arg[kVT], ex[kVT];
#pragma unroll
        for (int k = 0; k < kVT; ++k) {
          const float fk = float(k);
          arg[k] = (k == 0) ? arg0 : fmaf(fk, fmaf(d.y, fk, E), arg0);
          ex[k] = __builtin_amdgcn_exp2f(arg[k]);
        }
        masked_fma8(acc[w], p.w, arg, ex, d.z);
      }
    }
    wave_lds_sync();
  }
  // half 0 adds half 1's sums of the same rows (lane + 8); half 0 writes the first row, half 1 the second
  // (chosen from the sums: chosen from acc itself, the compiler indexed it by the lane, and
  // every entry of the lists went through memory)
  float sum[kVT];
#pragma unroll
  for (int k = 0; k < kVT; ++k) {
    const float s0 = acc[0][k] + __shfl_xor(acc[0][k], 8, kWave), s1 = acc[1][k] + __shfl_xor(acc[1][k], 8, kWave);
    sum[k] = half ? s1 : s0;
  }
  const int zw = z + half;
  if (y < G.dims[1] && zw < G.dims[2]) {
    float *row = vol + (uint64_t(zw) * G.dims[1] + y) * uint64_t(G.dims[0]);
#pragma unroll
    for (int k = 0; k < kVT; ++k) {
      const int x = tx * kVT + k;
      if (x < G.dims[0]) row[x] = sum[k];
    }
  }
}

// Moments of a pair, taken about the tile's centre, moved to the Gaussian's
// (q from the tile's centre: d = c - q) and written to its slot.
__device__ __forceinline__ void write_moments(float2 *__restrict__ out, float qx, float qy, float qz, float S0, float Sc,
                                              float Sy, float Sz, float Scc, float Sxy, float Sxz, float Syy,
                                              float Syz, float Szz) {
  const float Mx = fmaf(-qx, S0, Sc);
  const float My = fmaf(-qy, S0, Sy);
  const float Mz = fmaf(-qz, S0, Sz);
  const float Mxx = fmaf(qx * qx, S0, fmaf(-2.f * qx, Sc, Scc));
  const float Myy = fmaf(qy * qy, S0, fmaf(-2.f * qy, Sy, Syy));
  const float Mzz = fmaf(qz * qz, S0, fmaf(-2.f * qz, Sz, Szz));
  const float Mxy = fmaf(qx * qy, S0, fmaf(-qy, Sc, fmaf(-qx, Sy, Sxy)));
  const float Mxz = fmaf(qx * qz, S0, fmaf(-qz, Sc, fmaf(-qx, Sz, Sxz)));
  const float Myz = fmaf(qy * qz, S0, fmaf(-qz, Sy, fmaf(-qy, Sz, Syz)));
  out[0] = make_float2(S0, Mx);
  out[1] = make_float2(My, Mz);
  out[2] = make_float2(Mxx, Mxy);
  out[3] = make_float2(Mxz, Myy);
  out[4] = make_float2(Myz, Mzz);
}

// Backward over one 8^3 tile: lane j owns pair (tile, list[j]) and sums the
// ten moments over the 512 voxels. Coordinates are relative to the tile
// centre, (cx, cy, cz) in {-3.5, ..., 3.5}; along each x-row the exponent is
// a quadratic in cx with lane coefficients. The tile's g and g cx are staged
// in LDS, and each voxel adds g e into its column's sum (over y and z) and
// into the row's sums of g e and g e cx (three FMAs); the x-moments follow
// from the column sums, the others from the row sums, and all are moved to
// the Gaussian's centre once per pair. Branch-free loop body.
template <int TPB>
__global__ __launch_bounds__(kWave * TPB) void vox_bwd_kernel(const uint32_t *__restrict__ start,
                                                         const uint32_t *__restrict__ svals,
                                                         const float4 *__restrict__ prho,
                                                         const float4 *__restrict__ a0,
                                                         const float4 *__restrict__ a1,
                                                         const uint32_t *__restrict__ gid,
                                                         GridDev G, uint32_t n_tiles, int n_chunks, VoxPick pick,
                                                         const float *__restrict__ gvol,
                                                         float2 *__restrict__ partials) {
  if (!picked(pick, false)) return;
  __shared__ float4 s_g4_all[TPB][2][kVT * kVT * kVT / 4];
  const int wid = threadIdx.x / kWave;
  float4 *s_g4 = s_g4_all[wid][0];
  float *s_g = reinterpret_cast<float *>(s_g4);
  const float h = 0.5f * (kVT - 1);
  // work unit = (tile, chunk): chunk c takes batches c, c + n_chunks, ...
  // Natural order: blocks go round the XCDs, so on a wide grid an XCD keeps to
  // a few columns of tiles and their Gaussians (63.9 ms at 512^3 against 67.5
  // in turned order); on a narrow one the turned order keeps the load even.
  const uint32_t blk = G.nt[0] <= int(kXcds) * 4 ? turned_block(blockIdx.x, gridDim.x) : blockIdx.x;
  const uint32_t unit = blk * TPB + wid;
  if (unit >= n_tiles * uint32_t(n_chunks)) return;
  const uint32_t tile = unit / uint32_t(n_chunks);
  const uint32_t chunk = unit - tile * uint32_t(n_chunks);
  const int tx = int(tile % uint32_t(G.nt[0]));
  const int tyz = int(tile / uint32_t(G.nt[0]));
  const int ty = tyz % G.nt[1];
  const int tz = tyz / G.nt[1];
  const int lane = threadIdx.x & (kWave - 1);
  for (int q = lane; q < kVT * kVT * kVT; q += kWave) {
    const int x = tx * kVT + (q & 7), y = ty * kVT + ((q >> 3) & 7), z = tz * kVT + (q >> 6);
    const float g = (x < G.dims[0] && y < G.dims[1] && z < G.dims[2])
                        ? gvol[(uint64_t(z) * G.dims[1] + y) * uint64_t(G.dims[0]) + x]
                        : 0.f;
    s_g[q] = g;
    s_g[kVT * kVT * kVT + q] = g * (float(q & 7) - h);
  }
  wave_lds_sync();
  const uint32_t b0 = start[tile], e = start[tile + 1];
  const float ox = float(tx * kVT) + h, oy = float(ty * kVT) + h, oz = float(tz * kVT) + h;
  for (uint32_t b = b0 + chunk * kWave; b < e; b += kWave * uint32_t(n_chunks)) {
    const uint32_t k = b + lane;
    const bool active = k < e;
    float4 p = make_float4(ox, oy, oz, 0.f), c0 = make_float4(0.f, 0.f, 0.f, 0.f), c1 = c0;
    uint32_t q = 0;
    if (active) {
      q = svals[k];
      const uint32_t r = gid[q];
      p = prho[r];
      c0 = a0[r];
      c1 = a1[r];
    }
    const float qx = p.x - ox, qy = p.y - oy, qz = p.z - oz;
    const float m2aqx = -2.f * c0.x * qx;
    const float aqx2 = c0.x * qx * qx;
    float A[kVT];
#pragma unroll
    for (int u = 0; u < kVT; ++u) A[u] = 0.f;
    float Sy = 0.f, Sz = 0.f, Sxy = 0.f, Sxz = 0.f, Syy = 0.f, Syz = 0.f, Szz = 0.f;
    for (int zz = 0; zz < kVT; ++zz) {
      const float cz = float(zz) - h;
      const float dz = cz - qz;
#pragma unroll 2
      for (int yy = 0; yy < kVT; ++yy) {
        const float cy = float(yy) - h;
        const float dy = cy - qy;
        const float lin = fmaf(c0.y, dy, c0.z * dz);
        const float Cc = fmaf(dy, fmaf(c0.w, dy, c1.x * dz), c1.y * dz * dz);
        const float brow = lin + m2aqx;
        const float drow = fmaf(-lin, qx, aqx2 + Cc);
        const float4 *g4 = s_g4 + (zz * kVT + yy) * (kVT / 4);
        float R0 = 0.f, R1 = 0.f;
#pragma unroll
        for (int qd = 0; qd < kVT / 4; ++qd) {
          const float4 g0 = g4[qd];
          const float4 g1 = g4[kVT * kVT * kVT / 4 + qd];
          const float G0[4] = {g0.x, g0.y, g0.z, g0.w};
          const float G1[4] = {g1.x, g1.y, g1.z, g1.w};
          float arg[4], ex[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float cx = float(qd * 4 + u) - h;
            arg[u] = fmaf(cx, fmaf(c0.x, cx, brow), drow);
            ex[u] = __builtin_amdgcn_exp2f(arg[u]);
          }
          // (a call of few waves waits on the mask instead of on issue slots: 18.0
          // against 19.5 us for a 32^3 crop)
          if (TPB > 1) {
            masked_sums4(A, qd * 4, R0, R1, G0, G1, arg, ex, c1.z);
          } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const float e = (arg[u] >= c1.z) ? ex[u] : 0.f;
              A[qd * 4 + u] = fmaf(G0[u], e, A[qd * 4 + u]);
              R0 = fmaf(G0[u], e, R0);
              R1 = fmaf(G1[u], e, R1);
            }
          }
        }
        Sy = fmaf(R0, cy, Sy);
        Sz = fmaf(R0, cz, Sz);
        Sxy = fmaf(R1, cy, Sxy);
        Sxz = fmaf(R1, cz, Sxz);
        const float R0y = R0 * cy;
        Syy = fmaf(R0y, cy, Syy);
        Syz = fmaf(R0y, cz, Syz);
        Szz = fmaf(R0 * cz, cz, Szz);
      }
    }
    float S0 = 0.f, Sc = 0.f, Scc = 0.f;
#pragma unroll
    for (int u = 0; u < kVT; ++u) {
      const float cx = float(u) - h;
      S0 += A[u];
      Sc = fmaf(A[u], cx, Sc);
      Scc = fmaf(A[u], cx * cx, Scc);
    }
    if (active) {
      write_moments(partials + 5 * uint64_t(q), qx, qy, qz, S0, Sc, Sy, Sz, Scc, Sxy, Sxz, Syy, Syz, Szz);
    }
  }
}

// The ten moments of the pair (p, c0, c1) over a tile's 512 voxels, written to
// its slot. kInner: the tile lies inside the pair's support; a row then needs
// the exponentials of its first voxel and of its first step, and a voxel's
// factor is the running power p_{k+1} = p_k R times exp2(c k^2). Row sums are
// gathered per plane (over y) and folded into the z moments once per plane.
template <bool kInner>
__device__ __forceinline__ void tile_moments(const float4 &p, const float4 &c0, const float4 &c1, float ox, float oy,
                                             float oz, const float4 *__restrict__ s_g4, float2 *__restrict__ out,
                                             bool active) {
  const float h = 0.5f * (kVT - 1);
  const float qx = p.x - ox, qy = p.y - oy, qz = p.z - oz;
  const float m2aqx = -2.f * c0.x * qx;
  const float aqx2 = c0.x * qx * qx;
  float A[kVT], C[kVT];
#pragma unroll
  for (int u = 0; u < kVT; ++u) {
    A[u] = 0.f;
    if (kInner) C[u] = __builtin_amdgcn_exp2f(float(u * u) * c0.x);
  }
  float Sy = 0.f, Sz = 0.f, Sxy = 0.f, Sxz = 0.f, Syy = 0.f, Syz = 0.f, Szz = 0.f;
  TilePoly T;
  if (kInner) T = tile_poly(p, c0, c1, ox, oy, oz);
#pragma unroll 1
  for (int zz = 0; zz < kVT; ++zz) {
    const float cz = float(zz) - h;
    const float dz = cz - qz;
    float P0 = 0.f, P1 = 0.f, P2 = 0.f, Q0 = 0.f, Q1 = 0.f;
    // the plane's share of a row's first exponent and first step
    float u0 = 0.f, u1 = 0.f, v0 = 0.f;
    if (kInner) {
      u0 = fmaf(cz, fmaf(c1.y, cz, T.a01), T.a00);
      u1 = fmaf(c1.x, cz, T.a10);
      v0 = fmaf(c0.z, cz, T.e0);
    }
#pragma unroll
    for (int yy = 0; yy < kVT; ++yy) {
      const float cy = float(yy) - h;
      const float4 *g4 = s_g4 + (zz * kVT + yy) * (kVT / 4);
      float R0 = 0.f, R1 = 0.f, pk = 0.f, R = 0.f, brow = 0.f, drow = 0.f;
      if (kInner) {
        pk = __builtin_amdgcn_exp2f(fmaf(cy, fmaf(c0.w, cy, u1), u0));
        R = __builtin_amdgcn_exp2f(fmaf(c0.y, cy, v0));
      } else {
        const float dy = cy - qy;
        const float lin = fmaf(c0.y, dy, c0.z * dz);
        const float Cc = fmaf(dy, fmaf(c0.w, dy, c1.x * dz), c1.y * dz * dz);
        brow = lin + m2aqx;
        drow = fmaf(-lin, qx, aqx2 + Cc);
      }
#pragma unroll
      for (int qd = 0; qd < kVT / 4; ++qd) {
        const float4 g0 = g4[qd];
        const float4 g1 = g4[kVT * kVT * kVT / 4 + qd];
        const float G0[4] = {g0.x, g0.y, g0.z, g0.w};
        const float G1[4] = {g1.x, g1.y, g1.z, g1.w};
        if (kInner) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float ex = pk * C[qd * 4 + u];
            pk *= R;
            A[qd * 4 + u] = fmaf(G0[u], ex, A[qd * 4 + u]);
            R0 = fmaf(G0[u], ex, R0);
            R1 = fmaf(G1[u], ex, R1);
          }
        } else {
          float arg[4], ex[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float cx = float(qd * 4 + u) - h;
            arg[u] = fmaf(cx, fmaf(c0.x, cx, brow), drow);
            ex[u] = __builtin_amdgcn_exp2f(arg[u]);
          }
          masked_sums4(A, qd * 4, R0, R1, G0, G1, arg, ex, c1.z);
        }
      }
      P0 += R0;
      P1 = fmaf(R0, cy, P1);
      P2 = fmaf(R0, cy * cy, P2);
      Q0 += R1;
      Q1 = fmaf(R1, cy, Q1);
    }
    Sy += P1;
    Syy += P2;
    Sxy += Q1;
    Sz = fmaf(P0, cz, Sz);
    Szz = fmaf(P0 * cz, cz, Szz);
    Syz = fmaf(P1, cz, Syz);
    Sxz = fmaf(Q0, cz, Sxz);
  }
  float S0 = 0.f, Sc = 0.f, Scc = 0.f;
#pragma unroll
  for (int u = 0; u < kVT; ++u) {
    const float cx = float(u) - h;
    S0 += A[u];
    Sc = fmaf(A[u], cx, Sc);
    Scc = fmaf(A[u], cx * cx, Scc);
  }
  if (active) write_moments(out, qx, qy, qz, S0, Sc, Sy, Sz, Scc, Sxy, Sxz, Syy, Syz, Szz);
}

// Backward over one 8^3 tile where Gaussians span many tiles: as
// vox_bwd_kernel, one pair per lane, but the list is first sorted into pairs
// whose support holds the whole tile and the rest (the tests of
// quarter_masks, for the tile), through two rings in LDS, so that every round
// of 64 lanes is of one kind. The rows of a plane are unrolled, so their
// coordinates are constants (96 registers, 5 waves per SIMD: 1% faster than 6
// with 80). Bound by VALU issue: 6.4 instructions per voxel inside, 9 else.
// Measured with 500,000 Gaussians at 512^3 (half the pairs inside): 66.2 ms
// by vox_bwd_kernel, 57 ms now.
template <int TPB>
__global__ __launch_bounds__(kWave * TPB) __attribute__((amdgpu_waves_per_eu(5, 5))) void vox_bwd_product_kernel(const uint32_t *__restrict__ start,
                                                                      const uint32_t *__restrict__ svals,
                                                                      const float4 *__restrict__ prho,
                                                                      const float4 *__restrict__ a0,
                                                                      const float4 *__restrict__ a1,
                                                                      const uint32_t *__restrict__ gid, GridDev G,
                                                                      uint32_t n_tiles, float thr_widen, VoxPick pick,
                                                                      const float *__restrict__ gvol,
                                                                      float2 *__restrict__ partials) {
  if (!picked(pick, true)) return;
  __shared__ float4 s_g4_all[TPB][2][kVT * kVT * kVT / 4];
  __shared__ uint32_t s_ring_all[TPB][2][2 * kWave];
  const int wid = threadIdx.x / kWave;
  float4 *s_g4 = s_g4_all[wid][0];
  float *s_g = reinterpret_cast<float *>(s_g4);
  uint32_t(*s_ring)[2 * kWave] = s_ring_all[wid];
  const float h = 0.5f * (kVT - 1);
  const uint32_t blk = G.nt[0] <= int(kXcds) * TPB ? turned_block(blockIdx.x, gridDim.x) : blockIdx.x;
  const uint32_t tile = blk * TPB + wid;
  if (tile >= n_tiles) return;
  const int tx = int(tile % uint32_t(G.nt[0]));
  const int tyz = int(tile / uint32_t(G.nt[0]));
  const int ty = tyz % G.nt[1];
  const int tz = tyz / G.nt[1];
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  for (int q = lane; q < kVT * kVT * kVT; q += kWave) {
    const int x = tx * kVT + (q & 7), y = ty * kVT + ((q >> 3) & 7), z = tz * kVT + (q >> 6);
    const float g = (x < G.dims[0] && y < G.dims[1] && z < G.dims[2])
                        ? gvol[(uint64_t(z) * G.dims[1] + y) * uint64_t(G.dims[0]) + x]
                        : 0.f;
    s_g[q] = g;
    s_g[kVT * kVT * kVT + q] = g * (float(q & 7) - h);
  }
  wave_lds_sync();
  const uint32_t b0 = start[tile], e = start[tile + 1];
  const float ox = float(tx * kVT) + h, oy = float(ty * kVT) + h, oz = float(tz * kVT) + h;
  // a round over the first n <= 64 entries of a ring
  auto round = [&](auto kind, int n) {
    constexpr bool kInner = decltype(kind)::value;
    float4 p = make_float4(ox, oy, oz, 0.f), c0 = make_float4(0.f, 0.f, 0.f, 0.f), c1 = c0;
    uint32_t q = 0;
    if (lane < n) {
      q = svals[s_ring[kInner][lane]];
      const uint32_t r = gid[q];
      p = prho[r];
      c0 = a0[r];
      c1 = a1[r];
    }
    tile_moments<kInner>(p, c0, c1, ox, oy, oz, s_g4, partials + 5 * uint64_t(q), lane < n);
  };
  int n_ring[2] = {0, 0};
  for (uint32_t b = b0; b < e || n_ring[0] || n_ring[1]; b += kWave) {
    const bool more = b < e;  // after the list, one pass more empties the rings
    bool have = false, inside = false;
    const uint32_t k = b + lane;
    if (more && k < e) {
      const uint32_t r = gid[svals[k]];
      const float4 p = prho[r], c0 = a0[r], c1 = a1[r];
      const TilePoly T = tile_poly(p, c0, c1, ox, oy, oz);
      const float slope = h * (fabsf(T.g[0]) + fabsf(T.g[1]) + fabsf(T.g[2]));
      const float drop = h * h * (fabsf(c0.x) + fabsf(c0.y) + fabsf(c0.z) + fabsf(c0.w) + fabsf(c1.x) + fabsf(c1.y));
      have = true;
      inside = T.q - slope - drop >= c1.z - thr_widen + T.err && c1.z > -64.f && c0.x > -0.75f;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const bool mine = have && inside == (c == 1);
      const uint64_t bal = __ballot(mine);
      if (mine) s_ring[c][n_ring[c] + __popcll(bal & lt)] = k;
      n_ring[c] += __popcll(bal);
    }
    wave_lds_sync();
    if (n_ring[1] >= kWave || (!more && n_ring[1])) round(std::true_type(), min(n_ring[1], kWave));
    if (n_ring[0] >= kWave || (!more && n_ring[0])) round(std::false_type(), min(n_ring[0], kWave));
    // what is left (fewer than 64 entries) moves to the front
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (n_ring[c] < kWave && more) continue;
      const uint32_t v = s_ring[c][kWave + lane];
      wave_lds_sync();
      s_ring[c][lane] = v;
      n_ring[c] = max(0, n_ring[c] - kWave);
    }
    wave_lds_sync();
  }
}

// Per Gaussian: reduce its contiguous partial slots (ten moments each), then
// the chain rule. A block takes kGradGauss consecutive Gaussians; their slots
// are read by groups of kGradLanes lanes (consecutive lanes, consecutive
// slots) and summed across the group in a fixed butterfly order; one thread
// per Gaussian then applies the chain rule.
constexpr int kGradGauss = 64;
constexpr int kGradLanes = 32;

__global__ __launch_bounds__(256) void vox_grad_kernel(fgs_gaussians g, GridDev G,
                                                       const uint32_t *__restrict__ offset,
                                                       const float2 *__restrict__ partials,
                                                       const uint32_t *__restrict__ kdev,
                                                       fgs_gaussian_grads out, int accumulate) {
  __shared__ float s_sum[kGradGauss][11];
  __shared__ uint32_t s_off[kGradGauss + 1];
  // kdev[1]: the lists overflowed their capacity and hold nothing
  const bool none = kdev[1] != 0u;
  const int t = threadIdx.x;
  const int64_t i0 = int64_t(blockIdx.x) * kGradGauss;
  // the block's offsets in one coalesced read (offset has n + 1 entries)
  if (t <= kGradGauss && i0 + t <= g.n) s_off[t] = offset[i0 + t];
  __syncthreads();
  const int li = t % kGradLanes;
  for (int idx = t / kGradLanes; idx < kGradGauss; idx += 256 / kGradLanes) {
    if (i0 + idx >= g.n || none) break;
    const uint32_t o = s_off[idx], end = s_off[idx + 1];
    if (o == end) continue;  // the whole lane group agrees: no pairs, nothing to sum
    float acc[10];
#pragma unroll
    for (int c = 0; c < 10; ++c) acc[c] = 0.f;
    {
      for (uint32_t q = o + li; q < end; q += kGradLanes) {
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          const float2 v = partials[5 * uint64_t(q) + c];
          acc[2 * c] += v.x;
          acc[2 * c + 1] += v.y;
        }
      }
    }
#pragma unroll
    for (int d = 1; d < kGradLanes; d <<= 1)
#pragma unroll
      for (int c = 0; c < 10; ++c) acc[c] += __shfl_xor(acc[c], d, kGradLanes);
    if (li == 0)
#pragma unroll
      for (int c = 0; c < 10; ++c) s_sum[idx][c] = acc[c];
  }
  __syncthreads();
  if (t >= kGradGauss) return;
  const int64_t i = i0 + t;
  if (i >= g.n) return;
  const int64_t n = g.n;
  const uint32_t o = s_off[t], end = none ? o : s_off[t + 1];
  // a Gaussian with no pair adds nothing: when accumulating, leave it alone
  if (accumulate && o == end) return;
  float s[10];
#pragma unroll
  for (int c = 0; c < 10; ++c) s[c] = s_sum[t][c];
  float res[11];
#pragma unroll
  for (int c = 0; c < 11; ++c) res[c] = 0.f;
  if (o != end) {
    GaussParams P;
    load_gauss(g, i, P);
    VoxGauss V;
    vox_gauss(P, G, G.kappa, V);
    // s: S0, Sx, Sy, Sz, Sxx, Sxy, Sxz, Syy, Syz, Szz with d = voxel - centre
    const float rho = P.rho;
    const float Sd[3] = {s[1], s[2], s[3]};
    for (int a = 0; a < 3; ++a) {
      const float dpv = rho * (V.A[a][0] * Sd[0] + V.A[a][1] * Sd[1] + V.A[a][2] * Sd[2]);
      res[a] = dpv / G.h[a];
    }
    // dA_vox = -rho/2 M, M the symmetric second-moment matrix
    const float M[3][3] = {{s[4], s[5], s[6]}, {s[5], s[7], s[8]}, {s[6], s[8], s[9]}};
    // A_vox = W W^T: dW = 2 dA W
    float dR[9];
    for (int j = 0; j < 3; ++j) {
      float dls = 0.f;
      for (int a = 0; a < 3; ++a) {
        const float dW = -rho * (M[a][0] * V.W[0][j] + M[a][1] * V.W[1][j] + M[a][2] * V.W[2][j]);
        // W[a][j] = h_a R[a][j] / s_j
        dR[3 * a + j] = dW * G.h[a] / P.s[j];
        dls -= dW * V.W[a][j];
      }
      res[3 + j] = dls;
    }
    float dq[4];
    rot_grad_to_quat(P.qh, P.qnorm, dR, dq);
    res[6] = dq[0]; res[7] = dq[1]; res[8] = dq[2]; res[9] = dq[3];
    res[10] = s[0];
  }
  if (accumulate) {
    res[0] += out.mean[i]; res[1] += out.mean[n + i]; res[2] += out.mean[2 * n + i];
    res[3] += out.log_scale[i]; res[4] += out.log_scale[n + i]; res[5] += out.log_scale[2 * n + i];
    res[6] += out.quat[i]; res[7] += out.quat[n + i]; res[8] += out.quat[2 * n + i]; res[9] += out.quat[3 * n + i];
    res[10] += out.density[i];
  }
  out.mean[i] = res[0]; out.mean[n + i] = res[1]; out.mean[2 * n + i] = res[2];
  out.log_scale[i] = res[3]; out.log_scale[n + i] = res[4]; out.log_scale[2 * n + i] = res[5];
  out.quat[i] = res[6]; out.quat[n + i] = res[7]; out.quat[2 * n + i] = res[8]; out.quat[3 * n + i] = res[9];
  out.density[i] = res[10];
}

// ------------------------------------------------------------------ host

struct VoxLayout {
  uint64_t N, T, K;
  uint64_t total64, kdev, prho, radii, rect, offset, a0, a1, scan_scratch, start, hits;
  uint64_t fixed_end;
  uint64_t keys, vals, keys_alt, vals_alt, gid, sort_scratch, partials;
  uint64_t total;
  bool sorted_in_alt;
};

VoxLayout vox_layout(uint64_t N, uint64_t T, uint64_t K) {
  VoxLayout L{};
  L.N = N;
  L.T = T;
  L.K = K;
  Carver c(nullptr);
  c.take<unsigned long long>(1, &L.total64);
  c.take<uint32_t>(4, &L.kdev);
  c.take<float4>(N, &L.prho);
  c.take<float4>(N, &L.radii);
  c.take<Rect3>(N, &L.rect);
  c.take<uint32_t>(N + 1, &L.offset);
  c.take<float4>(N, &L.a0);
  c.take<float4>(N, &L.a1);
  c.take<uint32_t>(scan_scratch_words(N), &L.scan_scratch);
  c.take<uint32_t>(T + 1, &L.start);
  c.take<unsigned long long>(N * kHitWords, &L.hits);
  L.fixed_end = c.used;
  c.take<uint32_t>(K, &L.keys);
  c.take<uint32_t>(K, &L.vals);
  c.take<uint32_t>(K, &L.keys_alt);
  c.take<uint32_t>(K, &L.vals_alt);
  c.take<uint32_t>(K, &L.gid);
  c.take<uint32_t>(sort_scratch_words(K), &L.sort_scratch);
  c.take<float>(10 * K, &L.partials);
  L.total = c.used;
  const int bits = bits_for(T);
  const int passes = sort_passes(K, bits);
  L.sorted_in_alt = (passes & 1) != 0;
  return L;
}

// The culling tests' slack on the pre-scaled exponent (negative).
float cull_widening(const fgs_opts *o) { return -0.5f * kLog2e * o->kappa * o->kappa * (kCullSlack - 1.f); }

// Pairs from which a call takes the product kernels (one wave per tile only).
uint64_t product_from(const VoxLayout &L) {
  return chunks_per_tile(L.T) == 1 ? std::max(kProductKeysPerRecord * L.N, kProductKeysPerTile * L.T) : ~uint64_t(0);
}

// Whether the list-order forward takes its tiles longest list first: where
// lists average a batch of 64 or more and the chip holds a good share of the tiles
// at once (up to 65,536: 320^3). In grid order the longest lists end last: 200,000
// Gaussians in the middle of 256^3 0.67 ms, 0.46 longest first and 0.01 for
// the order; with more tiles the end weighs little and neighbours no longer
// share an L2 (sigma 3 voxels, 100 keys per tile in a body of 0.7 of the grid's width, grid
// order and longest first: 64,000 tiles 522 and 519 us, 110,592 tiles 880 and 898,
// 175,616 tiles 1,333 and 1,429; a narrower body gains up to 110,592 tiles too);
// with short lists the order costs what it gives (3,000 at 256^3 0.41 and 0.42 ms).
bool longest_first(const fgs_workspace *ws, const VoxLayout &L) {
  return ws->key_capacity == 0 && L.T <= 65536 && L.K >= kWave * L.T && L.K < product_from(L);
}

// Whether the forward without chunks takes whole tiles as vox_fwd_kernel does:
// below kShortLists pairs per tile on average there is little to skip, and the
// lists of quarters cost more than they save (256^3, Gaussians of sigma 3 voxels
// all over it: 9 pairs per tile 89 us and 98 by quarters, 28 pairs 108 and
// 112, 42 pairs 150 and 118). Large grids in workgroups of 16 tiles, since most of the
// time is the volume's writes and the dispatch (an empty 256^3: 76 us, 82 in
// workgroups of 4). The sums are the same either way.
constexpr uint64_t kShortLists = 16, kWideBlockTiles = 16384;
bool short_lists(const fgs_workspace *ws, const VoxLayout &L) {
  return ws->key_capacity == 0 && L.K < kShortLists * L.T;
}

// Waves per tile in the backward, whose pairs are independent of each other:
// as in the forward, but four also where lists average a batch of 64 or
// more. A wave per tile leaves the longest lists to the end: 200,000 Gaussians
// in the middle of 256^3, lists of some 500 to 800 in a fifth of the tiles: 0.79 ms
// with one, 0.56 ms with four (the CUs busy 58% and 93% of the time). From 2^24 tiles on
// four waves each would be 2^32 work-items, more than a launch holds.
int backward_chunks(const fgs_workspace *ws, const VoxLayout &L) {
  const int c = chunks_per_tile(L.T);
  const bool fits = L.T < (uint64_t(1) << 32) / (4 * kWave);
  return c == 1 && fits && ws->key_capacity == 0 && L.K >= kWave * L.T ? 4 : c;
}

template <typename T>
T *at(void *base, uint64_t off) {
  return reinterpret_cast<T *>(static_cast<char *>(base) + off);
}

// Calls list_order(pick) or product(pick) or, at a fixed key capacity that
// reaches the line, both.
template <typename F, typename P>
void with_vox_pick(const fgs_workspace *ws, void *b, const VoxLayout &L, F &&list_order, P &&product) {
  const bool reaches = L.K >= product_from(L), by_count = reaches && ws->key_capacity > 0;
  const VoxPick pick{by_count ? at<uint32_t>(b, L.kdev) : nullptr, product_from(L)};
  if (!reaches || by_count) list_order(pick);
  if (reaches) product(pick);
}

int validate(const fgs_gaussians *g, const fgs_grid *grid, const fgs_opts *o, fgs_workspace *ws) {
  if (!g || !grid || !o || !ws) return fail(FGS_E_INVALID, "null argument");
  if (g->n <= 0 || !g->mean || !g->log_scale || !g->quat || !g->density)
    return fail(FGS_E_INVALID, "invalid Gaussians");
  if (g->n > 0x7fffffff) return fail(FGS_E_UNSUPPORTED, "more than 2^31 Gaussians");
  for (int a = 0; a < 3; ++a) {
    if (grid->dims[a] <= 0 || grid->dims[a] > 65535 * kVT) return fail(FGS_E_INVALID, "grid dims");
    if (!(grid->spacing[a] > 0.f)) return fail(FGS_E_INVALID, "grid spacing");
  }
  if (!(o->kappa > 0.f)) return fail(FGS_E_INVALID, "kappa must be > 0");
  if (o->model != 0) return fail(FGS_E_INVALID, "opts.model must be 0 for the voxelizer");
  if (!(o->density_aabb_tau >= 0.f) || !std::isfinite(o->density_aabb_tau))
    return fail(FGS_E_INVALID, "density_aabb_tau must be finite and >= 0");
  return FGS_OK;
}

GridDev make_grid_dev(const fgs_grid *grid, const fgs_opts *o) {
  GridDev G{};
  for (int a = 0; a < 3; ++a) {
    G.origin[a] = grid->origin[a];
    G.h[a] = grid->spacing[a];
    G.dims[a] = grid->dims[a];
    G.nt[a] = (grid->dims[a] + kVT - 1) / kVT;
  }
  G.kappa = o->kappa;
  G.tau = o->density_aabb_tau;
  G.origin_dev = nullptr;
  return G;
}

// extra_bytes: room the caller needs after the lists (partial volumes).
int vox_build(const fgs_gaussians *g, const fgs_grid *grid, const fgs_opts *o, fgs_workspace *ws,
              hipStream_t s, VoxLayout *Lout, GridDev *Gout, uint64_t extra_bytes = 0,
              const float *origin_dev = nullptr) {
  GridDev G = make_grid_dev(grid, o);
  G.origin_dev = origin_dev;
  const uint64_t T = uint64_t(G.nt[0]) * G.nt[1] * G.nt[2];
  if (T >= 0xffffffffull) return fail(FGS_E_UNSUPPORTED, "too many voxel tiles");
  const uint64_t N = uint64_t(g->n);
  // key_capacity > 0: lists laid out for that many pairs, count kept on the device
  const uint64_t cap = ws->key_capacity;
  if (cap >= 0xffffffffull) return fail(FGS_E_UNSUPPORTED, "key_capacity must be below 2^32");
  VoxLayout L = vox_layout(N, T, cap);
  ws->kind = 0;
  if (cap > 0) {
    ws->needed = L.total + extra_bytes;
    ws->n_pairs = cap;
    ws->n_records = N;
    ws->n_tiles = T;
    if (!ws->ptr || ws->bytes < ws->needed) return fail(FGS_E_CAPACITY, "workspace too small for key_capacity pairs");
  } else if (!ws->ptr || ws->bytes < L.fixed_end + (uint64_t(1) << 20)) {
    ws->needed = L.fixed_end + (uint64_t(64) << 20);
    return fail(FGS_E_CAPACITY, "workspace too small for the per-Gaussian arrays");
  }
  void *b = ws->ptr;
  unsigned long long *total64 = at<unsigned long long>(b, L.total64);
  vox_record_kernel<<<grid_for(N, 256), 256, 0, s>>>(*g, G, at<float4>(b, L.prho), at<float4>(b, L.a0),
                                                      at<float4>(b, L.a1), at<float4>(b, L.radii),
                                                      at<Rect3>(b, L.rect));
  FGS_LAUNCH_CHECK("vox_record_kernel");
  const float thr_widen = cull_widening(o);
  with_wave_gauss(N, [&](auto per) {
    constexpr int PER = decltype(per)::value;
    vox_count_kernel<PER><<<grid_for(N, 4 * PER), 256, 0, s>>>(int64_t(N), at<float4>(b, L.prho), at<float4>(b, L.a0),
                                                               at<float4>(b, L.a1), at<Rect3>(b, L.rect), thr_widen,
                                                               at<uint32_t>(b, L.offset),
                                                               at<unsigned long long>(b, L.hits));
  });
  FGS_LAUNCH_CHECK("vox_count_kernel");
  // offsets, the 64-bit pair total and the device pair count (0 past the
  // capacity) in one scan
  uint32_t *kdev = at<uint32_t>(b, L.kdev);
  int st = scan_counts(at<uint32_t>(b, L.offset), N, at<uint32_t>(b, L.scan_scratch),
                       cap > 0 ? cap : uint64_t(0xfffffffeull), total64, kdev, cap > 0 ? ws->overflow : nullptr, s);
  if (st != FGS_OK) return st;
  if (cap == 0) {
    unsigned long long K64 = 0;
    FGS_HIP(hipMemcpyAsync(&K64, total64, sizeof(K64), hipMemcpyDeviceToHost, s));
    FGS_HIP(hipStreamSynchronize(s));
    if (K64 >= 0xffffffffull)
      return fail(FGS_E_UNSUPPORTED, "more than 2^32 (tile, Gaussian) pairs; split the grid into slabs");
    const uint64_t K = K64;
    L = vox_layout(N, T, K);
    ws->needed = L.total + extra_bytes;
    ws->n_pairs = K;
    ws->n_records = N;
    ws->n_tiles = T;
    if (ws->bytes < L.total + extra_bytes) return fail(FGS_E_CAPACITY, "workspace too small for the tile lists");
  }
  const uint64_t K = L.K;
  if (K > 0) {
    with_wave_gauss(N, [&](auto per) {
      constexpr int PER = decltype(per)::value;
      vox_emit_kernel<PER><<<grid_for(N, 4 * PER), 256, 0, s>>>(
          int64_t(N), G.nt[0], G.nt[1], at<float4>(b, L.prho), at<float4>(b, L.a0), at<float4>(b, L.a1),
          at<Rect3>(b, L.rect), thr_widen, at<uint32_t>(b, L.offset), at<unsigned long long>(b, L.hits),
          at<uint32_t>(b, L.keys), at<uint32_t>(b, L.vals), at<uint32_t>(b, L.gid), kdev);
    });
    FGS_LAUNCH_CHECK("vox_emit_kernel");
  }
  uint32_t *sk, *sv;
  st = radix_sort_pairs(at<uint32_t>(b, L.keys), at<uint32_t>(b, L.vals), at<uint32_t>(b, L.keys_alt),
                        at<uint32_t>(b, L.vals_alt), K, bits_for(T), at<uint32_t>(b, L.sort_scratch),
                        &sk, &sv, s, kSortMaxBits, cap > 0 ? kdev : nullptr);
  if (st != FGS_OK) return st;
  vox_ranges_kernel<<<grid_for(K + 1, 256), 256, 0, s>>>(sk, K, kdev, uint32_t(T), at<uint32_t>(b, L.start));
  FGS_LAUNCH_CHECK("vox_ranges_kernel");
  ws->kind = 2;
  *Lout = L;
  *Gout = G;
  return FGS_OK;
}

}  // namespace

// Workspace of a voxelizer call: as rast_workspace_bytes (the forward over
// few tiles also keeps one partial volume per chunk).
int vox_workspace_bytes(const fgs_gaussians *g, const fgs_grid *grid, bool forward, uint64_t *fixed_bytes,
                        uint64_t *bytes_per_key) {
  if (!g || !grid || g->n <= 0 || grid->dims[0] <= 0 || grid->dims[1] <= 0 || grid->dims[2] <= 0)
    return fail(FGS_E_INVALID, "workspace query: null argument, no Gaussians or grid dims");
  const uint64_t T = uint64_t((grid->dims[0] + kVT - 1) / kVT) * uint64_t((grid->dims[1] + kVT - 1) / kVT) *
                     uint64_t((grid->dims[2] + kVT - 1) / kVT);
  const uint64_t N = uint64_t(g->n);
  const uint64_t k_ref = uint64_t(1) << 24;
  const uint64_t base = vox_layout(N, T, 0).total;
  const uint64_t big = vox_layout(N, T, k_ref).total;
  const int chunks = chunks_per_tile(T);
  const uint64_t n_vox = uint64_t(grid->dims[0]) * uint64_t(grid->dims[1]) * uint64_t(grid->dims[2]);
  const uint64_t part = (forward && chunks > 1) ? uint64_t(chunks) * n_vox * sizeof(float) + 256 : 0;
  // (a call first asks for the per-record arrays plus 1 MiB before it knows K)
  *fixed_bytes = base + part + 8 * kAlign + (uint64_t(1) << 20);
  *bytes_per_key = (big - base + k_ref - 1) / k_ref;
  return FGS_OK;
}

int vox_binning_layout(const fgs_workspace *ws, uint64_t off[9], uint64_t counts[3]) {
  VoxLayout L = vox_layout(ws->n_records, ws->n_tiles, ws->n_pairs);
  off[0] = L.prho;
  off[1] = L.radii;
  off[2] = L.rect;
  off[3] = L.offset;
  off[4] = L.sorted_in_alt ? L.keys : L.keys_alt;
  off[5] = L.sorted_in_alt ? L.vals : L.vals_alt;
  off[6] = L.sorted_in_alt ? L.keys_alt : L.keys;
  off[7] = L.sorted_in_alt ? L.vals_alt : L.vals;
  off[8] = L.start;
  counts[0] = L.N;
  counts[1] = L.K;
  counts[2] = L.T;
  return FGS_OK;
}

}  // namespace fgs

namespace fgs {

int vox_forward(const fgs_gaussians *g, const fgs_grid *grid, const fgs_opts *opts, float *vol, fgs_workspace *ws,
                hipStream_t s, const float *origin_dev) {
  int st = validate(g, grid, opts, ws);
  if (st != FGS_OK) return st;
  if (!vol) return fail(FGS_E_INVALID, "null volume");
  const uint64_t n_tiles = uint64_t((grid->dims[0] + kVT - 1) / kVT) * uint64_t((grid->dims[1] + kVT - 1) / kVT) *
                           uint64_t((grid->dims[2] + kVT - 1) / kVT);
  const int chunks = chunks_per_tile(n_tiles);
  const uint64_t n_vox = uint64_t(grid->dims[0]) * uint64_t(grid->dims[1]) * uint64_t(grid->dims[2]);
  // partial volumes of the chunks, after the lists (only when chunked)
  const uint64_t part_bytes = chunks > 1 ? uint64_t(chunks) * n_vox * sizeof(float) + 256 : 0;
  VoxLayout L;
  GridDev G;
  st = vox_build(g, grid, opts, ws, s, &L, &G, part_bytes, origin_dev);
  if (st != FGS_OK) return st;
  void *b = ws->ptr;
  float *part = chunks > 1 ? at<float>(b, (L.total + 255) / 256 * 256) : vol;
  const uint32_t *sv = at<uint32_t>(b, L.sorted_in_alt ? L.vals_alt : L.vals);
  hipEvent_t *ev = static_cast<hipEvent_t *>(opts->events);
  if (ev) FGS_HIP(hipEventRecord(ev[0], s));
  const uint64_t units = L.T * uint64_t(chunks);
  const float thr_widen = cull_widening(opts);
  if (chunks == 1) {
    uint32_t *order = nullptr;
    if (longest_first(ws, L)) {
      // in the room of the backward's partial sums, 10 words per pair
      static_assert(10 * kWave >= 1 + kLengthClasses, "order and counts fit");
      const unsigned blocks = grid_for(L.T, 1024);
      order = at<uint32_t>(b, L.partials);
      uint32_t *counts = order + L.T;
      tile_classes_kernel<<<blocks, 1024, 0, s>>>(at<uint32_t>(b, L.start), uint32_t(L.T), counts);
      FGS_LAUNCH_CHECK("tile_classes_kernel");
      tile_order_kernel<<<blocks, 1024, 0, s>>>(at<uint32_t>(b, L.start), uint32_t(L.T), counts, order);
      FGS_LAUNCH_CHECK("tile_order_kernel");
    }
    auto whole = [&](auto tpb) {
      constexpr int TPB = decltype(tpb)::value;
      vox_fwd_kernel<false, TPB><<<grid_for(L.T, TPB), kWave * TPB, 0, s>>>(
          at<uint32_t>(b, L.start), sv, at<float4>(b, L.prho), at<float4>(b, L.a0), at<float4>(b, L.a1),
          at<uint32_t>(b, L.gid), G, uint32_t(L.T), 1, vol, nullptr);
    };
    with_vox_pick(
        ws, b, L,
        [&](const VoxPick &pick) {
          if (short_lists(ws, L) && L.T >= kWideBlockTiles)
            return whole(std::integral_constant<int, 16>());
          if (short_lists(ws, L)) return whole(std::integral_constant<int, 4>());
          vox_fwd_ordered_kernel<4><<<grid_for(L.T, 4), kWave * 4, 0, s>>>(
              at<uint32_t>(b, L.start), sv, at<float4>(b, L.prho), at<float4>(b, L.a0), at<float4>(b, L.a1),
              at<uint32_t>(b, L.gid), G, uint32_t(L.T), order, thr_widen, pick, vol);
        },
        [&](const VoxPick &pick) {
          vox_fwd_product_kernel<4><<<grid_for(L.T, 4), kWave * 4, 0, s>>>(
              at<uint32_t>(b, L.start), sv, at<float4>(b, L.prho), at<float4>(b, L.a0), at<float4>(b, L.a1),
              at<uint32_t>(b, L.gid), G, uint32_t(L.T), thr_widen, pick, vol);
        });
    FGS_LAUNCH_CHECK("vox_fwd_ordered_kernel / vox_fwd_product_kernel");
  } else {
    with_tiles_per_block(units, [&](auto tpb) {
      constexpr int TPB = decltype(tpb)::value;
      vox_fwd_kernel<false, TPB><<<grid_for(units, TPB), kWave * TPB, 0, s>>>(
          at<uint32_t>(b, L.start), sv, at<float4>(b, L.prho), at<float4>(b, L.a0), at<float4>(b, L.a1),
          at<uint32_t>(b, L.gid), G, uint32_t(L.T), chunks, part, nullptr);
    });
    FGS_LAUNCH_CHECK("vox_fwd_kernel");
    st = sum_chunks(part, chunks, n_vox, vol, s);
    if (st != FGS_OK) return st;
  }
  if (ev) FGS_HIP(hipEventRecord(ev[1], s));
  return FGS_OK;
}

}  // namespace fgs

using namespace fgs;

extern "C" int fgs_voxelize_fwd(const fgs_gaussians *g, const fgs_grid *grid, const fgs_opts *opts,
                                float *vol, fgs_workspace *ws, void *stream) {
  return vox_forward(g, grid, opts, vol, ws, static_cast<hipStream_t>(stream), nullptr);
}

extern "C" int fgs_voxelize_support(const fgs_gaussians *g, const fgs_grid *grid, const fgs_opts *opts,
                                    uint64_t *out, fgs_workspace *ws, void *stream) {
  int st = validate(g, grid, opts, ws);
  if (st != FGS_OK) return st;
  if (!out) return fail(FGS_E_INVALID, "null output");
  hipStream_t s = static_cast<hipStream_t>(stream);
  VoxLayout L;
  GridDev G;
  st = vox_build(g, grid, opts, ws, s, &L, &G);
  if (st != FGS_OK) return st;
  void *b = ws->ptr;
  unsigned long long *cnt = reinterpret_cast<unsigned long long *>(out);
  zero_u64_kernel<<<1, 1, 0, s>>>(cnt, 1);
  FGS_LAUNCH_CHECK("zero_u64_kernel");
  const uint32_t *sv = at<uint32_t>(b, L.sorted_in_alt ? L.vals_alt : L.vals);
  const int chunks = chunks_per_tile(L.T);
  const uint64_t units = L.T * uint64_t(chunks);
  with_tiles_per_block(units, [&](auto tpb) {
    constexpr int TPB = decltype(tpb)::value;
    vox_fwd_kernel<true, TPB><<<grid_for(units, TPB), kWave * TPB, 0, s>>>(
        at<uint32_t>(b, L.start), sv, at<float4>(b, L.prho), at<float4>(b, L.a0), at<float4>(b, L.a1),
        at<uint32_t>(b, L.gid), G, uint32_t(L.T), chunks, nullptr, cnt);
  });
  FGS_LAUNCH_CHECK("vox_fwd_kernel<count>");
  return FGS_OK;
}

namespace fgs {

int vox_backward(const fgs_gaussians *g, const fgs_grid *grid, const fgs_opts *opts, const float *grad_vol,
                 fgs_gaussian_grads *out, fgs_workspace *ws, hipStream_t s, const float *origin_dev) {
  int st = validate(g, grid, opts, ws);
  if (st != FGS_OK) return st;
  if (!grad_vol || !out || !out->mean || !out->log_scale || !out->quat || !out->density)
    return fail(FGS_E_INVALID, "null gradient buffer");
  VoxLayout L;
  GridDev G;
  if (opts->recompute) {
    st = vox_build(g, grid, opts, ws, s, &L, &G, 0, origin_dev);
    if (st != FGS_OK) return st;
  } else {
    G = make_grid_dev(grid, opts);
    G.origin_dev = origin_dev;
    const uint64_t T = uint64_t(G.nt[0]) * G.nt[1] * G.nt[2];
    if (ws->kind != 2 || ws->n_records != uint64_t(g->n) || ws->n_tiles != T || !ws->ptr)
      return fail(FGS_E_INVALID, "workspace does not hold this call's voxelizer lists");
    L = vox_layout(uint64_t(g->n), T, ws->n_pairs);
    if (ws->bytes < L.total) return fail(FGS_E_INVALID, "workspace lists do not match this call");
  }
  void *b = ws->ptr;
  const uint32_t *sv = at<uint32_t>(b, L.sorted_in_alt ? L.vals_alt : L.vals);
  hipEvent_t *ev = static_cast<hipEvent_t *>(opts->events);
  if (ev) FGS_HIP(hipEventRecord(ev[0], s));
  if (L.K > 0) {
    const int chunks = backward_chunks(ws, L);
    const uint64_t units = L.T * uint64_t(chunks);
    with_vox_pick(
        ws, b, L,
        [&](const VoxPick &pick) {
          with_tiles_per_block(units, [&](auto tpb) {
            constexpr int TPB = decltype(tpb)::value;
            vox_bwd_kernel<TPB><<<grid_for(units, TPB), kWave * TPB, 0, s>>>(
                at<uint32_t>(b, L.start), sv, at<float4>(b, L.prho), at<float4>(b, L.a0), at<float4>(b, L.a1),
                at<uint32_t>(b, L.gid), G, uint32_t(L.T), chunks, pick, grad_vol, at<float2>(b, L.partials));
          });
        },
        [&](const VoxPick &pick) {
          vox_bwd_product_kernel<4><<<grid_for(L.T, 4), kWave * 4, 0, s>>>(
              at<uint32_t>(b, L.start), sv, at<float4>(b, L.prho), at<float4>(b, L.a0), at<float4>(b, L.a1),
              at<uint32_t>(b, L.gid), G, uint32_t(L.T), cull_widening(opts), pick, grad_vol, at<float2>(b, L.partials));
        });
    FGS_LAUNCH_CHECK("vox_bwd_kernel / vox_bwd_product_kernel");
  }
  if (ev) FGS_HIP(hipEventRecord(ev[1], s));
  vox_grad_kernel<<<grid_for(uint64_t(g->n), kGradGauss), 256, 0, s>>>(*g, G, at<uint32_t>(b, L.offset),
                                                                at<float2>(b, L.partials),
                                                                at<uint32_t>(b, L.kdev), *out,
                                                                opts->accumulate);
  FGS_LAUNCH_CHECK("vox_grad_kernel");
  return FGS_OK;
}

}  // namespace fgs

extern "C" int fgs_voxelize_bwd(const fgs_gaussians *g, const fgs_grid *grid, const fgs_opts *opts,
                                const float *grad_vol, fgs_gaussian_grads *out, fgs_workspace *ws,
                                void *stream) {
  return vox_backward(g, grid, opts, grad_vol, out, ws, static_cast<hipStream_t>(stream), nullptr);
}
