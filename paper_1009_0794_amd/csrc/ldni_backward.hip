// ldni_backward.hip -- gfx950 kernels of the sampler's backward pass: the
// vertex gradient of a loss on the samples (depth and normal) of an LDNI,
// with the sample set held fixed.
#pragma clang fp contract(off)

#include <cmath>

#include "ldni_internal.hpp"

namespace ldni {
namespace {

constexpr int kBlock = 256;  // 4 wave64 per workgroup

inline unsigned grid_for(int64_t n, int per_block) { return (unsigned)((n + per_block - 1) / per_block); }

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
// For a sample on triangle (A,B,C) at pixel centre c, with barycentric
// weights lambda of c in the projected triangle and unit normal n:
//   depth:  moving vertex X moves the hit along the fixed ray by
//           lambda_X (n . dX) / n_a, so dL/dX += gd * lambda_X * n / n_a;
//   normal: n = N/|N|, N = (B-A)x(C-A): dL/dN = (gn - n (n.gn)) / |N| and
//           dL/dA = (B-C) x dL/dN, dL/dB = (C-A) x dL/dN, dL/dC = (A-B) x dL/dN.
// n / n_a and the normal Jacobian are constant per triangle, so the
// sample-parallel kernel only accumulates, per (triangle, image), the sums of
// gd * lambda_X and of gn; the triangle-parallel kernel applies the
// per-triangle factors and adds to the three vertices.
struct BackwardImage {
  int32_t a, u, v, w;
  double lo_u, h_u, lo_v, h_v;
  // bound, in pixels, on the distance between a float32 pixel centre and
  // its float64 position estimate (x - lo) / h - 0.5 for x within the image
  double margin_u, margin_v;
  const uint32_t* offsets;  // [w*w+1]
  const int32_t* tri;       // [n]
  const float* gd;          // [n] or null
  const float* gn;          // [n][3] or null
  float* acc;               // [T][6] sums of gd * lambda per vertex, then of gn
};

struct BackwardSet {
  BackwardImage img[kMaxImages];
  int32_t n;
  uint32_t block_start[kMaxImages + 1];  // pixel blocks per image
  const float* verts;
  int64_t n_verts;
  const int32_t* tris;
  int64_t n_tris;
};

// One workgroup per kBwdTile x kBwdTile pixel tile.  The tile's samples (one
// contiguous range per pixel row) are spread over the threads; each sample's
// six values (gd * lambda per vertex, gn) are summed per triangle in an LDS
// hash table, and every triangle of the tile then writes its sums once: with
// plain stores when every pixel centre its projection can cover lies in the
// tile (no other tile has samples of it on this image: the common case, and
// stores cost far less than global atomics), else with atomic additions.  A
// sample that finds no free slot adds its own directly (its triangle then has
// no slot in this tile, so nothing stores over it).
// Bound by the chain of dependent loads per sample and by the atomics, which
// go out to memory at 11 to 12 cache lines a nanosecond whatever they hold:
// so six neighbouring lanes write a triangle's six sums, and a tile borrows no
// pixel it need not (centres within the projection, not the pixels touched).
// 261,120 triangles at w = 512, 1.6 M samples: 234 us with a lane per triangle
// (1.7 M lines) and 256 threads, 125 us now; 512 threads because tiles at the
// mesh's poles hold 7,900 samples (256: 149 us), tiles of 12 pixels 123, of 8
// 154 us, 2,048 slots 161 us (fewer workgroups per CU), quartered deep tiles
// 157 us.
constexpr int kBwdTile = 16;
constexpr int kBwdBlock = 512;
constexpr int kBwdSlotBits = 10;
constexpr int kBwdSlots = 1 << kBwdSlotBits;
constexpr int kBwdProbe = 8;  // (32 steps took 5 % longer in full tables)
static_assert(kBwdSlots % kBwdBlock == 0, "the list of slots is made in whole steps of the workgroup");
constexpr uint32_t kBwdInside = 1u << 31;  // flag of a key: the tile holds all of the triangle

// The coordinates u and v of vertex i (its three floats in one load), clamped to the array.
__device__ __forceinline__ void load_uv(const BackwardSet& bs, const BackwardImage& im, int32_t i, double& u, double& v) {
  const float* P = bs.verts + 3 * (int64_t)min(max(i, 0), (int32_t)(bs.n_verts - 1));
  const float p0 = P[0], p1 = P[1], p2 = P[2];
  u = (double)(im.u == 0 ? p0 : im.u == 1 ? p1 : p2);
  v = (double)(im.v == 0 ? p0 : im.v == 1 ? p1 : p2);
}

// Whether every pixel whose centre can lie in the projection of triangle t
// on image im is a pixel of the tile (x0, y0, cw, ch): the centres within the
// projection's bounding box, its index range widened by the image's rounding
// margin.  Only then does the tile hold all of t's samples on im.
__device__ __forceinline__ bool projection_in_tile(const BackwardSet& bs, const BackwardImage& im, int64_t t,
                                                   int x0, int y0, int cw, int ch) {
  const int32_t* fv = bs.tris + 3 * t;
  double umin = HUGE_VAL, umax = -HUGE_VAL, vmin = HUGE_VAL, vmax = -HUGE_VAL;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    double u, v;
    load_uv(bs, im, fv[q], u, v);
    umin = fmin(umin, u);
    umax = fmax(umax, u);
    vmin = fmin(vmin, v);
    vmax = fmax(vmax, v);
  }
  // pixel i has centre f32(lo + (i + 0.5) h); a centre in [mn, mx] has i
  // within [tmn - m, tmx + m] for t = (x - lo) / h - 0.5 and m the margin
  const double iu0 = (umin - im.lo_u) / im.h_u - 0.5 - im.margin_u,
               iu1 = (umax - im.lo_u) / im.h_u - 0.5 + im.margin_u;
  const double iv0 = (vmin - im.lo_v) / im.h_v - 0.5 - im.margin_v,
               iv1 = (vmax - im.lo_v) / im.h_v - 0.5 + im.margin_v;
  return iu0 > (double)(x0 - 1) && iu1 < (double)(x0 + cw) && iv0 > (double)(y0 - 1) && iv1 < (double)(y0 + ch);
}

__global__ void __launch_bounds__(kBwdBlock) backward_samples_kernel(BackwardSet bs) {
  __shared__ uint32_t s_row[kBwdTile + 1][kBwdTile + 1];  // offsets of the tile's rows
  __shared__ uint32_t s_pre[kBwdTile + 1];                // samples before each row
  __shared__ alignas(16) uint32_t s_key[kBwdSlots];       // triangle + 1, 0 = free
  __shared__ alignas(16) float s_val[kBwdSlots][6];
  __shared__ uint16_t s_used[kBwdSlots];
  __shared__ uint32_t s_taken;
  const int lane = threadIdx.x & 63;
  int k = 0;
  while (k + 1 < bs.n && blockIdx.x >= bs.block_start[k + 1]) ++k;
  const BackwardImage& im = bs.img[k];
  const int ntx = (im.w + kBwdTile - 1) / kBwdTile;
  const int tile = (int)(blockIdx.x - bs.block_start[k]);
  const int x0 = (tile % ntx) * kBwdTile, y0 = (tile / ntx) * kBwdTile;
  const int cw = min(kBwdTile, im.w - x0), ch = min(kBwdTile, im.w - y0);
  // every wave by itself: the tile's samples, a row per lane
  uint32_t row = 0;
  if (lane < ch) {
    const uint32_t* o = im.offsets + (int64_t)(y0 + lane) * im.w + x0;
    row = o[cw] - o[0];
  }
  uint32_t upto = row;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)upto, d, 64);
    if (lane >= d) upto += y;
  }
  const uint32_t S = (uint32_t)__shfl((int)upto, 63, 64);
  if (S == 0) return;

  if (threadIdx.x < 64 && lane <= ch) s_pre[lane] = upto - row;  // (upto of the lanes from ch on: all)
  for (int q = threadIdx.x; q < ch * (cw + 1); q += kBwdBlock) {
    const int r = q / (cw + 1), x = q - r * (cw + 1);
    s_row[r][x] = im.offsets[(int64_t)(y0 + r) * im.w + x0 + x];
  }
  for (int q = threadIdx.x; q < kBwdSlots / 4; q += kBwdBlock) reinterpret_cast<uint4*>(s_key)[q] = make_uint4(0, 0, 0, 0);
  for (int q = threadIdx.x; q < kBwdSlots * 6 / 4; q += kBwdBlock)
    reinterpret_cast<float4*>(s_val)[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (threadIdx.x == 0) s_taken = 0;
  __syncthreads();
  float* const accp = im.acc;

  for (uint32_t f = threadIdx.x; f < S; f += kBwdBlock) {
    int r = 0;  // row of f: the last r with s_pre[r] <= f (binary search)
    for (int hi = ch - 1; r < hi;) {
      const int mid = (r + hi + 1) >> 1;
      if (s_pre[mid] <= f) r = mid; else hi = mid - 1;
    }
    const uint32_t s = s_row[r][0] + (f - s_pre[r]);
    const int32_t t = im.tri[s];
    // all loads of a sample that do not hang on another are under way at once
    const float g = im.gd ? im.gd[s] : 0.0f;
    float v[6] = {0, 0, 0, 0, 0, 0};
    if (im.gn) {
      const float* gv = im.gn + 3 * (int64_t)s;
      v[3] = gv[0];
      v[4] = gv[1];
      v[5] = gv[2];
    }
    if (t < 0 || t >= bs.n_tris) continue;  // not a triangle of this mesh
    if (g != 0.0f) {
      const int32_t* fv = bs.tris + 3 * (int64_t)t;
      double xu[3], xv[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) load_uv(bs, im, fv[q], xu[q], xv[q]);
      int lo = 0, hi = cw - 1;  // pixel of s in the row: the last x with s_row[r][x] <= s
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_row[r][mid] <= s) lo = mid; else hi = mid - 1;
      }
      const double cu = im.lo_u + ((double)(x0 + lo) + 0.5) * im.h_u;
      const double cv = im.lo_v + ((double)(y0 + r) + 0.5) * im.h_v;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        xu[q] -= cu;
        xv[q] -= cv;
      }
      const double e_bc = xu[1] * xv[2] - xv[1] * xu[2];
      const double e_ca = xu[2] * xv[0] - xv[2] * xu[0];
      const double e_ab = xu[0] * xv[1] - xv[0] * xu[1];
      const double den = e_ab + e_bc + e_ca;
      if (den != 0.0) {
        const double gs = (double)g / den;
        v[0] = (float)(gs * e_bc);
        v[1] = (float)(gs * e_ca);
        v[2] = (float)(gs * e_ab);
      }
    }
    if (v[0] == 0.0f && v[1] == 0.0f && v[2] == 0.0f && v[3] == 0.0f && v[4] == 0.0f && v[5] == 0.0f)
      continue;
    // slot of t in the table (linear probing, a bounded number of steps; none
    // for the one triangle whose key would be the flag)
    const uint32_t key = (uint32_t)t + 1u;
    uint32_t h = ((uint32_t)t * 2654435761u) >> (32 - kBwdSlotBits);
    int slot = -1;
    for (int step = key == kBwdInside ? kBwdProbe : 0; step < kBwdProbe; ++step) {
      const uint32_t old = atomicCAS(&s_key[h], 0u, key);
      if (old == 0u || old == key) {
        slot = (int)h;
        break;
      }
      h = (h + 1) & (kBwdSlots - 1);
    }
    if (slot >= 0) {
#pragma unroll
      for (int c = 0; c < 6; ++c)
        if (v[c] != 0.0f) atomicAdd(&s_val[slot][c], v[c]);
    } else {
      float* a6 = accp + 6 * (int64_t)t;
#pragma unroll
      for (int c = 0; c < 6; ++c)
        if (v[c] != 0.0f) atomicAdd(a6 + c, v[c]);
    }
  }
  __syncthreads();
  // list the slots taken and mark the triangles that the tile holds all of
  for (int q0 = 0; q0 < kBwdSlots; q0 += kBwdBlock) {
    const int q = q0 + (int)threadIdx.x;
    const uint32_t key = s_key[q];
    const uint64_t taken = __ballot(key != 0u);
    uint32_t to = 0;
    if (lane == 0 && taken != 0) to = atomicAdd(&s_taken, (uint32_t)__popcll(taken));
    to = __shfl(to, 0, 64);
    if (key != 0u) {
      s_used[to + (uint32_t)__popcll(taken & ((1ull << lane) - 1))] = (uint16_t)q;
      if (projection_in_tile(bs, im, (int64_t)(key - 1u), x0, y0, cw, ch)) s_key[q] = key | kBwdInside;
    }
  }
  __syncthreads();
  const int n_sums = 6 * (int)s_taken;
  for (int e = threadIdx.x; e < n_sums; e += kBwdBlock) {
    const int q = s_used[e / 6], c = e % 6;
    const uint32_t key = s_key[q];
    const float x = s_val[q][c];
    float* const to = accp + 6 * (int64_t)((key & ~kBwdInside) - 1u) + c;
    if (key & kBwdInside) *to = x;
    else if (x != 0.0f) atomicAdd(to, x);
  }
}

// The gradient of triangle t's three vertices (false: t is not a valid
// triangle, or degenerate, and adds nothing).
__device__ bool triangle_gradient(const BackwardSet& bs, int64_t t, int32_t (&vid)[3], double (&g)[3][3]) {
  const int32_t* f = bs.tris + 3 * t;
  for (int q = 0; q < 3; ++q) {
    vid[q] = f[q];
    if (f[q] < 0 || f[q] >= bs.n_verts) return false;  // not a valid triangle
  }
  double P[3][3];
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int c = 0; c < 3; ++c) P[q][c] = (double)bs.verts[3 * (int64_t)f[q] + c];
  double e1[3], e2[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    e1[c] = P[1][c] - P[0][c];
    e2[c] = P[2][c] - P[0][c];
  }
  const double N[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                       e1[0] * e2[1] - e1[1] * e2[0]};
  const double len = sqrt(N[0] * N[0] + N[1] * N[1] + N[2] * N[2]);
  if (!(len > 0.0)) return false;
  const double n[3] = {N[0] / len, N[1] / len, N[2] / len};
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int c = 0; c < 3; ++c) g[q][c] = 0.0;
  double G[3] = {0.0, 0.0, 0.0};
  for (int k = 0; k < bs.n; ++k) {
    const BackwardImage& im = bs.img[k];
    const float* acc = im.acc + 6 * t;
#pragma unroll
    for (int c = 0; c < 3; ++c) G[c] += (double)acc[3 + c];
    if (n[im.a] == 0.0) continue;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double s = (double)acc[q] / n[im.a];
#pragma unroll
      for (int c = 0; c < 3; ++c) g[q][c] += s * n[c];
    }
  }
  if (G[0] != 0.0 || G[1] != 0.0 || G[2] != 0.0) {
    const double dot = n[0] * G[0] + n[1] * G[1] + n[2] * G[2];
    double gN[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) gN[c] = (G[c] - n[c] * dot) / len;
    double ed[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      ed[0][c] = P[1][c] - P[2][c];
      ed[1][c] = P[2][c] - P[0][c];
      ed[2][c] = P[0][c] - P[1][c];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      g[q][0] += ed[q][1] * gN[2] - ed[q][2] * gN[1];
      g[q][1] += ed[q][2] * gN[0] - ed[q][0] * gN[2];
      g[q][2] += ed[q][0] * gN[1] - ed[q][1] * gN[0];
    }
  }
  return true;
}

// One thread per triangle, adding to its three vertices with global atomics,
// the bound: the nine values go through LDS so that neighbouring lanes add
// neighbouring floats (each lane its own nine: 40 us for 261,120 triangles, now
// 27; summing per vertex in an LDS table first was slower than either).
__global__ void __launch_bounds__(kBlock) backward_triangles_kernel(BackwardSet bs, int64_t n_tris,
                                                                    float* grad) {
  __shared__ float s_g[kBlock / 64][64 * 9];
  __shared__ int32_t s_to[kBlock / 64][64 * 3];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  int32_t vid[3];
  double g[3][3];
  const bool any = t < n_tris && triangle_gradient(bs, t, vid, g);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    s_to[wave][3 * lane + q] = any ? vid[q] : -1;
#pragma unroll
    for (int c = 0; c < 3; ++c) s_g[wave][9 * lane + 3 * q + c] = any ? (float)g[q][c] : 0.0f;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int e = 64 * k + lane;
    const int32_t v = s_to[wave][e / 3];
    const float x = s_g[wave][e];
    if (v >= 0 && x != 0.0f) atomicAdd(grad + 3 * (int64_t)v + e % 3, x);
  }
}

}  // namespace

hipError_t launch_backward(const BackwardArgs& args, hipStream_t s) {
  BackwardSet bs{};
  bs.n = args.n;
  bs.verts = args.verts;
  bs.n_verts = args.n_verts;
  bs.tris = args.tris;
  bs.n_tris = args.n_tris;
  bs.block_start[0] = 0;
  for (int k = 0; k < args.n; ++k) {
    const BackwardAxis& a = args.axis[k];
    BackwardImage& im = bs.img[k];
    im.a = a.a;
    im.u = (a.a + 1) % 3;
    im.v = (a.a + 2) % 3;
    im.w = args.w;
    im.lo_u = args.bbox[im.u];
    im.h_u = (args.bbox[3 + im.u] - args.bbox[im.u]) / (double)args.w;
    im.lo_v = args.bbox[im.v];
    im.h_v = (args.bbox[3 + im.v] - args.bbox[im.v]) / (double)args.w;
    // a centre's float32 rounding (2^-24 of its magnitude, at most
    // |lo| + (w + 1) h, or 2^-150 if subnormal) plus the float64 rounding of
    // the estimate, doubled
    const auto margin = [&](double lo, double h) {
      return 2.0 * ((std::ldexp(std::fabs(lo) + ((double)args.w + 1.0) * h, -24) + std::ldexp(1.0, -150)) / h +
                    std::ldexp((double)args.w + 1.0, -48)) + 1e-6;
    };
    im.margin_u = margin(im.lo_u, im.h_u);
    im.margin_v = margin(im.lo_v, im.h_v);
    im.offsets = a.offsets;
    im.tri = a.tri;
    im.gd = a.gd;
    im.gn = a.gn;
    im.acc = a.acc;
    const uint32_t nt = (uint32_t)((args.w + kBwdTile - 1) / kBwdTile);
    bs.block_start[k + 1] = bs.block_start[k] + nt * nt;
  }
  if (args.n > 0 && bs.block_start[args.n] > 0)
    hipLaunchKernelGGL(backward_samples_kernel, dim3(bs.block_start[args.n]), dim3(kBwdBlock), 0, s, bs);
  if (args.n_tris > 0)
    hipLaunchKernelGGL(backward_triangles_kernel, dim3(grid_for(args.n_tris, kBlock)), dim3(kBlock), 0, s,
                       bs, args.n_tris, args.grad);
  return hipGetLastError();
}

}  // namespace ldni
