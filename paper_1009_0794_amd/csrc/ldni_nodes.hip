// ldni_nodes.hip -- gfx950 kernels classifying the grid nodes of three LDNIs.
//
// The rays of the x-, y- and z-LDNI of one box and resolution w meet at the
// nodes of a w x w x w grid (Definition 3).  Along each of its rays a node is
// inside the solid when it lies in one of the ray's volumes (from a sample of
// odd rank to the next; Sec. 2 after Proposition 1); step 1 of the contouring
// algorithm (Sec. 5.1) classifies a node inside when at least two of its
// three LDNIs say so, which repairs disagreements caused by numerical error.
//
// Fixed readings: node t of an axis sits at the pixel centre
// f32(lo + (t + 0.5) h) and has depth f32(centre - lo) on that axis's LDNI
// (the depth a sample exactly there would get); a node is inside along a ray
// when an odd number of the ray's paired samples have depth <= its depth
// (half-open volumes [enter, exit); an unpaired last sample is ignored).
//
// Output: one bit per node in 32 x 32 x 32 bricks of 1024 words (4 KiB).
// Brick (bi, bj, bk) = (i/32, j/32, k/32) is brick number (bk*nb + bj)*nb + bi
// with nb = ceil(w/32); in a brick, word (k%32)*32 + (j%32) holds the nodes
// i = 32 bi .. 32 bi + 31 of row (j, k), node i in bit i%32.  Bits of nodes
// beyond w are zero.
//
// A sample changes the inside state of its ray at one node, the first at or
// behind it (a toggle); between samples nothing changes, so most bricks hold
// no toggle and are one value.  Two passes:
//  * bin: a workgroup owns 32 x 32 rays of one LDNI, the rays through nb
//    bricks, and sorts their toggles by brick (one 16-bit word each), with
//    each ray's inside state at the start of every brick as 32 words of bits
//    (left out where all 1024 rays agree);
//  * vote: a wave owns a brick.  The toggles of an axis are XORed into a
//    cleared 4 KB LDS matrix in the orientation of the output; a prefix XOR
//    along the axis and the start bits give the axis's inside words, and the
//    majority of the three is stored.  A brick without toggles takes its
//    words from the start bits alone.
// Nothing here is a contraction: nothing for MFMA.
#pragma clang fp contract(off)

#include "ldni_internal.hpp"

namespace ldni {
namespace {

constexpr int kNodeBlock = 256;
constexpr int kNodeWaves = kNodeBlock / 64;
constexpr int kUniformBlock = 512;
constexpr int kUniformWaves = kUniformBlock / 64;
// Grids of up to this many bricks (w <= 256) are voted on brick by brick: without
// a launch that lists those that are not one value and one that sums the totals.
// An icosphere at w = 64, 128 and 200: 50.5, 50.6 and 52.4 us with the two launches
// (and one more, which cleared the counters), 40.6, 40.6 and 42.2 now.
constexpr uint32_t kNodeAll = 512;
constexpr int kParityStride = 33;  // LDS words per brick of the start bits (no bank conflicts)

// What a brick's 1024 rays of one axis are at the brick's first node.
constexpr uint32_t kAllOutside = 0, kAllInside = 1, kMixed = 2;

// Depth of node t on an axis with origin lo and pixel size h.
__device__ __forceinline__ float node_depth(double lo, double h, int t) {
  const float c = (float)(lo + ((double)t + 0.5) * h);
  return (float)((double)c - lo);
}

// The first node whose depth is at or above s (w if none, as for NaN).  The
// estimate s / h - 0.5 is exact when it is farther than the axis's slack (the
// float32 roundings of the node depths, in pixels, and the estimate's own)
// from every integer: in float32 for nearly all samples, else in float64, else
// a binary search over the node depths decides.
__device__ __forceinline__ int first_node(const NodeArgs& g, int f, float s) {
  const float t = fmaf(s, g.inv_hf[f], -0.5f), c = ceilf(t);
  if (c - t > g.slackf[f] && c - t < 1.0f - g.slackf[f]) return (int)fminf(fmaxf(c, 0.0f), (float)g.w);
  const double td = (double)s * g.inv_h[f] - 0.5, cd = ceil(td);
  if (cd - td > g.slack[f] && cd - td < 1.0 - g.slack[f]) return (int)fmin(fmax(cd, 0.0), (double)g.w);
  int lo = 0, hi = g.w;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (node_depth(g.lo[f], g.h[f], mid) >= s) hi = mid; else lo = mid + 1;
  }
  return lo;
}

// One workgroup per 32 x 32 rays (u, v) of axis f = blockIdx.y; a wave takes
// a row of 32 rays at a time, whose samples are one contiguous range, a
// sample per lane (with a ray per lane, a 333^3 grid whose deepest ray has 160
// samples took 296 us here).  A first pass over the samples counts the toggles
// per brick and keeps the first kKept of them in LDS, a second places them
// (and reads what was not kept again).  Half bound by VALU issue (53 %; 180 instructions
// per wave of 64 samples over both passes), half by the latency of a patch's
// few serial steps, some 10 us: 0.33 ms for the 38.6 M samples of scene64 at
// w = 2048, 50 us for the flower at w = 333; the span codes it replaced took
// 0.46 ms and 103 us.  On one patch an axis (w = 32) it is longer than they were, 9
// against 4 us, and the call as long (41 us).
constexpr uint32_t kKept = 3072;

template <int kBinBlock>
__global__ void __launch_bounds__(kBinBlock) node_bin_kernel(NodeArgs g) {
  constexpr int kBinWaves = kBinBlock / 64, kSegs = kBinBlock / 32;
  extern __shared__ uint32_t s_node[];
  __shared__ uint32_t s_off[32][33];  // the rays' first samples
  __shared__ uint32_t s_falls[kBinWaves];  // rows whose offsets decrease
  __shared__ uint32_t s_at[33];       // samples of the rows before
  __shared__ uint32_t s_keep[kKept];  // brick << 15 | toggle, or ~0
  __shared__ uint32_t s_seg[kSegs][kParityStride];
  __shared__ uint32_t s_scan[kBinWaves];
  __shared__ unsigned long long s_base;
  const int f = blockIdx.y;
  const int w = g.w, nb = g.nb;
  uint32_t* s_cur = s_node;          // [nb] toggles per brick, then list positions
  uint32_t* s_par = s_node + nb;     // [nb][kParityStride] start bits: toggles of the brick before, then their prefix
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pu = (int)(blockIdx.x % (uint32_t)nb), pv = (int)(blockIdx.x / (uint32_t)nb);
  const AxisArrays& ax = g.axis[f];
  const int cols = min(32, w - 32 * pu), rows = min(32, w - 32 * pv);

  // brick number and its step along the axis
  const size_t nb2 = (size_t)nb * nb;
  const size_t brick0 = f == 0 ? (size_t)pv * nb2 + (size_t)pu * nb
                      : f == 1 ? (size_t)pu * nb2 + (size_t)pv
                               : (size_t)pv * nb + (size_t)pu;
  const size_t step = f == 0 ? 1 : f == 1 ? (size_t)nb : nb2;
  const size_t axis0 = (size_t)f * nb2 * nb;
  auto mismatch = [&] {
    __hip_atomic_store(g.host_fail, (uint32_t)kStatusMismatch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  };

  // the counters of the launches behind this one (it has none itself)
  if (blockIdx.x == 0 && f == 0)
    for (uint32_t q = tid; q < kNodeCounters; q += kBinBlock) g.n_mixed[q] = 0u;
  uint32_t falls = 0;  // rows whose offsets decrease
  for (int q = tid; q < 32 * 33; q += kBinBlock) {
    const int r = q / 33, c = q - 33 * r;
    // (rays beyond the grid are empty)
    uint32_t o0 = 0, o1 = 0;
    if (r < rows) {
      const uint32_t* o = ax.offsets + (size_t)(32 * pv + r) * w + 32 * pu;
      o0 = o[min(c, cols)];
      o1 = o[min(c + 1, cols)];
    }
    s_off[r][c] = o0;
    falls |= o0 > o1 ? 1u << r : 0u;
  }
  if (__ballot(falls != 0) != 0)
    for (int o = 32; o >= 1; o >>= 1) falls |= (uint32_t)__shfl_xor((int)falls, o, 64);
  if (lane == 0) s_falls[wave] = falls;
  uint32_t band = 0;  // first sample of the image's row
  if (wave == 1 && lane < rows) band = ax.offsets[(size_t)(32 * pv + lane) * w];
  for (int q = tid; q < nb * (1 + kParityStride); q += kBinBlock) s_node[q] = 0u;
  __syncthreads();
  // a row whose offsets decrease or pass the sample count is an error and
  // counts as empty, and so do all rows that name more samples than there are
  if (wave == 0) {
    const int r = lane & 31;
    uint32_t bad = 0;
    for (int k = 0; k < kBinWaves; ++k) bad |= s_falls[k];
    const bool ok = s_off[r][32] <= ax.n && !((bad >> r) & 1u);
    uint64_t incl = (ok && lane < 32) ? s_off[r][32] - s_off[r][0] : 0u;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
      const uint64_t y = __shfl_up((unsigned long long)incl, o, 64);
      if (lane >= o) incl += y;
    }
    const bool fits = __shfl((unsigned long long)incl, 31, 64) <= ax.n;
    if (lane < 32) {
      if (!ok || !fits) mismatch();
      s_at[r + 1] = fits ? (uint32_t)incl : 0u;
    }
    if (lane == 0) s_at[0] = 0u;
  } else if (wave == 1) {
    // The patch's part of its axis's list: the samples of the band's 32 rows
    // are one range, and the patches of the band share it in their order,
    // each as many entries as it has samples.
    uint64_t before = lane < rows ? (uint64_t)s_off[lane][0] - band : 0u;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor((unsigned long long)before, o, 64);
    if (lane == 0) s_base = band + before;
  }
  __syncthreads();
  const uint64_t base = s_base;
  const bool any = base <= ax.n && base + s_at[32] <= ax.n;  // (else offsets that decrease somewhere: an empty patch)
  if (!any && tid == 0) mismatch();
  if (s_at[32] == 0u) {  // no sample: all outside
    if (tid < nb) {
      g.range[axis0 + brick0 + (size_t)tid * step] = make_uint2(0u, 0u);
      g.kind[axis0 + brick0 + (size_t)tid * step] = kAllOutside;
    }
    return;
  }

  // calls on(place in the patch, row, column, brick, node in the brick, live)
  // for the samples of this wave's rows from r on; live: paired and in front of
  // some node.  Four loads are in flight, and a row's first four are on their
  // way while the row before it is searched.
  auto walk = [&](int r, auto&& on) {
    auto load = [&](int q, uint32_t s0, float (&d)[4]) {
      const uint32_t rest = s_at[q + 1] - s_at[q] - s0;
      const float* dep = ax.depth + s_off[q][0] + s0;
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) d[j] = 64 * j + lane < rest ? dep[64 * j + lane] : 0.0f;
    };
    float next[4] = {};
    if (r < rows) load(r, 0, next);
    for (; r < rows; r += kBinWaves) {
      const uint32_t* off = s_off[r];
      const uint32_t len = s_at[r + 1] - s_at[r], row0 = off[0];
      float d[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) d[j] = next[j];
      if (r + kBinWaves < rows) load(r + kBinWaves, 0, next);
      for (uint32_t s0 = 0; s0 < len; s0 += 256) {
        const uint32_t rest = len - s0;
        if (s0 > 0) load(r, s0, d);
#pragma unroll
        for (int j = 0; j < 4; j += 2) {  // two at a time: their chains of LDS reads overlap
          if (64u * j >= rest) break;
          uint32_t s[2];
          int c[2] = {0, 0}, t[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) s[i] = min(s0 + 64 * (j + i) + lane, len - 1);
          // the ray: the last column whose samples start at or before s
#pragma unroll
          for (int h = 16; h >= 1; h >>= 1)
#pragma unroll
            for (int i = 0; i < 2; ++i) c[i] += off[c[i] + h] <= row0 + s[i] ? h : 0;
#pragma unroll
          for (int i = 0; i < 2; ++i) t[i] = first_node(g, f, d[j + i]);
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const bool here = 64u * (j + i) + lane < rest;
            const bool live = t[i] < w && row0 + s[i] - off[c[i]] < ((off[c[i] + 1] - off[c[i]]) & ~1u);
            if (here) on(s_at[r] + s[i], r, c[i], t[i] >> 5, t[i] & 31, live);
          }
        }
        if (rest <= 256) break;
      }
    }
  };

  walk(wave, [&](uint32_t at, int r, int c, int b, int t, bool live) {
    if (at < kKept) s_keep[at] = live ? (uint32_t)(b << 15 | t | (c << 5) | (r << 10)) : ~0u;
    if (!live) return;
    atomicAdd(&s_cur[b], 1u);
    // x- and z-rays: a word per row, bits along the columns; y-rays: a word
    // per column (k), bits along the rows (i)
    if (b + 1 < nb) atomicXor(&s_par[(b + 1) * kParityStride + (f == 1 ? c : r)], 1u << (f == 1 ? r : c));
  });
  __syncthreads();

  // list positions: exclusive prefix of the bricks' counts from the range
  // this workgroup takes of the axis's list; nb <= 256
  const uint32_t n_b = tid < nb ? s_cur[tid] : 0u;
  uint32_t incl = n_b;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) s_scan[tid >> 6] = incl;
  __syncthreads();
  uint32_t first = (uint32_t)base;
  for (int k = 0; k < wave; ++k) first += s_scan[k];
  first += incl - n_b;
  if (tid < nb) s_cur[tid] = first;

  // start bits: prefix XOR over the bricks, kSegs segments of each of the 32 words
  const int col = tid & 31, seg = tid >> 5, len = (nb + kSegs - 1) / kSegs;
  const int b_lo = min(seg * len, nb), b_hi = min(b_lo + len, nb);
  uint32_t acc = 0;
  for (int b = b_lo; b < b_hi; ++b) {
    acc ^= s_par[b * kParityStride + col];
    s_par[b * kParityStride + col] = acc;
  }
  s_seg[seg][col] = acc;
  __syncthreads();
  uint32_t before = 0;
  for (int k = 0; k < seg; ++k) before ^= s_seg[k][col];
  for (int b = b_lo; b < b_hi; ++b) {
    const uint32_t word = s_par[b * kParityStride + col] ^ before;
    const uint64_t zero = __ballot(word == 0u), one = __ballot(word == ~0u);
    const int half = (lane >> 5) * 32;
    const bool all0 = (uint32_t)(zero >> half) == ~0u, all1 = (uint32_t)(one >> half) == ~0u;
    const size_t brick = axis0 + brick0 + (size_t)b * step;
    if (!all0 && !all1) g.parity[brick * 32 + col] = word;
    if (col == 0) g.kind[brick] = all0 ? kAllOutside : all1 ? kAllInside : kMixed;
  }
  if (tid < nb) g.range[axis0 + brick0 + (size_t)tid * step] = make_uint2(any ? first : 0u, any ? n_b : 0u);
  if (!any) return;
  __syncthreads();

  uint16_t* list = g.toggles[f];
  const uint32_t kept = min(s_at[32], kKept);
  for (uint32_t q = tid; q < kept; q += kBinBlock) {
    const uint32_t x = s_keep[q];
    if (x != ~0u) list[atomicAdd(&s_cur[x >> 15], 1u)] = (uint16_t)(x & 0x7fffu);
  }
  if (kept == s_at[32]) return;
  int r0 = wave;  // the first row with samples that were not kept
  while (r0 < rows && s_at[r0 + 1] <= kKept) r0 += kBinWaves;
  walk(r0, [&](uint32_t at, int r, int c, int b, int t, bool live) {
    if (live && at >= kKept) list[atomicAdd(&s_cur[b], 1u)] = (uint16_t)(t | (c << 5) | (r << 10));
  });
}

// One axis's part of a brick for the vote.
struct BrickAxis {
  uint32_t first, n, kind;
};
__device__ __forceinline__ BrickAxis brick_axis(const NodeArgs& g, size_t at) {
  const uint2 r = g.range[at];
  return BrickAxis{r.x, r.y, g.kind[at]};
}
// (the same in every lane)
__device__ __forceinline__ BrickAxis uniform(const BrickAxis& a) {
  return BrickAxis{(uint32_t)__builtin_amdgcn_readfirstlane((int)a.first), (uint32_t)__builtin_amdgcn_readfirstlane((int)a.n),
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)a.kind)};
}

// Stores four words of a brick as one 16-byte vector at any 4-byte address
// (the caller's buffer; gfx950 takes such a store whole.  A branch on the
// alignment was merged into four scattered words: 303 against 156 us below).
typedef uint32_t Words4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void store4(uint32_t* out, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  *reinterpret_cast<Words4*>(out) = Words4{a, b, c, d};
}

// Adds a wave's nodes (by lane 0) to one of the kNodeSlots pairs of totals.
__device__ __forceinline__ void add_totals(const NodeArgs& g, uint32_t wave_no, uint32_t inside, uint32_t split) {
  unsigned long long* slot = (unsigned long long*)g.partial + 2 * (wave_no % kNodeSlots);
  if (__lane_id() == 0 && inside != 0) atomicAdd(slot, (unsigned long long)inside);
  if (__lane_id() == 0 && split != 0) atomicAdd(slot + 1, (unsigned long long)split);
}

// Bricks that are one value: a wave looks at 64 consecutive bricks at once, a
// brick per lane, so that one round of loads is waited for before 64 bricks
// of stores; what remains is the writing: 0.96 GiB at w = 2048 in 156 us, the
// rate of a plain fill.  The others are listed for classify_nodes_kernel.
__global__ void __launch_bounds__(kUniformBlock) uniform_nodes_kernel(NodeArgs g, uint32_t per) {
  __shared__ uint32_t s_n[kUniformWaves], s_at;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t nb = (uint32_t)g.nb, n_bricks = nb * nb * nb;
  const uint32_t wave_no = blockIdx.x * kUniformWaves + wave;
  const uint32_t first = min(wave_no * per, n_bricks), end = min(first + per, n_bricks), brick = first + lane;
  bool in = false, split = false, plain = false;
  if (brick < end) {
    const BrickAxis x = brick_axis(g, brick), y = brick_axis(g, (size_t)n_bricks + brick),
                    z = brick_axis(g, 2 * (size_t)n_bricks + brick);
    const uint32_t bi = brick % nb, bj = brick / nb % nb, bk = brick / (nb * nb);
    in = x.kind + y.kind + z.kind >= 2;
    split = x.kind != y.kind || x.kind != z.kind;
    // (bricks that reach beyond the grid are masked: listed unless outside)
    plain = (x.n | y.n | z.n) == 0 && x.kind != kMixed && y.kind != kMixed && z.kind != kMixed &&
            ((!in && !split) || (32 * bi + 32 <= (uint32_t)g.w && 32 * bj + 32 <= (uint32_t)g.w && 32 * bk + 32 <= (uint32_t)g.w));
  }
  const uint64_t m_plain = __ballot(plain), m_in = __ballot(plain && in);
  const uint64_t m_list = __ballot(brick < end && !plain);
  // one atomic per workgroup: they queue at the counter
  if (lane == 0) s_n[wave] = (uint32_t)__popcll(m_list);
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t n = 0;
    for (int k = 0; k < kUniformWaves; ++k) {
      const uint32_t c = s_n[k];
      s_n[k] = n;
      n += c;
    }
    s_at = n != 0 ? atomicAdd(g.n_mixed, n) : 0u;
  }
  __syncthreads();
  if ((m_list >> lane) & 1u)
    g.mixed[s_at + s_n[wave] + (uint32_t)__popcll(m_list & ((1ull << lane) - 1ull))] = brick;
  add_totals(g, wave_no, 32768u * (uint32_t)__popcll(m_in), 32768u * (uint32_t)__popcll(__ballot(plain && split)));
  // (waves start at different bricks of theirs: in step they would all write
  // addresses a power of two apart, the same memory channels)
  const uint32_t turn = (wave_no * 5u) & 63u;
  for (uint64_t todo = turn ? m_plain >> turn | m_plain << (64 - turn) : m_plain; todo != 0; todo &= todo - 1) {
    const uint32_t b = ((uint32_t)__ffsll((unsigned long long)todo) - 1u + turn) & 63u;
    const uint32_t v = (m_in >> b) & 1u ? ~0u : 0u;
    uint32_t* out = g.bits + (size_t)(first + b) * 1024 + 4 * lane;
#pragma unroll
    for (int m = 0; m < 4; ++m) store4(out + 256 * m, v, v, v, v);
  }
}

// The listed bricks (kAll: every brick, and the last workgroup reports the
// totals), a wave each in turn; lane l holds the 16 words 4 l + 256 m + c (m, c = 0..3): rows k = 8 m + l / 8, j = 4 (l % 8) + c.
// One LDS matrix per wave serves the three axes in turn, four waves per SIMD
// (123 registers; held to 80 they spill: 0.70 ms for all bricks against 0.47).
// Bound by the latency of the list reads: 27,000 of scene64's 262,144 bricks
// at w = 2048 in 0.10 ms.  The vote it replaced transposed a 32 x 32 bit matrix
// per thread of every brick: 0.93 ms, and 1.05 ms for the flower at w = 333 (now 30
// us), whose spans with more than two samples it walked.
template <bool kAll>
__global__ void __launch_bounds__(kNodeBlock, 4) classify_nodes_kernel(NodeArgs g) {
  __shared__ uint4 s_mat[kNodeWaves][256];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = g.w, nb = g.nb;
  const uint32_t n_bricks = (uint32_t)nb * nb * nb;
  const int jq = lane & 7, kk = lane >> 3;
  uint4* mat = s_mat[wave];
  uint32_t* mat1 = reinterpret_cast<uint32_t*>(mat);
  auto sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  // The first toggles of an axis, loaded ahead of their use.
  struct Ahead {
    uint32_t x[2];
  };
  auto ahead = [&](const BrickAxis& a, const uint16_t* list) {
    Ahead r;
#pragma unroll
    for (int q = 0; q < 2; ++q) r.x[q] = 64u * q + lane < a.n ? list[(size_t)a.first + 64 * q + lane] : 0u;
    return r;
  };
  // XORs an axis's toggles into the matrix: bit(t, col, row) gives the word
  // and its bits
  auto scatter = [&](const BrickAxis& a, const Ahead& r, const uint16_t* list, auto&& bit) {
    auto put = [&](uint32_t e, uint32_t x) {
      uint32_t word, bits;
      bit(x & 31u, (x >> 5) & 31u, x >> 10, word, bits);
      if (e < a.n) atomicXor(&mat1[word], bits);
    };
#pragma unroll
    for (int q = 0; q < 2; ++q) put(64 * q + lane, r.x[q]);
    for (uint32_t e0 = 128; e0 < a.n; e0 += 256) {  // four loads in flight
      uint32_t x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = e0 + 64 * q + lane < a.n ? list[(size_t)a.first + e0 + 64 * q + lane] : 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) put(e0 + 64 * q + lane, x[q]);
    }
    sync();
  };
  // takes the lane's words out of the matrix and clears them
  auto take = [&](uint32_t (&v)[4][4]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const uint4 x = mat[64 * m + lane];
      v[m][0] = x.x; v[m][1] = x.y; v[m][2] = x.z; v[m][3] = x.w;
      mat[64 * m + lane] = make_uint4(0u, 0u, 0u, 0u);
    }
    sync();
  };
  // the start word of this lane (lane % 32) of an axis
  auto start = [&](const BrickAxis& a, size_t at) -> uint32_t {
    return a.kind == kMixed ? g.parity[at * 32 + (lane & 31)] : a.kind == kAllInside ? ~0u : 0u;
  };

  const uint32_t wave_no = blockIdx.x * kNodeWaves + wave, stride = gridDim.x * kNodeWaves;
  const uint32_t n_listed = kAll ? n_bricks : *g.n_mixed;
  uint32_t n_inside = 0, n_split = 0;
#pragma unroll
  for (int m = 0; m < 4; ++m) mat[64 * m + lane] = make_uint4(0u, 0u, 0u, 0u);
  sync();
  for (uint32_t at = wave_no; at < n_listed; at += stride) {
    const uint32_t brick = kAll ? at : (uint32_t)__builtin_amdgcn_readfirstlane((int)g.mixed[at]);
    const BrickAxis vx = brick_axis(g, brick), vy = brick_axis(g, (size_t)n_bricks + brick),
                    vz = brick_axis(g, 2 * (size_t)n_bricks + brick);
    const BrickAxis x = uniform(vx), y = uniform(vy), z = uniform(vz);
    const int bi = (int)(brick % (uint32_t)nb), bj = (int)(brick / (uint32_t)nb % (uint32_t)nb),
              bk = (int)(brick / ((uint32_t)nb * nb));
    // bits along i of nodes of the grid
    const int wi = w - 32 * bi;
    const uint32_t ibits = wi >= 32 ? ~0u : (1u << wi) - 1u;
    uint32_t* out = g.bits + (size_t)brick * 1024 + 4 * lane;
    const Ahead list_x = ahead(x, g.toggles[0]), list_y = ahead(y, g.toggles[1]), list_z = ahead(z, g.toggles[2]);
    uint32_t xw[4][4], yw[4][4];
    const uint32_t px = start(x, brick), py = start(y, (size_t)n_bricks + brick),
                   pz = start(z, 2 * (size_t)n_bricks + brick);
    // x: a ray is a word; its toggles flip the nodes from theirs on
    if (x.n > 0) {
      scatter(x, list_x, g.toggles[0], [](uint32_t t, uint32_t col, uint32_t row, uint32_t& word, uint32_t& bits) {
        word = row * 32 + col;
        bits = ~0u << t;
      });
      take(xw);
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int c = 0; c < 4; ++c) xw[m][c] = 0u;
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const uint32_t row = (uint32_t)__shfl((int)px, 8 * m + kk, 64) >> (4 * jq);
#pragma unroll
      for (int c = 0; c < 4; ++c) xw[m][c] ^= 0u - ((row >> c) & 1u);
    }
    // y: prefix along j, in the lane's four words and over the 8 lanes of a row
    if (y.n > 0) {
      scatter(y, list_y, g.toggles[1], [](uint32_t t, uint32_t col, uint32_t row, uint32_t& word, uint32_t& bits) {
        word = col * 32 + t;
        bits = 1u << row;
      });
      take(yw);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        yw[m][1] ^= yw[m][0];
        yw[m][2] ^= yw[m][1];
        yw[m][3] ^= yw[m][2];
        uint32_t s = yw[m][3];
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
          const uint32_t q = (uint32_t)__shfl_up((int)s, o, 64);
          if (jq >= o) s ^= q;
        }
        s ^= yw[m][3];  // the lanes before
#pragma unroll
        for (int c = 0; c < 4; ++c) yw[m][c] ^= s;
      }
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int c = 0; c < 4; ++c) yw[m][c] = 0u;
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const uint32_t p = (uint32_t)__shfl((int)py, 8 * m + kk, 64);
#pragma unroll
      for (int c = 0; c < 4; ++c) yw[m][c] ^= p;
    }
    // z: prefix along k, over the 8 lanes of a column and then the groups m,
    // straight into the majority of the three words; rays beyond the grid are
    // outside, so only the disagreements need the mask of the grid's nodes
    if (z.n > 0)
      scatter(z, list_z, g.toggles[2], [](uint32_t t, uint32_t col, uint32_t row, uint32_t& word, uint32_t& bits) {
        word = t * 32 + row;
        bits = 1u << col;
      });
    uint32_t p[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) p[c] = (uint32_t)__shfl((int)pz, 4 * jq + c, 64);
    uint32_t ni = 0, ns = 0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      uint32_t zw[4] = {p[0], p[1], p[2], p[3]};
      if (z.n > 0) {
        const uint4 v = mat[64 * m + lane];
        mat[64 * m + lane] = make_uint4(0u, 0u, 0u, 0u);
        const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          uint32_t s = u[c];
#pragma unroll
          for (int o = 8; o < 64; o <<= 1) {
            const uint32_t q = (uint32_t)__shfl_up((int)s, o, 64);
            if (lane >= o) s ^= q;
          }
          zw[c] = s ^ p[c];
          p[c] ^= (uint32_t)__shfl((int)s, 56 + jq, 64);
        }
      }
      uint32_t in[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t a = xw[m][c], b = yw[m][c], d = zw[c];
        const uint32_t live = (32 * bj + 4 * jq + c < w && 32 * bk + 8 * m + kk < w) ? ibits : 0u;
        in[c] = ((a & b) | (d & (a | b))) & live;
        ni += __popc(in[c]);
        ns += __popc(((a ^ b) | (a ^ d)) & live);
      }
      store4(out + 256 * m, in[0], in[1], in[2], in[3]);
    }
    n_inside += ni;
    n_split += ns;
  }
  if (kAll) {
    // one brick a wave at most: both counts of a wave fit 16 bits, and of a
    // grid 28; with the workgroups that are done in the upper 8 one atomic per
    // workgroup adds them up and finds the last, which reports
    static_assert(kNodeAll * 32768ull <= 1ull << 27 && kNodeAll / kNodeWaves < 256, "the fields of the sum");
    __shared__ uint32_t s_n[kNodeWaves];
    uint32_t n = n_inside | n_split << 16;
    for (int o = 32; o > 0; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o);
    if (lane == 0) s_n[wave] = n;
    __syncthreads();
    if (threadIdx.x != 0) return;
    unsigned long long sum = 1ull << 56;
    for (int q = 0; q < kNodeWaves; ++q) sum += (unsigned long long)(s_n[q] & 0xffffu) | (unsigned long long)(s_n[q] >> 16) << 28;
    sum += atomicAdd((unsigned long long*)g.partial, sum);
    if (sum >> 56 != gridDim.x) return;
    constexpr uint32_t field = (1u << 28) - 1u;
    g.host[0] = (uint32_t)sum & field;
    g.host[1] = 0u;
    g.host[2] = (uint32_t)(sum >> 28) & field;
    g.host[3] = 0u;
    return;
  }
  // (a lane sees fewer than 2^32 nodes: 512 of each brick)
  uint64_t a = n_inside, b = n_split;
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor((unsigned long long)a, o);
    b += __shfl_xor((unsigned long long)b, o);
  }
  unsigned long long* slot = (unsigned long long*)g.partial + 2 * (wave_no % kNodeSlots);
  if (lane == 0 && a != 0) atomicAdd(slot, (unsigned long long)a);
  if (lane == 0 && b != 0) atomicAdd(slot + 1, (unsigned long long)b);
}

// Sums the counts of the kNodeSlots slots and writes both (low, high word
// each) to pinned host memory (one block).
__global__ void __launch_bounds__(kNodeBlock) node_stats_kernel(const uint64_t* partial, uint32_t* host) {
  static_assert(kNodeSlots == kNodeBlock, "a slot per thread");
  __shared__ uint64_t s_sum[2][kNodeWaves];
  uint64_t a = partial[2 * threadIdx.x], b = partial[2 * threadIdx.x + 1];
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor((unsigned long long)a, o);
    b += __shfl_xor((unsigned long long)b, o);
  }
  if ((threadIdx.x & 63) == 0) {
    s_sum[0][threadIdx.x >> 6] = a;
    s_sum[1][threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  a = b = 0;
  for (int q = 0; q < kNodeWaves; ++q) {
    a += s_sum[0][q];
    b += s_sum[1][q];
  }
  host[0] = (uint32_t)a;
  host[1] = (uint32_t)(a >> 32);
  host[2] = (uint32_t)b;
  host[3] = (uint32_t)(b >> 32);
}

}  // namespace

hipError_t launch_node_bins(const NodeArgs& g, hipStream_t s) {
  const uint32_t lds = sizeof(uint32_t) * (uint32_t)g.nb * (1 + kParityStride);  // 34 KB at w = 8192
  const uint32_t patches = (uint32_t)g.nb * g.nb;
  // 1,024 threads a patch, two rows a wave, where all patches are resident at
  // once (two per CU): what counts then is a patch's own time.  Calls on an
  // icosphere at w = 64 and the flower at 333: 40.6 and 106 us, with 512 threads
  // 43.4 and 108; one at w = 2048 485 and 437 us.
  if (3 * patches <= 512) hipLaunchKernelGGL(node_bin_kernel<1024>, dim3(patches, 3), dim3(1024), lds, s, g);
  else hipLaunchKernelGGL(node_bin_kernel<512>, dim3(patches, 3), dim3(512), lds, s, g);
  return hipGetLastError();
}

hipError_t launch_classify_nodes(const NodeArgs& g, hipStream_t s) {
  const uint32_t bricks = (uint32_t)g.nb * g.nb * g.nb;
  const uint32_t blocks = (bricks + kNodeWaves - 1) / kNodeWaves;
  if (bricks <= kNodeAll) {
    hipLaunchKernelGGL(classify_nodes_kernel<true>, dim3(blocks), dim3(kNodeBlock), 0, s, g);
    return hipGetLastError();
  }
  // bricks per wave: up to 64, fewer where that leaves under 4096 waves (16 per CU)
  const uint32_t per = bricks / 4096 < 1 ? 1 : bricks / 4096 > 64 ? 64 : bricks / 4096;
  const uint32_t group = per * kUniformWaves;
  hipLaunchKernelGGL(uniform_nodes_kernel, dim3((bricks + group - 1) / group), dim3(kUniformBlock), 0, s, g, per);
  // as many workgroups as stay resident (four per CU), at most one wave a brick
  hipLaunchKernelGGL(classify_nodes_kernel<false>, dim3(blocks < 1024 ? blocks : 1024), dim3(kNodeBlock), 0, s, g);
  hipLaunchKernelGGL(node_stats_kernel, dim3(1), dim3(kNodeBlock), 0, s, g.partial, g.host);
  return hipGetLastError();
}

}  // namespace ldni
