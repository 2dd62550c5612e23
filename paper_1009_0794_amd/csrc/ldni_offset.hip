// ldni_offset.hip -- gfx950 kernels offsetting a solid given by its LDNIs.
//
// Sec. 4.2 approximates the offset of a solid H by a distance r by the
// Minkowski sum of H with a sphere of radius r: a sphere is centred at every
// depth-normal sample of H's LDNIs, sampled into LDNIs on the same grid, and
// united with H (an inner offset, r < 0, subtracts spheres of radius |r|),
// with the Boolean operations of Sec. 4.1 and the small interval removal of
// Sec. 4.1.1.
//
// Fixed readings: the spheres of all samples of the three LDNIs are applied
// at once; a sphere hits a ray when rho^2 < r^2 (float64), at centre -/+
// sqrt(r^2 - rho^2); per ray the events are H's paired samples and the
// spheres' chord ends; events of equal float32 depth form one group, after
// which H's state is the parity of its samples so far and the spheres' state
// is "some sphere entered and not left"; a group that changes the result
// (H or S, resp. H and not S) contributes its first event (H's samples by
// index, then spheres by generating sample, enter before exit); volumes with
// (double)exit - (double)enter <= 0 or < eps are removed.  Generating samples
// are numbered over the x-, y-, z-LDNI in storage order; a sphere's sample
// gets id -1 - g.
//
// Passes: the sphere centres; binning of the spheres into the lists of the
// rays they hit (count, scan, scatter); one wave per ray; and the result's
// samples.  The count pass (offset_union_kernel) merges the chords of a
// ray into the few intervals they cover together before it sorts anything, and
// keeps the result's end points for the write pass (offset_write_kernel, a
// sample per lane).  Rays that this leaves with
// too many events, and rays with more end points than are kept, go through the
// sweep over all events (sweep_ray): they go to a wave-private LDS buffer as
// 64-bit keys (orderable depth, order), window by window in depth when they do
// not fit, a bitonic sort orders them, and a sweep in chunks of 64 (wave prefix
// sums of H's parity and of the open spheres, group starts by a max-scan) finds
// the result's end points.
// Nothing is a contraction: the work is the exact chord tests and the sorts.
#pragma clang fp contract(off)

#include "ldni_internal.hpp"
#include "ldni_bin.hpp"

namespace ldni {
namespace {

constexpr int kOffBlock = 256;  // four waves, one ray each at a time
constexpr int kOffWaves = kOffBlock / 64;
constexpr uint32_t kSphereOrder = 0x80000000u;

__device__ __forceinline__ uint32_t orderable(float d) {
  uint32_t u = __float_as_uint(d);
  if (u == 0x80000000u) u = 0u;  // -0 groups with +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ double centre_of(const OffsetArgs& g, int b, int i) {
  return (double)(float)(g.lo[b] + ((double)i + 0.5) * g.h[b]);
}

// Centres of the spheres (world order), at the sample's number: a wave takes
// the samples of 64 pixels in a row, a sample per lane (a lane per pixel:
// 31 us for 405,002 samples at w = 256, now 21).
__global__ __launch_bounds__(kOffBlock) void offset_centres_kernel(OffsetArgs g) {
  __shared__ uint32_t s_off[kOffWaves][65];
  const int64_t npix = (int64_t)g.w * g.w;
  const int lane = threadIdx.x & 63;
  uint32_t* const off = s_off[threadIdx.x >> 6];
  const int64_t groups = (npix + 63) / 64;
  const int64_t group = (int64_t)blockIdx.x * kOffWaves + (threadIdx.x >> 6);
  if (group >= 3 * groups) return;
  const int a = (int)(group / groups);
  const int64_t p0 = (group - a * groups) * 64;
  const int n = (int)min((int64_t)64, npix - p0);
  const int u = (a + 1) % 3, v = (a + 2) % 3;
  const AxisArrays& ax = g.in[a];
  uint32_t o0 = 0, o1 = 0;
  if (lane < n) {
    o0 = ax.offsets[p0 + lane];
    o1 = ax.offsets[p0 + lane + 1];
    off[lane] = o0;
    if (lane == n - 1) off[n] = o1;
  }
  if (__ballot(lane < n && (o1 < o0 || (uint64_t)o1 > ax.n)) != 0) {
    if (lane == 0) atomicOr(g.status, kStatusMismatch);
    return;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const uint32_t first = off[0], last = off[n];
  for (uint32_t q = first + (uint32_t)lane; q < last; q += 64) {
    int k = 0;  // the last pixel with off[k] <= q
    for (int hi = n - 1; k < hi;) {
      const int mid = (k + hi + 1) >> 1;
      if (off[mid] <= q) k = mid; else hi = mid - 1;
    }
    const int64_t p = p0 + k;
    double* c = g.centres + 3 * (g.base[a] + q);
    c[a] = g.lo[a] + (double)ax.depth[q];
    c[u] = centre_of(g, u, (int)(p % g.w));
    c[v] = centre_of(g, v, (int)(p / g.w));
  }
}

// Pixel range [i0, i1] of an image axis whose centres may lie within r of x:
// a centre c_i with |c_i - x| < r has i within [t0 - m, t1 + m] for
// t = (x -+ r - lo) / h - 0.5 and m the axis's rounding margin in pixels;
// i0 > i1 if none.
__device__ __forceinline__ void pixel_range(const OffsetArgs& g, int b, double x, int& i0, int& i1) {
  const double t0 = (x - g.r - g.lo[b]) / g.h[b] - 0.5, t1 = (x + g.r - g.lo[b]) / g.h[b] - 0.5;
  const double f0 = ceil(t0 - g.margin[b]), f1 = floor(t1 + g.margin[b]);
  i0 = f0 < 0.0 ? 0 : f0 > (double)(g.w - 1) ? g.w : (int)f0;
  i1 = f1 < 0.0 ? -1 : f1 > (double)(g.w - 1) ? g.w - 1 : (int)f1;
}

// Binning: for sphere s and image a, the rays of the pixels in its range
// that the sphere hits (rho^2 < r^2, the test of the ray pass); count
// (kScatter false) or write the sphere into those rays' lists.  A workgroup
// (256 consecutive spheres of one image, which mostly hit the same rays)
// first adds its (sphere, ray) pairs per ray into an LDS table, and then
// touches each ray's global counter once: the count pass adds its pairs to
// ray_count; the scatter pass reserves a range of the ray's list from
// ray_cursor and, in a second sweep over the same pairs, fills it.  A ray that
// finds no free entry (kBinProbe probes) is counted and placed with global
// atomics; entries never free, so it misses the table in the second sweep as
// well.
// Bound by the exact tests and by the global atomics, which go out to memory
// a cache line each: an entry holds eight rays in a row, so that lanes in a row
// add to one line (405,002 spheres at w = 256: 0.72 M lines instead of 2.6 M).
// Count and scatter there: 169 and 264 us when every lane tested its next
// pixel and added in the same step, 130 and 180 us with the hits as masks, 51
// and 108 us with entries of eight rays (of sixteen: 61 and 171 us).
constexpr int kRayGroup = 8;  // rays in a row that share a table entry
constexpr int kRayGroupBits = 9;
constexpr int kRayGroups = 1 << kRayGroupBits;
struct RayTable {
  uint32_t key[kRayGroups];            // first ray / kRayGroup, or kBinEmpty
  uint32_t n[kRayGroups * kRayGroup];  // pairs counted; or the list position of the ray's next one
};

// The counter of a ray, its group claimed if new; -1 if no entry is free within kBinProbe probes.
__device__ __forceinline__ int ray_slot(RayTable& h, uint32_t ray) {
  const uint32_t k = ray / kRayGroup;
  uint32_t s = (k * 2654435761u) >> (32 - kRayGroupBits);
  for (int i = 0; i < kBinProbe; ++i) {
    uint32_t was = h.key[s];
    if (was == kBinEmpty) was = atomicCAS(&h.key[s], kBinEmpty, k);
    if (was == kBinEmpty || was == k) return (int)(s * kRayGroup + ray % kRayGroup);
    s = (s + 1) & (kRayGroups - 1);
  }
  return -1;
}

// kSmall: no sphere's range has more than eight pixels a side, so that its hits
// are a mask of 64 bits: the exact tests are made once, without a wave's other
// lanes, and then every step takes a hit of each lane.
template <bool kScatter, bool kSmall>
__global__ __launch_bounds__(kOffBlock) void offset_bin_kernel(OffsetArgs g) {
  __shared__ RayTable h;
  constexpr int kPer = kRayGroups * kRayGroup / kOffBlock;
  for (int i = threadIdx.x; i < kRayGroups; i += kOffBlock) h.key[i] = kBinEmpty;
#pragma unroll
  for (int i = 0; i < kPer; ++i) h.n[i * kOffBlock + threadIdx.x] = 0u;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * kOffBlock + threadIdx.x;
  int a = 0, u = 0, v = 0, ni = 0, nj = 0, n_my = 0, iu0 = 0, iv0 = 0;
  uint32_t s = 0;
  double pu = 0.0, pv = 0.0;
  if (t < 3 * (int64_t)g.n_spheres) {
    a = (int)(t / g.n_spheres);
    s = (uint32_t)(t - (int64_t)a * g.n_spheres);
    u = (a + 1) % 3;
    v = (a + 2) % 3;
    const double* c = g.centres + 3 * (size_t)s;
    pu = c[u];
    pv = c[v];
    int iu1, iv1;
    pixel_range(g, u, pu, iu0, iu1);
    pixel_range(g, v, pv, iv0, iv1);
    if (iu0 <= iu1 && iv0 <= iv1) {
      ni = iu1 - iu0 + 1;
      nj = iv1 - iv0 + 1;
      n_my = ni * nj;
    }
  }
  const double r2 = g.r * g.r;
  const int64_t npix = (int64_t)g.w * g.w;
  uint64_t hits = 0;  // kSmall: bit 8 j + i for pixel (iu0 + i, iv0 + j)
  if (kSmall) {
    double du2[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const double du = centre_of(g, u, iu0 + i) - pu;
      du2[i] = du * du;
    }
    for (int j = 0; __ballot(j < nj) != 0; ++j) {
      const double dv = centre_of(g, v, iv0 + j) - pv, dv2 = dv * dv;
      uint32_t m = 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) m |= du2[i] + dv2 < r2 ? 1u << i : 0u;
      if (j < nj) hits |= (uint64_t)(m & ((1u << ni) - 1u)) << (8 * j);
    }
  }
  // kSmall: every lane's next hit while any lane has one; else every lane's
  // j-th pixel, j = 0, 1, ...  The ray it hits (or -1) and the runs of equal
  // rays
  auto sweep = [&](auto&& on_ray) {
    if (kSmall) {
      for (uint64_t m = hits; __ballot(m != 0) != 0; m &= m - 1) {
        const int j = __ffsll((unsigned long long)m) - 1;
        const int my = m != 0 ? (int)(a * npix + (int64_t)(iv0 + (j >> 3)) * g.w + iu0 + (j & 7)) : -1;
        on_ray(my);
      }
      return;
    }
    for (int j = 0; __ballot(j < n_my) != 0; ++j) {
      int my = -1;
      if (j < n_my) {
        const int iu = iu0 + j % ni, iv = iv0 + j / ni;
        const double du = centre_of(g, u, iu) - pu, dv = centre_of(g, v, iv) - pv;
        if (du * du + dv * dv < r2) my = (int)(a * npix + (int64_t)iv * g.w + iu);
      }
      on_ray(my);
    }
  };
  sweep([&](int my) {
    if (my < 0) return;
    const int sl = ray_slot(h, (uint32_t)my);
    if (sl >= 0) atomicAdd(&h.n[sl], 1u);
    else if (!kScatter) atomicAdd(&g.ray_count[my], 1u);
  });
  __syncthreads();
  uint32_t ray[kPer], n[kPer], at[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int q = i * kOffBlock + (int)threadIdx.x;
    n[i] = h.n[q];
    ray[i] = h.key[q / kRayGroup] * kRayGroup + (uint32_t)(q % kRayGroup);
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (n[i] == 0) continue;
    if (!kScatter) atomicAdd(&g.ray_count[ray[i]], n[i]);
    else at[i] = g.ray_start[ray[i]] + atomicAdd(&g.ray_cursor[ray[i]], n[i]);
  }
  if (!kScatter) return;
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    if (n[i] != 0) h.n[i * kOffBlock + threadIdx.x] = at[i];
  __syncthreads();
  sweep([&](int my) {
    if (my < 0) return;
    const int sl = ray_slot(h, (uint32_t)my);
    g.list[sl >= 0 ? atomicAdd(&h.n[sl], 1u) : g.ray_start[my] + atomicAdd(&g.ray_cursor[my], 1u)] = s;
  });
}

// One event's world-order normal and depth for a sphere g on the ray of axis
// a through (cu, cv) (exactly the arithmetic of the hit test).
struct SphereHit {
  float depth;
  float n[3];
};
// the depth alone (the count pass's small-volume test needs no normal)
__device__ __forceinline__ float sphere_depth(const OffsetArgs& g, int a, double cu, double cv, uint32_t s,
                                              bool is_exit) {
  const int u = (a + 1) % 3, v = (a + 2) % 3;
  const double* c = g.centres + 3 * (size_t)s;
  const double du = cu - c[u], dv = cv - c[v];
  const double rho2 = du * du + dv * dv;
  const double t = sqrt(g.r * g.r - rho2);
  const double z = is_exit ? c[a] + t : c[a] - t;
  return (float)(z - g.lo[a]);
}
__device__ __forceinline__ SphereHit sphere_sample(const OffsetArgs& g, int a, double cu, double cv, uint32_t s,
                                                   bool is_exit) {
  const int u = (a + 1) % 3, v = (a + 2) % 3;
  const double* c = g.centres + 3 * (size_t)s;
  const double du = cu - c[u], dv = cv - c[v];
  const double rho2 = du * du + dv * dv;
  const double t = sqrt(g.r * g.r - rho2);
  const double z = is_exit ? c[a] + t : c[a] - t;
  const double sign = g.union_op ? 1.0 : -1.0;
  const float nu = (float)(sign * (du / g.r)), nv = (float)(sign * (dv / g.r)),
              na = (float)(sign * ((z - c[a]) / g.r));
  // to world order by selects (an array indexed by the axis would live in
  // scratch memory): x, y, z are (a, u, v) for a = 0, (v, a, u) for a = 1
  // and (u, v, a) for a = 2
  SphereHit h;
  h.depth = (float)(z - g.lo[a]);
  h.n[0] = a == 0 ? na : (a == 1 ? nv : nu);
  h.n[1] = a == 0 ? nu : (a == 1 ? na : nv);
  h.n[2] = a == 0 ? nv : (a == 1 ? nu : na);
  return h;
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// Inclusive wave prefix sum.
__device__ __forceinline__ int wave_scan_add(int x) {
  const int lane = (int)lane_id();
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  return x;
}

__device__ __forceinline__ int wave_scan_max(int x) {
  const int lane = (int)lane_id();
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x = max(x, y);
  }
  return x;
}

// Sort of key[0..n) ascending by one wave: a bitonic network over the next
// power of two in which every comparator puts the smaller key first (each
// merge of blocks of k starts with a mirrored stage, pairing blk + r with
// blk + k - 1 - r, followed by half-cleaners).  Keys beyond n count as
// larger than all, so no comparator ever moves them: comparators that reach
// beyond n are skipped, blocks wholly beyond n are not visited, and nothing
// beyond n is read or written.  A lane takes up to four comparators of a
// stage at a time, loading all of them before storing any (the comparators
// of a stage are disjoint), so their LDS round trips overlap.
__device__ __forceinline__ void wave_sort(uint64_t* key, uint32_t n) {
  const uint32_t lane = lane_id();
  constexpr int kPairs = 4;
  auto stage = [&](uint32_t pairs, auto&& pair_of) {
    for (uint32_t h0 = lane; h0 < pairs; h0 += 64 * kPairs) {
      uint64_t x[kPairs], y[kPairs];
      uint32_t lo[kPairs], hi[kPairs];
      bool act[kPairs];
#pragma unroll
      for (int j = 0; j < kPairs; ++j) {
        const uint32_t h = h0 + 64u * j;
        pair_of(h, lo[j], hi[j]);
        act[j] = h < pairs && hi[j] < n;
        if (act[j]) {
          x[j] = key[lo[j]];
          y[j] = key[hi[j]];
        }
      }
#pragma unroll
      for (int j = 0; j < kPairs; ++j) {
        if (act[j] && x[j] > y[j]) {
          key[lo[j]] = y[j];
          key[hi[j]] = x[j];
        }
      }
    }
    wave_sync();
  };
  for (uint32_t lk = 1; (1u << (lk - 1)) < n; ++lk) {  // blocks of k = 2^lk
    const uint32_t k = 1u << lk, hk = k >> 1;
    stage(((n + k - 1) >> lk) << (lk - 1), [&](uint32_t h, uint32_t& lo, uint32_t& hi) {
      const uint32_t blk = (h >> (lk - 1)) << lk, r = h & (hk - 1);
      lo = blk + r;
      hi = blk + k - 1 - r;
    });
    for (uint32_t lj = lk - 1; lj-- > 0;) {  // half-cleaners, j = 2^lj = k/4 .. 1
      const uint32_t jj = 1u << lj;
      stage(((n + 2 * jj - 1) >> (lj + 1)) << lj, [&](uint32_t h, uint32_t& lo, uint32_t& hi) {
        lo = ((h >> lj) << (lj + 1)) + (h & (jj - 1));
        hi = lo + jj;
      });
    }
  }
}

// The orderable depth of the event of the given rank (0-based) among
// key[0..n) by one wave: a radix select over the 32 depth bits, five bits a
// pass, with a 32-bin histogram in hist (32 words of the wave's own).
// A cut window keeps fewer than kOffsetKeep events and then takes one more
// step of the sphere loop (two events per lane).
static_assert(kOffsetKeep + 128 <= kOffsetBuf, "a cut window takes one more step of 128 events");
// a sweep step appends up to 64 end points after a flush that leaves one
static_assert(kOffsetEmit >= 65, "the emit buffer takes one step after a flush");
__device__ __forceinline__ uint32_t select_depth(const uint64_t* key, uint32_t n, uint32_t rank, uint32_t* hist) {
  const uint32_t lane = lane_id();
  uint32_t prefix = 0, mask = 0;
  for (int hi = 32; hi > 0; hi -= 5) {
    const int lo = hi > 5 ? hi - 5 : 0;
    const uint32_t digit_mask = (1u << (hi - lo)) - 1u;
    if (lane < 32) hist[lane] = 0;
    wave_sync();
    for (uint32_t q = lane; q < n; q += 64) {
      const uint32_t d = (uint32_t)(key[q] >> 32);
      if ((d & mask) == prefix) atomicAdd(&hist[(d >> lo) & digit_mask], 1u);
    }
    wave_sync();
    const uint32_t c = lane < 32 ? hist[lane] : 0u;
    const uint32_t cum = (uint32_t)wave_scan_add((int)c);
    const uint64_t over = __ballot(cum > rank);
    const int bucket = __ffsll((unsigned long long)over) - 1;
    rank -= __shfl(cum - c, bucket);
    prefix |= (uint32_t)bucket << lo;
    mask |= digit_mask << lo;
    wave_sync();
  }
  return prefix;
}

// Writes the result sample of event key k (a sample of the solid, or a
// sphere's chord end) of ray (a, p) at output position o.
__device__ __forceinline__ void write_event(const OffsetArgs& g, int a, int64_t p, double cu, double cv, uint64_t k,
                                            size_t o) {
  if (!(k & kSphereOrder)) {
    const uint32_t hq = g.in[a].offsets[p] + (uint32_t)(k & 0x7fffffffu);
    g.out_depth[a][o] = g.in[a].depth[hq];
    g.out_normal[a][3 * o] = g.in[a].normal[3 * (size_t)hq];
    g.out_normal[a][3 * o + 1] = g.in[a].normal[3 * (size_t)hq + 1];
    g.out_normal[a][3 * o + 2] = g.in[a].normal[3 * (size_t)hq + 2];
    g.out_tri[a][o] = g.in[a].tri[hq];
  } else {
    const uint32_t sph = (uint32_t)((k & 0x7fffffffu) >> 1);
    const SphereHit h = sphere_sample(g, a, cu, cv, sph, (k & 1u) != 0);
    g.out_depth[a][o] = h.depth;
    g.out_normal[a][3 * o] = h.n[0];
    g.out_normal[a][3 * o + 1] = h.n[1];
    g.out_normal[a][3 * o + 2] = h.n[2];
    g.out_tri[a][o] = -1 - (int32_t)sph;
  }
}

// Whether the write pass may take [o0, o1) as the output slot of ray (a, p): the
// offsets are in the caller's memory, and if they changed between the passes
// they must not lead beyond the outputs, nor leave any of them unwritten
// unnoticed.
__device__ __forceinline__ bool slot_ok(const OffsetArgs& g, int a, int64_t p, uint32_t o0, uint32_t o1) {
  return o0 <= o1 && o1 <= g.n_out[a] && (p > 0 || o0 == 0) && (p + 1 < (int64_t)g.w * g.w || o1 == g.n_out[a]);
}

// The per-ray pass: counts (kWrite false) or writes the ray's result.  The
// ray's events are taken in windows of depth: a window collects the events
// at or after its lower depth bound into a buffer of kOffsetBuf keys; when a
// chunk would not fit, the buffer is sorted and cut back to the events
// before the depth of its kOffsetKeep-th smallest, which becomes the
// window's (exclusive) upper bound.  Windows end between groups of equal
// depth, and the sweep carries H's parity, the open spheres and the result
// state from one window to the next.
struct RayLds {
  uint64_t key[kOffWaves][kOffsetBuf];
  uint64_t emit[kOffWaves][kOffsetEmit];
  uint32_t rbit[kOffWaves][kOffsetBuf / 32];
  uint32_t hist[kOffWaves][32];
};

// The ray of a wave: waves take the deep rays first (workgroups start in
// index order, so the longest rays do not end up as the launch's tail), then
// every ray in order, skipping the deep ones (-1: none).
__device__ __forceinline__ int64_t ray_of_wave(const OffsetArgs& g, int64_t wave_no) {
  if (wave_no < (int64_t)g.n_deep) return g.deep[wave_no];
  const int64_t ray = wave_no - g.n_deep;
  if (ray >= 3 * (int64_t)g.w * g.w) return -1;
  if (g.n_deep > 0 && g.ray_start[ray + 1] - g.ray_start[ray] > (uint32_t)kOffsetDeep) return -1;
  return ray;
}

template <bool kWrite>
__device__ void sweep_ray(const OffsetArgs& g, int64_t ray, RayLds& lds) {
  const int wv = threadIdx.x >> 6;
  const uint32_t lane = lane_id();
  const int64_t npix = (int64_t)g.w * g.w;
  const int a = (int)(ray / npix);
  const int64_t p = ray - a * npix;
  const int u = (a + 1) % 3, v = (a + 2) % 3;
  const int iu = (int)(p % g.w), iv = (int)(p / g.w);
  const double cu = centre_of(g, u, iu), cv = centre_of(g, v, iv);
  uint64_t* key = lds.key[wv];
  uint64_t* emit = lds.emit[wv];
  uint32_t* rbit = lds.rbit[wv];
  const AxisArrays& H = g.in[a];

  // the write pass's slot of the ray: out .. out + cnt
  uint32_t out = 0, cnt = 0;
  if (kWrite) {
    out = g.out_offsets[a][p];
    const uint32_t end = g.out_offsets[a][p + 1];
    if (!slot_ok(g, a, p, out, end)) {
      if (lane == 0) raise_mismatch(g.status, g.host_fail);
      return;
    }
    cnt = end - out;
    if (cnt == 0) return;
  }
  const uint32_t o0 = H.offsets[p], o1 = H.offsets[p + 1];
  uint32_t nh = 0;
  if (o1 < o0 || (uint64_t)o1 > H.n) {
    if (lane == 0) raise_mismatch(g.status, g.host_fail);
  } else {
    nh = (o1 - o0) & ~1u;
  }
  const uint32_t l0 = g.ray_start[ray], l1 = g.ray_start[ray + 1];
  const double r2 = g.r * g.r;

  uint32_t lower = 0;        // window: orderable depth >= lower ...
  bool more = true;          // ... and, if bounded, < upper
  int carry_h = 0, carry_s = 0;
  bool prev_res = false;
  uint32_t n_emit = 0;
  uint32_t kept = 0;         // end-point pairs kept so far
  uint32_t big = 0xffffffffu;  // a depth whose group was found larger than a window
  auto depth_of = [&](uint64_t k) -> float {
    if (!(k & kSphereOrder)) return H.depth[o0 + (uint32_t)(k & 0x7fffffffu)];
    return sphere_depth(g, a, cu, cv, (uint32_t)((k & 0x7fffffffu) >> 1), (k & 1u) != 0);
  };
  // Small interval removal over the first np end-point pairs of emit, which
  // are then counted or written (pairs are independent volumes, so the
  // emitted end points are taken in batches); an unpaired last end point
  // moves to the front.
  auto flush = [&](uint32_t np) {
    for (uint32_t m0 = 0; m0 < np; m0 += 64) {
      const uint32_t m = m0 + lane;
      bool keep = false;
      uint64_t ea = 0, eb = 0;
      if (m < np) {
        ea = emit[2 * m];
        eb = emit[2 * m + 1];
        const double th = (double)depth_of(eb) - (double)depth_of(ea);
        keep = th > 0.0 && th >= g.eps;
      }
      const uint64_t km = __ballot(keep);
      const uint32_t rank = kept + (uint32_t)__popcll(km & ((1ull << lane) - 1ull));
      // the sweep is deterministic, so the write pass keeps what the count
      // pass counted; a disagreement (checked at the end) never writes
      // outside the ray's slot
      if (kWrite && keep && 2 * rank + 1 < cnt) {
        write_event(g, a, p, cu, cv, ea, (size_t)out + 2 * rank);
        write_event(g, a, p, cu, cv, eb, (size_t)out + 2 * rank + 1);
      }
      if (!kWrite && keep && g.saved && 2 * rank + 1 < g.n_saved) {
        g.saved[(size_t)ray * g.n_saved + 2 * rank] = ea;
        g.saved[(size_t)ray * g.n_saved + 2 * rank + 1] = eb;
      }
      kept += (uint32_t)__popcll(km);
    }
    wave_sync();
    const uint32_t rest = n_emit - 2 * np;
    if (rest > 0 && lane == 0) emit[0] = emit[2 * np];
    n_emit = rest;
    wave_sync();
  };
  while (more) {
    if (big == lower) {
      // The group of equal depth `big`, from its sums over all the ray's
      // events: H's samples in it, the spheres entering minus those leaving
      // in it, and its first event (the smallest key).  The result state
      // after the group against the one before decides whether it emits,
      // exactly as the sweep decides for a group inside a window.
      uint32_t ch = 0;
      int cs = 0;
      uint64_t first = ~0ull;
      for (uint32_t k0 = 0; k0 < nh; k0 += 64) {
        const uint32_t k = k0 + lane;
        if (k < nh && orderable(H.depth[o0 + k]) == big) {
          ++ch;
          first = min(first, ((uint64_t)big << 32) | k);
        }
      }
      for (uint32_t base = l0; base < l1; base += 64) {
        const uint32_t e = base + lane;
        if (e < l1) {
          const uint32_t sph = g.list[e];
          const double* c = g.centres + 3 * (size_t)sph;
          const double du = cu - c[u], dv = cv - c[v];
          const double rho2 = du * du + dv * dv;
          if (rho2 < r2) {
            const double t = sqrt(r2 - rho2);
            const float d0 = (float)((c[a] - t) - g.lo[a]), d1 = (float)((c[a] + t) - g.lo[a]);
            if (orderable(d0) == big) {
              ++cs;
              first = min(first, ((uint64_t)big << 32) | kSphereOrder | (sph << 1));
            }
            if (orderable(d1) == big) {
              --cs;
              first = min(first, ((uint64_t)big << 32) | kSphereOrder | (sph << 1) | 1u);
            }
          }
        }
      }
      for (int d = 32; d >= 1; d >>= 1) {
        ch += (uint32_t)__shfl_xor((int)ch, d, 64);
        cs += __shfl_xor(cs, d, 64);
        const uint64_t o = __shfl_xor(first, d, 64);
        first = min(first, o);
      }
      carry_h += (int)ch;
      carry_s += cs;
      const bool res = g.union_op ? ((carry_h & 1) != 0 || carry_s > 0) : ((carry_h & 1) != 0 && carry_s <= 0);
      if (res != prev_res) {
        if (n_emit + 1 > (uint32_t)kOffsetEmit) flush(n_emit / 2);
        if (lane == 0) emit[n_emit] = first;
        ++n_emit;
        wave_sync();
      }
      prev_res = res;
      more = big != 0xffffffffu;
      lower = big + 1u;
      big = 0xffffffffu;
      continue;
    }
    uint32_t upper = 0;
    bool bounded = false;
    uint32_t n = 0;
    // append up to two events per lane (keys k0, k1; has0, has1) after filtering
    auto append = [&](uint64_t k0, bool has0, uint64_t k1, bool has1) {
      auto in_window = [&](uint64_t k) {
        const uint32_t d = (uint32_t)(k >> 32);
        return d >= lower && (!bounded || d < upper);
      };
      bool h0 = has0 && in_window(k0), h1 = has1 && in_window(k1);
      uint32_t total = (uint32_t)__popcll(__ballot(h0)) + (uint32_t)__popcll(__ballot(h1));
      if (n + total > (uint32_t)kOffsetBuf) {
        // the depth of the kOffsetKeep-th smallest event becomes the bound;
        // the events before it are compacted to the front (unsorted)
        const uint32_t cut = select_depth(key, n, (uint32_t)kOffsetKeep, lds.hist[wv]);
        uint32_t m = 0;
        for (uint32_t c0 = 0; c0 < n; c0 += 64) {
          const uint32_t q = c0 + lane;
          const uint64_t kq = q < n ? key[q] : 0ull;
          const bool keep = q < n && (uint32_t)(kq >> 32) < cut;
          const uint64_t bal = __ballot(keep);
          if (keep) key[m + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull))] = kq;
          m += (uint32_t)__popcll(bal);
        }
        bounded = true;
        upper = cut;
        n = m;
        // one group of equal depth fills the window: the window ends before
        // it and the group is taken whole, by its sums, when it is reached
        if (m == 0) big = cut;
        h0 = has0 && in_window(k0);
        h1 = has1 && in_window(k1);
        wave_sync();
      }
      const uint64_t m0 = __ballot(h0), m1 = __ballot(h1);
      const uint64_t below = (1ull << lane) - 1ull;
      uint32_t pos = n + (uint32_t)__popcll(m0 & below) + (uint32_t)__popcll(m1 & below);
      if (h0) key[pos++] = k0;
      if (h1) key[pos] = k1;
      n += (uint32_t)__popcll(m0) + (uint32_t)__popcll(m1);
    };
    for (uint32_t k0 = 0; k0 < nh; k0 += 64) {
      const uint32_t k = k0 + lane;
      const bool has = k < nh;
      const uint64_t kk = has ? (((uint64_t)orderable(H.depth[o0 + k]) << 32) | k) : 0ull;
      append(kk, has, 0ull, false);
    }
    // the ray's spheres, 64 at a time; loads run ahead (list entries two
    // chunks, centres one chunk) so that a chunk's tests do not wait for them
    uint32_t sph1 = 0, sph2 = 0;
    double cu1 = 0.0, cv1 = 0.0, ca1 = 0.0;
    if (l0 + lane < l1) {
      sph1 = g.list[l0 + lane];
      const double* c = g.centres + 3 * (size_t)sph1;
      cu1 = c[u];
      cv1 = c[v];
      ca1 = c[a];
    }
    if (l0 + 64 + lane < l1) sph2 = g.list[l0 + 64 + lane];
    for (uint32_t base = l0; base < l1; base += 64) {
      const uint32_t e = base + lane;
      const uint32_t sph = sph1;
      const double pu = cu1, pv = cv1, pa = ca1;
      if (e + 64 < l1) {
        const double* c = g.centres + 3 * (size_t)sph2;
        cu1 = c[u];
        cv1 = c[v];
        ca1 = c[a];
      }
      sph1 = sph2;
      if (e + 128 < l1) sph2 = g.list[e + 128];
      bool hit = false;
      uint64_t ka = 0, kb = 0;
      if (e < l1) {
        const double du = cu - pu, dv = cv - pv;
        const double rho2 = du * du + dv * dv;
        if (rho2 < r2) {
          hit = true;
          const double t = sqrt(r2 - rho2);
          const float d0 = (float)((pa - t) - g.lo[a]), d1 = (float)((pa + t) - g.lo[a]);
          ka = ((uint64_t)orderable(d0) << 32) | kSphereOrder | (sph << 1);
          kb = ((uint64_t)orderable(d1) << 32) | kSphereOrder | (sph << 1) | 1u;
        }
      }
      append(ka, hit, kb, hit);
    }
    wave_sync();
    if (n > 0) {
      wave_sort(key, n);
      // sweep: per event H's parity and the open spheres after it; at the
      // last event of each group the result state against the one after the
      // previous group; a change emits the group's first event
      int carry_first = -1;
      const bool window_prev = prev_res;  // result state before this window
      for (uint32_t c0 = 0; c0 < n; c0 += 64) {
        const uint32_t q = c0 + lane;
        const bool valid = q < n;
        const uint64_t kq = valid ? key[q] : ~0ull;
        const bool is_h = valid && !(kq & kSphereOrder);
        const int ph = carry_h + wave_scan_add(is_h ? 1 : 0);
        const int ps = carry_s + wave_scan_add((valid && !is_h) ? ((kq & 1u) ? -1 : 1) : 0);
        const uint32_t dq = (uint32_t)(kq >> 32);
        const bool first = valid && (q == 0 || (uint32_t)(key[q - 1] >> 32) != dq);
        const bool last = valid && (q + 1 == n || (uint32_t)(key[q + 1] >> 32) != dq);
        const int fq = max(carry_first, wave_scan_max(first ? (int)q : -1));
        const bool res = g.union_op ? ((ph & 1) != 0 || ps > 0) : ((ph & 1) != 0 && ps <= 0);
        const uint64_t rm = __ballot(valid && res);
        if (lane == 0) rbit[c0 >> 5] = (uint32_t)rm;
        if (lane == 32) rbit[(c0 >> 5) + 1] = (uint32_t)(rm >> 32);
        wave_sync();
        bool e = false;
        if (last) {
          const bool prev = fq > 0 ? ((rbit[(fq - 1) >> 5] >> ((fq - 1) & 31)) & 1u) != 0 : window_prev;
          e = prev != res;
        }
        const uint64_t em = __ballot(e);
        const uint32_t ne = (uint32_t)__popcll(em);
        if (n_emit + ne > (uint32_t)kOffsetEmit) flush(n_emit / 2);  // (then at most one is left)
        if (e) emit[n_emit + (uint32_t)__popcll(em & ((1ull << lane) - 1ull))] = key[fq];
        n_emit += ne;
        carry_h = __shfl(ph, 63);
        carry_s = __shfl(ps, 63);
        carry_first = __shfl(fq, 63);
        // state after the last event so far (after the window: the next one's start)
        const int last_q = (int)min(c0 + 63, n - 1);
        const uint64_t rm_last = __shfl(rm, 0);
        prev_res = ((rm_last >> (last_q - (int)c0)) & 1ull) != 0;
      }
      wave_sync();
    }
    more = bounded;
    lower = upper;
  }
  flush(n_emit / 2);
  if (!kWrite && lane == 0) g.counts[a][p] = 2 * kept;
  // more or fewer end points than the count pass kept: slots unwritten or
  // surplus ones dropped, so the call fails
  if (kWrite && lane == 0 && 2 * kept != cnt) raise_mismatch(g.status, g.host_fail);
}

template <bool kWrite>
__global__ __launch_bounds__(kOffBlock) void offset_ray_kernel(OffsetArgs g) {
  __shared__ RayLds lds;
  const int64_t ray = ray_of_wave(g, (int64_t)blockIdx.x * kOffWaves + (threadIdx.x >> 6));
  if (ray >= 0) sweep_ray<kWrite>(g, ray, lds);
}

// The rays that offset_union_kernel or offset_write_kernel left (g.rest), wave after wave.
template <bool kWrite>
__global__ __launch_bounds__(kOffBlock) void offset_rest_kernel(OffsetArgs g) {
  __shared__ RayLds lds;
  const uint32_t n = min(g.status[kWrite ? 18 : 17], (uint32_t)(3 * (int64_t)g.w * g.w));
  for (uint32_t q = blockIdx.x * kOffWaves + (threadIdx.x >> 6); q < n; q += gridDim.x * kOffWaves) {
    sweep_ray<kWrite>(g, g.rest[q], lds);
    wave_sync();
  }
}

// The write pass over the end points that the count pass kept: a wave takes
// the result samples of 64 rays in a row, a sample per lane.  Rays with more
// end points than are kept are listed for offset_rest_kernel.  Bound by the
// gathers of kept end points and centres: 16 us at w = 256 (a wave per ray,
// with most lanes idle: 124 us).
__global__ __launch_bounds__(kOffBlock) void offset_write_kernel(OffsetArgs g) {
  __shared__ uint32_t s_off[kOffWaves][65];
  const int64_t npix = (int64_t)g.w * g.w, groups = (npix + 63) / 64;
  const uint32_t lane = lane_id();
  uint32_t* const off = s_off[threadIdx.x >> 6];
  const int64_t group = (int64_t)blockIdx.x * kOffWaves + (threadIdx.x >> 6);
  if (group >= 3 * groups) return;
  const int a = (int)(group / groups), u = (a + 1) % 3, v = (a + 2) % 3;
  const int64_t p0 = (group - a * groups) * 64;
  const int n = (int)min((int64_t)64, npix - p0);
  bool deep = false, bad = false;
  if ((int)lane < n) {
    const uint32_t o0 = g.out_offsets[a][p0 + lane], o1 = g.out_offsets[a][p0 + lane + 1];
    off[lane] = o0;
    if ((int)lane == n - 1) off[n] = o1;
    deep = o1 - o0 > g.n_saved;
    bad = !slot_ok(g, a, p0 + lane, o0, o1) || (deep && g.most_out <= g.n_saved);  // (nothing takes the rest then)
  }
  if (__ballot(bad) != 0) {
    if (lane == 0) raise_mismatch(g.status, g.host_fail);
    return;
  }
  const uint64_t m = __ballot(deep);
  if (m != 0) {
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&g.status[18], (uint32_t)__popcll(m));
    at = (uint32_t)__shfl((int)at, 0);
    if (deep) g.rest[at + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = (uint32_t)(a * npix + p0 + lane);
  }
  wave_sync();
  const uint32_t first = off[0], last = off[n];
  for (uint32_t q = first + lane; q < last; q += 64) {
    int k = 0;  // the last ray with off[k] <= q
    for (int hi = n - 1; k < hi;) {
      const int mid = (k + hi + 1) >> 1;
      if (off[mid] <= q) k = mid; else hi = mid - 1;
    }
    if (off[k + 1] - off[k] > g.n_saved) continue;
    const int64_t p = p0 + k;
    const uint64_t key = g.saved[(size_t)(a * npix + p) * g.n_saved + (q - off[k])];
    // (an end point that the count pass did not keep: the offsets changed)
    const uint32_t from = (uint32_t)(key & 0x7fffffffu);
    if ((key & kSphereOrder) ? from >> 1 >= g.n_spheres : (uint64_t)g.in[a].offsets[p] + from >= g.in[a].n) {
      raise_mismatch(g.status, g.host_fail);
      continue;
    }
    write_event(g, a, p, centre_of(g, u, (int)(p % g.w)), centre_of(g, v, (int)(p / g.w)), key, q);
  }
}

// 64-bit words of LDS for a wave's cells: enter and leave keys (n + 4 each), a
// bit and a 16-bit list entry per cell.  They hold the sorted events afterwards.
__host__ __device__ constexpr int union_words(int n_cells) {
  const int cells = 2 * (n_cells + 4) + (n_cells / 64 + 1) + (n_cells / 4 + 1);
  return cells > kUnionEvents ? cells : kUnionEvents;
}

// The count pass of a ray, one wave: most of the spheres that hit a ray lie
// along the few places where the ray crosses or grazes the surface and overlap
// there, and only the ends of their union matter.  The ray's depth range is
// divided into cells of half a radius.  A chord at least a cell to either side
// of its centre (long) covers its whole cell, so the long chords of a cell
// together are one interval, and so are those of a run of neighbouring cells:
// nothing inside it can change the state of the spheres, which stays "one is
// open" throughout.  A cell keeps its first enter (depth, then order) and its
// last exit (depth, then the least order at that depth) by LDS min / max; a run
// of cells becomes two events, its first enter and its last exit.  The other
// chords (short, or outside the cells) are dropped when they lie strictly
// inside the interval of their cell and its neighbours and are events of their
// own otherwise.  An event that is dropped lies strictly inside an interval
// that is kept, so it could neither change the result nor be the first event of
// a group that does: the end points are those of the sweep over all events.
// The few events left are sorted (each finds its rank among at most 64 by
// reading them all, more by wave_sort) and swept as in sweep_ray.  A ray with
// more than kUnionEvents of them is listed for offset_rest_kernel.
// Bound by the latency of a ray's dependent loads (starts, list, centres) at the
// 25 waves that its LDS leaves a CU; a workgroup is one wave, so that a ray's LDS
// is free for the next as soon as it is done.  On the flower, r = 2 pixels: 0.196
// ms at w = 256 and 0.058 at 128 (with LDS of its own for the sorted events, 20
// waves: 0.24 and 0.063; with four rays a workgroup as well: 0.27 and 0.077), where
// sweeping every ray over all its events (one LDS sort of up to 1,024 keys a
// window) took 1.60 and 0.74 ms.  With four rays a workgroup, cells of three
// quarters of a radius took 0.31 and 0.096 (more short chords), and 256 events
// 0.36 ms at w = 256; with 160 one polar ray of w = 128 is left to the sweep,
// 0.02 ms.
__global__ __launch_bounds__(64) void offset_union_kernel(OffsetArgs g) {
  extern __shared__ uint64_t s_union[];
  __shared__ uint64_t buf[kUnionEvents];
  __shared__ uint32_t s_rbit[kUnionEvents / 32 + 2];
  const uint32_t lane = lane_id();
  const int64_t ray = ray_of_wave(g, blockIdx.x);
  if (ray < 0) return;
  const int64_t npix = (int64_t)g.w * g.w;
  const int a = (int)(ray / npix);
  const int64_t p = ray - a * npix;
  const int u = (a + 1) % 3, v = (a + 2) % 3;
  const AxisArrays& H = g.in[a];
  const uint32_t o0 = H.offsets[p], o1 = H.offsets[p + 1];
  const uint32_t l0 = g.ray_start[ray], l1 = g.ray_start[ray + 1];
  uint32_t nh = 0;
  if (o1 < o0 || (uint64_t)o1 > H.n) {
    if (lane == 0) atomicOr(g.status, kStatusMismatch);
  } else {
    nh = (o1 - o0) & ~1u;
  }
  if (nh == 0 && l0 == l1) {
    if (lane == 0) g.counts[a][p] = 0u;
    return;
  }
  auto give_up = [&] {
    if (lane == 0) g.rest[atomicAdd(&g.status[17], 1u)] = (uint32_t)ray;
  };
  const double cu = centre_of(g, u, (int)(p % g.w)), cv = centre_of(g, v, (int)(p / g.w));
  const double r2 = g.r * g.r, lo_a = g.lo[a];
  // cell c at index c + 1, empty cells before the first and behind the last
  const int n_cells = g.n_cells, n_slots = n_cells + 4;
  uint64_t* enter = s_union;
  uint64_t* leave = enter + n_slots;
  uint64_t* taken = leave + n_slots;                             // bit c: cell c holds a chord
  uint16_t* cells = reinterpret_cast<uint16_t*>(taken + n_cells / 64 + 1);  // the cells that do, in any order
  uint32_t n_taken = 0;
  uint64_t* buf2 = s_union;  // (once the cells are no longer needed)
  uint32_t n = 0;  // keys in buf
  const uint64_t below = (1ull << lane) - 1ull;

  if (l0 != l1) {
    for (int c = (int)lane; c < n_slots; c += 64) {
      enter[c] = ~0ull;
      leave[c] = 0ull;
    }
    if ((int)lane <= n_cells / 64) taken[lane] = 0ull;
    wave_sync();
    // whether the chord [d0, d1] (orderable depths) lies strictly inside the
    // interval of the cell of its middle and the cells beside it
    auto inside = [&](uint32_t d0, uint32_t d1) -> bool {
      auto depth = [](uint32_t b) -> double {
        return (double)__uint_as_float((b & 0x80000000u) ? (b & 0x7fffffffu) : ~b);
      };
      const double mid = 0.5 * (depth(d0) + depth(d1)) * g.inv_cell;
      if (!(mid >= 0.0 && mid < (double)n_cells)) return false;
      const int c = (int)mid + 1;
      const uint32_t e0 = (uint32_t)(enter[c - 1] >> 32), e1 = (uint32_t)(enter[c] >> 32), e2 = (uint32_t)(enter[c + 1] >> 32);
      const uint32_t x0 = (uint32_t)(leave[c - 1] >> 32), x1 = (uint32_t)(leave[c] >> 32), x2 = (uint32_t)(leave[c + 1] >> 32);
      // an empty cell's interval is (~0, 0) and holds nothing; a cell between
      // two joins them
      if (leave[c] != 0ull) return min(min(e0, e1), e2) < d0 && max(max(x0, x1), x2) > d1;
      return (e0 < d0 && x0 > d1) || (e2 < d0 && x2 > d1);
    };
    // drops the chords of buf that lie inside (pairs of keys), keeping order
    auto filter = [&] {
      wave_sync();
      uint32_t m = 0;
      for (uint32_t q0 = 0; q0 < n; q0 += 128) {
        const uint32_t q = q0 + 2 * lane;
        uint64_t k0 = 0, k1 = 0;
        bool keep = false;
        if (q < n) {
          k0 = buf[q];
          k1 = buf[q + 1];
          keep = !inside((uint32_t)(k0 >> 32), (uint32_t)(k1 >> 32));
        }
        const uint64_t bal = __ballot(keep);
        wave_sync();
        if (keep) {
          const uint32_t at = m + 2 * (uint32_t)__popcll(bal & below);
          buf[at] = k0;
          buf[at + 1] = k1;
        }
        m += 2 * (uint32_t)__popcll(bal);
      }
      n = m;
      wave_sync();
    };
    // Calls on(live, long, cell, enter key, exit key) for the chords of the
    // ray's spheres, 64 at a time; loads run ahead (list entries two chunks,
    // centres one chunk) so that a chunk's tests do not wait for them.
    auto chords = [&](auto&& on) {
      uint32_t sph1 = 0, sph2 = 0;
      double cu1 = 0.0, cv1 = 0.0, ca1 = 0.0;
      if (l0 + lane < l1) {
        sph1 = g.list[l0 + lane];
        const double* c = g.centres + 3 * (size_t)sph1;
        cu1 = c[u];
        cv1 = c[v];
        ca1 = c[a];
      }
      if (l0 + 64 + lane < l1) sph2 = g.list[l0 + 64 + lane];
      for (uint32_t base = l0; base < l1; base += 64) {
        const uint32_t e = base + lane;
        const uint32_t sph = sph1;
        const double pu = cu1, pv = cv1, pa = ca1;
        if (e + 64 < l1) {
          const double* c = g.centres + 3 * (size_t)sph2;
          cu1 = c[u];
          cv1 = c[v];
          ca1 = c[a];
        }
        sph1 = sph2;
        if (e + 128 < l1) sph2 = g.list[e + 128];
        const double du = cu - pu, dv = cv - pv;
        const double rho2 = du * du + dv * dv;
        const bool live = e < l1 && rho2 < r2;
        const double t = sqrt(live ? r2 - rho2 : 0.0);
        const float d0 = (float)((pa - t) - lo_a), d1 = (float)((pa + t) - lo_a);
        const uint64_t ka = ((uint64_t)orderable(d0) << 32) | kSphereOrder | (sph << 1),
                       kb = ((uint64_t)orderable(d1) << 32) | kSphereOrder | (sph << 1) | 1u;
        const double cell = (pa - lo_a) * g.inv_cell;
        const bool whole = t >= g.long_chord && cell >= 0.0 && cell < (double)n_cells && (ka >> 32) < (kb >> 32);
        on(live, whole, (int)cell, ka, kb);
      }
    };
    // appends a pair of keys; false: they do not fit
    auto append = [&](bool own, uint64_t ka, uint64_t kb) -> bool {
      const uint64_t bal = __ballot(own);
      const uint32_t more = 2 * (uint32_t)__popcll(bal);
      if (n + more > (uint32_t)kUnionEvents) return false;
      if (own) {
        const uint32_t at = n + 2 * (uint32_t)__popcll(bal & below);
        buf[at] = ka;
        buf[at + 1] = kb;
      }
      n += more;
      return true;
    };
    bool again = false;  // too many chords that are not long: taken once the cells are complete
    chords([&](bool live, bool whole, int c, uint64_t ka, uint64_t kb) {
      bool fresh = false;
      if (live && whole) {
        fresh = atomicMin((unsigned long long*)&enter[c + 1], (unsigned long long)ka) == ~0ull;
        // (the depth, then the complement of the order: the maximum has the least order)
        atomicMax((unsigned long long*)&leave[c + 1], (unsigned long long)(kb ^ 0xffffffffull));
      }
      const uint64_t bal = __ballot(fresh);
      if (fresh) {
        atomicOr((unsigned long long*)&taken[c >> 6], 1ull << (c & 63));
        cells[n_taken + (uint32_t)__popcll(bal & below)] = (uint16_t)c;
      }
      n_taken += (uint32_t)__popcll(bal);
      if (!again && !append(live && !whole, ka, kb)) again = true;
    });
    wave_sync();
    bool fits = true;
    if (again) {
      n = 0;
      chords([&](bool live, bool whole, int, uint64_t ka, uint64_t kb) {
        const bool own = live && !whole && !inside((uint32_t)(ka >> 32), (uint32_t)(kb >> 32));
        if (fits && !append(own, ka, kb)) fits = false;
      });
    } else {
      filter();
    }
    if (!fits) {
      give_up();
      return;
    }
    wave_sync();
    // runs of cells; the first enter of a run lies in one of its first three
    // cells and the last exit in one of its last three (a chord reaches at most
    // two cells beyond its own, and the run's end cells are covered whole)
    for (uint32_t q0 = 0; q0 < n_taken; q0 += 64) {
      bool first = false, last = false;
      uint64_t ke = 0, kx = 0;
      if (q0 + lane < n_taken) {
        const int c = (int)cells[q0 + lane] + 1;
        first = leave[c - 1] == 0ull;
        last = leave[c + 1] == 0ull;
        if (first) {
          ke = enter[c];
          if (!last) {
            ke = min(ke, enter[c + 1]);
            if (leave[c + 2] != 0ull) ke = min(ke, enter[c + 2]);
          }
        }
        if (last) {
          kx = leave[c];
          if (!first) {
            kx = max(kx, leave[c - 1]);
            if (leave[c - 2] != 0ull) kx = max(kx, leave[c - 2]);  // (c - 1 is a cell)
          }
          kx ^= 0xffffffffull;
        }
      }
      const uint64_t m0 = __ballot(first), m1 = __ballot(last);
      const uint32_t more = (uint32_t)__popcll(m0) + (uint32_t)__popcll(m1);
      if (more == 0) continue;
      if (n + more > (uint32_t)kUnionEvents) {
        give_up();
        return;
      }
      uint32_t at = n + (uint32_t)__popcll(m0 & below) + (uint32_t)__popcll(m1 & below);
      if (first) buf[at++] = ke;
      if (last) buf[at] = kx;
      n += more;
    }
  }
  wave_sync();
  // The solid's samples.  Strictly inside a run the result does not depend on
  // the solid (and every sample is, as a rule, inside the run of its own
  // sphere), so of consecutive samples inside one run only the parity counts:
  // one is kept if they are odd, none if they are even.
  {
    // the cell of a sample strictly inside the interval of its cell, else -1
    auto cell_of = [&](uint32_t k) -> int {
      if (k >= nh || l0 == l1) return -1;
      const float d = H.depth[o0 + k];
      const uint32_t b = orderable(d);
      const double cell = (double)d * g.inv_cell;
      if (!(cell >= 0.0 && cell < (double)n_cells)) return -1;
      const int c = (int)cell;
      return (uint32_t)(enter[c + 1] >> 32) < b && (uint32_t)(leave[c + 1] >> 32) > b ? c : -1;
    };
    // whether two such samples' cells are of one run: no empty cell between
    auto joined = [&](int c, int d) -> bool {
      if (c < 0 || d < 0) return false;
      if (c > d) {
        const int x = c;
        c = d;
        d = x;
      }
      for (int q = c >> 6; q <= d >> 6; ++q) {
        uint64_t gaps = ~taken[q];
        if (q == c >> 6) gaps &= ~0ull << (c & 63);
        if (q == d >> 6) gaps &= ~0ull >> (63 - (d & 63));
        if (gaps != 0) return false;
      }
      return true;
    };
    uint32_t start = 0;     // first sample of the group of the sample before the chunk
    int cell_before = -1;
    for (uint32_t k0 = 0; k0 < nh; k0 += 64) {
      const uint32_t k = k0 + lane;
      const int cell = cell_of(k), next = cell_of(k + 1);
      int prev = __shfl_up(cell, 1, 64);
      if (lane == 0) prev = cell_before;
      const bool head = !joined(prev, cell);
      const uint64_t heads = __ballot(head) & (below | (1ull << lane));
      const uint32_t first = heads ? k0 + 63u - (uint32_t)__clzll((long long)heads) : start;
      const bool keep = k < nh && (cell < 0 || (!joined(cell, next) && ((k - first) & 1u) == 0u));
      const uint64_t m = __ballot(keep);
      if (n + (uint32_t)__popcll(m) > (uint32_t)kUnionEvents) {
        give_up();
        return;
      }
      if (keep) buf[n + (uint32_t)__popcll(m & below)] = ((uint64_t)orderable(H.depth[o0 + k]) << 32) | k;
      n += (uint32_t)__popcll(m);
      start = (uint32_t)__shfl((int)first, 63);
      cell_before = __shfl(cell, 63);
    }
  }
  wave_sync();
  if (n == 0) {
    if (lane == 0) g.counts[a][p] = 0u;
    return;
  }
  uint64_t* key = buf;
  uint64_t* emit = buf2;
  if (n <= 64) {
    const uint64_t mine = lane < n ? buf[lane] : ~0ull;
    uint32_t rank = 0;
    for (uint32_t q = 0; q < n; ++q) rank += buf[q] < mine ? 1u : 0u;
    if (lane < n) buf2[rank] = mine;  // (every event has an order of its own)
    key = buf2;
    emit = buf;
    wave_sync();
  } else {
    wave_sort(buf, n);
  }
  // the sweep of sweep_ray, over one window that holds all events
  uint32_t* rbit = s_rbit;
  int carry_h = 0, carry_s = 0, carry_first = -1;
  uint32_t n_emit = 0;
  for (uint32_t c0 = 0; c0 < n; c0 += 64) {
    const uint32_t q = c0 + lane;
    const bool valid = q < n;
    const uint64_t kq = valid ? key[q] : ~0ull;
    const bool is_h = valid && !(kq & kSphereOrder);
    const uint64_t hm = __ballot(is_h), xm = __ballot(valid && !is_h && (kq & 1u)), sm = __ballot(valid && !is_h);
    const uint64_t upto = below | (1ull << lane);
    const int ph = carry_h + __popcll(hm & upto);
    const int ps = carry_s + __popcll(sm & upto) - 2 * __popcll(xm & upto);
    const uint32_t dq = (uint32_t)(kq >> 32);
    const bool first = valid && (q == 0 || (uint32_t)(key[q - 1] >> 32) != dq);
    const bool last = valid && (q + 1 == n || (uint32_t)(key[q + 1] >> 32) != dq);
    const uint64_t fm = __ballot(first) & upto;
    const int fq = fm ? (int)c0 + 63 - __clzll((long long)fm) : carry_first;
    const bool res = g.union_op ? ((ph & 1) != 0 || ps > 0) : ((ph & 1) != 0 && ps <= 0);
    const uint64_t rm = __ballot(valid && res);
    if (lane == 0) rbit[c0 >> 5] = (uint32_t)rm;
    if (lane == 32) rbit[(c0 >> 5) + 1] = (uint32_t)(rm >> 32);
    wave_sync();
    const bool prev = fq > 0 && ((rbit[(fq - 1) >> 5] >> ((fq - 1) & 31)) & 1u) != 0;
    const bool end = last && prev != res;
    const uint64_t em = __ballot(end);
    if (end) emit[n_emit + (uint32_t)__popcll(em & below)] = key[fq];
    n_emit += (uint32_t)__popcll(em);
    carry_h = __shfl(ph, 63);
    carry_s = __shfl(ps, 63);
    carry_first = __shfl(fq, 63);
  }
  wave_sync();
  // small interval removal (a key holds its event's depth)
  uint32_t kept = 0;
  for (uint32_t m0 = 0; m0 < n_emit / 2; m0 += 64) {
    const uint32_t m = m0 + lane;
    bool keep = false;
    uint64_t ea = 0, eb = 0;
    if (m < n_emit / 2) {
      ea = emit[2 * m];
      eb = emit[2 * m + 1];
      auto depth = [](uint64_t k) -> double {
        const uint32_t b = (uint32_t)(k >> 32);
        return (double)__uint_as_float((b & 0x80000000u) ? (b & 0x7fffffffu) : ~b);
      };
      const double th = depth(eb) - depth(ea);
      keep = th > 0.0 && th >= g.eps;
    }
    const uint64_t km = __ballot(keep);
    const uint32_t rank = kept + (uint32_t)__popcll(km & below);
    if (keep && g.saved && 2 * rank + 1 < g.n_saved) {
      g.saved[(size_t)ray * g.n_saved + 2 * rank] = ea;
      g.saved[(size_t)ray * g.n_saved + 2 * rank + 1] = eb;
    }
    kept += (uint32_t)__popcll(km);
  }
  if (lane == 0) g.counts[a][p] = 2 * kept;
}

}  // namespace

hipError_t launch_offset_centres(const OffsetArgs& g, hipStream_t s) {
  const int64_t groups = 3 * (((int64_t)g.w * g.w + 63) / 64);
  hipLaunchKernelGGL(offset_centres_kernel, dim3((unsigned)((groups + kOffWaves - 1) / kOffWaves)), dim3(kOffBlock), 0, s,
                     g);
  return hipGetLastError();
}

hipError_t launch_offset_bin(const OffsetArgs& g, bool scatter, hipStream_t s) {
  const int64_t n = 3 * (int64_t)g.n_spheres;
  if (n == 0) return hipSuccess;
  const dim3 grid((unsigned)((n + kOffBlock - 1) / kOffBlock));
  // a range lies within 2 (r / h + margin) pixels: less than eight of them hold
  // at most eight centres.  Whole offsets of the flower with masks and without:
  // 496 and 564 us at w = 256 and 2 pixels, 709 and 758 at w = 128 and 3.9
  bool small = true;
  for (int b = 0; b < 3; ++b) small = small && 2.0 * (g.r / g.h[b] + g.margin[b]) < 7.9;
  const auto kernel = small ? (scatter ? offset_bin_kernel<true, true> : offset_bin_kernel<false, true>)
                            : (scatter ? offset_bin_kernel<true, false> : offset_bin_kernel<false, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(kOffBlock), 0, s, g);
  return hipGetLastError();
}

// The workgroup that is done last reports the status, the lists' total and the
// number of deep rays to pinned memory (the atomics have returned by then).
__global__ __launch_bounds__(kOffBlock) void offset_deep_kernel(OffsetArgs g, uint32_t* host) {
  const int64_t ray = (int64_t)blockIdx.x * kOffBlock + threadIdx.x, n_rays = 3 * (int64_t)g.w * g.w;
  // (one atomic per wave: they queue at the counter)
  const bool deep = ray < n_rays && g.ray_start[ray + 1] - g.ray_start[ray] > (uint32_t)kOffsetDeep;
  const uint64_t m = __ballot(deep);
  if (m != 0) {
    uint32_t at = 0;
    const int lead = __ffsll((unsigned long long)m) - 1;
    if ((int)lane_id() == lead) at = atomicAdd(&g.status[16], (uint32_t)__popcll(m));
    at = (uint32_t)__shfl((int)at, lead, 64);
    if (deep) g.deep[at + (uint32_t)__popcll(m & ((1ull << lane_id()) - 1ull))] = (uint32_t)ray;
  }
  __syncthreads();
  if (threadIdx.x != 0 || atomicAdd(&g.status[19], 1u) + 1u != gridDim.x) return;
  host[0] = g.status[0];
  host[1] = g.ray_start[n_rays];
  host[2] = atomicAdd(&g.status[16], 0u);
}

hipError_t launch_offset_deep(const OffsetArgs& g, uint32_t* host, hipStream_t s) {
  const int64_t rays = 3 * (int64_t)g.w * g.w;
  hipLaunchKernelGGL(offset_deep_kernel, dim3((unsigned)((rays + kOffBlock - 1) / kOffBlock)), dim3(kOffBlock), 0, s,
                     g, host);
  return hipGetLastError();
}

hipError_t launch_offset_rays(const OffsetArgs& g, bool write, hipStream_t s) {
  const int64_t rays = 3 * (int64_t)g.w * g.w + g.n_deep;
  const dim3 grid((unsigned)((rays + kOffWaves - 1) / kOffWaves));
  const dim3 rest(grid.x < 1024 ? grid.x : 1024);  // (four workgroups of it fit a CU)
  if (write && g.saved) {
    const int64_t groups = 3 * (((int64_t)g.w * g.w + 63) / 64);
    hipLaunchKernelGGL(offset_write_kernel, dim3((unsigned)((groups + kOffWaves - 1) / kOffWaves)), dim3(kOffBlock), 0, s,
                       g);
    if (g.most_out > g.n_saved) hipLaunchKernelGGL(offset_rest_kernel<true>, rest, dim3(kOffBlock), 0, s, g);
  } else if (write) {
    hipLaunchKernelGGL(offset_ray_kernel<true>, grid, dim3(kOffBlock), 0, s, g);
  } else if (g.n_cells > 0) {
    const size_t lds = sizeof(uint64_t) * (size_t)union_words(g.n_cells);
    hipLaunchKernelGGL(offset_union_kernel, dim3((unsigned)rays), dim3(64), lds, s, g);
    hipLaunchKernelGGL(offset_rest_kernel<false>, rest, dim3(kOffBlock), 0, s, g);
  } else {
    hipLaunchKernelGGL(offset_ray_kernel<false>, grid, dim3(kOffBlock), 0, s, g);
  }
  return hipGetLastError();
}

}  // namespace ldni
