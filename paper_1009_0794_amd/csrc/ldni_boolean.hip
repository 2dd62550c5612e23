// ldni_boolean.hip -- gfx950 kernels of Boolean operations on two LDNIs.
//
// Sec. 4.1 (with Fig. 5) reduces a Boolean operation of two solids sampled on
// one grid to 1D work per pixel: each solid's samples bound its volumes as
// consecutive (enter, exit) pairs, and the result keeps the volumes where the
// operation holds; Sec. 4.1.1 then drops volumes thinner than eps.
//
// Each pixel is swept as a merge of its two sorted sample lists.  Events of
// equal depth form one group; a group flips a solid's inside state once per
// sample of that solid in it, and the result state is the operation of the two
// states after the group.  A group that changes the result state contributes
// one end point: A's first sample of the group if it has one, else B's (with
// its normal reversed for the difference).  So touching pieces merge, no
// zero-thickness gap or sliver can appear, and a pair's unpaired last sample
// (an odd count) is left out.  A volume is kept when its thickness
// (double)exit - (double)enter is positive and at least eps.
//
// Passes: count (the sweep: kept end points per pixel and the source of each),
// then the library's exclusive scan turns the counts into the result offsets
// in place (and finds the largest count), then write (a copy of each kept
// sample to its offset).  A wave owns 64 consecutive pixels, whose samples
// are contiguous ranges of both inputs and of the output: the count pass
// stages the depths in LDS with coalesced loads and merges them with
// all lanes at once, each an equal part of the merged samples, and the write pass copies the output range with coalesced stores.
// Nothing is a contraction; the passes stream the two inputs and the output
// (HBM).
#pragma clang fp contract(off)

#include "ldni_internal.hpp"

namespace ldni {
namespace {

constexpr int kBoolBlock = 256;
constexpr int kBoolWaves = kBoolBlock / 64;
constexpr int kBoolCap = 1024;  // depths of a wave's 64 pixels held in LDS (both inputs)
constexpr uint32_t kFromB = 0x80000000u;
// A batch whose deepest pixel has at most this many more (paired) samples than
// a 64th of the batch is merged a pixel per lane, else in 64 equal parts: the
// search, the compaction and the pairing of the parts cost about as many steps.
// Union of two scene64 LDNIs at w = 2048 / flower minus torus at 500: 8 steps 235 /
// 36 us, 16: 239 / 37, 32: 277 / 40, always a pixel per lane 357 / 117.
constexpr uint32_t kSerialSteps = 8;

__device__ __forceinline__ bool op_holds(int op, bool a, bool b) {
  return op == kBoolUnion ? (a | b) : op == kBoolIntersection ? (a & b) : (a & !b);
}

// The sweep of one pixel by one lane (a pixel deeper than LDS, or lists that
// are not ascending) over na (even) depths of A and nb of B; emit(enter,
// exit) receives the two end points of each kept volume as the index of the
// sample in its pixel list, | kFromB for B's.  Returns the kept samples.
template <class Emit>
__device__ __forceinline__ uint32_t sweep(const float* da, uint32_t na, const float* db, uint32_t nb,
                                          int op, double eps, Emit&& emit) {
  uint32_t ia = 0, ib = 0, n = 0;
  bool in_a = false, in_b = false, in_r = false;
  float enter = 0.0f;
  uint32_t enter_ref = 0;
  float za = na > 0 ? da[0] : 0.0f, zb = nb > 0 ? db[0] : 0.0f;
  while (ia < na || ib < nb) {
    // the group's depth: the smaller next depth (A first on ties and for
    // values that do not compare); its first event is always taken, so
    // every pass of the loop makes progress (when B's sample comes first,
    // A has none at its depth)
    const bool take_a = ia < na && (ib >= nb || !(zb < za));
    const float d = take_a ? za : zb;
    const uint32_t ref = take_a ? ia : (ib | kFromB);  // A's first sample of the group wins
    if (take_a) {
      in_a = !in_a;
      za = ++ia < na ? da[ia] : 0.0f;
    } else {
      in_b = !in_b;
      zb = ++ib < nb ? db[ib] : 0.0f;
    }
    while (ia < na && za == d) {
      in_a = !in_a;
      za = ++ia < na ? da[ia] : 0.0f;
    }
    while (ib < nb && zb == d) {
      in_b = !in_b;
      zb = ++ib < nb ? db[ib] : 0.0f;
    }
    const bool r = op_holds(op, in_a, in_b);
    if (r == in_r) continue;
    in_r = r;
    if (r) {
      enter = d;
      enter_ref = ref;
      continue;
    }
    const double th = (double)d - (double)enter;
    if (!(th > 0.0 && th >= eps)) continue;  // small interval removal
    emit(n, enter_ref, ref);
    n += 2;
  }
  return n;
}

// One input sample of A or B, read whole before anything is stored (the
// compiler cannot reorder loads past stores to other arrays, so reading and
// storing field by field would wait for each load in turn).
struct Sample {
  float d, nx, ny, nz;
  int32_t t;
};
__device__ __forceinline__ Sample get(const BooleanArgs& g, bool from_b, uint64_t src) {
  const AxisArrays& in = from_b ? g.b : g.a;
  Sample x;
  x.d = in.depth[src];
  x.nx = in.normal[3 * src];
  x.ny = in.normal[3 * src + 1];
  x.nz = in.normal[3 * src + 2];
  x.t = in.tri[src];
  return x;
}

// Stores result sample at (output index) from a sample of A or B.
__device__ __forceinline__ void put(const BooleanArgs& g, uint64_t at, bool from_b, const Sample& x) {
  const float sign = (from_b && g.op == kBoolDifference) ? -1.0f : 1.0f;
  g.out_depth[at] = x.d;
  g.out_normal[3 * at] = sign * x.nx;
  g.out_normal[3 * at + 1] = sign * x.ny;
  g.out_normal[3 * at + 2] = sign * x.nz;
  g.out_tri[at] = from_b ? -1 - x.t : x.t;
}

// A wave takes 64 consecutive pixels.  Their samples are contiguous in both
// inputs (and their results in the output), so the wave works through them in
// batches of consecutive pixels whose samples fit in LDS: it loads a batch's
// depths of both inputs with coalesced loads (all issued before any is waited
// for) and every lane of the batch sweeps its pixel from LDS.  A single pixel
// with more samples than LDS holds is swept straight from global memory.
// Offsets that decrease, pass the sample count, or do not chain from one pixel
// to the next raise the mismatch bit and empty the wave's pixels.
struct WavePixels {
  int64_t p;        // this lane's pixel
  bool live;        // p < npix
  bool ok;          // the whole wave's offsets are a valid prefix
  int nlive;        // live lanes (a prefix of the wave)
  uint32_t a0, a1, b0, b1;
};

__device__ __forceinline__ WavePixels wave_pixels(const BooleanArgs& g, int64_t p0, bool count_pass) {
  WavePixels w;
  const int lane = threadIdx.x & 63;
  w.p = p0 + lane;
  w.live = w.p < g.npix;
  w.nlive = (int)min<int64_t>(g.npix - p0, 64);
  w.a0 = w.a1 = w.b0 = w.b1 = 0;
  bool ok = true;
  if (w.live) {
    w.a0 = g.a.offsets[w.p];
    w.a1 = g.a.offsets[w.p + 1];
    w.b0 = g.b.offsets[w.p];
    w.b1 = g.b.offsets[w.p + 1];
    ok = w.a0 <= w.a1 && w.a1 <= g.a.n && w.b0 <= w.b1 && w.b1 <= g.b.n;
    if (!ok && count_pass)
      __hip_atomic_store(g.host_fail, (uint32_t)kStatusMismatch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  // consecutive pixels must also chain (each starts where the previous ends)
  const uint32_t pa1 = (uint32_t)__shfl_up((int)w.a1, 1, 64), pb1 = (uint32_t)__shfl_up((int)w.b1, 1, 64);
  const bool chained = lane == 0 || !w.live || (pa1 == w.a0 && pb1 == w.b0);
  w.ok = __ballot(!(ok && chained)) == 0;
  return w;
}

// The next batch from lane `first`: the lanes whose samples, counted from
// lane first's, fit in kBoolCap.  Returns its last lane, or first - 1 when
// lane first alone does not fit; sets the batch's first samples and counts.
struct Batch {
  int first, last;
  uint32_t A0, B0, nA, nB;
};
__device__ __forceinline__ Batch next_batch(const WavePixels& w, int first) {
  const int lane = threadIdx.x & 63;
  Batch bt;
  bt.first = first;
  bt.A0 = (uint32_t)__shfl((int)w.a0, first, 64);
  bt.B0 = (uint32_t)__shfl((int)w.b0, first, 64);
  const uint64_t need = (uint64_t)(w.a1 - bt.A0) + (w.b1 - bt.B0);
  const uint64_t fits = __ballot(lane >= first && lane < w.nlive && need <= (uint64_t)kBoolCap);
  bt.last = fits ? 63 - __clzll((long long)fits) : first - 1;
  const int l = bt.last >= first ? bt.last : first;
  bt.nA = (uint32_t)__shfl((int)w.a1, l, 64) - bt.A0;
  bt.nB = (uint32_t)__shfl((int)w.b1, l, 64) - bt.B0;
  return bt;
}

// Loads a batch's depths (A's, then B's) into s, eight per lane at a time,
// whose loads are issued before the stores to LDS wait for them.
__device__ __forceinline__ void load_batch(const BooleanArgs& g, const Batch& bt, float* s) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t tot = bt.nA + bt.nB;  // <= kBoolCap
  const float* da = g.a.depth + bt.A0;
  const float* db = g.b.depth + bt.B0;
  for (uint32_t i0 = 0; i0 < tot; i0 += 8 * 64) {
    float v[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      const uint32_t i = i0 + 64u * k + lane;
      v[k] = 0.0f;
      if (i < bt.nA) v[k] = da[i];
      else if (i < tot) v[k] = db[i - bt.nA];
    }
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      const uint32_t i = i0 + 64u * k + lane;
      if (i < tot) s[i] = v[k];
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The count pass: kept end points per pixel, and each one's source, in result
// order from refs[a0 + b0] of the wave's first pixel on (its index among the
// wave's samples of A, or of B | kFromB; a wave keeps at most its input
// samples, so these ranges never overlap).
//
// The samples of a batch, merged pixel by pixel, are cut into 64 equal parts,
// one per lane (the merge-path partition: Green, McColl, Bader, "GPU Merge Path",
// ICS 2012): a lane finds where its part begins (the pixel by its merged
// start, the place in both lists by a search along the merge's diagonal, and
// with them the parities so far), merges up to 16 samples, and decides the
// groups that begin in its part.  A change of the result state is marked at
// the group's place in the merged order, so the marks in order are the end
// points, enters and exits in turn (a pixel has an even number), and each pair
// decides by its thickness.
// Bound by the latency of the merge's dependent LDS reads (VALU issue 33 %): the union of two scene64
// LDNIs at w = 2048 (25.7 M samples) takes 0.236 ms against 0.305 with a pixel
// per lane throughout, the flower minus a torus at w = 500 36 us against 108
// (its polar pixels hold 160 samples, and a lane merged them while 63 waited).
__global__ void __launch_bounds__(kBoolBlock) boolean_count_kernel(BooleanArgs g) {
  __shared__ float s_dep[kBoolWaves][kBoolCap];
  __shared__ uint16_t s_mark[kBoolWaves][kBoolCap];
  // per pixel: its first samples in the batch, of A and of B, and the paired
  // samples of the pixels before it
  __shared__ uint32_t s_first[kBoolWaves][3][66];
  __shared__ uint32_t s_n[kBoolWaves][64];         // kept samples of the pixels
  // the status words of the launches behind this one (it has none itself)
  if (blockIdx.x == 0 && threadIdx.x < 64) g.status[threadIdx.x] = 0u;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t p0 = ((int64_t)blockIdx.x * kBoolWaves + wave) * 64;
  if (p0 >= g.npix) return;
  const WavePixels w = wave_pixels(g, p0, true);
  float* s = s_dep[wave];
  uint16_t* mark = s_mark[wave];
  uint32_t* fa = s_first[wave][0];
  uint32_t* fb = s_first[wave][1];
  uint32_t* merged = s_first[wave][2];
  uint32_t* count = s_n[wave];
  count[lane] = 0u;
  if (w.ok) {
    const uint32_t wa0 = (uint32_t)__shfl((int)w.a0, 0, 64), wb0 = (uint32_t)__shfl((int)w.b0, 0, 64);
    uint32_t* refs = g.refs + (uint64_t)wa0 + wb0;
    const uint32_t na = (w.a1 - w.a0) & ~1u, nb = (w.b1 - w.b0) & ~1u;  // whole pairs only
    // whether the operation holds, bit (inside A) * 2 + (inside B)
    const uint32_t holds = g.op == kBoolUnion ? 0xeu : g.op == kBoolIntersection ? 0x8u : 0x4u;
    uint64_t n_out = 0;  // kept samples of the wave so far
    // lanes [first, last] sweep their pixels one by one
    auto serial = [&](int first, int last, const float* da, const float* db) {
      const bool mine = lane >= first && lane <= last;
      uint32_t n = 0;
      if (mine) n = sweep(da, na, db, nb, g.op, g.eps, [](uint32_t, uint32_t, uint32_t) {});
      uint64_t incl = n;
      for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up((unsigned long long)incl, o, 64);
        if (lane >= o) incl += y;
      }
      uint32_t* to = refs + n_out + (incl - n);
      const uint32_t ra = w.a0 - wa0, rb = w.b0 - wb0;
      auto source = [&](uint32_t x) { return (x & kFromB) ? kFromB | (rb + (x & ~kFromB)) : ra + x; };
      if (mine) {
        sweep(da, na, db, nb, g.op, g.eps, [&](uint32_t k, uint32_t e, uint32_t x) {
          to[k] = source(e);
          to[k + 1] = source(x);
        });
        count[lane] = n;
      }
      n_out += __shfl((unsigned long long)incl, 63, 64);
    };
    for (int first = 0; first < w.nlive;) {
      const Batch bt = next_batch(w, first);
      if (bt.last < first) {  // one pixel deeper than LDS
        serial(first, first, g.a.depth + w.a0, g.b.depth + w.b0);
        first += 1;
        continue;
      }
      const uint32_t tot = bt.nA + bt.nB;
      if (tot == 0) {
        first = bt.last + 1;
        continue;
      }
      load_batch(g, bt, s);
      // (past the batch: its end)
      fa[lane] = lane > bt.last ? bt.nA : lane < first ? 0u : w.a0 - bt.A0;
      fb[lane] = lane > bt.last ? bt.nB : lane < first ? 0u : w.b0 - bt.B0;
      const uint32_t paired = lane >= first && lane <= bt.last ? na + nb : 0u;
      uint32_t upto = paired;
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)upto, o, 64);
        if (lane >= o) upto += y;
      }
      merged[lane] = upto - paired;
      const uint32_t all = (uint32_t)__shfl((int)upto, 63, 64);  // paired samples of the batch
      if (lane == 0) {
        fa[64] = bt.nA;
        fb[64] = bt.nB;
        merged[64] = all;
      }
      wave_sync();
      const uint32_t ra = bt.A0 - wa0, rb = bt.B0 - wb0;
      auto source = [&](uint32_t k) { return k >= bt.nA ? kFromB | (rb + (k - bt.nA)) : ra + k; };
      // the last pixel of the batch that starts at or before i
      auto pixel_of = [&](const uint32_t* f, uint32_t i) {
        int q = first;
#pragma unroll
        for (int h = 32; h >= 1; h >>= 1) {
          const int t = min(q + h, 64);
          if (t <= bt.last && f[t] <= i) q = t;
        }
        return q;
      };
      const uint32_t per = (all + 63) / 64;
      uint32_t deepest = paired;
      for (int o = 32; o >= 1; o >>= 1) deepest = max(deepest, (uint32_t)__shfl_xor((int)deepest, o, 64));
      if (deepest <= per + kSerialSteps) {
        // shallow pixels: a pixel per lane takes no more steps than the parts
        // and the search, the compaction and the pairing of the marks cost
        uint32_t n = 0;
        if (paired > 0) {
          const uint32_t xa = fa[lane], xb = bt.nA + fb[lane];
          uint16_t* mine = mark + merged[lane];
          n = sweep(s + xa, na, s + xb, nb, g.op, g.eps, [&](uint32_t k, uint32_t e, uint32_t x) {
            mine[k] = (uint16_t)((e & kFromB) ? xb + (e & ~kFromB) : xa + e);
            mine[k + 1] = (uint16_t)((x & kFromB) ? xb + (x & ~kFromB) : xa + x);
          });
        }
        uint32_t incl = n;
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t y = (uint32_t)__shfl_up((int)incl, o, 64);
          if (lane >= o) incl += y;
        }
        uint32_t* to = refs + n_out + (incl - n);
        for (uint32_t k = 0; k < n; ++k) to[k] = source(mark[merged[lane] + k]);
        if (n > 0) count[lane] = n;
        n_out += (uint32_t)__shfl((int)incl, 63, 64);
        wave_sync();
        first = bt.last + 1;
        continue;
      }
      for (uint32_t i = (uint32_t)lane; i < all; i += 64) mark[i] = 0xffffu;
      wave_sync();
      // Lists that do not ascend, or hold a NaN, are merged one sample after
      // the other.  There the search for a part's beginning may end elsewhere
      // than the part before it does: a lane checks the samples it merges, and
      // the parts must join, so that no sample is left unchecked between them.
      bool odd = false;
      uint32_t join = ~0u, end = 0;  // next sample of A where the part begins (inside a pixel), and where it ends
      const uint32_t m1 = min((lane + 1) * per, all);
      uint32_t m = (uint32_t)lane * per;
      if (m < m1) {
        int q = pixel_of(merged, m);
        uint32_t i, j, ea, eb;  // next samples of the pixel's lists in s, and their ends
        auto open = [&] {
          i = fa[q];
          j = bt.nA + fb[q];
          ea = i + ((fa[q + 1] - fa[q]) & ~1u);
          eb = j + ((fb[q + 1] - fb[q]) & ~1u);
        };
        open();
        uint32_t state;  // inside A: bit 1, inside B: bit 0
        float prev = 0.0f;  // depth of the sample before the part
        const uint32_t d0 = m - merged[q];
        {
          const uint32_t na_q = ea - i, nb_q = eb - j;
          uint32_t lo = d0 > nb_q ? d0 - nb_q : 0u, hi = min(d0, na_q);
          while (lo < hi) {  // A's samples among the first d0, A first on ties
            const uint32_t mid = (lo + hi) >> 1;
            if (!(s[j + d0 - 1 - mid] < s[i + mid])) lo = mid + 1; else hi = mid;
          }
          const uint32_t b_in = d0 - lo;
          state = (lo & 1u) << 1 | (b_in & 1u);
          const float pa = lo > 0 ? s[i + lo - 1] : 0.0f, pb = b_in > 0 ? s[j + b_in - 1] : 0.0f;
          prev = b_in == 0 || (lo > 0 && pb < pa) ? pa : pb;
          i += lo;
          j += b_in;
          if (d0 > 0) join = i;
        }
        float za = i < ea ? s[i] : 0.0f, zb = j < eb ? s[j] : 0.0f;
        // a group that began before this part is not ours: it is merged, not marked
        bool mine = !(d0 > 0 && ((i < ea && za == prev) || (j < eb && zb == prev)));
        bool was = (holds >> state) & 1u;
        uint32_t at = m, ref = 0;
        bool head = true;  // the next sample is the first of its group
        for (;;) {
          const bool of_a = i < ea && (j >= eb || !(zb < za));
          const uint32_t x = of_a ? i : j, e = of_a ? ea : eb;
          const float d = of_a ? za : zb;
          if (head) {
            ref = x;
            at = m;
          }
          const float z = x + 1 < e ? s[x + 1] : d;
          odd |= !(d <= z);
          i += of_a ? 1u : 0u;
          j += of_a ? 0u : 1u;
          za = of_a ? z : za;
          zb = of_a ? zb : z;
          state ^= of_a ? 2u : 1u;
          ++m;
          if (m == m1) end = i;
          head = !((i < ea && za == d) || (j < eb && zb == d));
          if (head) {  // the group is complete
            const bool is = (holds >> state) & 1u;
            if (mine && is != was) mark[at] = (uint16_t)ref;
            was = is;
            mine = true;
            if (m >= m1) break;
            if (i >= ea && j >= eb) {  // the next pixel with samples (there is one: m < all)
              do {
                ++q;
                open();
              } while (i >= ea && j >= eb);
              za = i < ea ? s[i] : 0.0f;
              zb = j < eb ? s[j] : 0.0f;
              state = 0;
              was = false;  // (nothing holds outside both)
            }
          }
        }
      }
      const uint32_t next = (uint32_t)__shfl_down((int)join, 1, 64);
      odd |= lane < 63 && next != ~0u && next != end;
      wave_sync();
      if (__ballot(odd) != 0) {
        serial(first, bt.last, s + (w.a0 - bt.A0), s + bt.nA + (w.b0 - bt.B0));
        wave_sync();
        first = bt.last + 1;
        continue;
      }
      // the marks, compacted in place (a mark only moves to the front)
      uint32_t n_ends = 0;
      for (uint32_t c = 0; c < all; c += 64) {
        const uint32_t m = c + lane < all ? mark[c + lane] : 0xffffu;
        const uint64_t bal = __ballot(m != 0xffffu);
        wave_sync();
        if (m != 0xffffu) mark[n_ends + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)m;
        n_ends += (uint32_t)__popcll(bal);
      }
      wave_sync();
      for (uint32_t m0 = 0; m0 < n_ends / 2; m0 += 64) {
        const uint32_t m = m0 + lane;
        uint32_t e = 0, x = 0;
        bool keep = false;
        if (m < n_ends / 2) {
          e = mark[2 * m];
          x = mark[2 * m + 1];
          const double th = (double)s[x] - (double)s[e];
          keep = th > 0.0 && th >= g.eps;  // small interval removal
        }
        const uint64_t bal = __ballot(keep);
        if (keep) {
          const uint64_t at = n_out + 2 * (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
          refs[at] = source(e);
          refs[at + 1] = source(x);
          atomicAdd(&count[e >= bt.nA ? pixel_of(fb, e - bt.nA) : pixel_of(fa, e)], 2u);
        }
        n_out += 2 * (uint32_t)__popcll(bal);
      }
      wave_sync();  // before the next batch replaces the depths
      first = bt.last + 1;
    }
  }
  wave_sync();
  if (w.live) g.counts[w.p] = count[lane];
}

// The write pass copies: the wave's output range [R0, R1) is contiguous, and
// so are its sources' entries in refs.  Four outputs per lane at a time, every
// load of the four issued before the stores.  Bound by HBM: whole lines of the
// inputs are read for the part that is kept (union of two scene64 LDNIs at w =
// 2048: 0.26 ms, 0.28 with a search for each output's pixel; flower minus torus
// at 500: 18 against 38 us).
__global__ void __launch_bounds__(kBoolBlock) boolean_write_kernel(BooleanArgs g) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t p0 = ((int64_t)blockIdx.x * kBoolWaves + wave) * 64;
  if (p0 >= g.npix) return;
  const uint32_t R0 = g.counts[p0], end = g.counts[min(p0 + 64, g.npix)];
  // (offsets in the caller's memory that changed between the passes do not lead
  // beyond the outputs, nor leave any of them unwritten unnoticed)
  const uint32_t R1 = (uint32_t)min((uint64_t)end, g.n_out);
  if (R0 > R1 || end != R1 || (p0 == 0 && R0 != 0) || (p0 + 64 >= g.npix && end != g.n_out))
    raise_mismatch(g.status, g.host_fail);
  const uint64_t a0 = g.a.offsets[p0], b0 = g.b.offsets[p0];
  const uint64_t n_refs = g.a.n + g.b.n;
  for (uint32_t k0 = R0; k0 < R1; k0 += 4 * 64) {
    uint32_t rf[4];
    bool from_b[4], ok[4], bad = false;
    uint64_t src[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint64_t k = (uint64_t)k0 + lane + 64u * u, at = a0 + b0 + (k - R0);
      ok[u] = k < R1 && at < n_refs;
      bad |= k < R1 && !ok[u];
      rf[u] = ok[u] ? g.refs[at] : 0u;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      from_b[u] = (rf[u] & kFromB) != 0;
      src[u] = (from_b[u] ? b0 : a0) + (rf[u] & ~kFromB);
      const bool in = src[u] < (from_b[u] ? g.b.n : g.a.n);
      bad |= ok[u] && !in;
      ok[u] = ok[u] && in;
    }
    Sample x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (ok[u]) x[u] = get(g, from_b[u], src[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (ok[u]) put(g, (uint64_t)k0 + lane + 64u * u, from_b[u], x[u]);
    // (inputs that changed between the passes do not lead out of bounds)
    if (bad) raise_mismatch(g.status, g.host_fail);
    if (R1 - k0 <= 4 * 64) break;
  }
}

}  // namespace

hipError_t launch_boolean(const BooleanArgs& g, bool write, hipStream_t s) {
  if (g.npix <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((g.npix + kBoolBlock - 1) / kBoolBlock);  // 64 pixels per wave
  if (write)
    hipLaunchKernelGGL(boolean_write_kernel, dim3(blocks), dim3(kBoolBlock), 0, s, g);
  else
    hipLaunchKernelGGL(boolean_count_kernel, dim3(blocks), dim3(kBoolBlock), 0, s, g);
  return hipGetLastError();
}

}  // namespace ldni
