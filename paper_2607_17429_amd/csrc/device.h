// Device helpers shared by the sector, block and H.V kernels: packed state
// labels, sector rank / unrank over digit-sum count tables, successor in
// label order, and the orbit search (candidate sets over the group).
//
// A packed label stores site k's digit a_k = m_k + s in bits [k*b, k*b+b),
// b = ceil(log2(2s+1)).  Comparing packed labels as integers gives the same
// order as comparing the labels n of Eq. (2), so "smallest label in the
// orbit" is the smallest packed word.  Also the start-vector generator of the
// Lanczos chains.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "ftlm.h"
#include "rank_word.h"

namespace ftlm {
namespace dev {

// Row map of the padded vector layouts: representative i starts at row
// (i / rpl) * rpline + (i % rpl) * dstride (dstride = d_Gamma).  rpl = 1:
// row i * rpline, with rpline = d_Gamma (plain padded rows) or a power of
// two above it (aligned rows); rpl > 1: rpl representatives packed into one
// 128-byte line of rpline rows, counted in 32 bits.
struct PadMap {
  uint32_t dstride, rpl, rpline;
  uint64_t n_reps;
};

__host__ __device__ __forceinline__ uint64_t padded_row(uint32_t dstride, uint32_t rpl, uint32_t rpline, uint64_t i) {
  if (rpl <= 1) return i * (uint64_t)rpline;
  const uint32_t i32 = (uint32_t)i;
  return (uint64_t)(i32 / rpl) * rpline + (uint64_t)(i32 % rpl) * dstride;
}

// The representative i and row k within it that stored row `row` holds;
// false for the rows between packed representatives and past the last one.
__host__ __device__ __forceinline__ bool padded_rep_of(const PadMap& m, uint64_t row, uint64_t& i, int& k) {
  if (m.rpl <= 1) {
    i = row / m.rpline;
    k = (int)(row - i * m.rpline);
    return i < m.n_reps;
  }
  const uint64_t g = row / m.rpline;
  const uint32_t w = (uint32_t)(row - g * m.rpline);
  const uint32_t slot = w / m.dstride;
  k = (int)(w - slot * m.dstride);
  i = g * m.rpl + slot;
  return slot < m.rpl && i < m.n_reps;
}

__device__ __forceinline__ uint64_t rank_bits(const RankWord& w) { return (uint64_t)w.hi << 32 | w.lo; }

template <typename W>
__device__ __forceinline__ int digit(W x, int k, int b, W mask) {
  return (int)((x >> (k * b)) & mask);
}

// Number of labels strictly below x in its sector (digits sum to A), in
// ascending label order.  cnt[k * stride + v] = ways for k digits to sum to v.
template <typename W>
__device__ __forceinline__ uint64_t sector_rank(W x, int N, int b, int d, int A, const uint64_t* cnt,
                                                int stride) {
  uint64_t r = 0;
  int rem = A;
  if (b == 1) {
    // one term per set bit, highest first, four table reads in flight
    for (; rem > 0; rem -= 4) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool on = x != 0 && rem > q;
        const int pos = on ? (int)(8 * sizeof(W)) - 1 - (sizeof(W) == 8 ? __clzll((long long)x) : __clz((int)x)) : 0;
        const uint64_t c = cnt[on ? pos * stride + rem - q : 0];
        r += on ? c : 0;
        x &= ~(W(on) << pos);
      }
    }
    return r;
  }
  const W mask = (W(1) << b) - 1;
  for (int pos = N - 1; pos >= 0; --pos) {
    int a = digit(x, pos, b, mask);
    for (int t = 0; t < a; ++t) {
      int v = rem - t;
      if (v >= 0) r += cnt[pos * stride + v];
    }
    rem -= a;
  }
  return r;
}

// The label of rank i in the sector.
template <typename W>
__device__ __forceinline__ W sector_unrank(uint64_t i, int N, int b, int d, int A, const uint64_t* cnt,
                                           int stride) {
  W x = 0;
  int rem = A;
  for (int pos = N - 1; pos >= 0; --pos) {
    int a = 0;
    for (; a < d - 1; ++a) {
      int v = rem - a;
      uint64_t c = v >= 0 ? cnt[pos * stride + v] : 0;
      if (i < c) break;
      i -= c;
    }
    x |= W(a) << (pos * b);
    rem -= a;
  }
  return x;
}

// Next larger label with the same digit sum.  For b == 1 the next bit
// permutation with equal popcount; otherwise move one unit up into the
// lowest raisable digit that has a non-zero digit sum below it and refill the
// lower digits with the smallest arrangement (largest digits lowest).
template <typename W>
__device__ __forceinline__ W sector_next(W x, int N, int b, int d) {
  if (b == 1) {
    if (x == 0) return x;
    W t = x | (x - 1);
    int tz = (sizeof(W) == 8) ? __builtin_ctzll((unsigned long long)x) : __builtin_ctz((unsigned)x);
    W nt = ~t;
    W low = nt & (W(0) - nt);
    return (t + 1) | (W((low - 1) >> (tz + 1)));
  }
  const W mask = (W(1) << b) - 1;
  int below = 0;
  for (int k = 0; k < N; ++k) {
    int a = digit(x, k, b, mask);
    if (k > 0 && below >= 1 && a < d - 1) {
      W y = x;
      // clear digits 0..k, set digit k to a + 1, refill 0..k-1 with below - 1
      W clear = (k + 1) * b >= (int)(8 * sizeof(W)) ? ~W(0) : ((W(1) << ((k + 1) * b)) - 1);
      y &= ~clear;
      y |= W(a + 1) << (k * b);
      int rem = below - 1;
      for (int j = 0; j < k && rem > 0; ++j) {
        int v = rem < d - 1 ? rem : d - 1;
        y |= W(v) << (j * b);
        rem -= v;
      }
      return y;
    }
    below += a;
  }
  return x;  // x was the largest label of the sector
}

// ---- orbit search ------------------------------------------------------------
// The orbit minimum of a label x is found bit by bit from the top: a set of
// candidate elements starts as the whole group, and at each image bit the
// candidates whose image has a 0 there stay (all stay when none has a 0).
// What is left maps x to the smallest image, and the lowest index in the set
// is the smallest element reaching it.  The set is a bit mask of GW 64-bit
// words (GW = 2, 5, 16 for groups of up to 128, 320, 1024 elements), and the
// set of elements with a 1 at an image bit is the OR of one mask per 4-site
// chunk of x: each position halves the candidates, so about log2 |G| + 2
// positions of N/4 mask lookups replace the |G| images of N b / 4 lookups
// each that a walk over the group costs (icosidodecahedron: about 10 x 8
// 16-byte reads instead of 130 x 8 4-byte ones).
//
// For labels of b > 1 bits per site the masks are those of the sites: the bit
// plane of digit bit `sub` (site s's bit at position s) is looked up.
//
// Mask table: mask[((p * NC + c) * 16 + v) * GW + w], p = 0 for the highest
// site, NC = chunks of 4 sites.  The first n_lds positions are read from LDS
// (lds), the others from memory (mask).  Image tables of the factored group G = T H (every g =
// t h exactly once): img[(row * nch + c) * 16 + v] = image of value v of the
// 4-bit chunk c of a label, rows = the |H| elements, then the |T| elements;
// split[g] = t << 16 | h.  PLAIN: one bit per site and no spin flip (every
// s = 1/2 sector but the flip-resolved ones), known at compile time.
template <typename W, int GW, bool PLAIN>
struct Orbit {
  const uint64_t* mask;
  const uint64_t* lds;
  int n_lds;
  const W* img;
  const uint32_t* split;
  int nH, nch, NC, N, b, G;
  bool zf_;  // resolve by the spin flip too (G x Z2)
  W full;    // packed label with every digit d - 1 (F x = full - x)
  __device__ __forceinline__ bool zf() const { return !PLAIN && zf_; }
  __device__ __forceinline__ int bits() const { return PLAIN ? 1 : b; }
};

// Image of x under the group element of table row `row` (a lane's own row).
template <typename W>
__device__ __forceinline__ W image_row(const W* __restrict__ img, int nch, int row, W x) {
  const W* t = img + (size_t)row * (nch * 16);
  W y = 0;
#pragma unroll 4
  for (int c = 0; c < nch; ++c) y |= t[c * 16 + (int)((x >> (4 * c)) & W(15))];
  return y;
}

template <typename W, int GW, bool PLAIN>
__device__ __forceinline__ W image(const Orbit<W, GW, PLAIN>& o, int g, W x) {
  if (o.nH == 1) return image_row<W>(o.img, o.nch, 1 + g, x);  // H = {e}, T in element order
  const uint32_t th = o.split[g];
  x = image_row<W>(o.img, o.nch, (int)(th & 0xffffu), x);
  return image_row<W>(o.img, o.nch, o.nH + (int)(th >> 16), x);
}

// The bits `sub` of every digit of x, site s's at position s.
template <typename W>
__device__ __forceinline__ W digit_plane(W x, int N, int b, int sub) {
  if (b == 1) return x;
  if (b == 2) {
    uint64_t y = ((uint64_t)x >> sub) & 0x5555555555555555ull;
    y = (y | (y >> 1)) & 0x3333333333333333ull;
    y = (y | (y >> 2)) & 0x0f0f0f0f0f0f0f0full;
    y = (y | (y >> 4)) & 0x00ff00ff00ff00ffull;
    y = (y | (y >> 8)) & 0x0000ffff0000ffffull;
    y = (y | (y >> 16)) & 0x00000000ffffffffull;
    return (W)y;
  }
  if (b == 3) {
    uint64_t y = ((uint64_t)x >> sub) & 0x1249249249249249ull;
    y = (y | (y >> 2)) & 0x10c30c30c30c30c3ull;
    y = (y | (y >> 4)) & 0x100f00f00f00f00full;
    y = (y | (y >> 8)) & 0x001f0000ff0000ffull;
    y = (y | (y >> 16)) & 0x001f00000000ffffull;
    y = (y | (y >> 32)) & 0x00000000001fffffull;
    return (W)y;
  }
  if (b == 4) {
    uint64_t y = ((uint64_t)x >> sub) & 0x1111111111111111ull;
    y = (y | (y >> 3)) & 0x0303030303030303ull;
    y = (y | (y >> 6)) & 0x000f000f000f000full;
    y = (y | (y >> 12)) & 0x000000ff000000ffull;
    y = (y | (y >> 24)) & 0x000000000000ffffull;
    return (W)y;
  }
  W y = 0;
  for (int k = 0; k < N; ++k) y |= ((x >> (k * b + sub)) & W(1)) << k;
  return y;
}

// The planes of a label: kept for b <= 4, formed on use above.
template <typename W>
struct Planes {
  W x, p0, p1, p2, p3;
  int N, b;
  __device__ __forceinline__ Planes(W x_, int N_, int b_) : x(x_), p1(0), p2(0), p3(0), N(N_), b(b_) {
    p0 = digit_plane<W>(x, N, b, 0);
    if (b > 1) p1 = digit_plane<W>(x, N, b, 1);
    if (b > 2) p2 = digit_plane<W>(x, N, b, 2);
    if (b > 3) p3 = digit_plane<W>(x, N, b, 3);
  }
  __device__ __forceinline__ W of(int sub) const {
    if (b > 4) return digit_plane<W>(x, N, b, sub);
    return sub < 2 ? (sub ? p1 : p0) : sub == 2 ? p2 : p3;
  }
};

// Elements whose image has a 1 at the plane's bit of position p's site.
template <typename W, int GW, bool PLAIN>
__device__ __forceinline__ void ones_at(const Orbit<W, GW, PLAIN>& o, W plane, int p, uint64_t (&ones)[GW]) {
#pragma unroll
  for (int w = 0; w < GW; ++w) ones[w] = 0;
  auto gather = [&](const uint64_t* t) {
    int c = 0;
    for (; c + 4 <= o.NC; c += 4) {  // four lookups in flight
      const uint64_t* e[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) e[q] = t + ((c + q) * 16 + (int)((plane >> (4 * (c + q))) & W(15))) * GW;
#pragma unroll
      for (int w = 0; w < GW; ++w) ones[w] |= (e[0][w] | e[1][w]) | (e[2][w] | e[3][w]);
    }
    if (c < o.NC) {
      // up to three more, the missing ones read the (empty) mask of value 0
      const uint64_t* e[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const bool in = c + q < o.NC;
        e[q] = t + (in ? (c + q) * 16 + (int)((plane >> (4 * (c + q))) & W(15)) : 0) * GW;
      }
#pragma unroll
      for (int w = 0; w < GW; ++w) ones[w] |= e[0][w] | e[1][w] | e[2][w];
    }
  };
  const size_t at = (size_t)p * o.NC * 16 * GW;
  if (p < o.n_lds)
    gather(o.lds + at);
  else
    gather(o.mask + at);
}

template <int GW>
__device__ __forceinline__ void all_elements(int G, uint64_t (&c)[GW]) {
#pragma unroll
  for (int w = 0; w < GW; ++w) {
    const int n = G - 64 * w;
    c[w] = n >= 64 ? ~0ull : n > 0 ? (1ull << n) - 1 : 0;
  }
}

template <int GW>
__device__ __forceinline__ int count(const uint64_t (&c)[GW]) {
  int n = 0;
#pragma unroll
  for (int w = 0; w < GW; ++w) n += __popcll(c[w]);
  return n;
}

// cand &= keep where that leaves any candidate
template <int GW>
__device__ __forceinline__ void keep_if_any(uint64_t (&cand)[GW], const uint64_t (&ones)[GW], bool of_ones) {
  uint64_t any = 0;
#pragma unroll
  for (int w = 0; w < GW; ++w) any |= cand[w] & (of_ones ? ones[w] : ~ones[w]);
  if (any) {
#pragma unroll
    for (int w = 0; w < GW; ++w) cand[w] &= of_ones ? ones[w] : ~ones[w];
  }
}

// Removes and returns the lowest element of a non-empty set.
template <int GW>
__device__ __forceinline__ int pop_lowest(uint64_t (&c)[GW]) {
  int g = 0;
  bool found = false;
#pragma unroll
  for (int w = 0; w < GW; ++w)
    if (!found && c[w]) {
      g = 64 * w + __builtin_ctzll(c[w]);
      c[w] &= c[w] - 1;
      found = true;
    }
  return g;
}

// Groups of up to this order are searched by the images of all elements (ring
// of 7 sites, s = 5/2, 14 elements, on-the-fly product: 80 us with the walk, 72
// so; rings of 18 and 20 sites, 36 and 40 elements: 70 us with the walk, 160
// and 133 by images).
constexpr int kFewElements = 16;

// Takes the flipped images into an orbit minimum: top is the largest image
// over G, reached first by topg and by top_ties elements.
template <typename W, int GW, bool PLAIN>
__device__ __forceinline__ void join_flipped(const Orbit<W, GW, PLAIN>& o, W top, int topg, int top_ties, W& best,
                                             int& bestg, int& ties) {
  if (o.full - top < best) {
    best = o.full - top;
    bestg = o.G + topg;
    ties = top_ties;
  } else if (o.full - top == best) {
    ties += top_ties;
  }
}

// Orbit minimum over G (over G x Z2 with zf) and the smallest group index h
// reaching it (U(h) a = best; index of (g, f) is f |G| + g).  Lanes that are
// not live do no search.  ties counts the elements that reach it, which is the
// order of the minimum's stabilizer.  The walk over positions stops when no
// lane of the wave has more than two candidates; two that are left are
// compared as images, a tie (non-trivial stabilizer) goes to the lower index.
// The spin flip F reverses label order (F x = full - x), so the flipped
// images' minimum is F of the G-orbit maximum: a second set keeps that one,
// and a G-element wins a tie with a flipped one.
template <typename W, int GW, bool PLAIN>
__device__ __forceinline__ void orbit_min(W a, bool live, const Orbit<W, GW, PLAIN>& o, W& best, int& bestg, int& ties) {
  uint64_t lo[GW], hi[GW];
  all_elements<GW>(o.G, lo);
#pragma unroll
  for (int w = 0; w < GW; ++w) {
    if (!live) lo[w] = w == 0 ? 1 : 0;
    hi[w] = o.zf() ? lo[w] : 0;
  }
  const Planes<W> planes(a, o.N, o.bits());
  if (o.G <= kFewElements) {
    // the images of all elements, which cost less than the walk's steps
    best = image<W, GW, PLAIN>(o, 0, a);
    W top = best;
    int topg = 0, top_ties = 1;
    bestg = 0;
    ties = 1;
#pragma unroll 4
    for (int g = 1; g < o.G; ++g) {
      const W y = image<W, GW, PLAIN>(o, g, a);
      ties = y < best ? 1 : ties + (y == best);
      bestg = y < best ? g : bestg;
      best = y < best ? y : best;
      top_ties = y > top ? 1 : top_ties + (y == top);
      topg = y > top ? g : topg;
      top = y > top ? y : top;
    }
    if (o.zf()) join_flipped(o, top, topg, top_ties, best, bestg, ties);
    return;
  }
  auto wide = [&] { return o.zf() ? max(count<GW>(lo), count<GW>(hi)) > 2 : count<GW>(lo) > 2; };
  bool more = __any(wide());
  for (int p = 0; p < o.N && more; ++p)
    for (int sub = o.bits() - 1; sub >= 0 && more; --sub) {
      uint64_t ones[GW];
      ones_at<W, GW, PLAIN>(o, planes.of(sub), p, ones);
      keep_if_any<GW>(lo, ones, false);
      if (o.zf()) keep_if_any<GW>(hi, ones, true);
      more = __any(wide());
    }
  // one or two are left, or, past the last position, all have the same image
  auto extreme = [&](uint64_t(&c)[GW], bool largest, W& y, int& g, int& n) {
    n = count<GW>(c);
    g = pop_lowest<GW>(c);
    const int g2 = n == 2 ? pop_lowest<GW>(c) : g;
    y = image<W, GW, PLAIN>(o, g, a);
    const W y2 = image<W, GW, PLAIN>(o, g2, a);
    if (n == 2 && y != y2) {
      n = 1;
      if (largest ? y2 > y : y2 < y) {
        y = y2;
        g = g2;
      }
    }
  };
  extreme(lo, false, best, bestg, ties);
  if (o.zf()) {
    W top;
    int topg, top_ties;
    extreme(hi, true, top, topg, top_ties);
    join_flipped(o, top, topg, top_ties, best, bestg, ties);
  }
}

// Whether x is the smallest label of its orbit (over G x Z2 with zf).  lo
// holds the elements whose image agrees with x so far, hi those whose image
// agrees with F x: x is not minimal once one of lo has a 0 where x has a 1,
// or one of hi a 1 where F x has a 0 (its flipped image is then below x).
template <typename W, int GW, bool PLAIN>
__device__ __forceinline__ bool is_orbit_min(W x, bool live, const Orbit<W, GW, PLAIN>& o) {
  uint64_t lo[GW], hi[GW];
  all_elements<GW>(o.G, lo);
#pragma unroll
  for (int w = 0; w < GW; ++w) hi[w] = o.zf() ? lo[w] : 0;
  const W fx = o.full - x;
  const Planes<W> planes(x, o.N, o.bits());
  bool open = live, minimal = live;
  for (int p = 0; p < o.N && __any(open); ++p)
    for (int sub = o.bits() - 1; sub >= 0 && __any(open); --sub) {
      uint64_t ones[GW];
      ones_at<W, GW, PLAIN>(o, planes.of(sub), p, ones);
      const int bit = (o.N - 1 - p) * o.bits() + sub;
      const bool xb = (x >> bit) & 1, fb = (fx >> bit) & 1;
      uint64_t below = 0;
#pragma unroll
      for (int w = 0; w < GW; ++w) {
        if (xb)
          below |= lo[w] & ~ones[w];
        else
          lo[w] &= ~ones[w];
        if (o.zf()) {
          if (!fb)
            below |= hi[w] & ones[w];
          else
            hi[w] &= ones[w];
        }
      }
      if (below) minimal = open = false;
      // only the identity (bit 0) follows x and nothing follows F x: no smaller image is left
      uint64_t rest = lo[0] & ~1ull;
#pragma unroll
      for (int w = 0; w < GW; ++w) rest |= hi[w] | (w ? lo[w] : 0);
      if (!rest) open = false;
    }
  return minimal;
}

// The elements that map x to itself (lo) and, with zf, to F x (hi).
template <typename W, int GW, bool PLAIN>
__device__ __forceinline__ void stabilizer(W x, bool live, const Orbit<W, GW, PLAIN>& o, uint64_t (&lo)[GW],
                                           uint64_t (&hi)[GW]) {
  all_elements<GW>(o.G, lo);
#pragma unroll
  for (int w = 0; w < GW; ++w) hi[w] = o.zf() ? lo[w] : 0;
  const W fx = o.full - x;
  const Planes<W> planes(x, o.N, o.bits());
  bool open = live;
  for (int p = 0; p < o.N && __any(open); ++p)
    for (int sub = o.bits() - 1; sub >= 0 && __any(open); --sub) {
      uint64_t ones[GW];
      ones_at<W, GW, PLAIN>(o, planes.of(sub), p, ones);
      const int bit = (o.N - 1 - p) * o.bits() + sub;
      const bool xb = (x >> bit) & 1, fb = (fx >> bit) & 1;
#pragma unroll
      for (int w = 0; w < GW; ++w) {
        lo[w] &= xb ? ones[w] : ~ones[w];
        if (o.zf()) hi[w] &= fb ? ones[w] : ~ones[w];
      }
      if (count<GW>(lo) <= 1 && count<GW>(hi) == 0) open = false;
    }
}

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Start-vector element j of the chain keyed by key (SplitMix64, Steele, Lea,
// Flood 2014): Rademacher takes the sign of the top bit of the (j+1)-th output;
// Gaussian draws outputs 2j+1, 2j+2 through the Box-Muller transform.
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ double start_value(uint64_t key, uint64_t j, int dist) {
  if (dist == FTLM_RADEMACHER) {
    const uint64_t x = mix64(key + (j + 1) * kGamma);
    return (x >> 63) ? -1.0 : 1.0;
  }
  const uint64_t x1 = mix64(key + (2 * j + 1) * kGamma);
  const uint64_t x2 = mix64(key + (2 * j + 2) * kGamma);
  const double u1 = ((double)(x1 >> 11) + 1.0) * 0x1.0p-53;
  const double u2 = (double)(x2 >> 11) * 0x1.0p-53;
  return sqrt(-2.0 * log(u1)) * cos(6.283185307179586476925286766559 * u2);
}

}  // namespace dev
}  // namespace ftlm
