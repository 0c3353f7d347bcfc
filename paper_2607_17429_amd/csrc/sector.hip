// Irrep-independent preprocessing of one magnetization sector (paper
// Section 3): orbit representatives, stabilizers, the rank lookup, Eq. (16)
// diagonal energies and the per-flip entry table (target representative,
// connecting element, flip), all built by GPU kernels.
//
// Representatives (Section 2.3: the smallest label of each orbit) come from a
// sweep over the sector in rank order: thread t owns ranks [64t, 64t + 64),
// unranks the first label, steps through the next 63 in label order and sets
// bit k of word t when no group element maps the label to a smaller one.  The
// bitmap over sector ranks, with per-word prefix counts, is also the lookup:
// index(r) = base[rank(r) >> 6] + popcount of the lower bits of that word.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <unordered_map>

#include "device.h"
#include "dispatch.h"
#include "internal.h"
#include "tune_cache.h"

namespace ftlm {

namespace {

constexpr int kThreads = 256;
// threads of the orbit-search kernels: their LDS tables (up to about 50 KiB)
// are shared by 8 waves, three workgroups to a CU
constexpr int kOrbitThreads = 512;

struct SecArgs {
  // orbit search (dev::Orbit): masks, image tables, element splits
  const uint64_t* mask;
  const void* img;
  const uint32_t* split;
  int n_lds, nH, nT, nch, NC;
  const uint64_t* cnt;
  int cnt_stride;
  int N, b, d, A, G;
  int zf;          // resolve by the spin flip too (G x Z2)
  uint64_t full;   // packed label with every digit d - 1 (F x = full - x)
  uint64_t D_M, n_words, n_reps;
  int transitive;  // the group moves every site to every other
};

template <typename E>
__device__ __forceinline__ void stage_copy(E* dst, const E* src, size_t n) {
  for (size_t i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

// The orbit-search tables of a kernel: the first n_lds mask positions in LDS,
// and with TABS the digit-sum counts and the image tables as well.
template <typename W, int GW, bool PLAIN, bool TABS>
__device__ __forceinline__ dev::Orbit<W, GW, PLAIN> stage_orbit(const SecArgs& a, uint64_t* smem, const uint64_t*& cnt) {
  const size_t pos = (size_t)a.NC * 16 * GW;
  stage_copy(smem, a.mask, (size_t)a.n_lds * pos);
  dev::Orbit<W, GW, PLAIN> o;
  o.mask = a.mask;
  o.lds = smem;
  o.n_lds = a.n_lds;
  o.split = a.split;
  o.nH = a.nH;
  o.nch = a.nch;
  o.NC = a.NC;
  o.N = a.N;
  o.b = a.b;
  o.G = a.G;
  o.zf_ = a.zf != 0;
  o.full = (W)a.full;
  if constexpr (TABS) {
    uint64_t* c = smem + (size_t)a.n_lds * pos;
    const size_t nc = (size_t)(a.N + 1) * a.cnt_stride;
    stage_copy(c, a.cnt, nc);
    W* t = (W*)(c + nc);
    stage_copy(t, (const W*)a.img, (size_t)(a.nH + a.nT) * a.nch * 16);
    cnt = c;
    o.img = t;
  } else {
    cnt = a.cnt;
    o.img = (const W*)a.img;
  }
  __syncthreads();
  return o;
}

// ---- representative sweep --------------------------------------------------
// Word w of the bitmap covers ranks [64 w, 64 w + 64).  WAVE = false: one
// thread per word unranks its first label and steps through the others in
// label order, 64 consecutive words per wave, so the lanes' labels share
// their high bits and mostly fail at the same position.  WAVE = true, for
// sectors of too few words to fill the device that way: one wave per word,
// every lane unranks its own label and the vote is the word.
// Bound by vector instructions (about 200 per label and wave, 61% busy) and
// branches.  1.55e8 labels of the s = 1/2 icosidodecahedron at M = 0: 1.19 ms
// against 1.53 ms with the images of all elements; the 924 labels of the
// icosahedron: 13 us (one wave per word) against 201 us.
template <typename W, int GW, bool PLAIN, bool TABS, bool WAVE>
__global__ void __launch_bounds__(kOrbitThreads) k_enum(SecArgs a, dev::RankWord* __restrict__ out) {
  extern __shared__ uint64_t smem_raw[];
  const uint64_t* cnt;
  const dev::Orbit<W, GW, PLAIN> o = stage_orbit<W, GW, PLAIN, TABS>(a, smem_raw, cnt);
  const uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  if constexpr (WAVE) {
    for (uint64_t w = t0 >> 6; w < a.n_words; w += stride >> 6) {
      const uint64_t rank = w * 64 + (threadIdx.x & 63);
      const bool live = rank < a.D_M;
      const W x = dev::sector_unrank<W>(live ? rank : 0, a.N, a.b, a.d, a.A, cnt, a.cnt_stride);
      const uint64_t bits = __ballot(dev::is_orbit_min<W, GW, PLAIN>(x, live, o));
      if ((threadIdx.x & 63) == 0) out[w] = dev::RankWord{(uint32_t)bits, (uint32_t)(bits >> 32), 0u};
    }
  } else {
    for (uint64_t w = t0; w < a.n_words; w += stride) {
      W x = dev::sector_unrank<W>(w * 64, a.N, a.b, a.d, a.A, cnt, a.cnt_stride);
      uint64_t bits = 0;
      // the top digit only grows along the word, and a transitive group can
      // bring any digit to the top: above the mean digit no label is minimal
      // (for d = 2 every label with the top bit set, half of them at M = 0)
      const int top = (int)(x >> ((a.N - 1) * a.b));
      for (int k = 0; k < 64 && !(a.transitive && a.A < a.N * top); ++k) {
        const bool live = w * 64 + k < a.D_M;
        if (dev::is_orbit_min<W, GW, PLAIN>(x, live, o)) bits |= 1ull << k;
        x = dev::sector_next<W>(x, a.N, a.b, a.d);
      }
      out[w] = dev::RankWord{(uint32_t)bits, (uint32_t)(bits >> 32), 0u};
    }
  }
}

// Representatives before each word, in place, in tiles of kRankTile words: the
// tiles' counts, their prefix sum (scan_exclusive_u64, 1/1536 of the records),
// then the words' own within each tile.  Building the records needs no other
// array of the sector's size.
constexpr int kRankItems = 4, kRankTile = kThreads * kRankItems;

// Inclusive sums of one count per thread over the workgroup (s: kThreads words).
__device__ __forceinline__ uint32_t wg_inclusive(uint32_t own, uint32_t* s) {
  const uint32_t t = threadIdx.x;
  s[t] = own;
  __syncthreads();
  for (uint32_t step = 1; step < kThreads; step <<= 1) {
    const uint32_t add = t >= step ? s[t - step] : 0;
    __syncthreads();
    s[t] += add;
    __syncthreads();
  }
  return s[t];
}

__global__ void __launch_bounds__(kThreads) k_rank_tiles(const dev::RankWord* __restrict__ ranks, uint64_t n,
                                                        uint64_t* __restrict__ tile_counts) {
  __shared__ uint32_t s[kThreads];
  const uint64_t w0 = (uint64_t)blockIdx.x * kRankTile;
  uint32_t own = 0;
#pragma unroll
  for (int i = 0; i < kRankItems; ++i) {
    const uint64_t w = w0 + i * kThreads + threadIdx.x;
    if (w < n) own += __popcll(dev::rank_bits(ranks[w]));
  }
  const uint32_t sum = wg_inclusive(own, s);
  if (threadIdx.x == kThreads - 1) tile_counts[blockIdx.x] = sum;
}

__global__ void __launch_bounds__(kThreads) k_rank_bases(dev::RankWord* __restrict__ ranks, uint64_t n,
                                                        const uint64_t* __restrict__ tile_base) {
  __shared__ uint32_t s[kThreads];
  const uint64_t w0 = (uint64_t)blockIdx.x * kRankTile + (uint64_t)threadIdx.x * kRankItems;
  uint32_t c[kRankItems], own = 0;
#pragma unroll
  for (int i = 0; i < kRankItems; ++i) {
    c[i] = w0 + i < n ? __popcll(dev::rank_bits(ranks[w0 + i])) : 0;
    own += c[i];
  }
  uint32_t base = (uint32_t)tile_base[blockIdx.x] + wg_inclusive(own, s) - own;
#pragma unroll
  for (int i = 0; i < kRankItems; ++i) {
    if (w0 + i < n) ranks[w0 + i].base = base;
    base += c[i];
  }
}

template <typename W>
__global__ void __launch_bounds__(kThreads) k_extract(SecArgs a, const dev::RankWord* __restrict__ ranks,
                                                     uint64_t* __restrict__ reps) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t w = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; w < a.n_words; w += stride) {
    const uint64_t m = dev::rank_bits(ranks[w]);
    if (!m) continue;
    W x = dev::sector_unrank<W>(w * 64, a.N, a.b, a.d, a.A, a.cnt, a.cnt_stride);
    uint64_t j = ranks[w].base;
    const int top = 63 - __clzll(m);
    for (int k = 0; k <= top; ++k) {
      if ((m >> k) & 1) reps[j++] = (uint64_t)x;
      if (k < top) x = dev::sector_next<W>(x, a.N, a.b, a.d);
    }
  }
}

// ---- stabilizers -----------------------------------------------------------
// flag[i] = 1 when some element other than e fixes representative i.
template <typename W, int GW, bool PLAIN, bool TABS>
__global__ void __launch_bounds__(kOrbitThreads) k_stab_flag(SecArgs a, const uint64_t* __restrict__ reps,
                                                            uint64_t* __restrict__ flag) {
  extern __shared__ uint64_t smem_raw[];
  const uint64_t* cnt;
  const dev::Orbit<W, GW, PLAIN> o = stage_orbit<W, GW, PLAIN, TABS>(a, smem_raw, cnt);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_reps; i += stride) {
    uint64_t lo[GW], hi[GW];
    dev::stabilizer<W, GW, PLAIN>((W)reps[i], true, o, lo, hi);
    flag[i] = dev::count<GW>(lo) + dev::count<GW>(hi) > 1 ? 1 : 0;
  }
}

// Full stabilizer masks of the representatives with a non-trivial stabilizer,
// written compacted (pos = exclusive scan of the flags, pos[n_reps] = count).
template <typename W, int GW, bool PLAIN, bool TABS>
__global__ void __launch_bounds__(kOrbitThreads) k_stab_mask(SecArgs a, const uint64_t* __restrict__ reps,
                                                            const uint64_t* __restrict__ pos, int mw,
                                                            uint64_t* __restrict__ masks,
                                                            uint64_t* __restrict__ idx_out) {
  extern __shared__ uint64_t smem_raw[];
  const uint64_t* cnt;
  const dev::Orbit<W, GW, PLAIN> o = stage_orbit<W, GW, PLAIN, TABS>(a, smem_raw, cnt);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_reps; i += stride) {
    const uint64_t p = pos[i];
    if (pos[i + 1] == p) continue;
    uint64_t lo[GW], hi[GW];
    dev::stabilizer<W, GW, PLAIN>((W)reps[i], true, o, lo, hi);
    // element (g, F) is bit |G| + g of the mask
    uint64_t* mk = masks + p * mw;
    for (int wq = 0; wq < mw; ++wq) {
      uint64_t m = 0;
#pragma unroll
      for (int q = 0; q < GW; ++q) {
        if (q == wq) m |= lo[q];
        const int at = a.G + 64 * q - 64 * wq;  // where hi's word q starts in this word
        if (at >= 0 && at < 64) m |= hi[q] << at;
        if (at < 0 && at > -64) m |= hi[q] >> -at;
      }
      mk[wq] = m;
    }
    idx_out[p] = i;
  }
}

__global__ void __launch_bounds__(kThreads) k_first_trivial(const uint64_t* __restrict__ pos, uint64_t n,
                                                           unsigned long long* out) {
  __shared__ unsigned long long red[kThreads];
  unsigned long long best = ~0ull;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    if (pos[i + 1] == pos[i]) {
      best = i;
      break;  // later i of this lane are larger
    }
  red[threadIdx.x] = best;
  __syncthreads();
  for (int off = kThreads / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] = min(red[threadIdx.x], red[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0 && red[0] != ~0ull) atomicMin(out, red[0]);
}

__global__ void k_assign_stab(const uint64_t* __restrict__ pos, uint64_t n, const uint16_t* __restrict__ ids_nt,
                              uint16_t trivial_id, uint16_t* __restrict__ stab_id) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t p = pos[i];
    stab_id[i] = (pos[i + 1] != p) ? ids_nt[p] : trivial_id;
  }
}

// ---- flips (Eq. 3) -----------------------------------------------------------
struct FlipArgs {
  const int32_t* bonds;
  const double* J;
  int nbonds;
};

template <typename W>
__device__ __forceinline__ bool admissible(W p, int cand, const FlipArgs& f, int b, int d, W mask) {
  const int bond = cand >> 1;
  const int i = f.bonds[2 * bond], j = f.bonds[2 * bond + 1];
  const int ai = dev::digit(p, i, b, mask), aj = dev::digit(p, j, b, mask);
  return (cand & 1) ? (ai > 0 && aj < d - 1) : (ai < d - 1 && aj > 0);
}

template <typename W>
__device__ __forceinline__ W apply_flip(W p, int cand, const FlipArgs& f, int b) {
  const int bond = cand >> 1;
  const int i = f.bonds[2 * bond], j = f.bonds[2 * bond + 1];
  const W ui = W(1) << (i * b), uj = W(1) << (j * b);
  return (cand & 1) ? (p - ui + uj) : (p + ui - uj);
}

template <typename W>
__global__ void __launch_bounds__(kThreads) k_entry_count(SecArgs a, FlipArgs f, const uint64_t* __restrict__ reps,
                                                         uint64_t* __restrict__ counts, double* __restrict__ ediag) {
  const W mask = (W(1) << a.b) - 1;
  const double s = 0.5 * (a.d - 1);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_reps; i += stride) {
    const W p = (W)reps[i];
    uint64_t c = 0;
    double e = 0;
    for (int bnd = 0; bnd < f.nbonds; ++bnd) {
      const int ai = dev::digit(p, f.bonds[2 * bnd], a.b, mask), aj = dev::digit(p, f.bonds[2 * bnd + 1], a.b, mask);
      c += (ai < a.d - 1 && aj > 0) + (ai > 0 && aj < a.d - 1);
      e += f.J[bnd] * (ai - s) * (aj - s);
    }
    counts[i] = c;
    ediag[i] = e;
  }
}

template <typename W>
__device__ __forceinline__ bool lookup(W r, const SecArgs& a, const dev::RankWord* __restrict__ ranks,
                                       const uint64_t* cnt, uint64_t& idx) {
  const uint64_t rk = dev::sector_rank<W>(r, a.N, a.b, a.d, a.A, cnt, a.cnt_stride);
  if (rk >= a.D_M) return false;
  const dev::RankWord w = ranks[rk >> 6];
  const int k = (int)(rk & 63);
  const uint64_t bits = dev::rank_bits(w);
  idx = w.base + (uint64_t)__popcll(bits & ((1ull << k) - 1));
  return (bits >> k) & 1;
}

// The entries of a workgroup's representatives (group i0 = blockIdx.x * rb,
// rb at most kFillReps, and so on by the grid): their admissible flips are
// listed in LDS in entry order, then one lane takes one flip, so every lane
// of the orbit search has work and neighbouring lanes write neighbouring
// entries (a lane per representative left the lanes of short rows idle and
// gave a sector of a few representatives to a few lanes, one flip after the
// other).  Bound by vector instructions (78% busy; the lookup is one random
// 12-byte read).  4.02e7 flips of the s = 1/2 icosidodecahedron at M = 0:
// 2.17 ms against 4.51 ms; the icosahedron's sectors 17 us against 257 us.
constexpr int kFillReps = 64;
constexpr int kFillList = 4096;  // listed flips per pass (16 KiB)

template <typename W, int GW, bool PLAIN, bool TABS>
__global__ void __launch_bounds__(kOrbitThreads) k_entry_fill(SecArgs a, FlipArgs f, int rb, const uint64_t* __restrict__ reps,
                                                             const uint64_t* __restrict__ row_ptr,
                                                             const dev::RankWord* __restrict__ ranks,
                                                             uint64_t* __restrict__ entries,
                                                             uint32_t* __restrict__ eidx, uint16_t* __restrict__ ehc,
                                                             int hbits) {
  extern __shared__ uint64_t smem_raw[];
  __shared__ uint32_t list[kFillList];       // representative in the group << 16 | flip
  __shared__ uint32_t from[kFillReps + 1];   // first listed flip of each representative
  __shared__ uint64_t done[kFillReps];       // entries written before this pass
  const uint64_t* cnt;
  const dev::Orbit<W, GW, PLAIN> o = stage_orbit<W, GW, PLAIN, TABS>(a, smem_raw, cnt);
  const W mask = (W(1) << a.b) - 1;
  const int ncand = 2 * f.nbonds;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int span = min(ncand, kFillList / rb);  // flips of one representative per pass
  for (uint64_t i0 = (uint64_t)blockIdx.x * rb; i0 < a.n_reps; i0 += (uint64_t)gridDim.x * rb) {
    const int n = (int)min((uint64_t)rb, a.n_reps - i0);
    for (int r = threadIdx.x; r < n; r += blockDim.x) done[r] = row_ptr[i0 + r];
    for (int q0 = 0; q0 < ncand; q0 += span) {
      const int q1 = min(q0 + span, ncand);
      __syncthreads();  // the last pass is through with list, from and done
      // count, offsets, list: one wave per representative
      for (int r = wave; r < n; r += waves) {
        const W p = (W)reps[i0 + r];
        uint32_t c = 0;
        for (int q = q0 + lane; __any(q < q1); q += 64)
          c += __popcll(__ballot(q < q1 && admissible(p, q, f, a.b, a.d, mask)));
        if (lane == 0) from[r + 1] = c;
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        from[0] = 0;
        for (int r = 0; r < n; ++r) from[r + 1] += from[r];
      }
      __syncthreads();
      for (int r = wave; r < n; r += waves) {
        const W p = (W)reps[i0 + r];
        uint32_t at = from[r];
        for (int q = q0 + lane; __any(q < q1); q += 64) {
          const bool ok = q < q1 && admissible(p, q, f, a.b, a.d, mask);
          const uint64_t m = __ballot(ok);
          if (ok) list[at + __popcll(m & ((1ull << lane) - 1))] = ((uint32_t)r << 16) | (uint32_t)q;
          at += __popcll(m);
        }
      }
      __syncthreads();
      const uint32_t total = from[n];
      for (uint32_t e0 = 0; e0 < total; e0 += blockDim.x) {
        const uint32_t e = e0 + threadIdx.x;
        const bool live = e < total;
        const uint32_t rq = list[live ? e : 0];
        const int r = (int)(rq >> 16), cur = (int)(rq & 0xffffu);
        W t;
        int h, ties;
        dev::orbit_min<W, GW, PLAIN>(apply_flip<W>((W)reps[i0 + r], cur, f, a.b), live, o, t, h, ties);
        if (live) {
          uint64_t idx = 0;
          const bool ok = lookup<W>(t, a, ranks, cnt, idx);
          // a canonical label of the sector is always a representative
          // top bit: the target's stabilizer is trivial, one element reaches it
          // (its n_Gamma, L and V are then known without its stabilizer id)
          const bool triv = ok && ties == 1;
          const uint64_t out = done[r] + (e - from[r]);
          if (eidx) {
            eidx[out] = ok ? (uint32_t)idx : 0xFFFFFFFFu;
            ehc[out] = (uint16_t)(h | (cur << hbits) | (triv ? 0x8000 : 0));
          } else {
            entries[out] = (ok ? idx : 0xFFFFFFFFull) | ((uint64_t)h << 32) | ((uint64_t)cur << 48) |
                           (triv ? (1ull << 63) : 0ull);
          }
        }
      }
      __syncthreads();
      for (int r = threadIdx.x; r < n; r += blockDim.x) done[r] += from[r + 1] - from[r];
    }
    __syncthreads();
  }
}

// ---- orbit search for arbitrary labels (test / export entry point) ---------
template <typename W, int GW, bool PLAIN, bool TABS>
__global__ void __launch_bounds__(kOrbitThreads) k_canon_labels(SecArgs a, const dev::RankWord* __restrict__ ranks,
                                                          const uint64_t* __restrict__ labels, int64_t n,
                                                          uint64_t* __restrict__ rep_out, int32_t* __restrict__ h_out,
                                                          int64_t* __restrict__ idx_out) {
  extern __shared__ uint64_t smem_raw[];
  const uint64_t* cnt;
  const dev::Orbit<W, GW, PLAIN> o = stage_orbit<W, GW, PLAIN, TABS>(a, smem_raw, cnt);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t n_iter = (n + stride - 1) / stride;
  for (int64_t it = 0; it < n_iter; ++it) {
    const int64_t i = it * stride + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = i < n;
    uint64_t lab = live ? labels[i] : 0;
    // Eq. (2) label -> packed digits
    W x = 0;
    int sum = 0;
    bool in_range = true;
    {
      uint64_t y = lab;
      for (int k = 0; k < a.N; ++k) {
        int dg = (int)(y % (uint64_t)a.d);
        y /= (uint64_t)a.d;
        x |= W(dg) << (k * a.b);
        sum += dg;
      }
      in_range = (y == 0) && (sum == a.A);
    }
    W r;
    int h, ties;
    dev::orbit_min<W, GW, PLAIN>(x, live, o, r, h, ties);
    if (live) {
      uint64_t idx = 0;
      bool ok = in_range && lookup<W>(r, a, ranks, cnt, idx);
      // packed -> Eq. (2)
      uint64_t outlab = 0;
      const W mask = (W(1) << a.b) - 1;
      for (int k = a.N - 1; k >= 0; --k) outlab = outlab * (uint64_t)a.d + (uint64_t)dev::digit(r, k, a.b, mask);
      rep_out[i] = in_range ? outlab : 0;
      h_out[i] = in_range ? h : -1;
      idx_out[i] = ok ? (int64_t)idx : -1;
    }
  }
}

unsigned grid_for(uint64_t n, int threads = kThreads, unsigned cap = 65536u * 4) {
  uint64_t g = (n + threads - 1) / threads;
  if (g < 1) g = 1;
  return (unsigned)std::min<uint64_t>(g, cap);
}

constexpr size_t kLdsLimit = 65536;
// dynamic LDS that leaves three workgroups of kOrbitThreads to a CU
constexpr size_t kLdsSoft = 36 * 1024;

// One launch of an orbit-search kernel template K<W, GW, PLAIN, TABS>.
#define FTLM_LAUNCH_ORBIT(K, s, static_lds, grid, st, a, ...)                                                  \
  {                                                                                                            \
    const OrbitLds ol = orbit_lds(s, kLdsSoft, kLdsLimit - (static_lds));                                      \
    (a).n_lds = ol.n_lds;                                                                                      \
    FTLM_DISPATCH_ORBIT((s).wide, (s).plain(), (s).gw, {                                                                    \
      if (ol.tabs)                                                                                             \
        hipLaunchKernelGGL((K<W, GW, PLAIN, true>), dim3(grid), dim3(kOrbitThreads), ol.bytes, st, a, __VA_ARGS__);   \
      else                                                                                                     \
        hipLaunchKernelGGL((K<W, GW, PLAIN, false>), dim3(grid), dim3(kOrbitThreads), ol.bytes, st, a, __VA_ARGS__);  \
    });                                                                                                        \
    FTLM_HIP(hipGetLastError());                                                                               \
  }

void orbit_args(const Sector& s, SecArgs& a) {
  a.mask = s.d_mask();
  a.img = s.d_img();
  a.split = s.d_split();
  a.nH = s.fac_nH;
  a.nT = s.fac_nT;
  a.nch = s.nch;
  a.NC = s.NC;
  a.cnt = s.d_cnt.p;
  a.cnt_stride = s.cnt_stride;
  a.N = s.N;
  a.b = s.bits;
  a.d = s.d;
  a.A = s.A;
  a.G = s.G->order;
  a.zf = s.zflip ? 1 : 0;
  a.full = s.full;
  a.D_M = s.D_M;
  a.n_words = s.n_words;
  a.n_reps = s.n_reps;
  // the sites that some element moves to the highest one
  std::vector<char> reach(s.N, 0);
  for (int g = 0; g < s.G->order; ++g)
    for (int k = 0; k < s.N; ++k)
      if (s.G->perms[(size_t)g * s.N + k] == s.N - 1) reach[k] = 1;
  a.transitive = std::count(reach.begin(), reach.end(), 1) == s.N;
}

}  // namespace

// Mask positions are read by every search, so at least two stay in LDS; the
// counts and image tables (read once or twice per search, at lane-dependent
// rows) join them where both fit; more positions take what is left up to the
// soft limit, which keeps three workgroups on a CU.
OrbitLds orbit_lds(const Sector& s, size_t soft, size_t limit) {
  OrbitLds o;
  const size_t pos = (size_t)s.NC * 16 * s.gw * 8;
  const size_t tabs = (size_t)(s.N + 1) * s.cnt_stride * 8 + s.img_bytes;
  o.tabs = tabs + 2 * pos <= limit;
  const size_t rest = o.tabs ? tabs : 0;
  const size_t room = std::max(std::min(soft, limit), std::min(limit, rest + 4 * pos));
  o.n_lds = room > rest ? (int)std::min<size_t>((size_t)s.N, (room - rest) / pos) : 0;
  o.bytes = rest + (size_t)o.n_lds * pos;
  return o;
}

std::shared_ptr<Sector> build_sector(const ftlm_cluster* cl, std::shared_ptr<const Group> G, int two_M,
                                     const ftlm_opts* opts) {
  if (!cl || !G) fail(FTLM_ERR_INVALID_ARG, "null cluster or group");
  auto S = std::make_shared<Sector>();
  Sector& s = *S;
  s.G = G;
  s.N = cl->N;
  s.two_s = cl->two_s;
  s.two_M = two_M;
  if (s.N != G->N) fail(FTLM_ERR_INVALID_ARG, "cluster N differs from the group's N");
  if (s.two_s < 1 || s.two_s > 62) fail(FTLM_ERR_INVALID_ARG, "two_s must be in 1..62");
  if (G->order > 1024) fail(FTLM_ERR_GROUP_TOO_LARGE, "sector tables support |G| <= 1024");
  s.d = s.two_s + 1;
  s.bits = 0;
  while ((1 << s.bits) < s.d) ++s.bits;
  if (s.N * s.bits > 64) fail(FTLM_ERR_UNSUPPORTED, "packed labels need more than 64 bits");
  s.wide = s.N * s.bits > 32;
  s.nch = (s.N * s.bits + 3) / 4;
  s.NC = (s.N + 3) / 4;
  s.gw = orbit_words(G->order);
  // spin flip (G x Z2) at M = 0
  s.zflip = opts && opts->spin_flip;
  if (s.zflip && two_M != 0) fail(FTLM_ERR_INVALID_ARG, "the spin flip resolves only the M = 0 sector");
  s.full = 0;
  for (int k = 0; k < s.N; ++k) s.full |= (uint64_t)(s.d - 1) << (k * s.bits);
  s.gorder = G->order * (s.zflip ? 2 : 1);
  if (cl->nbonds < 0 || (cl->nbonds > 0 && !cl->bonds)) fail(FTLM_ERR_INVALID_ARG, "bad bond list");
  if (cl->nbonds > 16000) fail(FTLM_ERR_INVALID_ARG, "too many bonds");
  s.nbonds = cl->nbonds;
  s.bonds.assign(cl->bonds, cl->bonds + 2 * (size_t)cl->nbonds);
  s.J.resize(s.nbonds);
  std::map<std::pair<int, int>, double> bondmap;
  for (int b = 0; b < s.nbonds; ++b) {
    int i = s.bonds[2 * b], j = s.bonds[2 * b + 1];
    if (i < 0 || j < 0 || i >= s.N || j >= s.N || i == j) fail(FTLM_ERR_INVALID_ARG, "bond site out of range");
    s.J[b] = cl->J ? cl->J[b] : 1.0;
    bondmap[{std::min(i, j), std::max(i, j)}] += s.J[b];
  }
  // bond invariance under every group element (weighted, Section 3)
  for (int g = 0; g < G->order; ++g) {
    const int32_t* p = &G->perms[(size_t)g * s.N];
    for (auto& kv : bondmap) {
      int a = p[kv.first.first], c = p[kv.first.second];
      auto it = bondmap.find({std::min(a, c), std::max(a, c)});
      if (it == bondmap.end() || std::fabs(it->second - kv.second) > 1e-12 * std::max(1.0, std::fabs(kv.second)))
        fail(FTLM_ERR_BONDS_NOT_INVARIANT, "bond list is not invariant under the group");
    }
  }
  {
    uint64_t h = fnv1a(&s.N, sizeof(s.N));
    h = fnv1a(&s.two_s, sizeof(s.two_s), h);
    h = fnv1a(s.bonds.data(), s.bonds.size() * sizeof(int32_t), h);
    h = fnv1a(s.J.data(), s.J.size() * sizeof(double), h);
    h = fnv1a(G->perms.data(), G->perms.size() * sizeof(int32_t), h);
    const int zf = s.zflip ? 1 : 0;
    s.cluster_hash = fnv1a(&zf, sizeof(zf), h);
  }
  // digit-sum counts
  const int Amax = s.N * (s.d - 1);
  s.cnt_stride = Amax + 1;
  s.cnt.assign((size_t)(s.N + 1) * s.cnt_stride, 0);
  s.cnt[0] = 1;
  for (int k = 1; k <= s.N; ++k)
    for (int v = 0; v <= Amax; ++v) {
      unsigned __int128 c = 0;
      for (int a = 0; a < s.d && a <= v; ++a) c += s.cnt[(size_t)(k - 1) * s.cnt_stride + v - a];
      s.cnt[(size_t)k * s.cnt_stride + v] = (uint64_t)c;
    }
  const int A2 = s.N * s.two_s + two_M;
  hipStream_t st = tl_alloc_stream;  // the caller's build stream, or the null stream
  if (A2 % 2 != 0 || A2 < 0 || A2 / 2 > Amax) {
    s.A = 0;
    s.D_M = 0;
  } else {
    s.A = A2 / 2;
    s.D_M = s.cnt[(size_t)s.N * s.cnt_stride + s.A];
  }
  s.n_words = (s.D_M + 63) / 64;
  // orbit-search tables (dev::Orbit): candidate masks, image tables of all |G|
  // elements when these take at most 16 KiB and of G = T H with |H| + |T|
  // tables otherwise, and each element's (t, h)
  const int G_ = G->order;
  const size_t wbytes = s.wide ? 8 : 4;
  std::vector<uint8_t> tab_host;                 // host copies of tables in flight to the device
  std::vector<double>& fac = s.fac;
  fac.assign(2 * s.d * s.d, 0.0);
  {
    const int max_plain = (int)std::max<size_t>(1, 16384 / ((size_t)s.nch * 16 * wbytes));
    const Factorization fz = factor_group(*G, max_plain);
    s.fac_nH = (int)fz.H.size();
    s.fac_nT = (int)fz.T.size();
    const size_t rows = (size_t)s.fac_nH + s.fac_nT;
    s.mask_words = (size_t)s.N * s.NC * 16 * s.gw;
    s.img_bytes = (rows * s.nch * 16 * wbytes + 7) / 8 * 8;
    std::vector<uint8_t> bytes(s.mask_words * 8 + s.img_bytes + (size_t)G_ * 4, 0);
    uint64_t* mask = (uint64_t*)bytes.data();
    for (int g = 0; g < G_; ++g)
      for (int site = 0; site < s.N; ++site) {
        // site `site` goes to position p (sites from the highest down)
        const int p = s.N - 1 - G->perms[(size_t)g * s.N + site];
        uint64_t* m = mask + ((size_t)p * s.NC + site / 4) * 16 * s.gw;
        for (int v = 0; v < 16; ++v)
          if ((v >> (site % 4)) & 1) m[(size_t)v * s.gw + g / 64] |= 1ull << (g % 64);
      }
    uint8_t* img_at = bytes.data() + s.mask_words * 8;
    for (size_t row = 0; row < rows; ++row) {
      const int g = row < (size_t)s.fac_nH ? fz.H[row] : fz.T[row - s.fac_nH];
      const int32_t* p = &G->perms[(size_t)g * s.N];
      for (int c = 0; c < s.nch; ++c)
        for (int v = 0; v < 16; ++v) {
          uint64_t img = 0;
          for (int t = 0; t < 4; ++t) {
            if (!((v >> t) & 1)) continue;
            int bit = 4 * c + t;
            if (bit >= s.N * s.bits) continue;
            int site = bit / s.bits, sub = bit % s.bits;
            img |= 1ull << (p[site] * s.bits + sub);
          }
          const size_t at = ((row * s.nch + c) * 16 + v) * wbytes;
          if (s.wide) {
            std::memcpy(img_at + at, &img, 8);
          } else {
            const uint32_t i32 = (uint32_t)img;
            std::memcpy(img_at + at, &i32, 4);
          }
        }
    }
    uint32_t* split = (uint32_t*)(img_at + s.img_bytes);
    for (int t = 0; t < s.fac_nT; ++t)
      for (int h = 0; h < s.fac_nH; ++h) split[fz.gidx[(size_t)t * s.fac_nH + h]] = (uint32_t)t << 16 | (uint32_t)h;
    s.d_tab.alloc((bytes.size() + 7) / 8);
    FTLM_HIP(hipMemcpyAsync(s.d_tab.p, bytes.data(), bytes.size(), hipMemcpyHostToDevice, st));
    tab_host.swap(bytes);  // kept until the stream has passed the copy
  }
  // the small tables go up without a wait each; the first synchronization
  // below (after the representative count) covers them
  s.d_cnt.upload_async(s.cnt, st);
  s.d_bonds.upload_async(s.bonds, st);
  s.d_J.upload_async(s.J, st);
  {
    const double sp = 0.5 * s.two_s, ss = sp * (sp + 1);
    for (int ai = 0; ai < s.d; ++ai)
      for (int aj = 0; aj < s.d; ++aj) {
        double mi = ai - sp, mj = aj - sp;
        // sign 0: s_i^+ s_j^-; sign 1: s_i^- s_j^+ (Eq. 3 with J = 1)
        fac[(0 * s.d + ai) * s.d + aj] = 0.5 * std::sqrt(std::max(0.0, ss - mi * (mi + 1))) *
                                         std::sqrt(std::max(0.0, ss - mj * (mj - 1)));
        fac[(1 * s.d + ai) * s.d + aj] = 0.5 * std::sqrt(std::max(0.0, ss - mi * (mi - 1))) *
                                         std::sqrt(std::max(0.0, ss - mj * (mj + 1)));
      }
  }
  SecArgs a{};
  orbit_args(s, a);
  FlipArgs f{s.d_bonds.p, s.d_J.p, s.nbonds};

  if (s.D_M == 0) {
    s.n_reps = 0;
    s.d_row_ptr.alloc(1);
    FTLM_HIP(hipMemsetAsync(s.d_row_ptr.p, 0, sizeof(uint64_t), st));
    FTLM_HIP(hipStreamSynchronize(st));
    return S;
  }
  const int64_t limit = opts ? opts->hbm_limit_bytes : 0;
  // representatives
  s.d_ranks.alloc(s.n_words);
  // one thread per word once the words fill the device (256 CUs x 1,024
  // threads); below that one wave per word: a sector of 924 states (15 words)
  // took 200 us with 15 threads stepping through 64 labels each
  const bool by_wave = s.n_words < (1ull << 18);
  {
    const OrbitLds ol = orbit_lds(s, kLdsSoft, kLdsLimit);
    a.n_lds = ol.n_lds;
    const unsigned grid = grid_for(by_wave ? s.n_words * 64 : s.n_words, kOrbitThreads, 8192);
    FTLM_DISPATCH_ORBIT(s.wide, s.plain(), s.gw, {
      if (by_wave && ol.tabs)
        hipLaunchKernelGGL((k_enum<W, GW, PLAIN, true, true>), dim3(grid), dim3(kOrbitThreads), ol.bytes, st, a, s.d_ranks.p);
      else if (by_wave)
        hipLaunchKernelGGL((k_enum<W, GW, PLAIN, false, true>), dim3(grid), dim3(kOrbitThreads), ol.bytes, st, a, s.d_ranks.p);
      else if (ol.tabs)
        hipLaunchKernelGGL((k_enum<W, GW, PLAIN, true, false>), dim3(grid), dim3(kOrbitThreads), ol.bytes, st, a, s.d_ranks.p);
      else
        hipLaunchKernelGGL((k_enum<W, GW, PLAIN, false, false>), dim3(grid), dim3(kOrbitThreads), ol.bytes, st, a, s.d_ranks.p);
    });
    FTLM_HIP(hipGetLastError());
  }
  {
    const uint64_t tiles = (s.n_words + kRankTile - 1) / kRankTile;
    DevBuf<uint64_t> tile_base;
    tile_base.alloc(tiles);
    hipLaunchKernelGGL(k_rank_tiles, dim3((unsigned)tiles), dim3(kThreads), 0, st, s.d_ranks.p, s.n_words, tile_base.p);
    FTLM_HIP(hipGetLastError());
    uint64_t total = 0;
    scan_exclusive_u64(tile_base.p, tile_base.p, tiles, &total, st);
    if (total >= 0xFFFFFFFFull) fail(FTLM_ERR_UNSUPPORTED, "more than 2^32 - 1 representatives");
    s.n_reps = total;
    hipLaunchKernelGGL(k_rank_bases, dim3((unsigned)tiles), dim3(kThreads), 0, st, s.d_ranks.p, s.n_words, tile_base.p);
    FTLM_HIP(hipGetLastError());
    FTLM_HIP(hipStreamSynchronize(st));
  }
  a.n_reps = s.n_reps;
  s.d_reps.alloc(s.n_reps);
  if (s.wide)
    hipLaunchKernelGGL((k_extract<uint64_t>), dim3(grid_for(s.n_words)), dim3(kThreads), 0, st, a, s.d_ranks.p,
                       s.d_reps.p);
  else
    hipLaunchKernelGGL((k_extract<uint32_t>), dim3(grid_for(s.n_words)), dim3(kThreads), 0, st, a, s.d_ranks.p,
                       s.d_reps.p);
  FTLM_HIP(hipGetLastError());

  // stabilizers: flags -> compaction -> host interning in first-appearance order
  {
    DevBuf<uint64_t> pos;
    pos.alloc(s.n_reps + 1);
    FTLM_HIP(hipMemsetAsync(pos.p + s.n_reps, 0, sizeof(uint64_t), st));
    FTLM_LAUNCH_ORBIT(k_stab_flag, s, 0, grid_for(s.n_reps, kOrbitThreads, 8192), st, a, s.d_reps.p, pos.p);
    uint64_t n_nt = 0;
    scan_exclusive_u64(pos.p, pos.p, s.n_reps + 1, &n_nt, st);
    const int mw = (s.gorder + 63) / 64;
    DevBuf<uint64_t> masks, idx;
    masks.alloc(std::max<uint64_t>(n_nt, 1) * mw);
    idx.alloc(std::max<uint64_t>(n_nt, 1));
    if (n_nt) {
      FTLM_LAUNCH_ORBIT(k_stab_mask, s, 0, grid_for(s.n_reps, kOrbitThreads, 8192), st, a, s.d_reps.p, pos.p, mw, masks.p,
                        idx.p);
    }
    DevBuf<unsigned long long> first;
    first.alloc(1);
    unsigned long long init = ~0ull;
    FTLM_HIP(hipMemcpyAsync(first.p, &init, sizeof(init), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_first_trivial, dim3(grid_for(s.n_reps)), dim3(kThreads), 0, st, pos.p, s.n_reps, first.p);
    FTLM_HIP(hipGetLastError());
    std::vector<uint64_t> h_masks(n_nt * mw), h_idx(n_nt);
    if (n_nt) {
      FTLM_HIP(hipMemcpyAsync(h_masks.data(), masks.p, n_nt * mw * 8, hipMemcpyDeviceToHost, st));
      FTLM_HIP(hipMemcpyAsync(h_idx.data(), idx.p, n_nt * 8, hipMemcpyDeviceToHost, st));
    }
    unsigned long long first_trivial = 0;
    FTLM_HIP(hipMemcpyAsync(&first_trivial, first.p, sizeof(first_trivial), hipMemcpyDeviceToHost, st));
    FTLM_HIP(hipStreamSynchronize(st));
    std::map<std::vector<uint64_t>, uint16_t> ids;
    std::vector<uint64_t> trivial_mask(mw, 0);
    trivial_mask[0] = 1;  // identity only
    std::vector<uint16_t> ids_nt(std::max<uint64_t>(n_nt, 1), 0);
    auto intern = [&](const std::vector<uint64_t>& m) -> uint16_t {
      auto it = ids.find(m);
      if (it != ids.end()) return it->second;
      if (ids.size() >= 65535) fail(FTLM_ERR_UNSUPPORTED, "too many distinct stabilizers");
      uint16_t id = (uint16_t)ids.size();
      ids.emplace(m, id);
      std::vector<int32_t> el;
      for (int g = 0; g < s.gorder; ++g)
        if ((m[g / 64] >> (g % 64)) & 1) el.push_back(g);
      s.stab_elems.push_back(el);
      s.stab_size.push_back((uint16_t)el.size());
      return id;
    };
    const bool has_trivial = first_trivial != ~0ull;
    bool trivial_done = !has_trivial;
    uint16_t trivial_id = 0;
    for (uint64_t q = 0; q < n_nt; ++q) {
      if (!trivial_done && h_idx[q] > first_trivial) {
        trivial_id = intern(trivial_mask);
        trivial_done = true;
      }
      std::vector<uint64_t> m(h_masks.begin() + q * mw, h_masks.begin() + (q + 1) * mw);
      ids_nt[q] = intern(m);
    }
    if (!trivial_done) trivial_id = intern(trivial_mask);
    s.trivial_sid = trivial_id;
    s.n_stab = (int32_t)ids.size();
    // representatives per stabilizer id (block dimensions follow from them)
    s.stab_count.assign(s.n_stab, 0);
    s.stab_count[trivial_id] += s.n_reps - n_nt;
    for (uint64_t q = 0; q < n_nt; ++q) s.stab_count[ids_nt[q]] += 1;
    DevBuf<uint16_t> d_ids;
    d_ids.upload_async(ids_nt, st);
    s.d_stab_id.alloc(s.n_reps);
    hipLaunchKernelGGL(k_assign_stab, dim3(grid_for(s.n_reps)), dim3(kThreads), 0, st, pos.p, s.n_reps, d_ids.p,
                       trivial_id, s.d_stab_id.p);
    FTLM_HIP(hipGetLastError());
    FTLM_HIP(hipStreamSynchronize(st));  // ids_nt and the temporaries go out of scope
  }

  // diagonal energies and the entry table
  s.d_ediag.alloc(s.n_reps);
  s.d_row_ptr.alloc(s.n_reps + 1);
  FTLM_HIP(hipMemsetAsync(s.d_row_ptr.p + s.n_reps, 0, sizeof(uint64_t), st));
  if (s.wide)
    hipLaunchKernelGGL((k_entry_count<uint64_t>), dim3(grid_for(s.n_reps)), dim3(kThreads), 0, st, a, f, s.d_reps.p,
                       s.d_row_ptr.p, s.d_ediag.p);
  else
    hipLaunchKernelGGL((k_entry_count<uint32_t>), dim3(grid_for(s.n_reps)), dim3(kThreads), 0, st, a, f, s.d_reps.p,
                       s.d_row_ptr.p, s.d_ediag.p);
  FTLM_HIP(hipGetLastError());
  uint64_t n_ent = 0;
  scan_exclusive_u64(s.d_row_ptr.p, s.d_row_ptr.p, s.n_reps + 1, &n_ent, st);
  s.n_entries = n_ent;
  // Entry format: 6 bytes (u32 target index + u16 holding h, the flip id and
  // the trivial-target bit) when they fit in 16 bits, 8 bytes (one u64:
  // idx | h << 32 | flip << 48 | trivial << 63) otherwise.
  {
    int hb = 1, cb = 1;
    while ((1 << hb) < s.gorder) ++hb;
    while ((1 << cb) < 2 * s.nbonds) ++cb;
    s.ent_hbits = hb;
    const bool compact_ok = hb + cb <= 15;
    const int fmt = opts ? opts->entry_format : FTLM_ENTRIES_AUTO;
    if (fmt < FTLM_ENTRIES_AUTO || fmt > FTLM_ENTRIES_COMPACT) fail(FTLM_ERR_INVALID_ARG, "bad entry_format");
    if (fmt == FTLM_ENTRIES_COMPACT && !compact_ok)
      fail(FTLM_ERR_UNSUPPORTED, "compact entries need |G| and the flip count to fit 15 bits");
    size_t free_b = 0, total_b = 0;
    FTLM_HIP(hipMemGetInfo(&free_b, &total_b));
    if (fmt == FTLM_ENTRIES_AUTO)
      s.entry_bytes = (compact_ok && (double)n_ent * 8.0 > (double)free_b / 4.0) ? 6 : 8;
    else
      s.entry_bytes = fmt == FTLM_ENTRIES_COMPACT ? 6 : 8;
  }
  int mode = opts ? opts->hv_mode : FTLM_HV_AUTO;
  if (mode == FTLM_HV_AUTO) {
    // the table must leave a third of the free memory for blocks and vectors
    size_t free_b = 0, total_b = 0;
    FTLM_HIP(hipMemGetInfo(&free_b, &total_b));
    mode = ((double)n_ent * s.entry_bytes <= (double)free_b * 2.0 / 3.0) ? FTLM_HV_ENTRIES : FTLM_HV_ONTHEFLY;
  }
  if (limit > 0 && (int64_t)(s.limited_bytes() + (mode == FTLM_HV_ENTRIES ? n_ent * s.entry_bytes : 0)) > limit)
    fail(FTLM_ERR_OUT_OF_MEMORY, "sector tables exceed the HBM limit");
  s.hv_mode = mode;
  if (mode == FTLM_HV_ENTRIES && n_ent) {
    if (s.entry_bytes == 6) {
      s.d_eidx.alloc(n_ent);
      s.d_ehc.alloc(n_ent);
    } else {
      s.d_entries.alloc(n_ent);
    }
    // representatives per workgroup: about two full rounds of its lanes (7%
    // under, as row lengths vary), fewer where the sector would leave the
    // device idle
    const double per_rep = std::max(1.0, (double)n_ent / (double)s.n_reps);
    const int64_t list_cap = std::max<int64_t>(1, kFillList / std::max(1, 2 * s.nbonds));
    const int rb = (int)std::max<int64_t>(
        1, std::min<int64_t>({(int64_t)kFillReps, list_cap, (int64_t)(0.93 * 2 * kOrbitThreads / per_rep),
                              (int64_t)(s.n_reps / 512)}));
    const size_t fill_lds = kFillList * 4 + (kFillReps + 1) * 4 + kFillReps * 8 + 64;
    FTLM_LAUNCH_ORBIT(k_entry_fill, s, fill_lds, grid_for((s.n_reps + rb - 1) / rb, 1, 8192), st, a, f, rb, s.d_reps.p,
                      s.d_row_ptr.p, s.d_ranks.p, s.d_entries.p, s.d_eidx.p, s.d_ehc.p, s.ent_hbits);
  }
  FTLM_HIP(hipStreamSynchronize(st));
  return S;
}

void sector_canonicalize(const Sector& s, const uint64_t* labels, int64_t n, uint64_t* rep, int32_t* h,
                         int64_t* index, hipStream_t st) {
  if (n < 0 || (n > 0 && (!labels || !rep || !h || !index))) fail(FTLM_ERR_INVALID_ARG, "bad canonicalize arguments");
  if (n == 0) return;
  // (an empty sector: nothing is in range; the search for rep and h still runs)
  SecArgs a{};
  orbit_args(s, a);
  FTLM_LAUNCH_ORBIT(k_canon_labels, s, 0, grid_for((uint64_t)n, kOrbitThreads, 8192), st, a, s.d_ranks.p, labels, n, rep, h, index);
}

std::vector<uint64_t> sector_export_labels(const Sector& s) {
  std::vector<uint64_t> packed = s.d_reps.download();
  if (s.d == (1 << s.bits)) return packed;  // packed digits are the Eq. (2) label
  const uint64_t mask = (1ull << s.bits) - 1;
  for (auto& x : packed) {
    uint64_t lab = 0;
    for (int k = s.N - 1; k >= 0; --k) lab = lab * (uint64_t)s.d + ((x >> (k * s.bits)) & mask);
    x = lab;
  }
  return packed;
}

}  // namespace ftlm
