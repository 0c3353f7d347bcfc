// H.V kernel template (paper Eqs. 15-16) shared by the per-dimension
// instantiation units hv_dg*.hip.  The host side (table layout, launch shape,
// dispatch) is in hv.hip.
//
// Gather form (from Eq. 15 with U(h) a = r for the flipped state
// a = flip_e(p) of output representative p):
//
//   Y[p] = E_diag(p) X[p]
//        + sqrt(L_p) V_p^T  sum_e  c_e(p) / sqrt(L_r)  rho(h)^T  V_r X[r]
//
// with c_e(p) the Eq. (3) coefficient of flip e evaluated on p's digits and
// L = |G| / |Stab|.
//
// Lane layout: a group of GL lanes owns one output representative; lane g of
// the group holds VPL vector columns (see HvVariant).  Every output element
// is written by exactly one lane and the sum over flips runs in a fixed
// order, so results are deterministic and do not depend on how many vectors
// share the launch.  Small GL with VPL vectors per lane keeps 64/GL
// representatives per wave in flight, which is what hides the latency of the
// dependent loads (flip -> target -> X rows): a chunk of GL flips is fetched
// and decoded (target offset, coefficient) with one flip per lane and
// exchanged by lane shuffles, then each flip's rows of X[r] are gathered for
// all VPL vectors.  rho^T, V_S, the stabilizer data and the bond coefficients
// sit in LDS when they fit; when only V_S does not (many stabilizer types),
// the kernels keep the others in LDS and read V_S, needed only for
// non-trivial stabilizers, through the caches (VG; table-driven H.V only).
//
// What bounds it: the rate of 128-byte lines the device delivers for random
// slices, about 5.4e10 per second whether they come from HBM or the Infinity
// Cache, and the waves that can wait for them.  Figures (MI355X, before ->
// after one decode per flip, four waves, adjacent columns in block rows and
// sweeps on one XCD; icosidodecahedron M = 0, 4.02e7 flips): plain product,
// d = 5, 24 FP32 columns 3.51 -> 2.71 ms, d = 3 3.32 -> 1.69 ms; one FP64
// column, d = 5 1.33 -> 0.62 ms; two FP32 columns 0.91 -> 0.67 ms; 24 FP16
// columns, d = 3 3.64 -> 1.40 ms; with the Lanczos epilogue in padded rows,
// 24 FP32 columns, d = 5 3.34 -> 2.85 ms, d = 4 2.54 -> 2.15, d = 3 1.98 ->
// 1.72 ms, d = 1 0.85 -> 0.75 ms.
// Arithmetic is FP64; FP32 and FP16 storage round once on the store.
//
// Flips come from the sector's entry table (target index, h, flip id; built
// once per sector and shared by all irreps) or are found on the fly (flip,
// orbit search over the group, rank lookup; the search's vector instructions
// bound it: 4.6e5 representatives of the icosidodecahedron at 2M = 8, d = 4,
// 7 FP32 vectors 1.55 ms, 9.15 ms with a walk over the group's images that
// also searched for inadmissible flips).
//
// Lanczos epilogue (partials != nullptr): the kernel writes
// w = s_j (H q_j) - bs_j q_prev over q_prev (Y holds q_prev on entry) and
// per-workgroup FP64 partial sums of q_j . w (w as stored).  With a shift
// e (eshift) the kernel applies H - e instead of H (the Chebyshev recursion
// of the kernel polynomial method); e = 0 otherwise.
#pragma once

#include <algorithm>
#include <cmath>

#include "device.h"
#include "dispatch.h"
#include "hv_rows.h"
#include "internal.h"

namespace ftlm {
namespace hvk {

constexpr int kThreads = 256;
// Waves per SIMD asked of the register allocator, by the accumulator's DG x
// VPL doubles.  The gathers' latency is hidden by other waves, so four waves
// with a few spilled registers beat three without (icosidodecahedron H_g, 24
// FP32 columns, 15 doubles: 2.96 against 3.10 ms); at 25 to 30 doubles three
// (six FP16 columns, d = 5: 2.50 against 2.73 ms with two); at 18 and 24 the
// spills cost more than the wave gives (1.40 against 1.44 ms).
constexpr int hv_waves(int width) { return width <= 15 ? 4 : width >= 25 && width <= 30 ? 3 : 1; }
// The general kernels: their clamped gathers need the registers from 11 on
// (d = 8, square 6 x 6; d = 3, four vectors on the fly: 324 us, 387 with four
// waves).
constexpr int hv_waves_general(int width) { return width <= 10 ? 4 : 1; }
constexpr uint64_t kOffMask = (1ull << 48) - 1;
constexpr uint32_t kInvalid = 0xffffffffu;

template <typename T>
struct HvArgs {
  const uint64_t* reps;
  const uint64_t* row_ptr;
  const uint64_t* entries;   // 8-byte entries, or
  const uint32_t* eidx;      // the 6-byte split form (eidx != nullptr)
  const uint16_t* ehc;
  int hbits;
  // vector layout: pad == 0: block rows (representative i at meta offset);
  // pad != 0: padded rows, representative i at dev::padded_row (i * dstride,
  // dstride = d_Gamma, or packed rpl to a line of rpline rows), and a
  // target's stabilizer id comes from the entry's trivial bit or sid[]
  int pad, dstride, triv_sid;
  uint32_t rpl, rpline;
  uint64_t rows;        // rows of X and Y
  const uint32_t* lack; // block rows: rows missing before every 32nd representative (Block::d_lack), or null
  const uint16_t* sid;
  const uint64_t* meta;
  const double* ediag;
  // small tables (Block::d_small): bytes to stage (from o_stab on where the
  // matrices stay in memory), where they go in dynamic LDS (behind the orbit
  // search's), offsets of the tables within
  const uint8_t* small;
  uint32_t small_bytes, o_small, o_stab, o_J, o_fac, o_bonds, o_V;
  int b, dloc, nbonds;
  uint64_t n_reps;
  const T* X;
  T* Y;
  int64_t ld;
  int nvec, GL, log2GL, tile_w;
  uint32_t sweep_w, sweep_k;  // workgroups and rounds of one sweep (k_hv); sweep_k = 0: workgroups in order
  int zero;  // always 0 (see the non-trivial stabilizer branch)
  // on-the-fly search (dev::Orbit; LDS: n_lds mask positions, counts, images)
  const uint64_t* mask;
  const void* img;
  const uint32_t* split;
  int n_lds, nH, nT, nch, NC;
  const uint64_t* cnt;
  const dev::RankWord* ranks;
  int cnt_stride, N, A_tot;
  int Gbase, zf;        // |G| and the spin flip of the on-the-fly search
  uint64_t full;
  double fpar;          // flip parity: element (g, F) acts as fpar * rho(g)
  uint64_t D_M;
  // Lanczos epilogue
  const double* scal;
  double* partials;
  double eshift;        // H - eshift is applied (0 except for the Chebyshev recursion)
};

// On-the-fly kernels: NCH is 8 (32-bit labels) or 16, and NCH - 1 marks the
// kernels of plain s = 1/2 sectors (dev::Orbit's PLAIN).
template <int NCH, int GW>
constexpr bool kPlain = GW > 0 && (NCH & 1);

struct LaunchCfg {
  dim3 grid;
  size_t shm;
  bool otf, lds_tab, slds, wide, plain;  // lds_tab: counts and images of the search in LDS
  int var;      // HvVariant
  bool vg;      // all small tables but V_S in LDS (table-driven H.V)
  int gw, vpl;
};

template <typename W>
__device__ __forceinline__ bool lookup_rep(W r, int N, int b, int d, int A, const uint64_t* cnt, int stride,
                                           uint64_t D_M, const dev::RankWord* ranks, uint64_t& idx) {
  const uint64_t rk = dev::sector_rank<W>(r, N, b, d, A, cnt, stride);
  if (rk >= D_M) return false;
  const dev::RankWord w = ranks[rk >> 6];
  const int k = (int)(rk & 63);
  const uint64_t bits = dev::rank_bits(w);
  idx = w.base + (uint64_t)__popcll(bits & ((1ull << k) - 1));
  return (bits >> k) & 1;
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src) {
  uint32_t lo = __shfl((unsigned)(v & 0xffffffffu), src);
  uint32_t hi = __shfl((unsigned)(v >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}

// Swap a value with the other lane of its lane pair (lanes 2i and 2i + 1):
// DPP quad permutation [1, 0, 3, 2], a register move with no LDS traffic.
__device__ __forceinline__ uint32_t pair_swap_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);
}
__device__ __forceinline__ float pair_swap(float v) { return __uint_as_float(pair_swap_u32(__float_as_uint(v))); }
__device__ __forceinline__ double pair_swap(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint64_t r = (uint64_t)pair_swap_u32((uint32_t)u) | ((uint64_t)pair_swap_u32((uint32_t)(u >> 32)) << 32);
  return __longlong_as_double((long long)r);
}
__device__ __forceinline__ _Float16 pair_swap(_Float16 v) {
  return __builtin_bit_cast(_Float16, (uint16_t)pair_swap_u32(__builtin_bit_cast(uint16_t, v)));
}

template <typename E>
__device__ __forceinline__ const E* stage(const E* src, uint32_t count, char* dst_bytes) {
  E* dst = (E*)dst_bytes;
  for (uint32_t i = threadIdx.x; i < count; i += blockDim.x) dst[i] = src[i];
  return dst;
}

struct HvTabs {
  const double* rhoT;
  const double* Vt;
  const double* stabf;
  const double* Jb;
  const double* fac;
  const int32_t* bonds;
};

// The small tables at `base` (LDS or memory); V possibly elsewhere.
template <typename T>
__device__ __forceinline__ HvTabs small_tabs(const HvArgs<T>& a, const uint8_t* base, const uint8_t* vbase) {
  return HvTabs{(const double*)base, (const double*)(vbase + a.o_V), (const double*)(base + a.o_stab),
                (const double*)(base + a.o_J), (const double*)(base + a.o_fac), (const int32_t*)(base + a.o_bonds)};
}

// Copies bytes (a multiple of 16) into LDS with eight 16-byte loads in flight
// per thread (with the kDeep ring, dodecahedron H_g at M = 0, 24 FP64 columns
// on 8 lanes: 45 -> 40 us).
__device__ __forceinline__ void stage_small(const uint8_t* src, uint32_t bytes, uint8_t* dst) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  const u4* s = (const u4*)src;
  u4* d = (u4*)dst;
  const uint32_t n = bytes / 16, step = blockDim.x;
  for (uint32_t i = threadIdx.x; i < n; i += 8 * step) {
    u4 v[8];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) v[u] = s[min(i + u * step, n - 1)];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u)
      if (i + u * step < n) d[i + u * step] = v[u];
  }
}

// Where the small tables are: all in LDS, all but V_S in LDS, the matrices in
// memory (the others in LDS all the same where they fit).
enum HvTables { kTabLds = 0, kTabV = 1, kTabMemory = 2 };

// use(i, row i) for the rows 0 .. N-1 of DG elements at(i, k), with A rows read
// ahead of the one in use and no more: left alone the compiler keeps whole
// matrices in registers that other waves need, or reads and waits element by
// element (fused jobs of 24 chains, d = 4 to 6: 1.2 to 1.6 times the time).
template <int N, int DG, int A, typename At, typename Use>
__device__ __forceinline__ void each_row(At at, Use use) {
  double r[A + 1][DG];
#pragma unroll
  for (int i = 0; i < A; ++i)
#pragma unroll
    for (int k = 0; k < DG; ++k) r[i][k] = i < N ? at(i, k) : 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + A < N) {
#pragma unroll
      for (int k = 0; k < DG; ++k) r[(i + A) % (A + 1)][k] = at(i + A, k);
    }
    use(i, r[i % (A + 1)]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The H.V over the representatives p = slot, slot + slot_stride, ... < p_end of
// one column tile: lane group of GL lanes per representative (see the file text).
// dot[j] accumulates q_j . w of this lane's column vcol + j * (column step).
// GW > 0: flips are found on the fly (orbit search with candidate sets of GW
// words; osearch, ocnt: its tables); GW = 0: flips come from the entry table.
template <typename T, int DG, int VPL, int GW, int NCH, int VAR = kGeneral, int TAB = kTabLds>
__device__ __forceinline__ void hv_pass(const HvArgs<T>& a, const HvTabs& tb,
                                        const dev::Orbit<word_t<NCH>, (GW > 0 ? GW : 1), kPlain<NCH, GW>>& osearch,
                                        const uint64_t* ocnt, int tile, uint64_t slot, uint64_t slot_stride, uint64_t p_end,
                                        double (&dot)[VPL], bool (&vok)[VPL], int& vcol) {
  using W = word_t<NCH>;
  constexpr bool OTF = GW > 0;
  constexpr bool ADJ = VAR != kGeneral;
  const bool EPI = a.partials != nullptr;
  const double* rhoT = tb.rhoT;
  const double* Vt = tb.Vt;
  const double* stabf = tb.stabf;
  const double* Jb = tb.Jb;
  const double* fac = tb.fac;
  const int32_t* bonds = tb.bonds;
  const int lane = threadIdx.x & 63;
  const int GL = VAR == kNarrow ? 1 : a.GL;
  const int lg = VAR == kNarrow ? 0 : lane & (GL - 1);
  const int gbase = lane - lg;
  // lane lg of the group owns columns vcol + j * vstep, those with vok[j]
  const int vstep = ADJ ? 1 : GL;
  vcol = lane_columns<VAR, VPL>(tile, a.tile_w, lg, GL, a.nvec, vok);
  bool full = true;
#pragma unroll
  for (int j = 0; j < VPL; ++j) full = full && vok[j];
  const SliceShape shape = slice_shape<VAR, VPL>(a.pad != 0, GL, lg, a.ld, a.nvec, vcol,
                                                 ((uintptr_t)a.X & (2 * sizeof(T) - 1)) == 0);
  const W lmask = (W(1) << a.b) - 1;
  const int ncand = 2 * a.nbonds;
#pragma unroll
  for (int j = 0; j < VPL; ++j) dot[j] = 0.0;

  for (uint64_t p = slot; p < p_end; p += slot_stride) {
    const uint64_t mp = a.meta[p];
    const int sp = (int)(mp >> 48);
    const int np_ = (int)stabf[4 * sp];
    if (np_ == 0) continue;
    const uint64_t offp = a.pad ? dev::padded_row((uint32_t)a.dstride, a.rpl, a.rpline, p) : (mp & kOffMask);
    const W plab = (W)a.reps[p];
    double acc[DG][VPL];
#pragma unroll
    for (int q = 0; q < DG; ++q)
#pragma unroll
      for (int j = 0; j < VPL; ++j) acc[q][j] = 0.0;

    // an entry (target index, h << 32, flip id << 48, trivial target << 63)
    auto load_entry = [&](uint64_t e) -> uint64_t {
      if (!a.eidx) return a.entries[e];
      const uint32_t hc = a.ehc[e];
      return (uint64_t)a.eidx[e] | ((uint64_t)(hc & ((1u << a.hbits) - 1)) << 32) |
             ((uint64_t)((hc & 0x7fffu) >> a.hbits) << 48) | ((uint64_t)(hc >> 15) << 63);
    };
    auto decode = [&](uint64_t ent) -> Flip {
      Flip f;
      const uint32_t idx = (uint32_t)(ent & 0xffffffffu);
      const bool triv = ent >> 63;
      f.c = 0.0;
      f.off = flip_word<VAR, DG>(offp, 0, false, a.pad != 0, a.rows, a.ld);
      f.info = 0;
      if (idx == kInvalid) return f;
      uint64_t row;
      int sr;
      if (a.pad) {
        sr = triv ? a.triv_sid : (int)a.sid[idx];
        row = dev::padded_row((uint32_t)a.dstride, a.rpl, a.rpline, idx);
      } else {
        // block rows: i * d minus the rows missing before representative i,
        // kept per 32 representatives; the metadata word only where one of
        // the 32 has fewer than d rows or the stabilizer is not trivial
        const uint32_t lack = triv && a.lack ? a.lack[idx >> 5] : 0x80000000u;
        if (lack & 0x80000000u) {
          const uint64_t m = a.meta[idx];
          sr = (int)(m >> 48);
          row = m & kOffMask;
        } else {
          sr = a.triv_sid;
          row = (uint64_t)idx * (uint32_t)a.dstride - lack;
        }
      }
      const int nr = (int)stabf[4 * sr];
      if (nr == 0) return f;
      int h = (int)((ent >> 32) & 0xffff);
      const int cand = (int)((ent >> 48) & 0x7fff);
      const int bond = cand >> 1;
      const int ai = dev::digit(plab, bonds[2 * bond], a.b, lmask);
      const int aj = dev::digit(plab, bonds[2 * bond + 1], a.b, lmask);
      const double c = Jb[bond] * fac[((cand & 1) * a.dloc + ai) * a.dloc + aj] * stabf[4 * sr + 2];
      // G x Z2: (g, F) has index |G| + g and matrix fpar * rho(g)
      const bool flipped = h >= a.Gbase;
      f.c = flipped ? c * a.fpar : c;
      f.info = (uint32_t)(flipped ? h - a.Gbase : h) | ((uint32_t)sr << 16);
      f.off = flip_word<VAR, DG>(row, nr, stabf[4 * sr + 3] != 0.0, a.pad != 0, a.rows, a.ld);
      return f;
    };
    auto gather = [&](const Flip& f, T (&xv)[DG][VPL]) {
      gather_slice<VAR>(a.X, f, shape, vok, xv, [](T v) { return pair_swap(v); });
    };
    // One flip's term: its coefficient times rho(h)^T (after V_r for a target
    // with a non-trivial stabilizer) applied to the gathered rows.  FP64
    // storage: the d x d product is summed by itself and added once per flip,
    // because summed into the accumulator term by term it rounds at the
    // accumulator's magnitude d times per flip (3.3e-16 off a 64-bit
    // reference instead of 2.1e-16).  FP32 and FP16 storage round the sum to
    // 6e-8 and 5e-4 anyway and take the form with fewer registers (1% faster
    // in FP32; six FP16 columns, d = 5: 2.5 against 5.5 ms).
    constexpr bool kPerFlip = sizeof(T) == 8 || DG > 6;
    // Rows of a matrix read ahead (each_row).  Trivial targets: one from LDS,
    // two from memory (square 6 x 6, d = 8, one FP64 vector 136 us with three,
    // 119 with two).  The others, which are few in large sectors: none in the
    // launches of many waves (one more row there spills 6 to 14 registers more
    // at d = 5), else the same.  The general kernels with the tables in LDS
    // have registers to spare and leave the schedule to the compiler, over
    // plain loops (fused jobs of one to 8 chains 3 to 15% faster so).
    constexpr bool kPlainLoops = !ADJ && TAB == kTabLds;
    constexpr bool kManyWaves = VAR == kAdjacent || VAR == kNarrow;
    constexpr int kAheadR = TAB == kTabMemory ? 2 : 1;
    constexpr int kAheadV = kManyWaves ? (TAB == kTabV && DG * VPL <= 4 ? 3 : 0) : kAheadR;
    auto accumulate = [&](const Flip& f, T (&xv)[DG][VPL]) {
      const double* R = rhoT + (size_t)f.h() * DG * DG;
      if (f.off & Flip::kTrivial) {
        if constexpr (kPlainLoops && kPerFlip) {
#pragma unroll
          for (int be = 0; be < DG; ++be)
#pragma unroll
            for (int j = 0; j < VPL; ++j) {
              double s = 0.0;
#pragma unroll
              for (int q = 0; q < DG; ++q) s = fma(R[be * DG + q], (double)xv[q][j], s);
              acc[be][j] = fma(f.c, s, acc[be][j]);
            }
        } else if constexpr (kPlainLoops) {
#pragma unroll
          for (int q = 0; q < DG; ++q)
#pragma unroll
            for (int j = 0; j < VPL; ++j) {
              const double x = f.c * (double)xv[q][j];
#pragma unroll
              for (int be = 0; be < DG; ++be) acc[be][j] = fma(R[be * DG + q], x, acc[be][j]);
            }
        } else if constexpr (kPerFlip) {
          each_row<DG, DG, kAheadR>([&](int be, int q) { return R[be * DG + q]; },
                                    [&](int be, const double (&r)[DG]) {
#pragma unroll
                                      for (int j = 0; j < VPL; ++j) {
                                        double s = r[0] * (double)xv[0][j];
#pragma unroll
                                        for (int q = 1; q < DG; ++q) s = fma(r[q], (double)xv[q][j], s);
                                        acc[be][j] = fma(f.c, s, acc[be][j]);
                                      }
                                    });
        } else {
          each_row<DG, DG, kAheadR>([&](int q, int be) { return R[be * DG + q]; },
                                    [&](int q, const double (&r)[DG]) {
                                      double x[VPL];
#pragma unroll
                                      for (int j = 0; j < VPL; ++j) x[j] = f.c * (double)xv[q][j];
#pragma unroll
                                      for (int be = 0; be < DG; ++be)
#pragma unroll
                                        for (int j = 0; j < VPL; ++j) acc[be][j] = fma(r[be], x[j], acc[be][j]);
                                    });
        }
      } else {
        if (ADJ && !a.pad) {
          const int nr = f.n();
#pragma unroll
          for (int q = 1; q < DG; ++q)
#pragma unroll
            for (int j = 0; j < VPL; ++j) xv[q][j] = q < nr ? xv[q][j] : T(0);
        }
        // The matrices are re-read for every vector (offset by the runtime
        // zero a.zero) so the compiler cannot keep both d x d matrices live
        // across the vector loop.
#pragma unroll
        for (int j = 0; j < VPL; ++j) {
          const double* Vr = Vt + (size_t)f.sr() * DG * DG + j * a.zero;
          const double* Rj = R + j * a.zero;
          double t[DG];
          if constexpr (kPlainLoops) {
#pragma unroll
            for (int q = 0; q < DG; ++q) {
              t[q] = 0.0;
#pragma unroll
              for (int k = 0; k < DG; ++k) t[q] = fma(Vr[q * DG + k], (double)xv[k][j], t[q]);
            }
#pragma unroll
            for (int be = 0; be < DG; ++be) {
              double s = 0.0;
#pragma unroll
              for (int q = 0; q < DG; ++q) s = fma(Rj[be * DG + q], t[q], s);
              acc[be][j] = fma(f.c, s, acc[be][j]);
            }
          } else {
            each_row<2 * DG, DG, kAheadV>([&](int i, int k) { return i < DG ? Vr[i * DG + k] : Rj[(i - DG) * DG + k]; },
                                          [&](int i, const double (&r)[DG]) {
                                            double s = 0.0;
#pragma unroll
                                            for (int k = 0; k < DG; ++k) s = fma(r[k], i < DG ? (double)xv[k][j] : t[k], s);
                                            if (i < DG)
                                              t[i] = s;
                                            else
                                              acc[i - DG][j] = fma(f.c, s, acc[i - DG][j]);
                                          });
          }
        }
      }
    };

    constexpr int kWords = (DG * VPL * (int)sizeof(T) + 3) / 4;  // registers of one gathered slice
    if constexpr (VAR == kNarrow) {
      // slices in flight per lane, by their registers
      constexpr int U = kWords <= 10 ? 4 : kWords <= 24 ? 2 : 1;
      const uint64_t e_end = a.row_ptr[p + 1];
      for (uint64_t e = a.row_ptr[p]; e < e_end; e += U) {
        Flip f[U];
        T xv[U][DG][VPL];
        uint64_t ent[U];
#pragma unroll
        for (int u = 0; u < U; ++u) ent[u] = load_entry(min(e + u, e_end - 1));
#pragma unroll
        for (int u = 0; u < U; ++u) f[u] = decode(e + u < e_end ? ent[u] : (uint64_t)kInvalid);
#pragma unroll
        for (int u = 0; u < U; ++u) gather(f[u], xv[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (f[u].n()) accumulate(f[u], xv[u]);
      }
    } else {
      uint64_t e_begin = OTF ? 0 : a.row_ptr[p];
      uint64_t e_end = OTF ? (uint64_t)ncand : a.row_ptr[p + 1];
      // on the fly: the admissible flips of p as a bit mask where it fits 128
      // bits, each lane of the group testing every GL-th one; e then counts
      // admissible flips, so no lane searches for an inadmissible one
      uint64_t adm0 = 0, adm1 = 0;
      const bool listed = OTF && ncand <= 128;
      if constexpr (OTF) {
        if (listed) {
          for (int q = lg; q < ncand; q += GL) {
            const int bond = q >> 1;
            const int ai = dev::digit(plab, bonds[2 * bond], a.b, lmask);
            const int aj = dev::digit(plab, bonds[2 * bond + 1], a.b, lmask);
            const uint64_t ok = (q & 1) ? (ai > 0 && aj < a.dloc - 1) : (ai < a.dloc - 1 && aj > 0);
            if (q < 64)
              adm0 |= ok << q;
            else
              adm1 |= ok << (q - 64);
          }
          for (int off = 1; off < GL; off <<= 1) {
            adm0 |= shfl64(adm0, lane ^ off);
            adm1 |= shfl64(adm1, lane ^ off);
          }
          e_end = (uint64_t)(__popcll(adm0) + __popcll(adm1));
          // lane lg starts at the lg-th admissible flip
          for (int q = 0; q < lg; ++q) {
            if (adm0)
              adm0 &= adm0 - 1;
            else
              adm1 &= adm1 - 1;
          }
        }
      }
      uint64_t next = kInvalid;
      if constexpr (!OTF) {
        if (e_begin + lg < e_end) next = load_entry(e_begin + lg);
      }
      for (uint64_t e = e_begin; e < e_end; e += GL) {
        // ---- one flip per lane, decoded by that lane; the next chunk's
        // entries are loaded while this one's slices are gathered
        uint64_t my = next;
        if constexpr (!OTF) {
          next = kInvalid;
          if (e + GL + lg < e_end) next = load_entry(e + GL + lg);
        } else {
          my = kInvalid;
          int cand = (int)e + lg;
          bool ok = cand < (int)e_end;
          if (listed) {
            cand = adm0 ? __builtin_ctzll(adm0) : adm1 ? 64 + __builtin_ctzll(adm1) : 0;
            for (int q = 0; q < GL; ++q) {
              if (adm0)
                adm0 &= adm0 - 1;
              else
                adm1 &= adm1 - 1;
            }
          }
          W x = plab;
          if (ok) {
            const int bond = cand >> 1;
            const int i = bonds[2 * bond], j = bonds[2 * bond + 1];
            const int ai = dev::digit(plab, i, a.b, lmask), aj = dev::digit(plab, j, a.b, lmask);
            ok = (cand & 1) ? (ai > 0 && aj < a.dloc - 1) : (ai < a.dloc - 1 && aj > 0);
            const W ui = W(1) << (i * a.b), uj = W(1) << (j * a.b);
            if (ok) x = (cand & 1) ? (plab - ui + uj) : (plab + ui - uj);
          }
          W r;
          int h, ties;
          dev::orbit_min<W, GW, kPlain<NCH, GW>>(x, ok, osearch, r, h, ties);
          uint64_t idx = 0;
          if (ok && lookup_rep<W>(r, a.N, a.b, a.dloc, a.A_tot, ocnt, a.cnt_stride, a.D_M, a.ranks, idx))
            my = idx | ((uint64_t)h << 32) | ((uint64_t)cand << 48) | ((uint64_t)(ties == 1) << 63);
        }
        const Flip mine = decode(my);
        const int cnt = (int)min((uint64_t)GL, e_end - e);
        auto flip_of = [&](int jj) -> Flip {
          Flip f;
          f.c = __longlong_as_double((long long)shfl64((uint64_t)__double_as_longlong(mine.c), gbase + jj));
          f.off = shfl64(mine.off, gbase + jj);
          f.info = (uint32_t)__shfl((int)mine.info, gbase + jj);
          return f;
        };
        // (a flip without a term gathers the output representative's own
        // rows, which flip_word keeps inside the array: a branch around the
        // loads made the launch 25% slower)
        if constexpr (VAR == kDeep) {
          // a ring of slices, each gathered kRing - 1 flips before its term
          // is added (terms in flip order)
          constexpr int kRing = kWords <= 16 ? 4 : 3;
          Flip f[kRing];
          T xv[kRing][DG][VPL];
#pragma unroll
          for (int k = 0; k < kRing - 1; ++k)
            if (k < cnt) {
              f[k] = flip_of(k);
              gather(f[k], xv[k]);
            }
#pragma unroll 1
          for (int jj = 0; jj < cnt; jj += kRing) {
#pragma unroll
            for (int k = 0; k < kRing; ++k) {
              const int ahead = jj + k + kRing - 1, at = (k + kRing - 1) % kRing;
              if (ahead < cnt) {
                f[at] = flip_of(ahead);
                gather(f[at], xv[at]);
              }
              if (jj + k < cnt && f[k].n()) accumulate(f[k], xv[k]);
            }
          }
        } else {
#pragma unroll 1
          for (int jj = 0; jj < cnt; ++jj) {
            const Flip f = flip_of(jj);
            if constexpr (!ADJ) {
              if (!f.n()) continue;
            }
            T xv[DG][VPL];
            gather(f, xv);
            if (f.n()) accumulate(f, xv);
          }
        }
      }
    }
    // ---- project with V_p, add the diagonal, write
    const double sqL = stabf[4 * sp + 1];
    const bool ptriv = stabf[4 * sp + 3] != 0.0;
    const double* Vp = Vt + (size_t)sp * DG * DG;
    const double ed = a.ediag[p] - a.eshift;
#pragma unroll
    for (int k = 0; k < DG; ++k) {
      if (k >= np_) break;
      __builtin_amdgcn_sched_barrier(0);
      const uint64_t at = (offp + k) * (uint64_t)a.ld + vcol;
      T xk[VPL], yk[VPL];
      if (ADJ) {
        const Elems<T, VPL> v = *reinterpret_cast<const Elems<T, VPL>*>(a.X + at);
#pragma unroll
        for (int j = 0; j < VPL; ++j) xk[j] = v.v[j];
        if (EPI) {
          const Elems<T, VPL> w = *reinterpret_cast<const Elems<T, VPL>*>(a.Y + at);
#pragma unroll
          for (int j = 0; j < VPL; ++j) yk[j] = w.v[j];
        }
      }
#pragma unroll
      for (int j = 0; j < VPL; ++j) {
        double y;
        if (ptriv) {
          y = acc[k][j];
        } else {
          double s = 0.0;
#pragma unroll
          for (int be = 0; be < DG; ++be) s = fma(Vp[be * DG + k], acc[be][j], s);
          y = s;
        }
        y *= sqL;
        if (ADJ || vok[j]) {
          const int v = vcol + j * vstep;
          const double xv = (double)(ADJ ? xk[j] : a.X[at + j * vstep]);
          const double hx = fma(ed, xv, y);
          if (!EPI) {
            yk[j] = (T)hx;
          } else {
            const double sj = a.scal[2 * v], bsj = a.scal[2 * v + 1];
            const T ws = (T)(sj * hx - bsj * (double)(ADJ ? yk[j] : a.Y[at + j * vstep]));
            yk[j] = ws;
            dot[j] += xv * (double)ws;
          }
          if (!ADJ) a.Y[at + j * vstep] = yk[j];
        }
      }
      if (ADJ) {
        if (full) {
          Elems<T, VPL> w;
#pragma unroll
          for (int j = 0; j < VPL; ++j) w.v[j] = yk[j];
          *reinterpret_cast<Elems<T, VPL>*>(a.Y + at) = w;
        } else {
#pragma unroll
          for (int j = 0; j < VPL; ++j)
            if (vok[j]) a.Y[at + j] = yk[j];
        }
      }
    }
  }
}

template <typename T, int DG, int VPL, int GW, int NCH, bool LDS_TAB, bool SLDS, int VAR = kGeneral,
          bool VG = false>
__global__ void __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(VAR == kDeep ? 1 : VAR == kGeneral ? hv_waves_general(DG * VPL) : hv_waves(DG * VPL))))
k_hv(HvArgs<T> a) {
  using W = word_t<NCH>;
  extern __shared__ uint64_t smem_raw[];
  char* sm = (char*)smem_raw;
  const bool EPI = a.partials != nullptr;
  dev::Orbit<W, (GW > 0 ? GW : 1), kPlain<NCH, GW>> osearch{};
  const uint64_t* ocnt = a.cnt;
  if constexpr (GW > 0) {
    const uint32_t pos = (uint32_t)(a.NC * 16 * GW), nc = (uint32_t)((a.N + 1) * a.cnt_stride);
    osearch.mask = a.mask;
    osearch.lds = stage<uint64_t>(a.mask, (uint32_t)a.n_lds * pos, sm);
    osearch.n_lds = a.n_lds;
    osearch.img = (const W*)a.img;
    if constexpr (LDS_TAB) {
      char* at = sm + (size_t)a.n_lds * pos * 8;
      ocnt = stage<uint64_t>(a.cnt, nc, at);
      osearch.img = stage<W>((const W*)a.img, (uint32_t)((a.nH + a.nT) * a.nch * 16), at + (size_t)nc * 8);
    }
    osearch.split = a.split;
    osearch.nH = a.nH;
    osearch.nch = a.nch;
    osearch.NC = a.NC;
    osearch.N = a.N;
    osearch.b = a.b;
    osearch.G = a.Gbase;
    osearch.zf_ = a.zf != 0;
    osearch.full = (W)a.full;
  }
  if constexpr (SLDS) stage_small(a.small, a.small_bytes, (uint8_t*)sm + a.o_small);
  const uint8_t* const tabs = SLDS ? (const uint8_t*)sm + a.o_small : a.small;
  HvTabs tb = small_tabs(a, tabs, VG ? a.small : tabs);
  if constexpr (!SLDS) {
    // stabilizer data and bonds (small_bytes from o_stab on): every flip's
    // decoding waits for three of their elements, one after the other
    if (a.small_bytes) {
      stage_small(a.small + a.o_stab, a.small_bytes, (uint8_t*)sm + a.o_small);
      const uint8_t* const mid = (const uint8_t*)sm + a.o_small;
      tb.stabf = (const double*)mid;
      tb.Jb = (const double*)(mid + (a.o_J - a.o_stab));
      tb.fac = (const double*)(mid + (a.o_fac - a.o_stab));
      tb.bonds = (const int32_t*)(mid + (a.o_bonds - a.o_stab));
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int GL = a.GL;
  const int slots_per_wave = 64 >> a.log2GL;
  const int waves = blockDim.x >> 6;
  // Workgroups run round-robin over the 8 XCDs.  Each XCD takes sweeps of
  // adjacent representatives (sweep_w workgroups, each striding over them
  // sweep_k times), because close representatives have many targets in common
  // and each XCD has its own L2: L2 misses of the d = 5, 24-column launch
  // 1.58e8 -> 1.38e8.  Sweeps of 64 workgroups measured best (16: 3% slower;
  // one eighth of the sector per XCD: 10% slower, its workgroups' fronts are
  // too far apart).
  const uint32_t per_wg = (uint32_t)(waves * slots_per_wave);
  const uint32_t in_wg = (threadIdx.x >> 6) * slots_per_wave + (lane >> a.log2GL);
  uint64_t slot = (uint64_t)blockIdx.x * per_wg + in_wg, slot_stride = (uint64_t)gridDim.x * per_wg, p_end = a.n_reps;
  if (a.sweep_k) {
    const uint32_t on_xcd = blockIdx.x >> 3;
    const uint32_t sweep = (on_xcd / a.sweep_w) * 8 + (blockIdx.x & 7);
    const uint64_t sweep_reps = (uint64_t)a.sweep_k * a.sweep_w * per_wg;
    slot = sweep * sweep_reps + (on_xcd % a.sweep_w) * per_wg + in_wg;
    slot_stride = (uint64_t)a.sweep_w * per_wg;
    p_end = min(a.n_reps, (sweep + 1) * sweep_reps);
  }
  double dot[VPL];
  bool vok[VPL];
  int vcol;
  constexpr int TAB = VG ? kTabV : SLDS ? kTabLds : kTabMemory;
  hv_pass<T, DG, VPL, GW, NCH, VAR, TAB>(a, tb, osearch, ocnt, (int)blockIdx.y, slot, slot_stride, p_end, dot, vok, vcol);
  if (EPI) {
    __shared__ double red[kThreads];
    // one vector slot j at a time: lanes with equal lg hold the same column
    const int vstep = VAR == kGeneral ? GL : 1;
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
      red[threadIdx.x] = dot[j];
      __syncthreads();
      if ((int)threadIdx.x < GL) {
        double s = 0.0;
        for (int q = 0; q < kThreads / GL; ++q) s += red[q * GL + threadIdx.x];
        // (threads below GL are the first group's lanes, their columns the sums')
        if (vok[j]) a.partials[(size_t)blockIdx.x * a.nvec + vcol + j * vstep] = s;
      }
      __syncthreads();
    }
  }
}

template <typename T, int DG, int VPL, int GW, int NCH, bool LDS_TAB>
void launch_k(const HvArgs<T>& a, const LaunchCfg& c, hipStream_t st) {
  // adjacent-column kernels for the dimension buckets 1-6 (buckets 8 and 12
  // take the general ones)
  if constexpr (GW == 0 && DG <= 6) {
    if (c.slds && c.var != kGeneral) {
      auto go = [&](auto var) {
        constexpr int V = decltype(var)::value;
        if (c.vg)
          hipLaunchKernelGGL((k_hv<T, DG, VPL, GW, NCH, LDS_TAB, true, V, true>), c.grid, dim3(kThreads), c.shm, st, a);
        else
          hipLaunchKernelGGL((k_hv<T, DG, VPL, GW, NCH, LDS_TAB, true, V>), c.grid, dim3(kThreads), c.shm, st, a);
      };
      if constexpr (VPL <= 4) {
        if (c.var == kDeep) {
          go(std::integral_constant<int, kDeep>{});
          return;
        }
        if (c.var == kNarrow) {
          go(std::integral_constant<int, kNarrow>{});
          return;
        }
      }
      go(std::integral_constant<int, kAdjacent>{});
      return;
    }
  }
  if constexpr (GW == 0) {
    if (c.slds && c.vg) {
      hipLaunchKernelGGL((k_hv<T, DG, VPL, GW, NCH, LDS_TAB, true, kGeneral, true>), c.grid, dim3(kThreads), c.shm, st, a);
      return;
    }
  }
  if (c.slds)
    hipLaunchKernelGGL((k_hv<T, DG, VPL, GW, NCH, LDS_TAB, true>), c.grid, dim3(kThreads), c.shm, st, a);
  else if constexpr (GW == 0)
    hipLaunchKernelGGL((k_hv<T, DG, VPL, GW, NCH, LDS_TAB, false>), c.grid, dim3(kThreads), c.shm, st, a);
  else
    fail(FTLM_ERR_UNSUPPORTED, "on-the-fly H.V needs the irrep tables in LDS");
}

template <typename T, int DG, int VPL>
void launch_vpl(const HvArgs<T>& a, const LaunchCfg& c, hipStream_t st) {
  if (!c.otf) {
    // the label word width still matters: flips read p's digits
    if (c.wide)
      launch_k<T, DG, VPL, 0, 16, false>(a, c, st);
    else
      launch_k<T, DG, VPL, 0, 8, false>(a, c, st);
    return;
  }
  if constexpr (VPL == 1 || VPL == 4) {
    FTLM_DISPATCH_ORBIT(c.wide, c.plain, c.gw, {
      constexpr int NCH = (sizeof(W) == 4 ? 8 : 16) - (PLAIN ? 1 : 0);
      // plain kernels only for groups of up to 320 elements with every search
      // table in LDS (c.plain); everything else takes the general ones
      if constexpr (!PLAIN || GW <= 5) {
        if (PLAIN || c.lds_tab)
          launch_k<T, DG, VPL, GW, NCH, true>(a, c, st);
        else if constexpr (!PLAIN)
          launch_k<T, DG, VPL, GW, NCH, false>(a, c, st);
      }
    });
  } else {
    fail(FTLM_ERR_INVALID_ARG, "on-the-fly H.V uses 1 or 4 vectors per lane");
  }
}

template <typename T, int DG>
void launch_t(const HvArgs<T>& a, const LaunchCfg& c, hipStream_t st) {
  switch (c.vpl) {
    case 1: launch_vpl<T, DG, 1>(a, c, st); break;
    case 2: launch_vpl<T, DG, 2>(a, c, st); break;
    case 3: launch_vpl<T, DG, 3>(a, c, st); break;
    case 4: launch_vpl<T, DG, 4>(a, c, st); break;
    case 6: launch_vpl<T, DG, 6>(a, c, st); break;
    case 8: launch_vpl<T, DG, 8>(a, c, st); break;
    default: fail(FTLM_ERR_INVALID_ARG, "unsupported vectors per lane");
  }
}

// one instantiation unit per irrep dimension bucket
template <int DG>
void launch_dg(const HvArgs<double>* a64, const HvArgs<float>* a32, const HvArgs<_Float16>* a16,
               const LaunchCfg& c, hipStream_t st);

#define FTLM_HV_INSTANTIATE(DGV)                                                                     \
  template <>                                                                                       \
  void launch_dg<DGV>(const HvArgs<double>* a64, const HvArgs<float>* a32,                         \
                      const HvArgs<_Float16>* a16, const LaunchCfg& c, hipStream_t st) {            \
    if (a64)                                                                                        \
      launch_t<double, DGV>(*a64, c, st);                                                           \
    else if (a32)                                                                                   \
      launch_t<float, DGV>(*a32, c, st);                                                            \
    else                                                                                            \
      launch_t<_Float16, DGV>(*a16, c, st);                                                         \
  }

}  // namespace hvk

// Launch shape, LDS layout and kernel arguments (all but X and Y) of one H.V
// over nvec vectors of leading dimension ld with gl lanes per representative
// (0: the default or autotuned layout).
template <typename T>
void hv_setup(const Block& b, int nvec, int64_t ld, int gl, const VecLayout& vl, const LanczosEpilogue* lz,
              hvk::LaunchCfg& c, hvk::HvArgs<T>& a);

}  // namespace ftlm
