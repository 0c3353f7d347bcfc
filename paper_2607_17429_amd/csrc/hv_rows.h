// Which elements of the vectors a lane of the H.V kernels reads: the lane
// layout of a launch, the columns of a lane and the loads of a flip's gather.
// Host and device code, so that the arithmetic the kernels run can be followed
// on the host for whole blocks (every load has to lie inside the vectors).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

namespace ftlm {
namespace hvk {

// Kernel variants (the host picks one, hv_variant):
//   kGeneral   lane g of a group holds columns g + j * GL; every element of a
//              gather has its own clamped address and a select.  Any launch.
//   kAdjacent  lane g holds the adjacent columns g * VPL + j (the last lanes
//              move back to end at column nvec - 1 and own only the columns
//              no other lane has), so a gathered row is one wide load per
//              lane.  Table-driven launches with d_Gamma equal to the
//              dimension bucket and nvec >= VPL.
//   kNarrow    kAdjacent with one lane per representative that holds every
//              column: no exchange between lanes, several flips' slices in
//              flight per lane, a slice of adjacent rows in 16-byte loads.
//   kDeep      kAdjacent with several flips' slices in flight per lane group,
//              for launches of so few waves that none waits for another.
//   kFused     kAdjacent in the fused Lanczos kernel, whose workgroup has the
//              registers of its CU to itself.
enum HvVariant { kGeneral = 0, kAdjacent = 1, kNarrow = 2, kDeep = 3, kFused = 4 };

// lanes of a launch up to which a wave seldom shares its SIMD (256 CUs x 4
// SIMDs x 64 lanes x 2): several slices in flight per group then hide what
// other waves cannot
constexpr uint64_t kDeepLanes = 131072;

struct Layout {
  int GL, log2GL, VPL, tile_w, tiles;
};

inline int pow2_at_least(int n) {
  int p = 1;
  while (p < n) p <<= 1;
  return p;
}

inline int vpl_bucket(int need, bool otf) {
  if (otf) return need <= 1 ? 1 : 4;
  const int opts[] = {1, 2, 3, 4, 6, 8};
  for (int o : opts)
    if (o >= need) return o;
  return 8;
}

// Lanes per output representative (GL) and vectors per lane (VPL) for gl lanes
// (the autotuner's choice or the default).
inline Layout choose_layout(int nvec, bool otf, int gl) {
  Layout L{};
  L.GL = std::min(64, pow2_at_least(gl));
  L.VPL = vpl_bucket((std::min(nvec, 64 * 8) + L.GL - 1) / L.GL, otf);
  if (L.GL * L.VPL > 64 && L.GL > 1) {
    // keep a tile within 64 vectors
    L.VPL = vpl_bucket(std::max(1, 64 / L.GL), otf);
  }
  L.log2GL = 0;
  while ((1 << L.log2GL) < L.GL) ++L.log2GL;
  L.tile_w = L.GL * L.VPL;
  L.tiles = (nvec + L.tile_w - 1) / L.tile_w;
  return L;
}

// The variant of a launch: adjacent columns wherever a gathered row is whole
// (adjacent_ok: no row of the bucket beyond d_Gamma, flips from the entry
// table) and every lane can own VPL columns.
inline int hv_variant(bool adjacent_ok, int nvec, const Layout& L, uint64_t n_reps) {
  return !adjacent_ok || nvec < L.VPL ? kGeneral
         : L.GL == 1 && L.tiles == 1 && L.VPL <= 4 && nvec == L.VPL ? kNarrow
         : L.VPL <= 4 && n_reps * (uint64_t)L.GL * L.tiles <= kDeepLanes ? kDeep : kAdjacent;
}

// Columns of lane lg: vcol + j * (1, or GL in kGeneral), those with vok[j];
// returns vcol.
template <int VAR, int VPL>
__host__ __device__ __forceinline__ int lane_columns(int tile, int tile_w, int lg, int GL, int nvec, bool (&vok)[VPL]) {
  constexpr bool ADJ = VAR != kGeneral;
  const int vbase = tile * tile_w + lg * (ADJ ? VPL : 1);
  const int last = nvec - VPL;
  const int vcol = ADJ && last < vbase ? last : vbase;
#pragma unroll
  for (int j = 0; j < VPL; ++j) vok[j] = ADJ ? vcol + j >= vbase : vbase + j * GL < nvec;
  return vcol;
}

// One flip as the gather and the accumulation need it, found by one lane:
// the coefficient c_e / sqrt(L_r) (sign of a flipped element included), the
// element offset of the target's first row, n_r, and h, stabilizer id, flags.
struct Flip {
  double c;
  uint64_t off;   // element offset (56 bits) | n_r << 56; n_r = 0: no term
  uint32_t info;  // h | stabilizer id << 16
  static constexpr uint64_t kOff = (1ull << 56) - 1;
  // flags above n_r (dimensions up to 12 need 4 bits)
  static constexpr uint64_t kTrivial = 1ull << 60;  // trivial stabilizer
  static constexpr uint64_t kEnd = 1ull << 61;      // rows beyond n_r may lie past the array
  __host__ __device__ __forceinline__ int n() const { return (int)(off >> 56) & 15; }
  __host__ __device__ __forceinline__ int h() const { return (int)(info & 0xffffu); }
  __host__ __device__ __forceinline__ int sr() const { return (int)(info >> 16); }
};

// Flip::off of a flip whose gather starts at row `row`: the target's first row,
// or for a flip without a term (nr = 0) the output representative's.  Whole
// rows are loaded for both, and on block rows either representative may have
// fewer than DG rows at the end of the array: both carry the end flag there.
template <int VAR, int DG>
__host__ __device__ __forceinline__ uint64_t flip_word(uint64_t row, int nr, bool trivial, bool pad, uint64_t rows,
                                                       int64_t ld) {
  return row * (uint64_t)ld | ((uint64_t)nr << 56) | (trivial ? Flip::kTrivial : 0) |
         (VAR != kGeneral && !pad && row + DG > rows ? Flip::kEnd : 0);
}

// What a gather's loads depend on besides the flip.
struct SliceShape {
  int64_t ld;
  int vcol, vstep, lg;
  bool pair;  // two lanes per representative, one of the two columns each, rows of two elements on a two-element boundary
  bool flat;  // a slice is DG * VPL adjacent elements
};

template <int VAR, int VPL>
__host__ __device__ __forceinline__ SliceShape slice_shape(bool pad, int GL, int lg, int64_t ld, int nvec, int vcol,
                                                           bool pair_aligned) {
  return SliceShape{ld, vcol, VAR == kGeneral ? GL : 1, lg,
                    (VAR == kAdjacent || VAR == kDeep) && VPL == 1 && pad && GL == 2 && nvec == 2 && ld == 2 &&
                        pair_aligned,
                    VAR == kNarrow && ld == VPL};
}

// Row-major elements loaded as one word of N elements at the element type's
// alignment (global loads of up to 16 bytes need no more than that).
template <typename T, int N>
struct __attribute__((packed, aligned(sizeof(T)))) Elems {
  T v[N];
};

template <int N, typename T>
__host__ __device__ __forceinline__ Elems<T, N> load_elems(const T* p) {
  return *reinterpret_cast<const Elems<T, N>*>(p);
}

// Gather of the target's rows into xv[row][column] (P: const T*, or a type
// with the same arithmetic and a load_elems of its own; swap exchanges a value
// with the other lane of the pair).  Every load is inside the array without a
// branch per row, and rows >= n_r are zeroed afterwards (padded rows hold zeros
// there), so all loads of a flip are in flight together; only a flip with the
// end flag, whose DG rows would pass the end of the array, loads its n_r rows
// alone (none for a flip without a term).
template <int VAR, typename P, typename T, int DG, int VPL, typename Swap>
__host__ __device__ __forceinline__ void gather_slice(P X, const Flip& f, const SliceShape& s, const bool (&vok)[VPL],
                                                      T (&xv)[DG][VPL], Swap swap) {
  const P x0 = X + (f.off & Flip::kOff);
  const P xr = x0 + s.vcol;
  if constexpr (VAR == kGeneral) {
    const int nr = f.n();
#pragma unroll
    for (int q = 0; q < DG; ++q)
#pragma unroll
      for (int j = 0; j < VPL; ++j) {
        const bool use = vok[j] && q < nr;
        const T val = load_elems<1>(xr + ((q < nr ? q : 0) * s.ld + (vok[j] ? j * s.vstep : -s.vcol))).v[0];
        xv[q][j] = use ? val : T(0);
      }
  } else if (s.pair) {
    // lane 0 loads rows 0 .. H-1 and lane 1 rows H .. DG-1 (H = ceil(DG / 2)),
    // both columns of a row in one load, then each lane hands the other
    // column to its partner: ceil(DG / 2) loads per flip instead of DG
    constexpr int H = (DG + 1) / 2;
#pragma unroll
    for (int k = 0; k < H; ++k) {
      const Elems<T, 2> v = load_elems<2>(x0 + 2 * (s.lg ? (k + H < DG ? k + H : DG - 1) : k));
      const T recv = swap(s.lg ? v.v[0] : v.v[1]);
      const T keep = s.lg ? v.v[1] : v.v[0];
      xv[k][0] = s.lg ? recv : keep;
      if (k + H < DG) xv[k + H][0] = s.lg ? keep : recv;
    }
  } else if (f.off & Flip::kEnd) {
    const int nr = f.n();
#pragma unroll
    for (int q = 0; q < DG; ++q)
#pragma unroll
      for (int j = 0; j < VPL; ++j) {
        xv[q][j] = T(0);
        if (q < nr) xv[q][j] = load_elems<1>(xr + (q * s.ld + j)).v[0];
      }
  } else if (s.flat) {
    const Elems<T, DG * VPL> v = load_elems<DG * VPL>(xr);
#pragma unroll
    for (int q = 0; q < DG; ++q)
#pragma unroll
      for (int j = 0; j < VPL; ++j) xv[q][j] = v.v[q * VPL + j];
  } else {
#pragma unroll
    for (int q = 0; q < DG; ++q) {
      const Elems<T, VPL> v = load_elems<VPL>(xr + q * s.ld);
#pragma unroll
      for (int j = 0; j < VPL; ++j) xv[q][j] = v.v[j];
    }
  }
}

}  // namespace hvk
}  // namespace ftlm
