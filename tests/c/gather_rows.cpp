// Host-side check of the H.V gathers' addresses: for every block read from
// stdin ("d n_reps" and n_Gamma of every representative), every vector layout,
// column count, leading dimension and lane layout, the loads that every lane
// makes for a flip to each representative, and for a flip without a term (an
// inadmissible target, or the padding of the one-lane kernel) at each output
// representative, have to lie inside the vector.  The loads are those of the
// kernels' own gather_slice, run here on a pointer type that records them.
// Prints "fail ..." for the first loads outside, and the totals.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "device.h"
#include "hv_rows.h"

namespace ftlm {
namespace hvk {

struct Extent {
  int64_t lo = 0, hi = 0;  // elements touched: [lo, hi)
  uint64_t loads = 0;
};

struct Probe {
  Extent* e;
  int64_t at;
};
inline Probe operator+(Probe p, int64_t n) { return Probe{p.e, p.at + n}; }
inline Probe operator+(Probe p, uint64_t n) { return Probe{p.e, p.at + (int64_t)n}; }
inline Probe operator+(Probe p, int n) { return Probe{p.e, p.at + n}; }

template <int N>
Elems<float, N> load_elems(const Probe& p) {
  p.e->lo = std::min(p.e->lo, p.at);
  p.e->hi = std::max(p.e->hi, p.at + N);
  p.e->loads += 1;
  return Elems<float, N>{};
}

}  // namespace hvk
}  // namespace ftlm

namespace {

using namespace ftlm::hvk;

int fails = 0;
uint64_t loads = 0, variants[4];

struct Case {
  int d;
  std::vector<int> n;            // n_Gamma per representative
  std::vector<uint64_t> offset;  // block rows
  uint64_t D;
};

struct Rows {
  bool pad;
  uint32_t rpl, rpline;
  uint64_t rows;
};

template <int VAR, int DG, int VPL>
void run(const Case& c, const Rows& r, int nvec, int64_t ld, const Layout& L) {
  const int64_t size = (int64_t)(r.rows - 1) * ld + nvec;  // the smallest array a caller may pass
  ++variants[VAR];
  auto check = [&](uint64_t first, int nr, const char* what, size_t i) {
    Flip f;
    f.c = 0;
    f.info = 0;
    f.off = flip_word<VAR, DG>(first, nr, nr == c.d, r.pad, r.rows, ld);
    for (int tile = 0; tile < L.tiles; ++tile)
      for (int lg = 0; lg < L.GL; ++lg) {
        bool vok[VPL];
        const int vcol = lane_columns<VAR, VPL>(tile, L.tile_w, lg, L.GL, nvec, vok);
        const SliceShape s = slice_shape<VAR, VPL>(r.pad, L.GL, lg, ld, nvec, vcol, true);
        Extent e;
        float xv[DG][VPL];
        gather_slice<VAR>(Probe{&e, 0}, f, s, vok, xv, [](float v) { return v; });
        loads += e.loads;
        if ((e.lo < 0 || e.hi > size) && fails++ < 8)
          std::printf("fail %s variant=%d d=%d vpl=%d lanes=%d lane=%d nvec=%d ld=%lld pad=%d rep=%zu of %zu: [%lld, %lld) of %lld\n",
                      what, VAR, c.d, VPL, L.GL, lg, nvec, (long long)ld, (int)r.pad, i, c.n.size(), (long long)e.lo,
                      (long long)e.hi, (long long)size);
      }
  };
  for (size_t i = 0; i < c.n.size(); ++i) {
    if (c.n[i] == 0) continue;
    const uint64_t first = r.pad ? ftlm::dev::padded_row((uint32_t)c.d, r.rpl, r.rpline, i) : c.offset[i];
    check(first, c.n[i], "target", i);
    check(first, 0, "no term", i);
  }
}

template <int DG, int VPL>
void run_variants(const Case& c, const Rows& r, int nvec, int64_t ld, const Layout& L) {
  run<kGeneral, DG, VPL>(c, r, nvec, ld, L);
  if constexpr (DG <= 6) {
    // the variants the rule takes for this sector and for a large one
    for (uint64_t n : {(uint64_t)c.n.size(), (uint64_t)1 << 30}) {
      const int var = hv_variant(DG == c.d, nvec, L, n);
      if (var == kAdjacent) run<kAdjacent, DG, VPL>(c, r, nvec, ld, L);
      if constexpr (VPL <= 4) {
        if (var == kNarrow) run<kNarrow, DG, VPL>(c, r, nvec, ld, L);
        if (var == kDeep) run<kDeep, DG, VPL>(c, r, nvec, ld, L);
      }
    }
  }
}

template <int DG>
void run_dim(const Case& c, const Rows& r, int nvec, int64_t ld, const Layout& L) {
  switch (L.VPL) {
    case 1: run_variants<DG, 1>(c, r, nvec, ld, L); break;
    case 2: run_variants<DG, 2>(c, r, nvec, ld, L); break;
    case 3: run_variants<DG, 3>(c, r, nvec, ld, L); break;
    case 4: run_variants<DG, 4>(c, r, nvec, ld, L); break;
    case 6: run_variants<DG, 6>(c, r, nvec, ld, L); break;
    case 8: run_variants<DG, 8>(c, r, nvec, ld, L); break;
  }
}

void run_block(const Case& c) {
  for (int nvec : {1, 2, 3, 4, 5, 7, 13, 24, 25, 32, 65})
    for (int64_t ld : {(int64_t)nvec, (int64_t)nvec + 1, (int64_t)nvec + 3}) {
      std::vector<Rows> rows{{false, 1, 0, c.D}, {true, 1, (uint32_t)c.d, (uint64_t)c.n.size() * c.d}};
      uint32_t S = 1;
      while (S < (uint32_t)c.d) S <<= 1;
      if (S > (uint32_t)c.d) rows.push_back({true, 1, S, (uint64_t)c.n.size() * S});
      if (const uint32_t line = (uint32_t)(128 / (4 * ld)), p = line / c.d; p >= 2 && p * c.d < line)
        rows.push_back({true, p, line, (c.n.size() + p - 1) / p * line});
      for (const Rows& r : rows)
        for (int gl = 1; gl <= 64; gl <<= 1) {
          const Layout L = choose_layout(nvec, false, gl);
          switch (c.d) {
            case 1: run_dim<1>(c, r, nvec, ld, L); break;
            case 2: run_dim<2>(c, r, nvec, ld, L); break;
            case 3: run_dim<3>(c, r, nvec, ld, L); break;
            case 4: run_dim<4>(c, r, nvec, ld, L); break;
            case 5: run_dim<5>(c, r, nvec, ld, L); break;
            case 6: run_dim<6>(c, r, nvec, ld, L); break;
            case 7: case 8: run_dim<8>(c, r, nvec, ld, L); break;
            default: run_dim<12>(c, r, nvec, ld, L); break;
          }
        }
    }
}

}  // namespace

int main() {
  int d, blocks = 0;
  long long n_reps;
  while (std::scanf("%d %lld", &d, &n_reps) == 2) {
    Case c;
    c.d = d;
    c.D = 0;
    for (long long i = 0; i < n_reps; ++i) {
      int n;
      if (std::scanf("%d", &n) != 1) return 2;
      c.offset.push_back(c.D);
      c.n.push_back(n);
      c.D += (uint64_t)n;
    }
    run_block(c);
    ++blocks;
  }
  std::printf("blocks %d loads %llu general %llu adjacent %llu one-lane %llu deep %llu\nfails %d\n", blocks,
              (unsigned long long)loads, (unsigned long long)variants[0], (unsigned long long)variants[1],
              (unsigned long long)variants[2], (unsigned long long)variants[3], fails);
  return fails == 0 ? 0 : 1;
}
