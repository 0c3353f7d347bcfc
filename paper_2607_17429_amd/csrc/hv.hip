// Host side of the H.V (paper Eqs. 15-16): LDS layout of the small tables,
// lane layout (lanes per representative, vectors per lane) and dispatch to the
// kernel instantiations in hv_dg*.hip.  The kernel itself is in hv_kernel.h.
#include <map>
#include <mutex>
#include <string>

#include "hv_kernel.h"
#include "tune_cache.h"

namespace ftlm {

using namespace hvk;

namespace {

constexpr uint32_t kSmallLdsBudget = 48 * 1024;
constexpr uint32_t kLdsLimit = 65536 - 2048;  // dynamic LDS; 2 KiB stay for the epilogue reduction

// Lanes of a launch up to which more lanes per representative are taken
// (default_lanes): 4 x 4 torus, s = 1, 2M = 4, 3.6e4 representatives, d = 1,
// one FP32 vector 29 us on 4 lanes, 44 on two; square 6 x 6, 2M = 20, 1.1e5
// representatives 35 us on 4, 31 on two.
constexpr uint64_t kFewLanes = 163840;

// Whether the adjacent-column kernels can run the block (hv_setup's rule)
bool adjacent_ok(const Block& b) { return b.sec->hv_mode != FTLM_HV_ONTHEFLY && b.dg == b.dgp && b.dgp <= 6; }

// Default lanes per output representative (ms on MI355X, s = 1/2
// icosidodecahedron at M = 0 unless stated):
//   one lane that holds every column for rows of up to 8 bytes (two FP32,
//   d = 5: 0.67 against 0.69 with two lanes; one FP64, d = 3: 0.50 against
//   0.58); wider rows cost it more registers than the exchange it saves (two
//   FP64: 1.01 against 0.85; four: 1.74 against 1.07).  From d = 5 on two
//   lanes that share the decoding are the better for one column (one FP64,
//   d = 5: 0.65 against 0.74, padded rows 0.57 against 0.75) and, in padded
//   rows, for two, whose row pairs they split (0.58 against 0.63; the s = 3/2
//   dodecahedron, 7.2e8 representatives: 520 against 633);
//   up to 4 vectors one lane each;
//   above, 3 vectors per lane, 4 in FP32 and FP16 where that halves the lanes
//   of a large sector (13 FP32 vectors, d = 5: 1.77 against 1.95; 7: 1.28
//   against 1.14, so not below 8 lanes; s = 3/2 cuboctahedron 2M = 4, 3.2e4
//   representatives, d = 3: 62 us against 49 with 8 lanes), and 6 for more than 12 FP16 vectors, whose rows are then
//   whole 4-byte words (24 vectors, d = 3: 1.40 against 1.67), where the sector
//   is large (not for fewer: 2M = 8, 4.6e5 representatives, d = 4, five FP16
//   vectors 0.54 on one lane against 0.32 on two; square 6 x 6, 1.1e5, d = 4,
//   eight 0.19 on two against 0.14 on four);
//   16 lanes for 9 to 32 vectors from d = 4 on in sectors of 2e4 to 6.5e4
//   representatives, whose targets with a non-trivial stabilizer read their
//   matrices for every vector of a lane again (4 x 4 torus, s = 1, 2M = 4,
//   3.6e4 representatives, 13 FP32 vectors: 96 us against 130 with 8 lanes, 142
//   with 4; 24: 128 against 170; at 1.4e4 72 against 67, at d = 2 as fast);
//   more lanes, up to 32, where the sector's representatives leave the device
//   idle otherwise: few waves wait for one another's flips, and many lanes
//   decode a row's flips at once (dodecahedron H_g at M = 0, 1,648
//   representatives, FP64: 24 vectors 19 us against 40 with 8 lanes, one
//   vector 19 against 36 us; 17,238 representatives, one vector: 30 us with 4
//   lanes, 44 with one); up to kFewLanes lanes in all.
int default_lanes(const Block& b, int nvec, int dtype, bool pad) {
  if (b.sec->hv_mode == FTLM_HV_ONTHEFLY)
    return nvec <= 4 ? pow2_at_least(nvec) : std::min(16, pow2_at_least((nvec + 3) / 4));
  const int elem = dtype == FTLM_F64 ? 8 : dtype == FTLM_F32 ? 4 : 2;
  int gl = nvec <= 4 ? pow2_at_least(nvec) : pow2_at_least((nvec + 2) / 3);
  if (!adjacent_ok(b) || nvec > 64) return gl;
  const bool large = b.sec->n_reps >= (1u << 16);
  if (nvec * elem <= 8)
    gl = b.dg >= 5 && (pad || nvec == 1) ? 2 : 1;
  else if (elem == 2 && nvec > 12 && large)
    gl = pow2_at_least((nvec + 5) / 6);
  else if (elem < 8 && gl >= 8 && gl * 2 >= nvec && large)
    gl /= 2;
  if (!large && b.sec->n_reps > 20000 && b.dg >= 4 && nvec > 8 && nvec <= 32) gl = std::max(gl, 16);
  if (nvec <= 32)
    while (gl < 32 && b.sec->n_reps * (uint64_t)(2 * gl) <= kFewLanes) gl *= 2;
  return gl;
}

struct Sweep {
  uint32_t w, k;   // workgroups and rounds of one sweep (k = 0: workgroups in order)
  uint64_t need;   // workgroups that give every representative a lane group
  dim3 grid;
};

Sweep hv_grid(const Block& b, const Layout& L) {
  constexpr uint64_t TW = 64;    // workgroups of a sweep
  constexpr uint64_t TG = 8064;  // workgroups asked for: the grid stays within 8192
  const uint64_t slots_per_block = (uint64_t)(kThreads / 64) * (64 / L.GL);
  const uint64_t need = std::max<uint64_t>(1, (b.sec->n_reps + slots_per_block - 1) / slots_per_block);
  Sweep s{};
  s.need = need;
  if (need <= 512) {
    // one round of at most two workgroups a CU: nothing to sweep, and no
    // workgroup without a representative
    s.w = 1;
    s.grid = dim3((unsigned)need, (unsigned)L.tiles, 1);
    return s;
  }
  s.k = (uint32_t)((need + TG - 1) / TG);
  const uint64_t per_xcd = ((need + s.k - 1) / s.k + 7) / 8;
  const uint64_t sweeps = (per_xcd + TW - 1) / TW;
  s.w = (uint32_t)((per_xcd + sweeps - 1) / sweeps);
  s.grid = dim3((unsigned)(8 * sweeps * s.w), (unsigned)L.tiles, 1);
  return s;
}

uint32_t align16(uint64_t x) { return (uint32_t)((x + 15u) & ~uint64_t(15)); }

// Architecture name of the current device (cached per device ordinal): part
// of every autotuner key, so that a cache loaded from a file tuned on other
// hardware is never used here.
std::string current_arch() {
  static std::mutex mu;
  static std::map<int, std::string> names;
  int dev = 0;
  FTLM_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(mu);
  auto it = names.find(dev);
  if (it != names.end()) return it->second;
  hipDeviceProp_t prop{};
  FTLM_HIP(hipGetDeviceProperties(&prop, dev));
  return names[dev] = std::string(prop.gcnArchName);
}

// Size class of a sector for the tuned lanes, with default_lanes' thresholds:
// sectors of one class have the same default for every vector count, so lanes
// timed on one of them do not replace another class's.
int size_class(uint64_t n_reps) {
  int c = 0;
  for (uint64_t gl = 32; gl > 1 && n_reps * gl > kFewLanes; gl /= 2) ++c;
  return c;
}

TuneKey tune_key(const Block& b, int nvec, int dtype, const VecLayout& vl, bool epi) {
  const Sector& s = *b.sec;
  TuneKey k;
  k.arch = current_arch();
  k.cluster = s.cluster_hash;
  k.N = s.N;
  k.two_s = s.two_s;
  k.G = s.gorder;
  k.dgp = b.dgp;
  k.nvec = nvec;
  k.dtype = dtype;
  k.mode = s.hv_mode;
  k.pad = vl.kind();
  k.epi = epi ? 1 : 0;
  k.kernels = kTuneKernels;
  k.size = size_class(s.n_reps);
  return k;
}

int tuned_gl(const Block& b, int nvec, int dtype, const VecLayout& vl, bool epi) {
  const int gl = tune_lookup(tune_key(b, nvec, dtype, vl, epi));
  return gl > 0 ? gl : default_lanes(b, nvec, dtype, vl.pad);
}

// Column sums of a (ng x nvec) array of per-workgroup partials, one workgroup
// per column, in a fixed order.
__global__ void __launch_bounds__(256) k_col_sums(const double* __restrict__ partials, int ng, int nvec,
                                                 double* __restrict__ out) {
  __shared__ double red[256];
  const int v = blockIdx.x;
  double s = 0.0;
  for (int g = threadIdx.x; g < ng; g += blockDim.x) s += partials[(size_t)g * nvec + v];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = blockDim.x / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[v] = red[0];
}

__global__ void k_fill_f64(double* __restrict__ p, int n, double x) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = x;
}

}  // namespace

std::string device_arch() { return current_arch(); }

int irrep_dim_bucket(int d) {
  if (d >= 1 && d <= 6) return d;
  if (d <= 8) return 8;
  if (d <= 12) return 12;
  return -1;
}

int hv_layout_lanes(const Block& b, int nvec, int dtype, const VecLayout& vl, bool epi) {
  return choose_layout(nvec, b.sec->hv_mode == FTLM_HV_ONTHEFLY, tuned_gl(b, nvec, dtype, vl, epi)).GL;
}

int hv_partial_groups(const Block& b, int nvec, int gl) {
  return (int)hv_grid(b, choose_layout(nvec, b.sec->hv_mode == FTLM_HV_ONTHEFLY, gl)).grid.x;
}

void apply_hv(const Block& b, const void* X, void* Y, int nvec, int64_t ld, int dtype, hipStream_t st,
              const LanczosEpilogue* lz) {
  apply_hv_gl(b, X, Y, nvec, ld, dtype, st, lz, tuned_gl(b, nvec, dtype, VecLayout{}, lz != nullptr));
}

std::vector<std::pair<int, double>> autotune_hv(const Block& b, int nvec, int dtype, hipStream_t st, int reps,
                                                const VecLayout& vl, bool epi, int* chosen) {
  std::vector<std::pair<int, double>> out;
  if (chosen) *chosen = -1;
  if (b.D == 0 || b.sec->n_reps == 0) return out;
  const size_t elem = dtype == FTLM_F64 ? 8 : dtype == FTLM_F32 ? 4 : 2;
  const uint64_t rows = vec_rows(b, vl);
  DevBuf<uint8_t> X, Y;
  DevBuf<double> scal, partials;
  X.alloc((size_t)rows * nvec * elem);
  Y.alloc((size_t)rows * nvec * elem);
  FTLM_HIP(hipMemsetAsync(X.p, 0, X.bytes(), st));
  FTLM_HIP(hipMemsetAsync(Y.p, 0, Y.bytes(), st));
  if (epi) {
    // the Lanczos epilogue with s = b = 0 (the work of a step; the values do not matter)
    scal.alloc(2 * (size_t)nvec);
    hipLaunchKernelGGL(k_fill_f64, dim3((2 * nvec + 255) / 256), dim3(256), 0, st, scal.p, 2 * nvec, 0.0);
    size_t most = 0;
    for (int gl = 1; gl <= 64; gl <<= 1) most = std::max<size_t>(most, (size_t)hv_partial_groups(b, nvec, gl));
    partials.alloc(most * nvec);
  }
  hipEvent_t e0, e1;
  FTLM_HIP(hipEventCreate(&e0));
  FTLM_HIP(hipEventCreate(&e1));
  // VPL <= 8, and no more lanes than columns but where the default has more
  // (small sectors: idle columns' lanes decode flips)
  const int deflt = choose_layout(nvec, b.sec->hv_mode == FTLM_HV_ONTHEFLY, default_lanes(b, nvec, dtype, vl.pad)).GL;
  const int most_lanes = std::max(pow2_at_least(nvec), deflt);
  int best = -1, at_default = -1;
  for (int gl = 1; gl <= 64; gl <<= 1) {
    if (gl * 8 < nvec || gl > most_lanes) continue;
    LanczosEpilogue lz{scal.p, partials.p, hv_partial_groups(b, nvec, gl)};
    const LanczosEpilogue* lzp = epi ? &lz : nullptr;
    apply_hv_gl(b, X.p, Y.p, nvec, nvec, dtype, st, lzp, gl, vl);  // warm
    // launches below a millisecond are timed four times and the best counts
    double per = 1e300;
    for (int round = 0; round == 0 || (round < 4 && per < 1.0); ++round) {
      FTLM_HIP(hipEventRecord(e0, st));
      for (int r = 0; r < reps; ++r) apply_hv_gl(b, X.p, Y.p, nvec, nvec, dtype, st, lzp, gl, vl);
      FTLM_HIP(hipEventRecord(e1, st));
      FTLM_HIP(hipEventSynchronize(e1));
      float ms = 0;
      FTLM_HIP(hipEventElapsedTime(&ms, e0, e1));
      per = std::min(per, (double)ms / reps);
    }
    if (gl == deflt) at_default = (int)out.size();
    if (best < 0 || per < out[best].second) best = (int)out.size();
    out.push_back({gl, per});
  }
  // the default stays unless another layout is faster by more than runs differ
  if (at_default >= 0 && out[best].second > 0.97 * out[at_default].second) best = at_default;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (best >= 0) tune_store(tune_key(b, nvec, dtype, vl, epi), out[best].first);
  if (chosen) *chosen = best;
  return out;
}

HvExPlan plan_hv_ex(const Block& b, int nvec, int64_t ld, int dtype, const ftlm_hv_opts* o) {
  HvExPlan p{};
  if (nvec <= 0 || ld < nvec) fail(FTLM_ERR_INVALID_ARG, "need 0 < nvec <= ld");
  const int64_t elem = dtype == FTLM_F64 ? 8 : dtype == FTLM_F32 ? 4 : 2;
  const int layout = o ? o->layout : FTLM_LAYOUT_BLOCK;
  if (layout == FTLM_LAYOUT_AUTO)
    p.vl = run_layout(b, ld * elem);
  else if (layout == FTLM_LAYOUT_BLOCK || layout == FTLM_LAYOUT_PADDED || layout == FTLM_LAYOUT_PACKED ||
           layout == FTLM_LAYOUT_ALIGNED)
    p.vl = vec_layout(b, layout, ld * elem);
  else
    fail(FTLM_ERR_INVALID_ARG, "layout must be FTLM_LAYOUT_AUTO, _BLOCK, _PADDED, _PACKED or _ALIGNED");
  p.rows = vec_rows(b, p.vl);
  p.epi = o && o->scale;
  if (o && o->dots && !o->scale) fail(FTLM_ERR_INVALID_ARG, "dots need scale");
  const int lanes = o ? o->lanes : 0;
  if (lanes != 0 && (lanes < 0 || lanes > 64 || (lanes & (lanes - 1))))
    fail(FTLM_ERR_INVALID_ARG, "lanes must be 0 or a power of two up to 64");
  const bool otf = b.sec->hv_mode == FTLM_HV_ONTHEFLY;
  const Layout L = choose_layout(nvec, otf, lanes ? lanes : tuned_gl(b, nvec, dtype, p.vl, p.epi));
  p.gl = L.GL;
  p.ng = (b.D && b.sec->n_reps) ? hv_partial_groups(b, nvec, p.gl) : 0;
  p.ng_asked = p.ng ? (int)std::min<uint64_t>(hv_grid(b, L).need, 8192) : 0;
  if (b.D && b.sec->n_reps) {
    LaunchCfg c{};
    HvArgs<double> a{};
    hv_setup(b, nvec, nvec, p.gl, p.vl, nullptr, c, a);
    p.adjacent = p.vl.pad && c.var != kGeneral && c.slds;
  }
  return p;
}

void apply_hv_ex(const Block& b, const void* X, void* Y, int nvec, int64_t ld, int dtype, const ftlm_hv_opts* o,
                 const HvExPlan& p, double* partials, hipStream_t st) {
  if (p.epi && p.ng > 0 && !partials) fail(FTLM_ERR_INVALID_ARG, "no scratch for the partial sums");
  if (p.rows == 0 || b.sec->n_reps == 0) {
    if (o && o->dots) hipLaunchKernelGGL(k_fill_f64, dim3((nvec + 255) / 256), dim3(256), 0, st, o->dots, nvec, 0.0);
    FTLM_HIP(hipGetLastError());
    return;
  }
  if (!X || !Y) fail(FTLM_ERR_INVALID_ARG, "null vector");
  LanczosEpilogue lz{p.epi ? o->scale : nullptr, partials, p.ng, o ? o->shift : 0.0};
  if (p.epi) {
    apply_hv_gl(b, X, Y, nvec, ld, dtype, st, &lz, p.gl, p.vl);
    if (o->dots) hipLaunchKernelGGL(k_col_sums, dim3(nvec), dim3(256), 0, st, partials, p.ng, nvec, o->dots);
  } else if (lz.eshift != 0.0) {
    // a shift without the epilogue: the same kernel with scale (1, 0) would
    // need a scale array; the plain pass takes the shift directly
    apply_hv_gl(b, X, Y, nvec, ld, dtype, st, nullptr, p.gl, p.vl, lz.eshift);
  } else {
    apply_hv_gl(b, X, Y, nvec, ld, dtype, st, nullptr, p.gl, p.vl);
  }
  FTLM_HIP(hipGetLastError());
}

template <typename T>
void hv_setup(const Block& b, int nvec, int64_t ld, int gl, const VecLayout& vl, const LanczosEpilogue* lz,
              LaunchCfg& c, HvArgs<T>& a) {
  const bool pad = vl.pad;
  const Sector& s = *b.sec;
  const bool otf = s.hv_mode == FTLM_HV_ONTHEFLY;
  const Layout L = choose_layout(nvec, otf, gl);
  c = LaunchCfg{};
  const Sweep sw = hv_grid(b, L);
  c.grid = sw.grid;
  c.otf = otf;
  c.wide = s.wide;
  c.gw = s.gw;
  c.vpl = L.VPL;
  c.var = hv_variant(adjacent_ok(b), nvec, L, s.n_reps);
  // small tables first priority; the orbit search's tables take what they
  // leave (up to the soft limit that keeps two workgroups on a CU), the rest
  // of them is read through the caches
  const uint64_t small = b.small_bytes;
  OrbitLds ol;
  if (otf) {
    const size_t room = kLdsLimit - 32 - (small <= kSmallLdsBudget ? small : 0);
    ol = orbit_lds(s, room, room);
  }
  c.lds_tab = ol.tabs;
  c.plain = s.plain() && s.gw <= 5 && ol.tabs;
  const uint32_t base = align16(ol.bytes);
  c.slds = small <= kSmallLdsBudget && base + small <= kLdsLimit;
  // the kernels without V_S in LDS (VG): rho^T and the small tables only;
  // V_S, used only for non-trivial stabilizers, is read through the caches
  // (a 6x6-torus sector has up to 324 stabilizer types)
  c.vg = !c.slds && !otf && b.o_V <= kSmallLdsBudget;
  if (c.vg) c.slds = true;
  // neither: the matrices are read from memory, the tables between them still
  // go to LDS where they fit
  const uint32_t mid = b.o_V - b.o_stab;
  const uint32_t staged = c.vg ? b.o_V : c.slds ? (uint32_t)small : !otf && mid <= kSmallLdsBudget ? mid : 0;
  c.shm = base + staged;
  {
    a.reps = s.d_reps.p;
    a.row_ptr = s.d_row_ptr.p;
    a.entries = s.d_entries.p;
    a.eidx = s.d_eidx.p;
    a.ehc = s.d_ehc.p;
    a.hbits = s.ent_hbits;
    a.pad = pad ? 1 : 0;
    a.dstride = b.dg;
    a.rpl = vl.rpl;
    a.rpline = vl.rpl > 1 || vl.aligned ? vl.rpline : (uint32_t)b.dg;
    a.rows = vec_rows(b, vl);
    a.lack = b.use_lack ? b.d_lack.p : nullptr;
    a.triv_sid = s.trivial_sid;
    a.sid = s.d_stab_id.p;
    a.meta = b.d_meta.p;
    a.ediag = s.d_ediag.p;
    a.small = b.d_small.p;
    a.small_bytes = staged;
    a.o_small = base;
    a.o_stab = b.o_stab;
    a.o_J = b.o_J;
    a.o_fac = b.o_fac;
    a.o_bonds = b.o_bonds;
    a.o_V = b.o_V;
    a.b = s.bits;
    a.dloc = s.d;
    a.nbonds = s.nbonds;
    a.Gbase = s.G->order;
    a.fpar = b.fpar;
    a.zf = s.zflip ? 1 : 0;
    a.full = s.full;
    a.mask = s.d_mask();
    a.img = s.d_img();
    a.split = s.d_split();
    a.n_lds = ol.n_lds;
    a.nH = s.fac_nH;
    a.nT = s.fac_nT;
    a.nch = s.nch;
    a.NC = s.NC;
    a.n_reps = s.n_reps;
    a.ld = ld;
    a.nvec = nvec;
    a.GL = L.GL;
    a.log2GL = L.log2GL;
    a.tile_w = L.tile_w;
    a.sweep_w = sw.w;
    a.sweep_k = sw.k;
    a.zero = 0;
    a.cnt = s.d_cnt.p;
    a.ranks = s.d_ranks.p;
    a.cnt_stride = s.cnt_stride;
    a.N = s.N;
    a.A_tot = s.A;
    a.D_M = s.D_M;
    a.scal = lz ? lz->scal : nullptr;
    a.partials = lz ? lz->partials : nullptr;
    a.eshift = lz ? lz->eshift : 0.0;
  }
}

template void hv_setup<double>(const Block&, int, int64_t, int, const VecLayout&, const LanczosEpilogue*,
                               LaunchCfg&, HvArgs<double>&);
template void hv_setup<float>(const Block&, int, int64_t, int, const VecLayout&, const LanczosEpilogue*, LaunchCfg&,
                              HvArgs<float>&);
template void hv_setup<_Float16>(const Block&, int, int64_t, int, const VecLayout&, const LanczosEpilogue*,
                                 LaunchCfg&, HvArgs<_Float16>&);

void apply_hv_gl(const Block& b, const void* X, void* Y, int nvec, int64_t ld, int dtype, hipStream_t st,
                 const LanczosEpilogue* lz, int gl, const VecLayout& vl, double shift) {
  const Sector& s = *b.sec;
  if (nvec <= 0 || ld < nvec) fail(FTLM_ERR_INVALID_ARG, "need 0 < nvec <= ld");
  if (b.D == 0 || s.n_reps == 0) return;
  if (!X || !Y) fail(FTLM_ERR_INVALID_ARG, "null vector");
  LaunchCfg c{};
  HvArgs<double> a64{};
  HvArgs<float> a32{};
  HvArgs<_Float16> a16{};
  const HvArgs<double>* p64 = nullptr;
  const HvArgs<float>* p32 = nullptr;
  const HvArgs<_Float16>* p16 = nullptr;
  if (dtype == FTLM_F64) {
    hv_setup(b, nvec, ld, gl, vl, lz, c, a64);
    a64.X = (const double*)X;
    a64.Y = (double*)Y;
    if (!lz) a64.eshift = shift;
    p64 = &a64;
  } else if (dtype == FTLM_F32) {
    hv_setup(b, nvec, ld, gl, vl, lz, c, a32);
    a32.X = (const float*)X;
    a32.Y = (float*)Y;
    if (!lz) a32.eshift = shift;
    p32 = &a32;
  } else if (dtype == FTLM_F16) {
    hv_setup(b, nvec, ld, gl, vl, lz, c, a16);
    a16.X = (const _Float16*)X;
    a16.Y = (_Float16*)Y;
    if (!lz) a16.eshift = shift;
    p16 = &a16;
  } else {
    fail(FTLM_ERR_INVALID_ARG, "dtype must be FTLM_F64, FTLM_F32 or FTLM_F16");
  }
  switch (b.dgp) {
    case 1: launch_dg<1>(p64, p32, p16, c, st); break;
    case 2: launch_dg<2>(p64, p32, p16, c, st); break;
    case 3: launch_dg<3>(p64, p32, p16, c, st); break;
    case 4: launch_dg<4>(p64, p32, p16, c, st); break;
    case 5: launch_dg<5>(p64, p32, p16, c, st); break;
    case 6: launch_dg<6>(p64, p32, p16, c, st); break;
    case 8: launch_dg<8>(p64, p32, p16, c, st); break;
    case 12: launch_dg<12>(p64, p32, p16, c, st); break;
    default: fail(FTLM_ERR_DIM_GT_12, "irrep dimension above 12");
  }
  FTLM_HIP(hipGetLastError());
}

}  // namespace ftlm
