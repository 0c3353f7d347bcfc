// Fused Lanczos kernel for small blocks (paper Sections 2.2 and 3): one
// workgroup runs every step of the R chains of one block job (start vectors,
// H.V with the Lanczos epilogue, alpha, update, beta) with workgroup barriers
// between the phases, so a whole campaign of small, uneven blocks is one launch
// per kernel shape instead of four launches per step and block.
//
// The recurrence, the scaling of the stored vectors and the stopping rule are
// those of the per-step kernels in lanczos.hip: w = s_j H q_j - beta_j s_{j-1}
// q_{j-1} written over q_{j-1} by the H.V pass (hv_pass, shared with k_hv),
// alpha_j = s_j <q_j, w>, w -= alpha_j s_j q_j, beta_{j+1} = |w|, q_{j+1} = w,
// s_{j+1} = 1 / beta_{j+1}.  Reductions run over the workgroup in a fixed order
// (deterministic; the order differs from the per-step kernels', so the two
// agree to rounding).  Vectors use the block row layout; the irrep tables and
// the bond data sit in LDS, and so do the two vectors when they fit.
#pragma once

#include "hv_kernel.h"

namespace ftlm {
namespace hvk {

constexpr int kWgMaxR = kWgMaxChains;
// threads per job: 512 (two waves per SIMD, so twice the representatives in
// flight as with 256) for irrep dimension buckets up to 6, whose registers fit
// the 256 per lane this allows; 256 for the 8 and 12 buckets
template <int DG>
constexpr int kWgThreads = DG <= 6 ? 512 : 256;

template <typename T>
struct WgJob {
  HvArgs<T> a;          // tables of the block (X, Y and scal are set by the kernel)
  T* q0;                // D x R, row-major (chain fastest)
  T* q1;                // D x R
  const uint64_t* keys; // R chain keys
  double* alpha;        // R x steps
  double* beta;         // R x steps
  int32_t* nsteps;      // R
  uint64_t D;
  int R, steps, target, dist;
  double sigma;         // storage scale of the stored vectors (1 for FP32 / FP64)
  int dgp;              // irrep dimension bucket
  int lds_vec;          // 1: q0, q1 live in dynamic LDS at byte offset o_q (q0 and q1 unused)
  uint32_t o_q;
};

struct WgChain {
  double s, bs, beta, scale, ca, a;
  int n, done;
};

// Column sums of red[q * W + c], q < n, by pairwise halving (a fixed order,
// log2(n) barrier steps instead of n serial reads); the sum of column c ends
// in red[c].  Called by every thread after red is written and synchronized.
__device__ __forceinline__ void wg_col_sum(double* red, int W, int n) {
  for (int m = n; m > 1;) {
    const int half = (m + 1) >> 1;
    for (int i = threadIdx.x; i < (m - half) * W; i += blockDim.x) {
      const int q = half + i / W, c = i - (i / W) * W;
      red[(q - half) * W + c] += red[q * W + c];
    }
    __syncthreads();
    m = half;
  }
}

// Per-chain sums of one value per thread (thread t holds chain t % R, rows
// t / R + k * RB); out[v] for v < R, in a fixed order.
__device__ __forceinline__ void wg_chain_sum(double x, int R, int RB, double* red, double* out) {
  red[threadIdx.x] = x;
  __syncthreads();
  wg_col_sum(red, R, RB);
  if ((int)threadIdx.x < R) out[threadIdx.x] = red[threadIdx.x];
  __syncthreads();
}

struct WgShared {
  double red[512];
  double scal[2 * kWgMaxR];
  double csum[kWgMaxR];
  WgChain ch[kWgMaxR];
};

// LV: the two Lanczos vectors are in LDS (decided per job on the host), known
// at compile time so their accesses are LDS instructions.
template <typename T, int DG, int VPL, bool LV>
__device__ __forceinline__ void wg_run(const WgJob<T>& J, char* sm, WgShared& sh) {
  constexpr int NT = kWgThreads<DG>;
  // adjacent columns for the buckets that equal d_Gamma (R >= VPL always); one
  // column per lane takes the general gather (one chain 7% faster over 24
  // blocks than with whole-row loads, which have nothing to join there)
  constexpr int kVar = DG <= 6 && VPL > 1 ? kFused : kGeneral;
  constexpr int NCH = 16;  // 64-bit label words serve every label
  using W = word_t<NCH>;
  double* const red = sh.red;
  double* const scal = sh.scal;
  double* const csum = sh.csum;
  WgChain* const ch = sh.ch;

  HvArgs<T> a = J.a;
  T* const q0 = LV ? (T*)(sm + J.o_q) : J.q0;
  T* const q1 = LV ? q0 + J.D * (uint64_t)J.R : J.q1;
  double* const alpha = J.alpha;
  double* const beta = J.beta;
  const uint64_t D = J.D;
  const int R = J.R, steps = J.steps, target = J.target, dist = J.dist;
  const double sigma = J.sigma;
  const int t = threadIdx.x;

  stage_small(a.small, a.small_bytes, (uint8_t*)sm + a.o_small);
  const HvTabs tb = small_tabs(a, (const uint8_t*)sm + a.o_small, (const uint8_t*)sm + a.o_small);
  const dev::Orbit<W, 1, false> none{};  // flips come from the entry table
  for (int i = t; i < R * steps; i += NT) {
    alpha[i] = 0.0;
    beta[i] = 0.0;
  }

  // ---- start vectors: FP64 norm of the draw, then the stored q_0 and its norm
  const int RB = NT / R;
  const int v = t % R, r0 = t / R;
  const bool act = r0 < RB;
  const uint64_t key = J.keys[v];
  double acc = 0.0;
  if (act)
    for (uint64_t row = (uint64_t)r0; row < D; row += (uint64_t)RB) {
      const double x = dev::start_value(key, row, dist);
      acc += x * x;
    }
  wg_chain_sum(acc, R, RB, red, csum);  // also the barrier after the table staging
  const double inv = csum[v] > 0 ? sigma / sqrt(csum[v]) : 0.0;  // stored q_0 has norm sigma
  acc = 0.0;
  if (act)
    for (uint64_t row = (uint64_t)r0; row < D; row += (uint64_t)RB) {
      const T q = (T)(dev::start_value(key, row, dist) * inv);
      q0[row * R + v] = q;
      q1[row * R + v] = T(0);
      acc += (double)q * (double)q;
    }
  wg_chain_sum(acc, R, RB, red, csum);
  if (t < R) {
    WgChain c{};
    c.s = csum[t] > 0 ? 1.0 / sqrt(csum[t]) : 0.0;
    ch[t] = c;
  }
  __syncthreads();

  // H.V lane layout: slots of GL lanes over the workgroup, one column tile
  a.scal = scal;
  a.partials = csum;  // non-null: hv_pass applies the Lanczos epilogue (sums are reduced below)
  const int GL = a.GL;
  const int lane = t & 63;
  const uint64_t slot = (uint64_t)(t >> 6) * (uint64_t)(64 >> a.log2GL) + (uint64_t)(lane >> a.log2GL);
  const uint64_t slot_stride = (uint64_t)(NT / 64) * (uint64_t)(64 >> a.log2GL);

  for (int j = 0; j < target; ++j) {
    if (t < R) {
      scal[2 * t] = ch[t].s * sigma;
      scal[2 * t + 1] = ch[t].bs * sigma;
    }
    __syncthreads();
    T* const qj = (j & 1) ? q1 : q0;
    T* const qp = (j & 1) ? q0 : q1;
    a.X = qj;
    a.Y = qp;
    double dot[VPL];
    bool vok[VPL];
    int vcol;
    hv_pass<T, DG, VPL, 0, NCH, kVar>(a, tb, none, nullptr, 0, slot, slot_stride, a.n_reps, dot, vok, vcol);
    // column sums of q_j . w: lanes with equal (lane mod GL) hold the same column
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
      red[t] = vok[k] ? dot[k] : 0.0;
      __syncthreads();
      wg_col_sum(red, GL, NT / GL);
      if (t < GL && vok[k]) csum[vcol + k * (kVar == kGeneral ? GL : 1)] = red[t];
      __syncthreads();
    }
    if (t < R) {
      WgChain c = ch[t];
      const double al = c.s * csum[t] / sigma;
      c.ca = al * c.s * sigma;
      c.a = al;
      if (!c.done) alpha[(size_t)t * steps + j] = al;
      ch[t] = c;
    }
    __syncthreads();
    // ---- w -= alpha_j s_j q_j, |w|^2
    const double ca = ch[v].ca;
    acc = 0.0;
    if (act)
      for (uint64_t row = (uint64_t)r0; row < D; row += (uint64_t)RB) {
        const uint64_t at = row * R + v;
        const T w = (T)((double)qp[at] - ca * (double)qj[at]);
        qp[at] = w;
        acc += (double)w * (double)w;
      }
    wg_chain_sum(acc, R, RB, red, csum);
    if (t < R) {
      WgChain c = ch[t];
      if (!c.done) {
        const double b = sqrt(csum[t]) / sigma;
        beta[(size_t)t * steps + j] = b;
        c.scale = fmax(c.scale, fabs(c.a) + c.beta + b);
        c.n = j + 1;
        if (j + 1 >= target || b <= 1e-10 * c.scale) {
          c.done = 1;
        } else {
          c.bs = b * c.s;
          c.s = 1.0 / (b * sigma);
          c.beta = b;
        }
      }
      if (c.done) {
        c.s = 0.0;
        c.bs = 0.0;
      }
      ch[t] = c;
    }
    __syncthreads();
    int live = 0;
    for (int c = 0; c < R; ++c) live |= !ch[c].done;
    if (!live) break;  // uniform: every thread reads the same chain states
  }
  if (t < R) J.nsteps[t] = ch[t].n;
}

template <typename T, int DG, int VPL>
__device__ __forceinline__ void wg_job(const WgJob<T>& J, char* sm, WgShared& sh) {
  if (J.lds_vec)
    wg_run<T, DG, VPL, true>(J, sm, sh);
  else
    wg_run<T, DG, VPL, false>(J, sm, sh);
}

// The jobs of dimension buckets up to 6 share one launch, whatever their
// dimension (uniform per workgroup): a launch per bucket ran one after the
// other, each waiting for its longest job, with most of the device idle.
template <typename T, int VPL>
__global__ void __launch_bounds__(kWgThreads<1>) k_lanczos_wg(const WgJob<T>* __restrict__ jobs) {
  extern __shared__ uint64_t smem_raw[];
  __shared__ WgShared sh;
  const WgJob<T>& J = jobs[blockIdx.x];
  switch (J.dgp) {
    case 1: wg_job<T, 1, VPL>(J, (char*)smem_raw, sh); break;
    case 2: wg_job<T, 2, VPL>(J, (char*)smem_raw, sh); break;
    case 3: wg_job<T, 3, VPL>(J, (char*)smem_raw, sh); break;
    case 4: wg_job<T, 4, VPL>(J, (char*)smem_raw, sh); break;
    case 5: wg_job<T, 5, VPL>(J, (char*)smem_raw, sh); break;
    case 6: wg_job<T, 6, VPL>(J, (char*)smem_raw, sh); break;
  }
}

template <typename T, int DG, int VPL>
__global__ void __launch_bounds__(kWgThreads<DG>) k_lanczos_wg_wide(const WgJob<T>* __restrict__ jobs) {
  extern __shared__ uint64_t smem_raw[];
  __shared__ WgShared sh;
  wg_run<T, DG, VPL, false>(jobs[blockIdx.x], (char*)smem_raw, sh);
}

// One launch: grid = one workgroup per job; wide = 0 (buckets 1 to 6), 8 or 12.
template <typename T, int VPL>
void wg_launch(int wide, const void* jobs, int njobs, size_t shm, hipStream_t st);

#define FTLM_WG_INSTANTIATE(T, V)                                                                                  \
  template <>                                                                                                     \
  void wg_launch<T, V>(int wide, const void* jobs, int njobs, size_t shm, hipStream_t st) {                       \
    const WgJob<T>* j = (const WgJob<T>*)jobs;                                                                    \
    if (wide == 0)                                                                                                \
      hipLaunchKernelGGL((k_lanczos_wg<T, V>), dim3(njobs), dim3(kWgThreads<1>), shm, st, j);                     \
    else if (wide == 8)                                                                                           \
      hipLaunchKernelGGL((k_lanczos_wg_wide<T, 8, V>), dim3(njobs), dim3(kWgThreads<8>), shm, st, j);             \
    else                                                                                                          \
      hipLaunchKernelGGL((k_lanczos_wg_wide<T, 12, V>), dim3(njobs), dim3(kWgThreads<12>), shm, st, j);           \
  }

}  // namespace hvk
}  // namespace ftlm
