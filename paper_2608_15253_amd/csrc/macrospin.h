// Replica-resident steps of single-cell systems (device code).
//
// A one-cell grid without the demag term has only cell-local field terms
// (anisotropy, Zeeman, thermal; exchange and DMI vanish with one cell), so a
// replica's whole run of Heun or rotation steps stays in registers: fields,
// torque with the spin-transfer term, predictor and corrector, and the
// switching time, with the per-cell arithmetic of the field kernels in the
// same order (results equal the staged path to round-off; the compiler may
// contract multiply-adds differently in the two kernels).  The thermal noise
// of a step is drawn once and used by both stages, as there.  Retire/refill
// runs here too, with the trial bookkeeping in registers.
//
// The steps of a replica are one serial chain, bound by the instructions of a
// wave (about 8 cycles each at one or two waves per SIMD).  G lanes share a
// replica: each draws the noise of every G-th step (a third of a step's
// instructions, and independent of the state), hands it round by shuffles,
// and all of them carry the state.  G fills the chip: 10 000 replicas on one
// lane each were 157 waves on 40 of 256 CUs.  10 000 macrospins with the
// spin-transfer torque, 2000 rotation steps, FP32: 3.98 -> 1.53 ms, 0.76 us
// per step (the rotation's series in place of its sines give half of it).
#pragma once
#include "common.h"
#include "kernels.h"
#include "philox.h"

namespace mmx {

// The cell-local terms of local_terms (a one-cell axis has no neighbours)
// and the noise.
template <typename T, bool EXT>
__device__ inline void macrospin_field(const FArgs<T>& a, const T mc[3], T sigma,
                                       const T eta[3], T H[3]) {
  H[0] = H[1] = H[2] = T(0);
  if (a.terms & T_ANIS) {
    const T mu = mc[0] * a.u[0] + mc[1] * a.u[1] + mc[2] * a.u[2];
#pragma unroll
    for (int c = 0; c < 3; ++c) H[c] = a.can * mu * a.u[c];
  }
  if (EXT && (a.terms & T_CUBIC)) {
    T Hc[3], dens;
    cubic_terms(a, mc, Hc, dens);
#pragma unroll
    for (int c = 0; c < 3; ++c) H[c] += Hc[c];
  }
  if (a.terms & T_ZEEMAN) {
#pragma unroll
    for (int c = 0; c < 3; ++c) H[c] += a.hz[c];
  }
  if (sigma != T(0)) {
#pragma unroll
    for (int c = 0; c < 3; ++c) H[c] += sigma * eta[c];
  }
}

// Retire/refill state of the replicas (null: plain run): initial states, the
// trial generation and first step of the running trial (carried between
// launches), finished-trial counts and the recorded trial lengths.
template <typename T>
struct MacroRefill {
  const T* m_init;
  int* tgen;
  unsigned long long* tstart;
  int* counts;
  double* times;
  int cap;
};

// m: replicas' states (3 values each, D1 layout with one cell); tsw: switching
// times or null.  G lanes per replica (a power of two dividing 64); a refilled
// trial's noise depends on when it starts, so retire/refill takes G = 1.  EXT:
// with the cubic anisotropy.
template <typename T, bool ROT, bool EXT, int G>
__global__ void __launch_bounds__(64) k_macrospin(FArgs<T> a, T* m, double dt_d, int nsteps,
                                                  uint64_t step0, double* tsw, int R,
                                                  MacroRefill<T> rf) {
  const int id = blockIdx.x * 64 + threadIdx.x;
  const int r = min(id / G, R - 1), q = id % G;  // surplus lanes repeat the last replica
  const bool write = id / G < R && q == 0;
  const bool refill = G == 1 && rf.tgen != nullptr;
  uint32_t gen = refill ? (uint32_t)rf.tgen[r] : 0u;
  unsigned long long start = refill ? rf.tstart[r] : 0ull;
  int count = refill ? rf.counts[r] : 0;
  const T dt = (T)dt_d;
  T sigma = 0;
  if ((a.terms & T_THERMAL) && a.Trep) {
    const double Tr = a.Trep[r];
    if (Tr > 0) sigma = (T)sqrt(a.sig2pref * Tr / a.dt_th);
  }
  const uint64_t seed = sigma != T(0) ? a.seeds[r] : 0;
  const T bJ = stt_bj(a, r);
  T mv[3] = {m[(size_t)r * 3], m[(size_t)r * 3 + 1], m[(size_t)r * 3 + 2]};
  double ts = tsw ? tsw[r] : 0.0;
  for (int s0 = 0; s0 < nsteps; s0 += G) {
    T mine[3] = {0, 0, 0};
    if (sigma != T(0)) {
      const uint64_t step = step0 + (uint64_t)(s0 + q);
      thermal_eta<T>(seed, 0u, refill ? step - start : step, mine, gen);
    }
    const int run = min(G, nsteps - s0);
    T next[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) next[c] = G > 1 ? __shfl(mine[c], 0, G) : mine[c];
    for (int i = 0; i < run; ++i) {
      const uint64_t step = step0 + (uint64_t)(s0 + i);
      const T eta[3] = {next[0], next[1], next[2]};
      if constexpr (G > 1) {  // the next step's noise arrives while this one is computed
#pragma unroll
        for (int c = 0; c < 3; ++c) next[c] = __shfl(mine[c], i + 1, G);
      }
      T H[3], k[3], tau[3], k1v[3], mp[3];
      macrospin_field<T, EXT>(a, mv, sigma, eta, H);
      cell_torque(a, bJ, mv, H, k, tau);
      heun_predict(a, ROT, mv, H, k, tau, dt, k1v, mp);
      macrospin_field<T, EXT>(a, mp, sigma, eta, H);
      cell_torque(a, bJ, mp, H, k, tau);
      T mn[3];
      heun_correct(a, ROT, mp, H, k, tau, mv, k1v, dt, mn);
#pragma unroll
      for (int c = 0; c < 3; ++c) mv[c] = mn[c];
      if (tsw && ts < 0 && (double)mv[2] < 0) ts = (double)(step + 1) * dt_d;
      if (refill && (double)mv[2] < 0) {
        // the trial ends: record its length, restart from the initial state
        if (count < rf.cap)
          rf.times[(size_t)r * rf.cap + count] = (double)(step + 1 - start) * dt_d;
        ++count;
        ++gen;
        start = step + 1;
#pragma unroll
        for (int c = 0; c < 3; ++c) mv[c] = rf.m_init[(size_t)r * 3 + c];
      }
    }
  }
  // a non-finite state stays non-finite through later steps and resets
  if (a.nonfinite && !(fabs(mv[0]) + fabs(mv[1]) + fabs(mv[2]) <= T(3))) *a.nonfinite = 1;
  if (!write) return;
#pragma unroll
  for (int c = 0; c < 3; ++c) m[(size_t)r * 3 + c] = mv[c];
  if (tsw) tsw[r] = ts;
  if (refill) {
    rf.tgen[r] = (int)gen;
    rf.tstart[r] = start;
    rf.counts[r] = count;
  }
}

}  // namespace mmx
