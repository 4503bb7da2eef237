// One-off setup kernels: Newell kernel in FP64 on the padded grid, FP64 line
// FFTs of the kernel and parity compression of its (real) spectrum; plus the
// small integrator bookkeeping kernels.
#pragma once
#include "common.h"
#include "fft_lds.h"
#include "kernels.h"
#include "newell.h"

namespace mmx {

struct AxisMap {   // per axis of the padded grid
  int n, P, periodic, images;
};

// For FFT index k on one axis: number of representative offsets (1 or 2) and
// their values.  Open axis of size 2n: k < n -> k, k > n -> k - 2n, k == n
// (Nyquist) -> none.  Periodic: minimum image; for even n the offset n/2 is
// averaged with -n/2.
__device__ inline int axis_reps(const AxisMap& m, int k, long o[2]) {
  if (m.n == 1) { o[0] = 0; return 1; }
  if (m.periodic) {
    const long v = (k < m.n - k) ? k : (long)k - m.n;
    o[0] = v;
    if (m.n % 2 == 0 && (v == m.n / 2 || v == -m.n / 2)) { o[1] = -v; return 2; }
    return 1;
  }
  if (k < m.n) { o[0] = k; return 1; }
  if (k > m.n) { o[0] = (long)k - 2 * m.n; return 1; }
  return 0;
}

// K (complex FP64, [6][Pz][Py][Px], imaginary part 0): real-space kernel.
__global__ void k_newell_kernel(cpx<double>* K, AxisMap ax, AxisMap ay, AxisMap az, double dx,
                                double dy, double dz, GaussRules rules) {
  const long total = (long)ax.P * ay.P * az.P;
  const long id = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= total) return;
  const int kx = id % ax.P;
  const int ky = (id / ax.P) % ay.P;
  const int kz = id / ((long)ax.P * ay.P);
  long ox[2], oy[2], oz[2];
  const int nxr = axis_reps(ax, kx, ox), nyr = axis_reps(ay, ky, oy), nzr = axis_reps(az, kz, oz);
  double acc[6] = {0, 0, 0, 0, 0, 0};
  if (nxr && nyr && nzr) {
    const double w = 1.0 / (nxr * nyr * nzr);
    const int px = (ax.periodic && ax.n > 1) ? ax.images : 0;
    const int py = (ay.periodic && ay.n > 1) ? ay.images : 0;
    const int pz = (az.periodic && az.n > 1) ? az.images : 0;
    for (int a = 0; a < nxr; ++a)
      for (int b = 0; b < nyr; ++b)
        for (int c = 0; c < nzr; ++c)
          for (int iz = -pz; iz <= pz; ++iz)
            for (int iy = -py; iy <= py; ++iy)
              for (int ix = -px; ix <= px; ++ix)
                tensor_add(ox[a] + (long)ix * ax.n, oy[b] + (long)iy * ay.n,
                           oz[c] + (long)iz * az.n, dx, dy, dz, rules, w, acc);
  }
  for (int c = 0; c < 6; ++c) K[(size_t)c * total + id] = {acc[c], 0.0};
}

// In-place FP64 FFT of lines: element k of line (o, i) at o*os + i*is + k*stride.
__global__ void k_line_fft(cpx<double>* data, long os, long is, long stride, FftPlan plan,
                           const cpx<double>* tw) {
  extern __shared__ unsigned char smem_raw[];
  cpx<double>* A = reinterpret_cast<cpx<double>*>(smem_raw);
  cpx<double>* Bf = A + plan.n;
  const long base = (long)blockIdx.y * os + (long)blockIdx.x * is;
  for (int k = threadIdx.x; k < plan.n; k += blockDim.x) A[k] = data[base + k * stride];
  __syncthreads();
  const cpx<double>* X = lds_fft<double, false, 128>(A, Bf, 1, plan, tw);
  for (int k = threadIdx.x; k < plan.n; k += blockDim.x) data[base + k * stride] = X[k];
}

// Nt[((tz Ty + ty) Kx + kx) 8 + c] = scale * Re Khat[c][tz][ty][kx] for
// kx <= Px/2, ty <= Py/2, tz <= Pz/2: the six components of one frequency are
// adjacent (slots 6, 7 unused), one aligned vector load per frequency.
template <typename T>
__global__ void k_compress(T* Nt, const cpx<double>* K, int Px, int Py, int Pz, int Kx, int Ty,
                           int Tz, double scale) {
  const long tot = (long)6 * Tz * Ty * Kx;
  const long id = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= tot) return;
  const int kx = id % Kx;
  const int ty = (id / Kx) % Ty;
  const int tz = (id / ((long)Kx * Ty)) % Tz;
  const int c = id / ((long)Kx * Ty * Tz);
  const long full = (long)Px * Py * Pz;
  const long f = ((long)tz * Ty + ty) * Kx + kx;
  Nt[f * kTensorStride + c] = (T)(scale * K[(size_t)c * full + ((long)tz * Py + ty) * Px + kx].re);
}

// ---------------------------------------------------------------------------
// integrator bookkeeping
// ---------------------------------------------------------------------------
// The controller's decision on the attempt that ended in state s: the state of
// the next attempt, and whether this one is accepted.
__device__ inline double rk_error(const RkState& s) {
  return s.nonfinite ? __builtin_nan("") : __longlong_as_double((long long)s.err_bits);
}
__device__ inline bool rk_accept(const RkState& s, const double* replay) {
  return replay || rk_error(s) <= s.tol;
}
__device__ inline RkState rk_decide(const RkState& s, const double* replay) {
  RkState n = s;
  const double err = rk_error(s);
  const bool accept = rk_accept(s, replay);
  n.err_bits = 0ull;
  n.nonfinite = 0;
  n.last_err = err;
  double next;
  if (replay) {
    n.replay_idx = s.replay_idx + 1;
    next = (n.replay_idx < s.n_replay) ? replay[n.replay_idx] : 0.0;
  } else {
    double fac = 0.2;
    if (err == err)
      fac = (err == 0.0) ? 5.0 : fmin(5.0, fmax(0.2, 0.9 * pow(s.tol / err, 0.2)));
    next = fmin(s.dt * fac, s.dt_max);
  }
  if (accept) {
    n.accepted = s.accepted + 1;
    n.t = (s.final_flag && !replay) ? s.t_end : s.t + s.dt;
  } else {
    n.rejected = s.rejected + 1;
  }
  n.accepted_flag = accept ? 1 : 0;
  if (replay) {
    n.dt = next;
    if (n.replay_idx >= n.n_replay) n.done = 1;
    return n;
  }
  n.dt_prop = next;
  n.final_flag = (n.t + next >= n.t_end) ? 1 : 0;
  if (n.final_flag) next = n.t_end - n.t;
  n.dt = next;
  if (n.t >= n.t_end) n.done = 1;
  else if (next < n.dt_min) { n.done = 1; n.dtmin_hit = 1; }
  return n;
}

// the decision alone: from *in to *out (may be the same)
__global__ void k_rk_controller(const RkState* in, RkState* out, const double* replay, double* dts,
                                long long dts_cap) {
  const RkState s = *in;
  if (s.done) {
    if (out != in) *out = s;
    return;
  }
  if (rk_accept(s, replay) && s.accepted < dts_cap) dts[s.accepted] = s.dt;
  *out = rk_decide(s, replay);
}

// Between two attempts in one pass: the decision on the attempt in *in, its
// commit (m <- m7, k1 <- k7 if accepted) and the next attempt's second-stage state
// m + dt a21 k1 with its x transform (the work of k_xfwd; x.m = m, x.kk[0] =
// k1).  The first wave of every workgroup computes the decision for its
// workgroup; the first workgroup of the leading group writes the new state
// to *out, which is not *in, so that every reader sees the old one.
// Separately (controller on one thread, copy of both arrays, combine) these
// took 19 of the 200 us of an attempt on the 512 x 512 film.
template <typename T>
struct NextArgs {
  XArgs<T> x;
  const RkState* in;
  RkState* out;
  const double* replay;
  double* dts;
  long long dts_cap;
  T* m;
  T* k1;
  const T* m7;
  const T* k7;
  int lead;
};

template <typename T, int HX>
__global__ void __launch_bounds__(kBlock) k_rk_next(NextArgs<T> a) {
  const XArgs<T>& x = a.x;
  const RkState s = *a.in;
  const bool first = blockIdx.x + blockIdx.y + blockIdx.z == 0 && threadIdx.x == 0 && a.lead;
  if (s.done) {
    if (first) *a.out = s;
    return;
  }
  const bool accept = rk_accept(s, a.replay);
  extern __shared__ unsigned char smem_raw[];
  __shared__ double dt_next;
  __shared__ int done_next;
  cpx<T>* A = reinterpret_cast<cpx<T>*>(smem_raw);
  const int hx = HX ? HX : x.hx, ld = HX ? Line<HX>::LD : hx, L = x.L, nl = 3 * L;
  cpx<T>* Bf = A + nl * ld;
  cpx<T>* tw = Bf + nl * ld;
  cpx<T>* wpost = tw + hx;
  auto tw_m = table_mover<T>(tw, x.tw, hx);
  auto wp_m = table_mover<T>(wpost, x.wpost, hx + 1);
  tw_m.issue();
  wp_m.issue();
  if (threadIdx.x < 64) {
    const RkState n = rk_decide(s, a.replay);
    if (threadIdx.x == 0) {
      dt_next = n.dt;
      done_next = n.done;
    }
    if (first) {
      if (accept && s.accepted < a.dts_cap) a.dts[s.accepted] = s.dt;
      *a.out = n;
    }
  }
  int bx, by, bz;
  xcd_block(x.map, bx, by, bz);
  const int r = bz, z = by, y0 = bx * L;
  const size_t rb = (size_t)r * 3 * x.N;
  const unsigned N = (unsigned)x.N;
  const int npair = x.xone ? 1 : (x.nx + 1) / 2;
  const int kw = x.kw;
  const T* __restrict__ ms = (accept ? a.m7 : a.m) + rb;
  const T* __restrict__ ks = (accept ? a.k7 : a.k1) + rb;
  __syncthreads();
  const T dt = (T)dt_next;
  for (int t = threadIdx.x; t < L * kw; t += kBlock) {
    const int l = mdiv(t, x.mkw), k = t - l * kw, y = y0 + l;
    cpx<T> v[3] = {{0, 0}, {0, 0}, {0, 0}};
    if (y < x.ny && k < npair) {
      const bool two = 2 * k + 1 < x.nx;
      const unsigned c0 = (unsigned)(2 * k) + (unsigned)x.nx * (unsigned)(y + x.ny * z);
      const unsigned cell[2] = {c0, two ? c0 + 1 : c0};
      T mv[2][3], pk[2][3];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        ld3(ms, N, cell[h], mv[h]);
        ld3(ks, N, cell[h], pk[h]);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h == 1 && !two) break;
        if (accept) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            a.m[rb + (size_t)c * x.N + cell[h]] = mv[h][c];
            a.k1[rb + (size_t)c * x.N + cell[h]] = pk[h][c];
          }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) mv[h][c] += dt * x.coef[0] * pk[h][c];
#pragma unroll
        for (int c = 0; c < 3; ++c) x.mout[rb + (size_t)c * x.N + cell[h]] = mv[h][c];
        if (x.msr) {  // the convolution acts on M = Ms_i m
          const T w = x.msr[cell[h]];
          mv[h][0] *= w; mv[h][1] *= w; mv[h][2] *= w;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if (h == 0) v[c].re = mv[h][c]; else v[c].im = mv[h][c];
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) A[(c * L + l) * ld + Line<HX>::at(k)] = v[c];
  }
  if (done_next) return;  // the run ended with this attempt: nothing follows
  tw_m.finish();
  wp_m.finish();
  __syncthreads();
  const cpx<T>* X = line_fft<T, false, HX>(A, Bf, nl, x.plan, tw);
  xfwd_store<T, HX>(X, wpost, x.S, r, z, y0, L, hx, x.Kx, x.ny, x.nz, x.Sy, x.xone, x.mL, x.mKx);
}

template <typename T>
__global__ void k_rk_commit(const RkState* st, T* m, const T* m7, T* k1, const T* k7, size_t n) {
  if (!st->accepted_flag) return;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x) {
    m[i] = m7[i];
    k1[i] = k7[i];
  }
}

// Sums of NV interleaved workgroup partials of replica r, in their order
// whatever the number of threads: one thread per replica (lanes = 1), or a wave
// (a workgroup of 64 lanes per replica) that loads a tile of them at once and adds
// each sum in one lane.  A thread that loads each partial before it adds it takes
// some 0.1 us for one: the energies of a 128 x 128 x 8 FP64 block (1024 workgroups)
// 214 us, 81 with the wave, of a 256 x 256 x 32 one (4096) 739 and 237.  Few partials
// of many replicas stay with the threads.
// Returns whether this lane holds the sums; with lanes = 64 the whole workgroup
// calls it.
constexpr int kSumTile = 512;
template <int NV>
__device__ inline bool replica_sums(const double* __restrict__ partial, int nblk, int r, int lanes,
                                    double s[NV]) {
  const double* p = partial + (size_t)r * nblk * NV;
#pragma unroll
  for (int v = 0; v < NV; ++v) s[v] = 0;
  if (lanes == 1) {
    for (int b = 0; b < nblk; ++b)
#pragma unroll
      for (int v = 0; v < NV; ++v) s[v] += p[(size_t)b * NV + v];
    return true;
  }
  __shared__ double tile[kSumTile * NV], sums[NV];
  const int t = threadIdx.x;
  double acc = 0;  // lane v < NV: sum v
  for (int base = 0; base < nblk; base += kSumTile) {
    const int n = min(kSumTile, nblk - base);
    double v[kSumTile / 64 * NV];  // a tile's loads in flight at once
#pragma unroll
    for (int i = 0; i < kSumTile / 64 * NV; ++i)
      v[i] = p[(size_t)base * NV + min(t + 64 * i, n * NV - 1)];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSumTile / 64 * NV; ++i) tile[t + 64 * i] = v[i];
    __syncthreads();
    if (t < NV) {
      int b = 0;
      for (; b + 16 <= n; b += 16) {  // sixteen reads in flight, added in order
        double x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = tile[(b + i) * NV + t];
#pragma unroll
        for (int i = 0; i < 16; ++i) acc += x[i];
      }
      for (; b < n; ++b) acc += tile[b * NV + t];
    }
  }
  if (t < NV) sums[t] = acc;
  __syncthreads();
#pragma unroll
  for (int v = 0; v < NV; ++v) s[v] = sums[v];
  return t == 0;
}
// lanes per replica for nblk partials, the grid of 64-thread workgroups for R
// replicas, and the replica of a thread
inline int sum_lanes(int nblk) { return nblk >= 32 ? 64 : 1; }
inline unsigned sum_grid(int nblk, int R) {
  return sum_lanes(nblk) == 1 ? (unsigned)(R + 63) / 64 : (unsigned)R;
}
__device__ inline int sum_replica(int lanes) {
  return lanes == 1 ? (int)(blockIdx.x * blockDim.x + threadIdx.x) : (int)blockIdx.x;
}

// per-replica fixed-order sums of workgroup partials; the check's time is
// step_after dt, step_after = (*stepdev if set) + the given count
__global__ void k_switch_reduce(const double* partial, int nblk, int R, int lanes, int N,
                                double* tsw, unsigned long long step_after,
                                const unsigned long long* stepdev, double dt) {
  const int r = sum_replica(lanes);
  if (r >= R) return;
  double s[1];
  if (!replica_sums<1>(partial, nblk, r, lanes, s)) return;
  const unsigned long long st = (stepdev ? *stepdev : 0ull) + step_after;
  if (tsw[r] < 0 && s[0] / N < 0) tsw[r] = (double)st * dt;
}

// Retire/refill bookkeeping after a step: a replica whose mean m_z is
// negative ends its trial, records the trial's duration (while fewer than cap
// are recorded), starts trial g + 1 at the next step and is flagged for a
// reset to its initial state.
__global__ void k_refill_check(const double* partial, int nblk, int R, int lanes, int N, int* tgen,
                               unsigned long long* tstart, int* flag, int* counts, double* times,
                               int cap, unsigned long long step_host,
                               const unsigned long long* stepdev, double dt) {
  const int r = sum_replica(lanes);
  if (r >= R) return;
  double sum[1];
  if (!replica_sums<1>(partial, nblk, r, lanes, sum)) return;
  const double s = sum[0];
  const unsigned long long step = (stepdev ? *stepdev : 0ull) + step_host;
  int f = 0;
  if (s / N < 0) {
    const int c = counts[r];
    if (c < cap) times[(size_t)r * cap + c] = (double)(step + 1 - tstart[r]) * dt;
    counts[r] = c + 1;
    tgen[r] += 1;
    tstart[r] = step + 1;
    f = 1;
  }
  flag[r] = f;
}

// Reset of flagged replicas: state (n per replica) and, if present, its half
// spectrum (ns per replica) from the saved initial copies.  Grid (x, R).
template <typename T>
__global__ void k_refill_copy(const int* flag, T* m, const T* m_init, size_t n, cpx<T>* S,
                              const cpx<T>* S_init, size_t ns) {
  const int r = blockIdx.y;
  if (!flag[r]) return;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    m[(size_t)r * n + i] = m_init[(size_t)r * n + i];
  if (S)
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < ns; i += stride)
      S[(size_t)r * ns + i] = S_init[(size_t)r * ns + i];
}

__global__ void k_fill_i32(int* p, size_t n, int v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_u64(unsigned long long* p, size_t n, unsigned long long v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_f64(double* p, size_t n, double v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// max over cells of |v| for vectors stored component-major per replica
// (n cells per replica, R replicas): per-workgroup maxima, then one workgroup
// folds them (part: gridDim.x doubles).
template <typename T>
__global__ void k_norm_max(const T* v, size_t n, int R, double* part) {
  __shared__ double red[256];
  double mx = 0;
  const size_t total = n * (size_t)R;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (size_t)gridDim.x * blockDim.x) {
    const size_t r = i / n, c = i - r * n;
    const T* b = v + r * 3 * n + c;
    const double x = (double)b[0], y = (double)b[n], z = (double)b[2 * n];
    mx = fmax(mx, sqrt(x * x + y * y + z * z));
  }
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void k_max_fold(double* part, int n) {
  __shared__ double red[256];
  double mx = 0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) mx = fmax(mx, part[i]);
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[n] = red[0];
}

// step counter of captured graphs: set before a replay, advanced inside it
__global__ void k_set_u64(unsigned long long* p, unsigned long long v) { *p = v; }
__global__ void k_inc_u64(unsigned long long* p, unsigned long long d) { *p += d; }

__global__ void k_energy_reduce(const double* partial, int nblk, int R, int lanes, double cq,
                                double cz, double* E) {
  const int r = sum_replica(lanes);
  if (r >= R) return;
  double s[5];
  if (!replica_sums<5>(partial, nblk, r, lanes, s)) return;
  double tot = 0;
  for (int v = 0; v < 5; ++v) {
    const double e = (v == 4 ? cz : cq) * s[v];
    E[(size_t)r * 6 + v] = e;
    tot += e;
  }
  E[(size_t)r * 6 + 5] = tot;
}

// trace[accepted] = sum over replicas of E[.][5] when the last attempt was accepted
__global__ void k_trace_store(const RkState* st, const double* E, int R, double* trace,
                              long long cap, int force0) {
  if (!force0 && !st->accepted_flag) return;
  const long long idx = force0 ? 0 : st->accepted;
  if (idx >= cap) return;
  double s = 0;
  for (int r = 0; r < R; ++r) s += E[(size_t)r * 6 + 5];
  trace[idx] = s;
}

template <typename T>
__global__ void k_topo(const T* m, int nx, int ny, int N, int pbcx, int pbcy, double i2dx,
                       double i2dy, double* partial, int nblk) {
  __shared__ double red[kBlock];
  const int r = blockIdx.y;
  const size_t rb = (size_t)r * 3 * N;
  double acc = 0;
  for (int cell = blockIdx.x * blockDim.x + threadIdx.x; cell < nx * ny;
       cell += gridDim.x * blockDim.x) {
    const int x = cell % nx, y = cell / nx;
    double mc[3], xm[3], xp[3], ym[3], yp[3];
    for (int c = 0; c < 3; ++c) mc[c] = m[rb + (size_t)c * N + cell];
    auto get = [&](int xx, int yy, double v[3]) {
      for (int c = 0; c < 3; ++c) v[c] = m[rb + (size_t)c * N + xx + (size_t)nx * yy];
    };
    if (nx > 1) {
      if (x > 0) get(x - 1, y, xm); else if (pbcx) get(nx - 1, y, xm); else get(x, y, xm);
      if (x < nx - 1) get(x + 1, y, xp); else if (pbcx) get(0, y, xp); else get(x, y, xp);
    } else { get(x, y, xm); get(x, y, xp); }
    if (ny > 1) {
      if (y > 0) get(x, y - 1, ym); else if (pbcy) get(x, ny - 1, ym); else get(x, y, ym);
      if (y < ny - 1) get(x, y + 1, yp); else if (pbcy) get(x, 0, yp); else get(x, y, yp);
    } else { get(x, y, ym); get(x, y, yp); }
    double a[3], b[3];
    for (int c = 0; c < 3; ++c) { a[c] = (xp[c] - xm[c]) * i2dx; b[c] = (yp[c] - ym[c]) * i2dy; }
    acc += mc[0] * (a[1] * b[2] - a[2] * b[1]) + mc[1] * (a[2] * b[0] - a[0] * b[2]) +
           mc[2] * (a[0] * b[1] - a[1] * b[0]);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[(size_t)r * nblk + blockIdx.x] = red[0];
}

__global__ void k_topo_reduce(const double* partial, int nblk, int R, double scale, double* Q) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  double s = 0;
  for (int b = 0; b < nblk; ++b) s += partial[(size_t)r * nblk + b];
  Q[r] = s * scale;
}

}  // namespace mmx
