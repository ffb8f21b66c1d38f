// Plant of closed-loop studies: the robot integrated with classical RK4 on its
// continuous dynamics (the simulations of Sec. IV-E run the plant at 1 kHz with
// RK4), one 16-lane group per instance (for very many instances one thread,
// launch_plant), FP64 arithmetic on FP32 states.
//
// A step is one serial chain of 4 substeps forward dynamics, so its time is one
// evaluation's latency. Lane j < n runs the recursive Newton-Euler pass for unit
// acceleration of joint j (column j of the inertia matrix), lane n the pass for the
// bias forces, all at once; the sines and cosines are one evaluation per lane and
// the n x n system is eliminated with one row per lane, entries passing between
// lanes by row broadcasts. 256 7-DoF instances, 10 substeps: 208 us with one
// thread per instance (inertia matrix, bias forces, Cholesky and solves in
// sequence), 82 us.
#include <type_traits>
#include <utility>

#include "gato_launch.hpp"

namespace gato {

namespace {

// Entry of lane I of the 16-lane row.
template <int CTRL>
__device__ __forceinline__ double row_dpp(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
template <int I>
__device__ __forceinline__ double from_lane(double v) {
  return row_dpp<0x150 + I>(v);   // row_newbcast:I
}
template <class F, int... I>
__device__ __forceinline__ void unrolled(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

// The chain's constants in FP64 (products as the FP32 routines round them).
template <int ND>
struct PlantChain {
  double L[ND], m[ND], mc[ND], I[ND][3], fe[3], Lt, g, ks;
  bool spring, has_fe;
};

// Generalised force of one Newton-Euler pass (the recursion of rnea, gato_rbd.hpp)
// for joint velocities qd, unit acceleration of joint `unit` (none: outside 0..ND-1)
// and base acceleration g.
template <int ND>
__device__ __forceinline__ void newton_euler(const PlantChain<ND> &ch, const double *c, const double *s,
                                             const double *qd, int unit, double g, bool force, double *tau) {
  double fn[ND][3], ff[ND][3];
  double w[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0}, aw[3] = {0.0, 0.0, 0.0}, av[3] = {0.0, 0.0, g};
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const double L = ch.L[i], a = unit == i ? 1.0 : 0.0;
    if (i & 1) {
      v[0] += L * w[1];
      v[1] -= L * w[0];
      rot_E<true>(c[i], s[i], w[0], w[1], w[2]);
      rot_E<true>(c[i], s[i], v[0], v[1], v[2]);
      av[0] += L * aw[1];
      av[1] -= L * aw[0];
      rot_E<true>(c[i], s[i], aw[0], aw[1], aw[2]);
      rot_E<true>(c[i], s[i], av[0], av[1], av[2]);
      w[1] += qd[i];
      aw[1] += a;
      aw[0] -= w[2] * qd[i];
      aw[2] += w[0] * qd[i];
      av[0] -= v[2] * qd[i];
      av[2] += v[0] * qd[i];
    } else {
      v[0] += L * w[1];
      v[1] -= L * w[0];
      rot_E<false>(c[i], s[i], w[0], w[1], w[2]);
      rot_E<false>(c[i], s[i], v[0], v[1], v[2]);
      av[0] += L * aw[1];
      av[1] -= L * aw[0];
      rot_E<false>(c[i], s[i], aw[0], aw[1], aw[2]);
      rot_E<false>(c[i], s[i], av[0], av[1], av[2]);
      w[2] += qd[i];
      aw[2] += a;
      aw[0] += w[1] * qd[i];
      aw[1] -= w[0] * qd[i];
      av[0] += v[1] * qd[i];
      av[1] -= v[0] * qd[i];
    }
    const double m = ch.m[i], mc = ch.mc[i], Ix = ch.I[i][0], Iy = ch.I[i][1], Iz = ch.I[i][2];
    const double hvn[3] = {Ix * w[0] - mc * v[1], Iy * w[1] + mc * v[0], Iz * w[2]};
    const double hvf[3] = {m * v[0] + mc * w[1], m * v[1] - mc * w[0], m * v[2]};
    const double han[3] = {Ix * aw[0] - mc * av[1], Iy * aw[1] + mc * av[0], Iz * aw[2]};
    const double haf[3] = {m * av[0] + mc * aw[1], m * av[1] - mc * aw[0], m * av[2]};
    fn[i][0] = han[0] + (w[1] * hvn[2] - w[2] * hvn[1]) + (v[1] * hvf[2] - v[2] * hvf[1]);
    fn[i][1] = han[1] + (w[2] * hvn[0] - w[0] * hvn[2]) + (v[2] * hvf[0] - v[0] * hvf[2]);
    fn[i][2] = han[2] + (w[0] * hvn[1] - w[1] * hvn[0]) + (v[0] * hvf[1] - v[1] * hvf[0]);
    ff[i][0] = haf[0] + (w[1] * hvf[2] - w[2] * hvf[1]);
    ff[i][1] = haf[1] + (w[2] * hvf[0] - w[0] * hvf[2]);
    ff[i][2] = haf[2] + (w[0] * hvf[1] - w[1] * hvf[0]);
  }
  // The wrench against the external force starts at the tip: (-(r x f), -f), r = (0, 0, Lt).
  double n[3] = {0.0, 0.0, 0.0}, f[3] = {0.0, 0.0, 0.0};
  if (force) {
    double e[3] = {ch.fe[0], ch.fe[1], ch.fe[2]};
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      if (i & 1) rot_E<true>(c[i], s[i], e[0], e[1], e[2]);
      else rot_E<false>(c[i], s[i], e[0], e[1], e[2]);
    }
    n[0] = ch.Lt * e[1];
    n[1] = -(ch.Lt * e[0]);
#pragma unroll
    for (int a = 0; a < 3; ++a) f[a] = -e[a];
  }
#pragma unroll
  for (int i = ND - 1; i >= 0; --i) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      n[a] += fn[i][a];
      f[a] += ff[i][a];
    }
    tau[i] = (i & 1) ? n[1] : n[2];
    if (i > 0) {
      if (i & 1) rot_R<true>(c[i], s[i], n[0], n[1], n[2]), rot_R<true>(c[i], s[i], f[0], f[1], f[2]);
      else rot_R<false>(c[i], s[i], n[0], n[1], n[2]), rot_R<false>(c[i], s[i], f[0], f[1], f[2]);
      n[0] -= ch.L[i] * f[1];
      n[1] += ch.L[i] * f[0];
    }
  }
}

// Forward dynamics of one instance, lane i < ND holding q_i, qd_i and tau_i and
// receiving qdd_i. ok becomes false for an inertia matrix that is not positive
// definite (a pivot of the elimination that is not positive).
template <int ND>
__device__ __forceinline__ double lane_dynamics(const PlantChain<ND> &ch, int lane, double q, double qd, double tau,
                                                bool &ok) {
  if (ch.spring) {
    const double l = row_dpp<0x111>(q), r = row_dpp<0x101>(q);   // lanes - 1 and + 1
    return tau - ch.ks * (2.0 * q - (lane > 0 ? l : 0.0) - (lane < ND - 1 ? r : 0.0));
  }
  const bool bias = lane == ND;
  double sq, cq;
  sincos(q, &sq, &cq);
  double c[ND], s[ND], v[ND], t[ND];
  constexpr auto joints = std::make_integer_sequence<int, ND>{};
  unrolled([&](auto i) {
    c[i] = from_lane<i>(cq);
    s[i] = from_lane<i>(sq);
    v[i] = from_lane<i>(qd);
    v[i] = bias ? v[i] : 0.0;
  }, joints);
  newton_euler<ND>(ch, c, s, v, lane, bias ? ch.g : 0.0, bias && ch.has_fe, t);
  // Row `lane` of the inertia matrix (symmetric) and the right-hand side.
  double rhs = 0.0, inv = 0.0;
  unrolled([&](auto i) {
    const double b = from_lane<ND>(t[i]);
    rhs = lane == i ? tau - b : rhs;
  }, joints);
  unrolled([&](auto p) {
    const double piv = from_lane<p>(t[p]);
    ok = ok && piv > 0.0;
    const double pinv = 1.0 / piv;
    inv = lane == p ? pinv : inv;
    const double f = lane == p ? 0.0 : t[p] * pinv;
    rhs -= f * from_lane<p>(rhs);
#pragma unroll
    for (int j = p + 1; j < ND; ++j) t[j] -= f * from_lane<p>(t[j]);
  }, joints);
  return rhs * inv;
}

// RK4 over h; returns whether the result is finite and every inertia matrix was
// positive definite. q, qd: lane i < ND its joint's state, in and out.
template <int ND>
__device__ __forceinline__ bool plant_rk4(const Chain &c, const float *fe, bool has_fe, int lane, double h, int substeps,
                                          double &q, double &qd, double tau) {
  PlantChain<ND> ch;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    ch.L[i] = c.Lp[i];
    ch.m[i] = c.m[i];
    ch.mc[i] = c.m[i] * c.cz[i];
#pragma unroll
    for (int a = 0; a < 3; ++a) ch.I[i][a] = c.Io[i][a];
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) ch.fe[a] = fe[a];
  ch.Lt = c.Lt;
  ch.g = c.g;
  ch.ks = c.ks;
  ch.spring = c.model == 1;
  ch.has_fe = has_fe;
  const double d = h / substeps;
  bool ok = true;
  for (int i = 0; i < substeps; ++i) {
    // The four stages: slopes at (q, qd), at half a step twice, at a whole step.
    double aq = 0.0, av = 0.0, zq = q, zv = qd;
#pragma unroll 1
    for (int st = 0; st < 4; ++st) {
      const double kq = zv, kv = lane_dynamics<ND>(ch, lane, zq, zv, tau, ok);
      const double wt = st == 0 || st == 3 ? 1.0 : 2.0, dt = st == 2 ? d : 0.5 * d;
      aq += wt * kq;
      av += wt * kv;
      zq = q + dt * kq;
      zv = qd + dt * kv;
    }
    q += d / 6.0 * aq;
    qd += d / 6.0 * av;
  }
  return ok && isfinite(q) && isfinite(qd);
}

__global__ __launch_bounds__(64) void plant_kernel(PlantArgs a) {
  const int lane = threadIdx.x & 15;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 4);
  if (r >= a.n) return;
  const int sid = a.slots ? a.slots[r] : r;
  if (sid < 0 || sid >= a.M) {
    if (lane == 0) a.status[r] = GATO_ST_NONFINITE;
    return;
  }
  const Chain &ch = a.desc[sid].chain;
  float fe[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) fe[c] = a.fext ? a.fext[(size_t)r * 3 + c] : ch.fe[c];
  const bool has_fe = a.fext ? (fe[0] != 0.f || fe[1] != 0.f || fe[2] != 0.f) && ch.model == 0 : ch.has_fe != 0;
  const int n = ch.n;
  const bool own = lane < n;
  const size_t xo = (size_t)r * a.nx_max;
  double q = own ? (double)a.x[xo + lane] : 0.0, qd = own ? (double)a.x[xo + n + lane] : 0.0;
  const double tau = own ? (double)a.tau[(size_t)r * a.nu_max + lane] : 0.0;
  bool fine = false;
  switch (n) {
    case 3: fine = plant_rk4<3>(ch, fe, has_fe, lane, a.h, a.substeps, q, qd, tau); break;
    case 6: fine = plant_rk4<6>(ch, fe, has_fe, lane, a.h, a.substeps, q, qd, tau); break;
    case 7: fine = plant_rk4<7>(ch, fe, has_fe, lane, a.h, a.substeps, q, qd, tau); break;
    default: break;
  }
  if (own) {
    a.xn[xo + lane] = (float)q;
    a.xn[xo + n + lane] = (float)qd;
  }
  const unsigned long long bad = __ballot(own && !fine) >> (threadIdx.x & 48);
  if (lane == 0) a.status[r] = (bad & 0xffffull) ? GATO_ST_NONFINITE : 0u;
}

// The same with one thread per instance: about twice the latency, but a sixteenth of
// the wavefronts.
template <int ND>
__device__ __forceinline__ bool plant_rk4_thread(const Chain &ch, double h, int substeps, const float *x,
                                                 const float *tau, float *xn) {
  constexpr int NX = 2 * ND;
  double y[NX], k[NX], acc[NX], z[NX], u[ND], L[ND][ND];
#pragma unroll
  for (int i = 0; i < NX; ++i) y[i] = (double)x[i];
#pragma unroll
  for (int i = 0; i < ND; ++i) u[i] = (double)tau[i];
  const double d = h / substeps;
  bool fine = true;
  for (int s = 0; s < substeps; ++s) {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      acc[i] = 0.0;
      z[i] = y[i];
    }
#pragma unroll 1
    for (int st = 0; st < 4; ++st) {
#pragma unroll
      for (int i = 0; i < ND; ++i) k[i] = z[ND + i];
      fine = forward_dynamics<ND, double>(ch, z, z + ND, u, k + ND, L) && fine;
      const double wt = st == 0 || st == 3 ? 1.0 : 2.0, dt = st == 2 ? d : 0.5 * d;
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        acc[i] += wt * k[i];
        z[i] = y[i] + dt * k[i];
      }
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) y[i] += d / 6.0 * acc[i];
  }
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    xn[i] = (float)y[i];
    fine = fine && isfinite(y[i]);
  }
  return fine;
}

__global__ __launch_bounds__(64) void plant_thread_kernel(PlantArgs a) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= a.n) return;
  const int sid = a.slots ? a.slots[r] : r;
  if (sid < 0 || sid >= a.M) {
    a.status[r] = GATO_ST_NONFINITE;
    return;
  }
  Chain ch = a.desc[sid].chain;
  if (a.fext) {
    for (int c = 0; c < 3; ++c) ch.fe[c] = a.fext[(size_t)r * 3 + c];
    ch.has_fe = (ch.fe[0] != 0.f || ch.fe[1] != 0.f || ch.fe[2] != 0.f) && ch.model == 0;
  }
  const float *x = a.x + (size_t)r * a.nx_max;
  const float *tau = a.tau + (size_t)r * a.nu_max;
  float *xn = a.xn + (size_t)r * a.nx_max;
  bool fine = false;
  switch (ch.n) {
    case 3: fine = plant_rk4_thread<3>(ch, a.h, a.substeps, x, tau, xn); break;
    case 6: fine = plant_rk4_thread<6>(ch, a.h, a.substeps, x, tau, xn); break;
    case 7: fine = plant_rk4_thread<7>(ch, a.h, a.substeps, x, tau, xn); break;
    default: break;
  }
  a.status[r] = fine ? 0u : GATO_ST_NONFINITE;
}

// Tip position of every knot of every solve, one thread per (solve, knot);
// zero beyond a solve's horizon and for the double-integrator model.
__global__ __launch_bounds__(256) void tip_kernel(const SolveDesc *desc, int M, int N_max, int nx_max,
                                                  const float *X, float *P) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= M * N_max) return;
  const int sid = t / N_max, k = t % N_max;
  const SolveDesc &D = desc[sid];
  float p[3] = {0.f, 0.f, 0.f};
  if (k < D.N && D.chain.model == 0) {
    const float *q = X + (size_t)t * nx_max;
    switch (D.n) {
      case 3: tip_position<3>(D.chain, q, p); break;
      case 6: tip_position<6>(D.chain, q, p); break;
      case 7: tip_position<7>(D.chain, q, p); break;
      default: break;
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) P[(size_t)t * 3 + c] = p[c];
}

// Fills n doubles with v (a kernel, so that callers may capture it in a graph).
__global__ __launch_bounds__(256) void fill_kernel(double *p, size_t n, double v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Shifts the resident trajectory and multipliers of slot slots[b] one knot
// towards the start, the last knot repeated; one workgroup per slot, staged
// through LDS so that the in-place update reads only old values.
__global__ __launch_bounds__(256) void shift_kernel(const SolveDesc *desc, int M, int n, const int *slots, int N_max,
                                                    int nx_max, int nu_max, float *X, float *U, double *lam) {
  __shared__ float xs[GATO_MAX_KNOTS * 2 * kMaxDof];
  __shared__ float us[GATO_MAX_KNOTS * kMaxDof];
  __shared__ double ls[GATO_MAX_KNOTS * 2 * kMaxDof];
  if ((int)blockIdx.x >= n) return;
  const int sid = slots[blockIdx.x];
  if (sid < 0 || sid >= M) return;   // uniform across the workgroup
  const int N = desc[sid].N;
  float *Xs = X + (size_t)sid * N_max * nx_max;
  float *Us = U + (size_t)sid * (N_max - 1) * nu_max;
  double *Ls = lam + (size_t)sid * N_max * nx_max;
  const int nxe = N * nx_max, nue = (N - 1) * nu_max;
  for (int t = threadIdx.x; t < nxe; t += blockDim.x) {
    xs[t] = Xs[t];
    ls[t] = Ls[t];
  }
  for (int t = threadIdx.x; t < nue; t += blockDim.x) us[t] = Us[t];
  __syncthreads();
  for (int t = threadIdx.x; t < nxe; t += blockDim.x) {
    const int k = t / nx_max, j = t - k * nx_max;
    const int ks = min(k + 1, N - 1);
    Xs[t] = xs[ks * nx_max + j];
    Ls[t] = ls[ks * nx_max + j];
  }
  for (int t = threadIdx.x; t < nue; t += blockDim.x) {
    const int k = t / nu_max, j = t - k * nu_max;
    Us[t] = us[min(k + 1, N - 2) * nu_max + j];
  }
}

// Hypothesis selection (gato_select_hypotheses): one wavefront per instance p.
// Lane l scores hypotheses j = l, l + 64, ... by the Euclidean distance between
// their one-step predictions and the measured state (FP64 sums in index
// order), a butterfly takes the smallest distance (the smaller j on ties), the
// estimate moves to that hypothesis and the instance's hypotheses are
// re-centred on it in the device descriptors.
__global__ __launch_bounds__(64) void select_kernel(SolveDesc *desc, int P, int H, int nx_max, const float *pred,
                                                    const float *meas, const double *off, double *est, int *sel,
                                                    double *dist) {
  __shared__ double e[3];
  const int p = blockIdx.x;
  if (p >= P) return;   // uniform across the workgroup
  const int lane = threadIdx.x;
  const size_t first = (size_t)p * H;
  const int nx = 2 * desc[first].n;
  const float *ms = meas + (size_t)p * nx_max;
  double best = INFINITY;
  int bj = H;   // none yet
  for (int j = lane; j < H; j += 64) {
    const float *q = pred + (first + j) * nx_max;
    double s = 0.0;
    for (int i = 0; i < nx; ++i) {
      const double d = (double)q[i] - (double)ms[i];
      s += d * d;
    }
    const double dj = sqrt(s);
    if (dist) dist[first + j] = dj;
    if (dj < best) {   // j ascends per lane, so ties keep the smaller j; NaN never wins
      best = dj;
      bj = j;
    }
  }
  for (int w = 32; w >= 1; w >>= 1) {
    const double ob = __shfl_xor(best, w);
    const int oj = __shfl_xor(bj, w);
    if (ob < best || (ob == best && oj < bj)) {
      best = ob;
      bj = oj;
    }
  }
  const int j = bj < H ? bj : 0;   // every distance non-finite: keep the estimate
  if (lane < 3) {
    const double v = est[(size_t)p * 3 + lane] + off[(size_t)j * 3 + lane];
    est[(size_t)p * 3 + lane] = v;
    e[lane] = v;
  }
  if (lane == 0 && sel) sel[p] = j;
  __syncthreads();
  for (int jj = lane; jj < H; jj += 64) {
    Chain &c = desc[first + jj].chain;
    float f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      f[a] = (float)(e[a] + off[(size_t)jj * 3 + a]);
      c.fe[a] = f[a];
    }
    c.has_fe = (f[0] != 0.f || f[1] != 0.f || f[2] != 0.f) ? 1 : 0;
  }
}

}  // namespace

hipError_t launch_select(SolveDesc *desc, int P, int H, int nx_max, const float *pred, const float *meas,
                         const double *off, double *est, int *sel, double *dist, hipStream_t s) {
  hipLaunchKernelGGL(select_kernel, dim3(P), dim3(64), 0, s, desc, P, H, nx_max, pred, meas, off, est, sel, dist);
  return hipGetLastError();
}

const void *fill_kernel_fn() { return reinterpret_cast<const void *>(&fill_kernel); }

hipError_t launch_fill(double *p, size_t n, double v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_shift(const SolveDesc *desc, int M, int n, const int *slots, int N_max, int nx_max, int nu_max,
                        float *X, float *U, double *lam, hipStream_t s) {
  hipLaunchKernelGGL(shift_kernel, dim3(n), dim3(256), 0, s, desc, M, n, slots, N_max, nx_max, nu_max, X, U, lam);
  return hipGetLastError();
}

hipError_t launch_tips(const SolveDesc *desc, int M, int N_max, int nx_max, const float *X, float *P,
                       hipStream_t s) {
  const int n = M * N_max;
  hipLaunchKernelGGL(tip_kernel, dim3((n + 255) / 256), dim3(256), 0, s, desc, M, N_max, nx_max, X, P);
  return hipGetLastError();
}

// Lane groups as long as their rounds of the device (256 CUs of four wavefronts of
// four groups) take less time than the one round of a thread per instance. us per
// call of 10 substeps, groups / threads, at 4096, 8192, 12288 and 65536 instances:
// 3 DoF 53 / 81, 90 / 82, 128 / 82, 609 / 96; 6 DoF 88 / 171, 161 / 172, 235 / 172,
// 1125 / 206; 7 DoF 107 / 205, 197 / 206, 289 / 209, 1343 / 251. (nu_max: the
// batch's largest robot, which sets the time.)
hipError_t launch_plant(const PlantArgs &a, hipStream_t s) {
  const int rounds = a.nu_max <= 3 ? 1 : 2;
  if (a.n > rounds * 4096) hipLaunchKernelGGL(plant_thread_kernel, dim3((a.n + 63) / 64), dim3(64), 0, s, a);
  else hipLaunchKernelGGL(plant_kernel, dim3((a.n + 3) / 4), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace gato
