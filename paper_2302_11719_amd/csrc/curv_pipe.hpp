// Curvilinear model: sampled rollouts as a pipeline of three waves per 64 samples
// (as pipe.hpp): noise and controls; the body states (v_x, v_y, r, omega_F,
// omega_R), whose forces depend on no path coordinate; the path states (e_psi,
// e_y, s) and the cost.  Same operations in the same order as rollout_sample_c8,
// so the costs are the same bits.
#pragma once

#include "adjoint_pipe.hpp"
#include "curv8.hpp"

namespace smppi {

constexpr int C8P_D = 4;             // ring slots
constexpr int C8P_BLK = 3 * WAVE;

template <class R>
struct C8PipeLds {
  R ctl[C8P_D][5][WAVE];       // delta, sin, cos, throttle, control cost
  Quad<R> vel[C8P_D][3][WAVE];  // v_x, v_y, r at the four RK4 stages
  R vxT[WAVE];                 // v_x of x_T
  int cnt[8];                  // steps: [0] noise, [1] body written; [4] read by the path wave
};

template <class R>
__device__ __forceinline__ void c8_put_ctl(C8PipeLds<R>& P, const DevCost<R>& C, int t, int s, R v0, R v1, R u0, R u1) {
  const Ctl8<R> c = ctl8(u0, u1);
  R(*o)[WAVE] = P.ctl[t % C8P_D];
  o[0][s] = c.delta;
  o[1][s] = c.sd;
  o[2][s] = c.cd;
  o[3][s] = c.thr;
  o[4][s] = pipe_ctl_cost(C, v0, v1, u0, u1);
}

// RK4 combination k1 + 2 k2 + 2 k3 + k4 (as rk4_c8).
template <class R>
__device__ __forceinline__ R c8_comb(R h6, R a1, R a2, R a3, R a4, R xv) {
  return fma_r(h6, fma_r(R(2), a2 + a3, a1) + a4, xv);
}

// The body wave.  put(t, x): called with the body states of x_{t+1}.
template <class R, class Put>
__device__ void c8_pipe_body(const DevModel<R>& M, const DevWheels<R>& Wh, C8<R> x, int T, C8PipeLds<R>& P,
                             uint32_t* err, Put put) {
  const int lane = threadIdx.x % WAVE;
  const R h = M.dt, h2 = R(0.5) * M.dt, h6 = M.dt * R(1.0 / 6.0);
  int seen = 0;
  for (int t = 0; t < T; ++t) {
    wave_wait(&P.cnt[0], t, seen, err);
    const R(*cr)[WAVE] = P.ctl[t % C8P_D];
    Ctl8<R> c;
    c.delta = cr[0][lane];
    c.sd = cr[1][lane];
    c.cd = cr[2][lane];
    c.thr = cr[3][lane];
    C8<R> k1 = zero8<R>(), k2 = zero8<R>(), k3 = zero8<R>(), k4 = zero8<R>();
    deriv_c8_body(M, Wh, c, x, k1);
    const C8<R> X2 = axpy8(h2, k1, x);
    R f2, f4;
    deriv_c8_body(M, Wh, c, X2, k2, &f2);
    const C8<R> X3 = axpy8(h2, k2, x);
    deriv_c8_body(M, Wh, c, X3, k3);
    const C8<R> X4 = axpy8(h, k3, x);
    deriv_c8_body(M, Wh, c, X4, k4, &f4);
    Quad<R>(*o)[WAVE] = P.vel[t % C8P_D];
    o[0][lane] = Quad<R>{{x.vx, X2.vx, X3.vx, X4.vx}};
    o[1][lane] = Quad<R>{{x.vy, X2.vy, X3.vy, X4.vy}};
    o[2][lane] = Quad<R>{{x.r, X2.r, X3.r, X4.r}};
    x.vx = c8_comb(h6, k1.vx, k2.vx, k3.vx, k4.vx, x.vx);
    x.vy = c8_comb(h6, k1.vy, k2.vy, k3.vy, k4.vy, x.vy);
    x.r = c8_comb(h6, k1.r, k2.r, k3.r, k4.r, x.r);
    // (the products of omega_F' fused into the sums, as in rollout_sample_c8)
    x.wF = fma_r(h6, fma_r(-Wh.rw_Iw, f4, fma_r(R(2), fma_r(Wh.rw_Iw, -f2, k3.wF), k1.wF)), x.wF);
    x.wR = c8_comb(h6, k1.wR, k2.wR, k3.wR, k4.wR, x.wR);
    if (t == T - 1) P.vxT[lane] = x.vx;
    wave_publish(&P.cnt[1], t + 1);
    put(t, x);
  }
}

// The path part of a step from the stage velocities: advances (e_psi, e_y, s).
template <class R>
__device__ __forceinline__ void c8_path_step(const DevModel<R>& M, const CurvView<R>& cv, const Quad<R>& vx,
                                             const Quad<R>& vy, const Quad<R>& r, C8<R>& x) {
  const R h = M.dt, h2 = R(0.5) * M.dt, h6 = M.dt * R(1.0 / 6.0);
  C8<R> k1 = zero8<R>(), k2 = zero8<R>(), k3 = zero8<R>(), k4 = zero8<R>();
  C8<R> X = x;
  X.vx = vx.v[0]; X.vy = vy.v[0]; X.r = r.v[0];
  deriv_c8_path(cv, X, k1);
  X.vx = vx.v[1]; X.vy = vy.v[1]; X.r = r.v[1];
  X.ep = fma_r(h2, k1.ep, x.ep); X.ey = fma_r(h2, k1.ey, x.ey); X.s = fma_r(h2, k1.s, x.s);
  deriv_c8_path(cv, X, k2);
  X.vx = vx.v[2]; X.vy = vy.v[2]; X.r = r.v[2];
  X.ep = fma_r(h2, k2.ep, x.ep); X.ey = fma_r(h2, k2.ey, x.ey); X.s = fma_r(h2, k2.s, x.s);
  deriv_c8_path(cv, X, k3);
  X.vx = vx.v[3]; X.vy = vy.v[3]; X.r = r.v[3];
  X.ep = fma_r(h, k3.ep, x.ep); X.ey = fma_r(h, k3.ey, x.ey); X.s = fma_r(h, k3.s, x.s);
  deriv_c8_path(cv, X, k4);
  x.ep = c8_comb(h6, k1.ep, k2.ep, k3.ep, k4.ep, x.ep);
  x.ey = c8_comb(h6, k1.ey, k2.ey, k3.ey, k4.ey, x.ey);
  x.s = c8_comb(h6, k1.s, k2.s, k3.s, k4.s, x.s);
}

// Sampled costs of 64 samples per workgroup, grid (ceil(k_max / 64), B).
template <class R>
__global__ __launch_bounds__(C8P_BLK) void k_rollout_c8_pipe(C8Args<R> a, R* S_out, R* eps_out) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int b = blockIdx.y;
  C8Dims d;
  if (!c8_dims(a, b, d)) return;
  const int m_base = blockIdx.x * WAVE;
  if (m_base >= d.K) return;
  R* Vs;
  const CurvView<R> cv = c8_stage(a, b, d, reinterpret_cast<R*>(smem), &Vs);
  C8PipeLds<R>& P = *reinterpret_cast<C8PipeLds<R>*>(smem + c8_stage_bytes<R>(a.n_max, a.t_max));
  if (threadIdx.x < 8) P.cnt[threadIdx.x] = 0;
  __syncthreads();
  const int w = threadIdx.x / WAVE, lane = threadIdx.x % WAVE, T = d.T, m = m_base + lane;
  const DevModel<R> M = model_in_vgprs(a.M);
  const DevCost<R> C = cost_in_vgprs(a.C);
  const C8<R> x0 = load_c8(a.x0 + 8 * (size_t)b);
  if (w == 0) {
    R* eo = (eps_out && m < d.K) ? eps_out + (size_t)(d.k0 + m) * a.t_max * 2 : nullptr;
    pipe_noise<R, 64, C8P_D, 1>(M, C, Vs, T, a.seed, (uint32_t)m, (uint32_t)(a.pid_base + b), a.iter[b], a.nominal != 0,
                                P.cnt, a.err, [&](int t, int s, R v0, R v1, R, R, R u0, R u1) {
                                  c8_put_ctl(P, C, t, s, v0, v1, u0, u1);
                                  if (eo) {
                                    eo[2 * t] = u0 - v0;
                                    eo[2 * t + 1] = u1 - v1;
                                  }
                                });
  } else if (w == 1) {
    c8_pipe_body(M, a.Wh, x0, T, P, a.err, [](int, const C8<R>&) {});
  } else {
    C8<R> x = x0;
    R h0 = fma_r(-x.ey, x.ey, cv.w2);
    bool outside = h0 < R(0);
    R S = C.C_cbf * fmax((C.alpha - R(1)) * h0, R(0));
    int seen = 0;
    for (int t = 0; t < T; ++t) {
      wave_wait(&P.cnt[1], t, seen, a.err);
      const Quad<R>(*o)[WAVE] = P.vel[t % C8P_D];
      const Quad<R> vx = o[0][lane], vy = o[1][lane], r = o[2][lane];
      const R ctl = P.ctl[t % C8P_D][4][lane];
      wave_publish(&P.cnt[4], t + 1);
      const R dv = vx.v[0] - C.v_g;
      R q = fma_r(C.q_ey, x.ey * x.ey, C.q_v * dv * dv);
      if (outside) q += C.C_obs;
      S += q + ctl;
      c8_path_step(M, cv, vx, vy, r, x);
      const R h1 = fma_r(-x.ey, x.ey, cv.w2);
      S = fma_r(C.C_cbf, fmax(fma_r(C.alpha, h0, -h1), R(0)), S);
      h0 = h1;
      outside = h1 < R(0);
    }
    const R dv = P.vxT[lane] - C.v_g;
    R q = fma_r(C.q_ey, x.ey * x.ey, C.q_v * dv * dv);
    if (outside) q += C.C_obs;
    S = fma_r(C.phi_w, q, S);
    if (m < d.K) S_out[d.k0 + m] = S;
  }
}

}  // namespace smppi
