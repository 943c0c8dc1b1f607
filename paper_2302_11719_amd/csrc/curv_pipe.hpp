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

// ---------------------------------------------------------------- adjoint
// As k_backward_pipe: the forward pass stores every state, and the reverse sweep
// follows the model's cascade backwards; the path's cotangent (e_psi, e_y, s) depends
// on no other, the body's takes the path's contribution per RK4 stage:
//   wave 0: body states and tyre terms of the four stages, from the stored state;
//   wave 1: path states of the stages, barrier gradient, the path's cotangent;
//   wave 2: the body's cotangent and the control gradient;
//   wave 3: the clip, the control cost, the sum over the 64 samples.
// The path wave bounds both sweeps (two curvature lookups in LDS per stage on its
// chain: about 1400 cycles per step forward, 2000 reverse).  Against one wave per
// 64 samples with recomputation: K = 4096, T = 50 191 -> 79.5 us (FP64 458 -> 148),
// K = 65536, T = 100 388 -> 261 us, 146 us when all but 100 samples have zero
// upstream.
template <class R>
struct C8RevLds {
  // per stage: v_x, v_y, r, 1/v, F_xF, F_yF, the forces' derivatives with respect to
  // v_x through 1/v (q, p, z, a), a cos - v_x sin (wave 0); path parts of the v_x,
  // v_y, r cotangents (wave 1)
  Quad<R> q[REV_D][14][WAVE];
  R c[REV_D][2][WAVE];   // sin(delta), cos(delta)
  R gd[REV_DS][2][WAVE];  // control gradient (steer, throttle)
  int cnt[8];            // steps: [0..2] written by the waves, [4] read by wave 2, [5] of gd
};

template <class R>
union C8AdjPipeLds {
  C8PipeLds<R> fwd;
  C8RevLds<R> rev;
};

template <class R>
struct C8BackwardPipeArgs {
  C8BackwardArgs<R> b;
  unsigned char* rows;  // [B][nblk_max] blocks of adj_rows_bytes_per_wg(t_max)
};

template <class R>
__global__ __launch_bounds__(RP_BLK) void k_backward_c8_pipe(C8BackwardPipeArgs<R> ba) {
  const C8BackwardArgs<R>& g = ba.b;
  const C8Args<R>& a = g.a;
  extern __shared__ __align__(16) unsigned char smem[];
  const int b = blockIdx.y;
  C8Dims d;
  const bool ok = c8_dims(a, b, d);
  if (blockIdx.x == 0 && threadIdx.x == 0) g.valid[b] = ok ? 1u : 0u;
  if (!ok) return;
  if (d.K == 0) {
    R* gVb = g.grad_V + 2 * (size_t)d.t0;
    if (blockIdx.x == 0)
      for (int i = threadIdx.x; i < 2 * d.T; i += blockDim.x) gVb[i] = R(0);
    return;
  }
  const int m_base = blockIdx.x * WAVE;
  if (m_base >= d.K) return;
  const int w = threadIdx.x / WAVE, lane = threadIdx.x % WAVE, T = d.T, m = m_base + lane;
  const R gs = m < d.K ? g.grad_S[d.k0 + m] : R(0);
  R* gp = g.part + ((size_t)b * g.nblk_max + blockIdx.x) * 2 * a.t_max;
  if (__ballot(gs != R(0)) == 0ull) {  // the same in every wave
    for (int i = threadIdx.x; i < 2 * T; i += blockDim.x) gp[i] = R(0);
    return;
  }
  R* Vs;
  const CurvView<R> cv = c8_stage(a, b, d, reinterpret_cast<R*>(smem), &Vs);
  C8AdjPipeLds<R>& L = *reinterpret_cast<C8AdjPipeLds<R>*>(smem + c8_stage_bytes<R>(a.n_max, a.t_max));
  if (threadIdx.x < 8) L.fwd.cnt[threadIdx.x] = 0;
  __syncthreads();
  const DevModel<R> M = model_in_vgprs(a.M);
  const DevCost<R> C = cost_in_vgprs(a.C);
  const DevWheels<R> Wh = a.Wh;
  const DevObjective<R> ob = g.ob;
  const C8<R> x0 = load_c8(a.x0 + 8 * (size_t)b);
  R* rows = reinterpret_cast<R*>(ba.rows + ((size_t)b * g.nblk_max + blockIdx.x) * adj_rows_bytes_per_wg<R>(a.t_max, true)) + lane;
  // ---- forward
  if (w == 0) {
    pipe_noise<R, 64, C8P_D, 1>(M, C, Vs, T, a.seed, (uint32_t)m, (uint32_t)(a.pid_base + b), a.iter[b], a.nominal != 0,
                                L.fwd.cnt, a.err, [&](int t, int s, R v0, R v1, R r0, R r1, R u0, R u1) {
                                  c8_put_ctl(L.fwd, C, t, s, v0, v1, u0, u1);
                                  rows[((size_t)t * ADJ_ROW8 + 8) * WAVE] = r0;
                                  rows[((size_t)t * ADJ_ROW8 + 9) * WAVE] = r1;
                                });
  } else if (w == 1) {
    auto put = [&](int t, const C8<R>& x) {
      R* o = rows + (size_t)(t + 1) * ADJ_ROW8 * WAVE;
      o[0 * WAVE] = x.vx; o[1 * WAVE] = x.vy; o[2 * WAVE] = x.r; o[3 * WAVE] = x.wF; o[4 * WAVE] = x.wR;
    };
    put(-1, x0);
    c8_pipe_body(M, Wh, x0, T, L.fwd, a.err, put);
  } else if (w == 2) {
    C8<R> x = x0;
    int seen = 0;
    auto put = [&](int t) {
      R* o = rows + (size_t)t * ADJ_ROW8 * WAVE;
      o[5 * WAVE] = x.ep; o[6 * WAVE] = x.ey; o[7 * WAVE] = x.s;
    };
    put(0);
    for (int t = 0; t < T; ++t) {
      wave_wait(&L.fwd.cnt[1], t, seen, a.err);
      const Quad<R>(*o)[WAVE] = L.fwd.vel[t % C8P_D];
      const Quad<R> vx = o[0][lane], vy = o[1][lane], r = o[2][lane];
      wave_publish(&L.fwd.cnt[4], t + 1);
      c8_path_step(M, cv, vx, vy, r, x);
      put(t + 1);
    }
  }
  __syncthreads();  // (also completes the stores of the rows)
  C8RevLds<R>& P = L.rev;
  if (threadIdx.x < 8) P.cnt[threadIdx.x] = 0;
  __syncthreads();
  // ---- reverse: step i of the pipeline is t = T - 1 - i
  const R h = M.dt, h2 = R(0.5) * M.dt, h6 = M.dt * R(1.0 / 6.0), h3 = R(2) * h6;
  auto row = [&](int t, int c) { return rows[((size_t)max(t, 0) * ADJ_ROW8 + c) * WAVE]; };
  if (w == 0) {
    struct In { R vx, vy, r, wF, wR, r0, r1; };
    auto load = [&](int t) {
      return In{row(t, 0), row(t, 1), row(t, 2), row(t, 3), row(t, 4), row(t, 8), row(t, 9)};
    };
    In cur = load(T - 1), n1 = load(T - 2);
    int seen = 0;
    for (int i = 0; i < T; ++i) {
      const In n2 = load(T - 3 - i);
      const R u0 = clamp_r(cur.r0, M.u_lo[0], M.u_hi[0]), u1 = clamp_r(cur.r1, M.u_lo[1], M.u_hi[1]);
      R sd, cd;
      sincos_r(u0, &sd, &cd);
      const R dr = Wh.drive_Iw * u1;
      Quad<R> vx, vy, r, inv, fx, fy, dq, dp, dz, da, va;
      R wF = cur.wF, wR = cur.wR;
      vx.v[0] = cur.vx;
      vy.v[0] = cur.vy;
      r.v[0] = cur.r;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const R x = vx.v[k], y = vy.v[k], o = r.v[k];
        const R iv = rcp_r(fmax(x, M.v_min));
        const R av = fma_r(M.lf, o, y), z = fma_r(M.lr, o, -y);
        const R p = fma_r(Wh.r_w, wF, -fma_r(x, cd, av * sd)), q = fma_r(Wh.r_w, wR, -x);
        const R ai = av * iv, zi = z * iv, pi = p * iv, qi = q * iv;
        const R FyF = M.Cf * (u0 - ai), FyR = M.Cr * zi, FxF = Wh.C_x * pi, FxR = Wh.C_x * qi;
        const R gi = x >= M.v_min ? iv : R(0);
        inv.v[k] = iv;
        fx.v[k] = FxF;
        fy.v[k] = FyF;
        dq.v[k] = gi * FxR;
        dp.v[k] = gi * FxF;
        dz.v[k] = gi * FyR;
        da.v[k] = gi * (M.Cf * ai);
        va.v[k] = fma_r(cd, av, -(sd * x));
        if (k < 3) {
          const R f = k == 2 ? h : h2;
          const R fl = fma_r(FxF, sd, FyF * cd);
          vx.v[k + 1] = fma_r(f, fma_r(FxR + fma_r(FxF, cd, -(FyF * sd)), M.inv_m, fma_r(-M.c_v, x, y * o)), cur.vx);
          vy.v[k + 1] = fma_r(f, fma_r(FyR + fl, M.inv_m, -(x * o)), cur.vy);
          r.v[k + 1] = fma_r(f, fma_r(M.lf_Iz, fl, -(M.lr_Iz * FyR)), cur.r);
          wF = fma_r(-f, Wh.rw_Iw * FxF, cur.wF);
          wR = fma_r(f, fma_r(-Wh.rw_Iw, FxR, dr), cur.wR);
        }
      }
      if (i >= REV_D) wave_wait(&P.cnt[4], i - REV_D, seen, a.err);
      Quad<R>(*o)[WAVE] = P.q[i % REV_D];
      o[0][lane] = vx;
      o[1][lane] = vy;
      o[2][lane] = r;
      o[3][lane] = inv;
      o[4][lane] = fx;
      o[5][lane] = fy;
      o[6][lane] = dq;
      o[7][lane] = dp;
      o[8][lane] = dz;
      o[9][lane] = da;
      o[10][lane] = va;
      P.c[i % REV_D][0][lane] = sd;
      P.c[i % REV_D][1][lane] = cd;
      wave_publish(&P.cnt[0], i + 1);
      cur = n1;
      n1 = n2;
    }
  } else if (w == 1) {
    struct In { R ep, ey, s; };
    auto load = [&](int t) { return In{row(t, 5), row(t, 6), row(t, 7)}; };
    In cur = load(T - 1), n1 = load(T - 2);
    R yn = row(T, 6);
    const R q2 = R(2) * ob.w_S * C.q_ey, cw = ob.w_S * C.C_cbf;
    R le = R(0), ly = C.phi_w * q2 * yn, ls = R(0);
    int seen = 0;
    for (int i = 0; i < T; ++i) {
      const int t = T - 1 - i;
      const In n2 = load(t - 2);
      // barrier of transition t: r = alpha h(x_t) - h(x_{t+1}), h = w^2 - e_y^2
      const R yp = cur.ey;
      const R rr = C.alpha * (cv.w2 - yp * yp) - (cv.w2 - yn * yn);
      const R gr = rr > R(0) ? R(2) * fma_r(R(2) * ob.w_sq, rr, cw + (t < ob.n_lin ? ob.w_lin : R(0))) : R(0);
      ly = fma_r(gr, yn, ly);
      const R ay = (q2 - gr * C.alpha) * yp;
      wave_wait(&P.cnt[0], i, seen, a.err);
      Quad<R>(*o)[WAVE] = P.q[i % REV_D];
      const Quad<R> vx = o[0][lane], vy = o[1][lane], r = o[2][lane];
      // path states of the stages
      R k_[4], sl[4], se[4], ce[4], rd[4], sd_[4], ys[4];
      R e = cur.ep, y = cur.ey, s = cur.s;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        k_[k] = kappa_cell(cv, s, sl[k]);
        sincos_r(e, &se[k], &ce[k]);
        rd[k] = rcp_r(fma_r(-k_[k], y, R(1)));
        sd_[k] = fma_r(vx.v[k], ce[k], -(vy.v[k] * se[k])) * rd[k];
        ys[k] = y;
        if (k < 3) {
          const R f = k == 2 ? h : h2;
          e = fma_r(f, fma_r(-k_[k], sd_[k], r.v[k]), cur.ep);
          y = fma_r(f, fma_r(vx.v[k], se[k], vy.v[k] * ce[k]), cur.ey);
          s = fma_r(f, sd_[k], cur.s);
        }
      }
      Quad<R> qa, qb, qr;
      R oe = R(0), oy = R(0), os = R(0), te = R(0), ty = R(0), ts = R(0);
#pragma unroll
      for (int k = 3; k >= 0; --k) {
        const R wk = (k == 0 || k == 3) ? h6 : h3, f = k == 2 ? h : h2;
        const R ge = k == 3 ? wk * le : fma_r(f, oe, wk * le);
        const R gy = k == 3 ? wk * ly : fma_r(f, oy, wk * ly);
        const R gl = k == 3 ? wk * ls : fma_r(f, os, wk * ls);
        const R gn = fma_r(-k_[k], ge, gl) * rd[k];  // cotangent of v_x cos - v_y sin
        const R gden = -(gn * sd_[k]);
        const R gk = -fma_r(sd_[k], ge, ys[k] * gden);
        qa.v[k] = fma_r(se[k], gy, ce[k] * gn);
        qb.v[k] = fma_r(ce[k], gy, -(se[k] * gn));
        qr.v[k] = ge;
        const R gce = fma_r(vx.v[k], gn, vy.v[k] * gy), gse = fma_r(vx.v[k], gy, -(vy.v[k] * gn));
        oy = -(k_[k] * gden);
        oe = fma_r(ce[k], gse, -(se[k] * gce));
        os = sl[k] * gk;
        te += oe;
        ty += oy;
        ts += os;
      }
      o[11][lane] = qa;
      o[12][lane] = qb;
      o[13][lane] = qr;
      wave_publish(&P.cnt[1], i + 1);
      le += te;
      ly += ty + ay;
      ls += ts;
      yn = yp;
      cur = n1;
      n1 = n2;
    }
  } else if (w == 2) {
    const R sv = ob.w_S * R(2) * C.q_v;
    R lx = C.phi_w * sv * (row(T, 0) - C.v_g), ly = R(0), lr = R(0), lf = R(0), lw = R(0);
    int seen = 0, seen3 = 0;
    for (int i = 0; i < T; ++i) {
      wave_wait(&P.cnt[1], i, seen, a.err);
      const Quad<R>(*o)[WAVE] = P.q[i % REV_D];
      const Quad<R> vx = o[0][lane], vy = o[1][lane], r = o[2][lane], inv = o[3][lane], fx = o[4][lane],
                    fy = o[5][lane], dq = o[6][lane], dp = o[7][lane], dz = o[8][lane], da = o[9][lane],
                    va = o[10][lane], qa = o[11][lane], qb = o[12][lane], qr = o[13][lane];
      const R sd = P.c[i % REV_D][0][lane], cd = P.c[i % REV_D][1][lane];
      wave_publish(&P.cnt[4], i + 1);
      R gd = R(0), gt = R(0), ox = R(0), oy = R(0), orr = R(0), of = R(0), ow = R(0);
      R sx = R(0), sy = R(0), sr = R(0), sf = R(0), sw = R(0);
#pragma unroll
      for (int k = 3; k >= 0; --k) {
        const R wk = (k == 0 || k == 3) ? h6 : h3, f = k == 2 ? h : h2;
        const R gx = k == 3 ? wk * lx : fma_r(f, ox, wk * lx);
        const R gy = k == 3 ? wk * ly : fma_r(f, oy, wk * ly);
        const R gr = k == 3 ? wk * lr : fma_r(f, orr, wk * lr);
        const R gf = k == 3 ? wk * lf : fma_r(f, of, wk * lf);
        const R gw = k == 3 ? wk * lw : fma_r(f, ow, wk * lw);
        // cotangents of the tyre forces
        const R Gx = M.inv_m * gx, Gy = fma_r(M.lf_Iz, gr, M.inv_m * gy);
        const R ge = fma_r(cd, Gx, sd * Gy);
        const R gFxF = fma_r(-Wh.rw_Iw, gf, ge), gFyF = fma_r(cd, Gy, -(sd * Gx));
        const R gFxR = fma_r(-Wh.rw_Iw, gw, Gx), gFyR = fma_r(M.inv_m, gy, -(M.lr_Iz * gr));
        const R cx = Wh.C_x * inv.v[k];
        const R gq = cx * gFxR, gp_ = cx * gFxF, gz = M.Cr * inv.v[k] * gFyR;
        const R ga = -fma_r(sd, gp_, M.Cf * inv.v[k] * gFyF);
        ox = fma_r(-M.c_v, gx, fma_r(-r.v[k], gy, qa.v[k])) - fma_r(cd, gp_, gq) -
             fma_r(dq.v[k], gFxR, fma_r(dp.v[k], gFxF, fma_r(dz.v[k], gFyR, -(da.v[k] * gFyF))));
        oy = fma_r(r.v[k], gx, qb.v[k]) + (ga - gz);
        orr = fma_r(vy.v[k], gx, fma_r(-vx.v[k], gy, fma_r(M.lr, gz, fma_r(M.lf, ga, qr.v[k]))));
        of = Wh.r_w * gp_;
        ow = Wh.r_w * gq;
        gd += fma_r(M.Cf + fx.v[k], gFyF, -fma_r(fy.v[k], ge, va.v[k] * gp_));
        gt += gw;
        sx += ox;
        sy += oy;
        sr += orr;
        sf += of;
        sw += ow;
      }
      if (i >= REV_DS) wave_wait(&P.cnt[5], i - REV_DS, seen3, a.err);
      P.gd[i % REV_DS][0][lane] = gd;
      P.gd[i % REV_DS][1][lane] = Wh.drive_Iw * gt;
      wave_publish(&P.cnt[2], i + 1);
      lx += fma_r(sv, vx.v[0] - C.v_g, sx);
      ly += sy;
      lr += sr;
      lf += sf;
      lw += sw;
    }
  } else {
    RevSum<R, ADJ_ROW8> sum(rows, Vs, gp, T, lane, gs, M, C, ob);
    for (int i = 0; i < T; ++i) sum.step(P.gd, P.cnt, i, a.err);
  }
}

}  // namespace smppi
