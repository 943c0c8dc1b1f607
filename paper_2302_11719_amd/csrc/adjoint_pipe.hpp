// Adjoint of the sampled rollout as two pipelines of four waves, 64 samples per
// workgroup: a forward pass that stores every state, then the reverse sweep.
//
// One wave that does a whole step of both sweeps issues 1500 to 1650
// instructions per step (a third of them to recompute states and noise), at one
// instruction per five cycles.  Here the states, the unclipped controls and the
// window segments are stored by the forward pass (nothing is recomputed from
// checkpoints), and each step of the reverse sweep is split over four waves, one
// per SIMD, along the model's cascade: the velocities (v_x, v_y, omega) evolve on
// their own and the pose (p, psi) integrates them, so in reverse the pose's
// cotangent depends on no other and the velocities' cotangent takes the pose's
// contribution per RK4 stage:
//   wave 0: the step's constants, the velocities of the four RK4 stages and their
//           tyre terms, from the stored state;
//   wave 1: barrier and lateral cost gradients, the pose's cotangent;
//   wave 2: the velocities' cotangent and the control gradient;
//   wave 3: the clip, the control cost, the sum over the 64 samples
// (with obstacles, whose gradients fill a wave of their own, wave 3 takes all
// barrier gradients and wave 1 the sums).
// Steps pass through LDS rings with step counters (wave_publish / wave_wait).
// Each wave then issues 100 to 200 instructions per step and a step of both sweeps
// takes about 2300 cycles, at four workgroups per compute unit (40 KB of LDS each)
// 4500.  Against one wave per 64 samples with recomputation: 8 x (K = 2048, T = 50)
// 147 -> 54 us, K = 65536, T = 100 with 64 obstacles 362 -> 237 us (131 us when all
// but 100 samples have zero upstream), FP64 8 x 2048 371 -> 125 us.
// Workgroups whose upstream gradients are all zero (softmax weights underflow)
// write zeros and leave: a sample with zero upstream contributes exactly zero.
#pragma once

#include "pipe.hpp"

namespace smppi {

// Stored rows of a workgroup: p_x, p_y, psi, v_x, v_y, omega of x_t and the two
// unclipped controls of step t, [t_max + 1][8][64], then the window segment of
// x_t, [t_max + 1][64]; curvilinear model: the eight states and two controls,
// [t_max + 1][10][64].
constexpr int ADJ_ROW = 8, ADJ_ROW8 = 10;
template <class R>
__host__ __device__ inline size_t adj_rows_bytes_per_wg(int t_max, bool curvilinear) {
  return (size_t)(t_max + 1) * WAVE * (curvilinear ? ADJ_ROW8 * sizeof(R) : ADJ_ROW * sizeof(R) + sizeof(int));
}

constexpr int REV_D = 2;   // ring slots of the stage rows
constexpr int REV_DS = 4;  // ring slots of the small rows

template <class R>
struct RevLds {
  Quad<R> q[REV_D][10][WAVE];  // per stage: v_x, v_y, omega, 1/v, t_1, p_a, p_z (wave 0); A, B, g_psi (wave 1)
  R c[REV_D][2][WAVE];         // C_f sin(delta)/m, C_f cos(delta)/m
  R gd[REV_DS][2][WAVE];        // control gradient (steer, throttle)
  Quad<R> bar[REV_DS][WAVE];   // with obstacles: barrier and lateral cotangents of p_{t+1} and p_t (wave 3)
  int cnt[8];  // steps: [0..3] written by the waves, [4] read by wave 2, [5] of gd, [6] of bar read
};

template <class R>
union AdjPipeLds {
  typename RolloutPipe<R, 64>::Lds fwd;
  RevLds<R> rev;
};

// e_y^2 and its gradient at (px, py) on segment idx (or the circle).
template <class R>
__device__ __forceinline__ R track_e2_grad(const TrackView<R>& tr, R px, R py, int idx, R& gx, R& gy) {
  if (tr.n == 0) {
    const R dx = px - tr.cx, dy = py - tr.cy;
    const R rho = sqrt_r(dx * dx + dy * dy);
    const R e = rho - tr.rad;
    const R f = R(2) * e / rho;
    gx = f * dx;
    gy = f * dy;
    return e * e;
  }
  R ex, ey;
  const R e2 = seg_dist2(tr, idx, px, py, &ex, &ey);
  gx = R(2) * ex;
  gy = R(2) * ey;
  return e2;
}

// Obstacle slots staged in LDS: FP32 reads its obstacles per wave (wave_obstacles).
template <class R>
__host__ __device__ inline int adj_pipe_obs(int obs_max) {
  return sizeof(R) == 4 ? 0 : obs_max;
}

template <class R>
struct BackwardPipeArgs {
  BackwardArgs<R> b;
  unsigned char* rows;  // [B][nblk_max] blocks of adj_rows_bytes_per_wg(t_max)
};

// Barrier and lateral cost gradients, transition by transition from the last one
// (the whole wave active): step(t) returns the cotangents of p_{t+1} and p_t, the
// latter with the lateral cost of x_t; rows are read two steps ahead.
template <class R, int NOBS>
struct RevBarrier {
  struct In { R px, py; int idx; };
  const R* rows;
  const int* segs;
  int lane;
  TrackView<R> tr;
  R alpha, cw, w_sq2, w_lin, qe, hn, gnx, gny, pnx, pny;
  int n_lin;
  In cur, n1;
  WaveObstacles wob;
  __device__ __forceinline__ In load(int t) const {
    const R* r = rows + (size_t)max(t, 0) * ADJ_ROW * WAVE;
    return In{r[0], r[WAVE], segs[(size_t)max(t, 0) * WAVE + lane]};
  }
  __device__ __forceinline__ RevBarrier(const BackwardArgs<R>& a, const TrackView<R>& tr_, const R* rows_,
                                        const int* segs_, int b, int T, int lane_, const DevCost<R>& C,
                                        const DevObjective<R>& ob)
      : rows(rows_), segs(segs_), lane(lane_), tr(tr_) {
    alpha = C.alpha;
    cw = ob.w_S * C.C_cbf;
    w_sq2 = R(2) * ob.w_sq;
    w_lin = ob.w_lin;
    n_lin = ob.n_lin;
    qe = ob.w_S * C.q_ey;
    const In xT = load(T);
    cur = load(T - 1);
    n1 = load(T - 2);
    pnx = xT.px;
    pny = xT.py;
    hn = tr.w2 - track_e2_grad(tr, pnx, pny, xT.idx, gnx, gny);
    if constexpr (NOBS > 0 && sizeof(R) == 4) wob = wave_obstacles(a.p, b, (float)C.alpha);
  }
  __device__ __forceinline__ Quad<R> step(int t) {
    const In n2 = load(t - 2);
    // r = alpha h(x_t) - h(x_{t+1}) per barrier
    R gpx, gpy;
    const R hp = tr.w2 - track_e2_grad(tr, cur.px, cur.py, cur.idx, gpx, gpy);
    const R base = cw + (t < n_lin ? w_lin : R(0));
    const R r = alpha * hp - hn;
    const R gr = r > R(0) ? fma_r(w_sq2, r, base) : R(0);
    const R ep = qe - gr * alpha;  // weight of grad e_y^2(x_t)
    R lx = gr * gnx, ly = gr * gny, ax = ep * gpx, ay = ep * gpy;
    if constexpr (NOBS > 0 && sizeof(R) == 4) {
      wob.grad(cur.px, cur.py, pnx, pny, alpha, base, w_sq2, lx, ly, ax, ay);
    } else if constexpr (NOBS > 0) {
#pragma unroll 2
      for (int k = 0; k < tr.n_obs; ++k) {
        const Obs<R> o = obs_at(tr, k);
        const R bx = cur.px - o.cx, by = cur.py - o.cy, cx = pnx - o.cx, cy = pny - o.cy;
        const R rr = alpha * (bx * bx + by * by - o.re2) - (cx * cx + cy * cy - o.re2);
        const R go = rr > R(0) ? R(2) * fma_r(w_sq2, rr, base) : R(0);
        lx = fma_r(-go, cx, lx);
        ly = fma_r(-go, cy, ly);
        ax = fma_r(go * alpha, bx, ax);
        ay = fma_r(go * alpha, by, ay);
      }
    }
    hn = hp;
    gnx = gpx;
    gny = gpy;
    pnx = cur.px;
    pny = cur.py;
    cur = n1;
    n1 = n2;
    Quad<R> q;
    q.v[0] = lx;
    q.v[1] = ly;
    q.v[2] = ax;
    q.v[3] = ay;
    return q;
  }
};

// Clip, control cost and the sum over the samples of step i (t = T - 1 - i), once
// wave 2 has written its control gradient.
template <class R, int ROW>
struct RevSum {
  struct In { R r0, r1; };
  const R* rows;
  const R* Vs;
  R* gp;
  int T, lane, seen;
  R g, c0, c1, lo0, hi0, lo1, hi1;
  In cur, n1;
  __device__ __forceinline__ In load(int t) const {
    const R* r = rows + ((size_t)max(t, 0) * ROW + ROW - 2) * WAVE;
    return In{r[0], r[WAVE]};
  }
  __device__ __forceinline__ RevSum(const R* rows_, const R* Vs_, R* gp_, int T_, int lane_, R g_,
                                    const DevModel<R>& M, const DevCost<R>& C, const DevObjective<R>& ob)
      : rows(rows_), Vs(Vs_), gp(gp_), T(T_), lane(lane_), seen(0), g(g_) {
    c0 = ob.w_S * C.ctrl_w[0];
    c1 = ob.w_S * C.ctrl_w[1];
    lo0 = M.u_lo[0]; hi0 = M.u_hi[0];
    lo1 = M.u_lo[1]; hi1 = M.u_hi[1];
    cur = load(T - 1);
    n1 = load(T - 2);
  }
  // ring: [REV_DS][2][64]; cnt[2] steps written, cnt[5] read
  __device__ __forceinline__ void step(const R (*ring)[2][WAVE], int* cnt, int i, uint32_t* err) {
    const int t = T - 1 - i;
    const In n2 = load(t - 2);
    const R v0 = Vs[t], v1 = Vs[T + t];
    const R u0 = clamp_r(cur.r0, lo0, hi0), u1 = clamp_r(cur.r1, lo1, hi1);
    const bool pass0 = cur.r0 >= lo0 && cur.r0 <= hi0, pass1 = cur.r1 >= lo1 && cur.r1 <= hi1;
    wave_wait(cnt + 2, i, seen, err);
    const R gd = ring[i % REV_DS][0][lane], gt = ring[i % REV_DS][1][lane];
    wave_publish(cnt + 5, i + 1);
    const R gv0 = (pass0 ? fma_r(c0, v0, gd) : R(0)) + c0 * u0;
    const R gv1 = (pass1 ? fma_r(c1, v1, gt) : R(0)) + c1 * u1;
    // a sample with zero upstream contributes exactly zero, even when it diverged
    const R s0 = wave_sum(g != R(0) ? g * gv0 : R(0));
    const R s1 = wave_sum(g != R(0) ? g * gv1 : R(0));
    if (lane == 0) {
      gp[t] = s0;
      gp[T + t] = s1;
    }
    cur = n1;
    n1 = n2;
  }
};

template <class R, int NOBS>
__global__ __launch_bounds__(RP_BLK) void k_backward_pipe(BackwardPipeArgs<R> ba) {
  const BackwardArgs<R>& a = ba.b;
  extern __shared__ __align__(16) unsigned char smem[];
  const int b = blockIdx.y;
  ProblemDims d;
  const bool ok = load_dims(a.p, b, d);
  if (blockIdx.x == 0 && threadIdx.x == 0) a.valid[b] = ok ? 1u : 0u;
  if (!ok) return;
  if (d.K == 0) {
    R* gVb = a.grad_V + 2 * (size_t)d.t0;
    if (blockIdx.x == 0)
      for (int i = threadIdx.x; i < 2 * d.T; i += blockDim.x) gVb[i] = R(0);
    return;
  }
  const int m_base = blockIdx.x * WAVE;
  if (m_base >= d.K) return;
  const int w = threadIdx.x / WAVE, lane = threadIdx.x % WAVE, T = d.T, m = m_base + lane;
  const R g = m < d.K ? a.grad_S[d.k0 + m] : R(0);
  R* gp = a.part + ((size_t)b * a.nblk_max + blockIdx.x) * 2 * a.p.t_max;
  if (__ballot(g != R(0)) == 0ull) {  // the same in every wave
    for (int i = threadIdx.x; i < 2 * T; i += blockDim.x) gp[i] = R(0);
    return;
  }
  R* Vs;
  ProblemArgs<R> sp = a.p;
  sp.obs_max = adj_pipe_obs<R>(a.p.obs_max);
  const TrackView<R> tr = stage_problem(sp, b, d, a.V, smem, &Vs);
  AdjPipeLds<R>& L =
      *reinterpret_cast<AdjPipeLds<R>*>(smem + stage_lds_bytes<R>(sp.poly_max, sp.t_max, sp.obs_max));
  if (threadIdx.x < 8) L.fwd.cnt[threadIdx.x] = 0;
  __syncthreads();
  const DevModel<R> M = model_in_vgprs(a.M);
  const DevCost<R> C = cost_in_vgprs(a.C);
  const DevObjective<R> ob = a.ob;
  const State<R> x0 = load_state(a.p.x0 + 6 * (size_t)b);
  unsigned char* wg = ba.rows + ((size_t)b * a.nblk_max + blockIdx.x) * adj_rows_bytes_per_wg<R>(a.p.t_max, false);
  R* rows = reinterpret_cast<R*>(wg) + lane;
  int* segs = reinterpret_cast<int*>(wg + (size_t)(a.p.t_max + 1) * ADJ_ROW * WAVE * sizeof(R));
  // ---- forward: every state, unclipped control and window segment
  if (w == 0) {
    pipe_noise<R, 64, RolloutPipe<R, 64>::D, 2>(
        M, C, Vs, T, a.p.seed, (uint32_t)m, (uint32_t)(a.p.pid_base + b), a.p.iter[b], a.p.nominal != 0, L.fwd.cnt,
        a.p.err, [&](int t, int s, R v0, R v1, R r0, R r1, R u0, R u1) {
          pipe_put_ctl<R, 64>(L.fwd, M, C, t, s, v0, v1, u0, u1);
          rows[((size_t)t * ADJ_ROW + 6) * WAVE] = r0;
          rows[((size_t)t * ADJ_ROW + 7) * WAVE] = r1;
        });
  } else if (w == 1) {
    auto put = [&](int t, const State<R>& x) {
      R* o = rows + (size_t)(t + 1) * ADJ_ROW * WAVE;
      o[0 * WAVE] = x.px; o[1 * WAVE] = x.py; o[2 * WAVE] = x.psi;
      o[3 * WAVE] = x.vx; o[4 * WAVE] = x.vy; o[5 * WAVE] = x.om;
    };
    put(-1, x0);
    pipe_rk4<R>(M, x0, T, L.fwd, a.p.err, put);
  } else {
    constexpr int LT = 2;
    const int tt = (int)threadIdx.x - 2 * WAVE, j = tt / LT, part = tt % LT;
    int idx = tr.idx0, seen = 0;
    (void)lateral_sq(tr, x0.px, x0.py, idx);
    const bool w4 = tr.n > 0 && tr.window == 4;
    WindowSlots<WindowRows<R, LT>::N> off;
#pragma unroll
    for (int k = 0; k < WindowRows<R, LT>::N; ++k) off.v[k] = window_slot<LT>(part, k);
    WindowRows<R, LT> wr;
    if (w4) wr = window_rows<R, LT>(tr, idx, off);
    if (part == 0) segs[j] = idx;
    for (int t = 0; t < T; ++t) {
      wave_wait(&L.fwd.cnt[2], t, seen, a.p.err);
      const R(*qp)[64] = L.fwd.pos[t % RolloutPipe<R, 64>::D];
      const R px = qp[0][j], py = qp[1][j];
      wave_publish(&L.fwd.cnt[2 + w], t + 1);
      if (w4) {
        (void)window4_lanes<R, LT>(tr, wr, off, part, idx, px, py);
        wr = window_rows<R, LT>(tr, idx, off);
      } else {
        (void)lateral_sq(tr, px, py, idx);
      }
      if (part == 0) segs[(size_t)(t + 1) * WAVE + j] = idx;
    }
  }
  __syncthreads();  // (also completes the stores of the rows)
  RevLds<R>& P = L.rev;
  if (threadIdx.x < 8) P.cnt[threadIdx.x] = 0;
  __syncthreads();
  // ---- reverse: step i of the pipeline is t = T - 1 - i
  const R h = M.dt, h2 = R(0.5) * M.dt, h6 = M.dt * R(1.0 / 6.0), h3 = R(2) * h6;
  const R kz = M.lf_Iz / M.inv_m;  // C_f cos l_f/I_z as a multiple of C_f cos/m
  const R crm = M.Cr * M.inv_m, crl = M.Cr * M.lr_Iz;
  auto row = [&](int t, int c) { return rows[((size_t)max(t, 0) * ADJ_ROW + c) * WAVE]; };
  if (w == 0) {
    // stage velocities and tyre terms; rows read two steps ahead
    struct In { R vx, vy, om, r0, r1; };
    auto load = [&](int t) { return In{row(t, 3), row(t, 4), row(t, 5), row(t, 6), row(t, 7)}; };
    In cur = load(T - 1), n1 = load(T - 2);
    int seen = 0;
    for (int i = 0; i < T; ++i) {
      const In n2 = load(T - 3 - i);
      R u0 = clamp_r(cur.r0, M.u_lo[0], M.u_hi[0]), u1 = clamp_r(cur.r1, M.u_lo[1], M.u_hi[1]);
      R sd, cd;
      sincos_r(u0, &sd, &cd);
      const R cfm = M.Cf * M.inv_m, csd = cfm * sd, ccd = cfm * cd, at = M.a_max * u1;
      Quad<R> vx, vy, om, inv, t1, pa, pz;
      vx.v[0] = cur.vx;
      vy.v[0] = cur.vy;
      om.v[0] = cur.om;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const R x = vx.v[k], y = vy.v[k], o = om.v[k];
        const R iv = rcp_r(fmax(x, M.v_min));
        const R ta = fma_r(M.lf, o, y) * iv, tz = fma_r(M.lr, o, -y) * iv, tf = u0 - ta;
        const bool above = x >= M.v_min;
        inv.v[k] = iv;
        t1.v[k] = tf;
        pa.v[k] = above ? ta * iv : R(0);
        pz.v[k] = above ? tz * iv : R(0);
        if (k < 3) {
          const R f = k == 2 ? h : h2, fc = tf * ccd;
          const R dvx = fma_r(y, o, fma_r(-tf, csd, fma_r(-M.c_v, x, at)));
          const R dvy = fma_r(-x, o, fma_r(tz, crm, fc));
          const R dom = fma_r(kz, fc, -(tz * crl));
          vx.v[k + 1] = fma_r(f, dvx, cur.vx);
          vy.v[k + 1] = fma_r(f, dvy, cur.vy);
          om.v[k + 1] = fma_r(f, dom, cur.om);
        }
      }
      if (i >= REV_D) wave_wait(&P.cnt[4], i - REV_D, seen, a.p.err);
      Quad<R>(*o)[WAVE] = P.q[i % REV_D];
      o[0][lane] = vx;
      o[1][lane] = vy;
      o[2][lane] = om;
      o[3][lane] = inv;
      o[4][lane] = t1;
      o[5][lane] = pa;
      o[6][lane] = pz;
      P.c[i % REV_D][0][lane] = csd;
      P.c[i % REV_D][1][lane] = ccd;
      wave_publish(&P.cnt[0], i + 1);
      cur = n1;
      n1 = n2;
    }
  } else if (w == 1) {
    // cotangent of (p_x, p_y, psi), and the barrier gradients or (with obstacles) the sums
    struct In { R psi; };
    auto load = [&](int t) { return In{row(t, 2)}; };
    In cur = load(T - 1), n1 = load(T - 2);
    RevBarrier<R, 0> bar(a, tr, rows, segs, b, T, lane, C, ob);
    RevSum<R, ADJ_ROW> sum(rows, Vs, gp, T, lane, g, M, C, ob);
    R lx = C.phi_w * bar.qe * bar.gnx, ly = C.phi_w * bar.qe * bar.gny, lp = R(0);
    int seen = 0, seenb = 0;
    for (int i = 0; i < T; ++i) {
      const In n2 = load(T - 3 - i);
      Quad<R> db;
      if (NOBS > 0) {
        wave_wait(&P.cnt[3], i, seenb, a.p.err);
        db = P.bar[i % REV_DS][lane];
        wave_publish(&P.cnt[6], i + 1);
      } else {
        db = bar.step(T - 1 - i);
      }
      lx += db.v[0];
      ly += db.v[1];
      wave_wait(&P.cnt[0], i, seen, a.p.err);
      Quad<R>(*o)[WAVE] = P.q[i % REV_D];
      const Quad<R> vx = o[0][lane], vy = o[1][lane], om = o[2][lane];
      Quad<R> qa, qb, qp;
      R os = R(0), of = R(0);  // sum of the stages' psi cotangents, and the last one's
#pragma unroll
      for (int k = 3; k >= 0; --k) {
        const R psi = k == 0 ? cur.psi : fma_r(k == 3 ? h : h2, om.v[k - 1], cur.psi);
        R sp, cp;
        sincos_r(psi, &sp, &cp);
        const R wk = (k == 0 || k == 3) ? h6 : h3;
        qa.v[k] = wk * fma_r(lx, cp, ly * sp);
        qb.v[k] = wk * fma_r(ly, cp, -(lx * sp));
        // stage k's psi is psi_t + f omega of the stage before: its cotangent goes there
        qp.v[k] = k == 3 ? wk * lp : fma_r(k == 2 ? h : h2, of, wk * lp);
        of = fma_r(vx.v[k], qb.v[k], -(vy.v[k] * qa.v[k]));
        os += of;
      }
      o[7][lane] = qa;
      o[8][lane] = qb;
      o[9][lane] = qp;
      wave_publish(&P.cnt[1], i + 1);
      lp += os;
      lx += db.v[2];
      ly += db.v[3];
      cur = n1;
      n1 = n2;
      if (NOBS > 0 && i >= 1) sum.step(P.gd, P.cnt, i - 1, a.p.err);
    }
    if (NOBS > 0) sum.step(P.gd, P.cnt, T - 1, a.p.err);
  } else if (w == 2) {
    // cotangent of (v_x, v_y, omega) and the control gradient
    const R sv = ob.w_S * R(2) * C.q_v;
    R lx = C.phi_w * sv * (row(T, 3) - C.v_g), ly = R(0), lo = R(0);
    int seen = 0, seen3 = 0;
    for (int i = 0; i < T; ++i) {
      wave_wait(&P.cnt[1], i, seen, a.p.err);
      const Quad<R>(*o)[WAVE] = P.q[i % REV_D];
      const Quad<R> vx = o[0][lane], vy = o[1][lane], om = o[2][lane], inv = o[3][lane], t1 = o[4][lane],
                    pa = o[5][lane], pz = o[6][lane], qa = o[7][lane], qb = o[8][lane], qp = o[9][lane];
      const R csd = P.c[i % REV_D][0][lane], ccd = P.c[i % REV_D][1][lane];
      wave_publish(&P.cnt[4], i + 1);
      R gd = R(0), gt = R(0), ox = R(0), oy = R(0), oo = R(0), sx = R(0), sy = R(0), so = R(0);
#pragma unroll
      for (int k = 3; k >= 0; --k) {
        const R wk = (k == 0 || k == 3) ? h6 : h3, f = k == 2 ? h : h2;
        const R gx = k == 3 ? wk * lx : fma_r(f, ox, wk * lx);
        const R gy = k == 3 ? wk * ly : fma_r(f, oy, wk * ly);
        const R go = k == 3 ? wk * lo : fma_r(f, oo, wk * lo);
        const R gw = fma_r(kz, go, gy);
        const R gaf = fma_r(ccd, gw, -(csd * gx));
        const R gar = fma_r(crm, gy, -(crl * go));
        const R g1 = inv.v[k] * gaf, g2 = inv.v[k] * gar;
        gd = fma_r(-t1.v[k], fma_r(ccd, gx, csd * gw), gd + gaf);
        gt += gx;
        ox = fma_r(-M.c_v, gx, fma_r(-om.v[k], gy, fma_r(pa.v[k], gaf, fma_r(-pz.v[k], gar, qa.v[k]))));
        oy = fma_r(om.v[k], gx, qb.v[k]) - (g1 + g2);
        oo = fma_r(vy.v[k], gx, fma_r(-vx.v[k], gy, fma_r(M.lr, g2, fma_r(-M.lf, g1, qp.v[k]))));
        sx += ox;
        sy += oy;
        so += oo;
      }
      if (i >= REV_DS) wave_wait(&P.cnt[5], i - REV_DS, seen3, a.p.err);
      P.gd[i % REV_DS][0][lane] = gd;
      P.gd[i % REV_DS][1][lane] = M.a_max * gt;
      wave_publish(&P.cnt[2], i + 1);
      lx += fma_r(sv, vx.v[0] - C.v_g, sx);
      ly += sy;
      lo += so;
    }
  } else {
    if constexpr (NOBS > 0) {
      // barrier gradients of the track and the obstacles
      RevBarrier<R, NOBS> bar(a, tr, rows, segs, b, T, lane, C, ob);
      int seen = 0;
      for (int i = 0; i < T; ++i) {
        const Quad<R> db = bar.step(T - 1 - i);
        if (i >= REV_DS) wave_wait(&P.cnt[6], i - REV_DS, seen, a.p.err);
        P.bar[i % REV_DS][lane] = db;
        wave_publish(&P.cnt[3], i + 1);
      }
    } else {
      RevSum<R, ADJ_ROW> sum(rows, Vs, gp, T, lane, g, M, C, ob);
      for (int i = 0; i < T; ++i) sum.step(P.gd, P.cnt, i, a.p.err);
    }
  }
}

}  // namespace smppi
