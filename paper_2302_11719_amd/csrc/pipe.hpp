// Sampled rollouts of small batches as a pipeline of specialised waves.
//
// A batch with fewer sample-waves than the chip has SIMDs is bound by each
// wave's own chain of instructions per step (one wave issues about one VALU
// instruction per five cycles, whatever its dependencies), so a workgroup here
// splits every step of its NS samples over four waves, one per SIMD:
//   noise: Philox and Box-Muller, clipped controls, the step constants of the
//          held control and the control cost.  64 / NS lanes per sample, each
//          lane two steps (one Philox call), so a pass yields 2 * 64 / NS steps;
//   NS = 64: the RK4 step (one lane per sample), and two waves for the lateral
//          offset and the cost, two lanes per sample;
//   NS = 16: the velocity part of the RK4 step (one lane per sample), the pose
//          part (four lanes per sample, one RK4 stage each), and one wave for
//          the lateral offset and the cost, four lanes per sample.
// Steps pass from wave to wave through rings of D slots in LDS with step counters
// (wave_publish / wave_wait).  All rings have the same depth and the last waves
// count the steps they have read, so only the noise wave waits for room: when it
// has written step t, step t - D has left the pipeline.
// The pipeline runs at its slowest wave's rate: with 16 samples the velocity wave
// (about 105 VALU instructions, 800 cycles per step; it never waits), with 64 the
// RK4 wave (980 cycles), where one wave per 64 samples takes 2200 cycles per step.
// Every operation of rollout_sample is done once per sample, by one of the
// waves, in the same form and order (S receives the same terms in the same
// order), so the costs are the same bits.
#pragma once

#include "kernels.hpp"

namespace smppi {

constexpr int RP_BLK = 4 * WAVE;

template <class R, int NS>
struct RolloutPipe {
  static constexpr int LN = WAVE / NS;           // noise lanes per sample
  static constexpr int D = NS == 64 ? 8 : 16;    // ring slots
  static constexpr int LT = NS == 64 ? 2 : 4;    // lanes per sample of the offset/cost waves
  static constexpr int NCTL = 6;                 // delta, sin/m, cos/m, cos l_f/I_z, a tau, control cost
  struct Lds {
    R ctl[D][NCTL][NS];
    R stg[NS == 64 ? 1 : D][NS == 64 ? 1 : NS][12];  // NS = 16: velocities of the four RK4 stages (v_x, v_y, omega)
    R pos[D][3][NS];                  // p_x, p_y, v_x of x_{t+1}
    int cnt[8];                       // steps: [0] noise, [1] velocity, [2] pose (NS = 64: RK4) written; [4], [5] read
  };
};

template <class R>
struct alignas(4 * sizeof(R)) Quad {
  R v[4];
};

// Lane q of a quad (or pair) to all its lanes' neighbours, by DPP.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, false);
}

// The window rule with half width 4 on LT lanes per sample (part = lane % LT).
// The offsets in the rule's order (0, -1, +1, -2, +2, -3, +3, -4, +4) are dealt
// out in consecutive runs, LT = 2: five and four, LT = 4: three and three times
// two; each lane keeps the first strict minimum of its run, and runs merge in
// order, a later run winning only when strictly smaller: the rule's result.
// The rows depend on the centre alone, so they are read before the wave waits for
// the next position.
template <class R, int LT>
struct WindowRows {
  static constexpr int N = LT == 2 ? 5 : 3;
  R s[N][4], il[N];
};
template <int N>
struct WindowSlots {
  int v[N];
  __device__ __forceinline__ int operator[](int k) const { return v[k]; }
};
// Offset of slot k of a lane's run; a run's missing last slot repeats another.
template <int LT>
__device__ __forceinline__ int window_slot(int part, int k) {
  const int first = LT == 2 ? 5 * part : (part ? 2 * part + 1 : 0);  // position in the rule's order
  const int p = min(first + k, 8);
  return (p & 1) ? -((p + 1) >> 1) : (p >> 1);
}
template <class R, int LT>
__device__ __forceinline__ WindowRows<R, LT> window_rows(const TrackView<R>& tr, int c,
                                                          const WindowSlots<WindowRows<R, LT>::N>& off) {
  WindowRows<R, LT> r;
#pragma unroll
  for (int k = 0; k < WindowRows<R, LT>::N; ++k) {
    const int i = c + off[k];
    const R* sg = static_cast<const R*>(__builtin_assume_aligned(tr.seg + 4 * i, 4 * sizeof(R) > 16 ? 16 : 4 * sizeof(R)));
#pragma unroll
    for (int q = 0; q < 4; ++q) r.s[k][q] = sg[q];
    r.il[k] = tr.il2[i];
  }
  return r;
}
// e_y^2 at (px, py) and the new centre c, on every lane of the sample.
template <class R, int LT>
__device__ __forceinline__ R window4_lanes(const TrackView<R>& tr, const WindowRows<R, LT>& r,
                                           const WindowSlots<WindowRows<R, LT>::N>& off, int part, int& c, R px, R py) {
  constexpr int N = WindowRows<R, LT>::N;
  R bd;
  int bo;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const R rx = px - r.s[k][0], ry = py - r.s[k][1];
    const R dx = r.s[k][2], dy = r.s[k][3];
    const R lam = clamp_r((rx * dx + ry * dy) * r.il[k], R(0), R(1));
    const R ex = rx - lam * dx, ey = ry - lam * dy;
    const R d = ex * ex + ey * ey;
    if (k == 0) {
      bd = d;
      bo = off[0];
    } else {
      // the last slot belongs to the first run only
      const bool take = d < bd && (k < N - 1 || part == 0);
      bd = take ? d : bd;
      bo = take ? off[k] : bo;
    }
  }
  {  // with the neighbouring lane: runs 0|1 (and 2|3)
    const R od = dpp_move<0xB1>(bd);
    const int oo = dpp_move<0xB1>(bo);
    const bool odd = (part & 1) != 0;
    const bool take = odd ? !(bd < od) : od < bd;  // the later run only when strictly smaller
    bd = take ? od : bd;
    bo = take ? oo : bo;
  }
  if (LT == 4) {  // runs 0-1 | 2-3
    const R od = dpp_move<0x4E>(bd);
    const int oo = dpp_move<0x4E>(bo);
    const bool hi = (part & 2) != 0;
    const bool take = hi ? !(bd < od) : od < bd;
    bd = take ? od : bd;
    bo = take ? oo : bo;
  }
  int i = c + bo;
  i += (i < 0) ? tr.n : 0;
  i -= (i >= tr.n) ? tr.n : 0;
  c = i;
  return bd;
}

// The noise wave: 64 / NS lanes per sample, rings of D slots, cnt[0] the steps
// written, cnt[4] (and, ROOM = 2, cnt[5]) the steps that have left the pipeline.
// put(t, s, v0, v1, r0, r1, u0, u1): the lane that owns step t of sample s
// writes its rows (controls v, with noise r, clipped u) before they are published.
template <class R, int NS, int D, int ROOM, class Put>
__device__ void pipe_noise(const DevModel<R>& M, const DevCost<R>& C, const R* Vs, int T, uint32_t seed, uint32_t m,
                           uint32_t pid, uint32_t it, bool nominal, int* cnt, uint32_t* err, Put put) {
  constexpr int LN = WAVE / NS, PASS = 2 * LN;
  static_assert(D >= 2 * PASS && (D & (D - 1)) == 0, "ring too short");
  const int lane = threadIdx.x % WAVE, s = lane / LN, l = lane % LN;
  int seen0 = 0, seen1 = 0;
  for (int tp = 0; tp < T; tp += PASS) {
    const int t0 = tp + 2 * l;
    R z[4] = {R(0), R(0), R(0), R(0)};
    if (!nominal) normals4<R>(seed, (uint32_t)(t0 >> 1), m, pid, it, z);
    const int last = min(tp + PASS, T) - 1 - D;  // the pass's last step reuses this step's slot
    if (last >= 0) {
      wave_wait(cnt + 4, last, seen0, err);
      if (ROOM == 2) wave_wait(cnt + 5, last, seen1, err);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int t = t0 + k;
      if (t < T) {
        const R v0 = Vs[t], v1 = Vs[T + t];
        // (rounded before the sum, as where the noise comes from NoiseStream::get)
        R e0 = C.sigma[0] * z[2 * k], e1 = C.sigma[1] * z[2 * k + 1];
        asm volatile("" : "+v"(e0), "+v"(e1));
        const R r0 = v0 + e0, r1 = v1 + e1;
        put(t, s, v0, v1, r0, r1, clamp_r(r0, M.u_lo[0], M.u_hi[0]), clamp_r(r1, M.u_lo[1], M.u_hi[1]));
      }
    }
    wave_publish(cnt, min(tp + PASS, T));
  }
}
// Control cost of a step, lambda_u v^T Sigma^-1 u.
template <class R>
__device__ __forceinline__ R pipe_ctl_cost(const DevCost<R>& C, R v0, R v1, R u0, R u1) {
  return fma_r(C.ctrl_w[0] * v0, u0, C.ctrl_w[1] * v1 * u1);
}
// Ring row of a step (six-state model).
template <class R, int NS>
__device__ __forceinline__ void pipe_put_ctl(typename RolloutPipe<R, NS>::Lds& P, const DevModel<R>& M,
                                             const DevCost<R>& C, int t, int s, R v0, R v1, R u0, R u1) {
  const StepCtl<R> c = step_ctl(M, u0, u1);
  R(*o)[NS] = P.ctl[t % RolloutPipe<R, NS>::D];
  o[0][s] = c.delta;
  o[1][s] = c.sd_m;
  o[2][s] = c.cd_m;
  o[3][s] = c.lfcd_Iz;
  o[4][s] = c.a_tau;
  o[5][s] = pipe_ctl_cost(C, v0, v1, u0, u1);
}

template <class R, int NS>
__device__ __forceinline__ StepCtl<R> pipe_ctl(const typename RolloutPipe<R, NS>::Lds& P, int t, int s) {
  const R(*c)[NS] = P.ctl[t % RolloutPipe<R, NS>::D];
  StepCtl<R> sc;
  sc.delta = c[0][s];
  sc.sd_m = c[1][s];
  sc.cd_m = c[2][s];
  sc.lfcd_Iz = c[3][s];
  sc.a_tau = c[4][s];
  sc.sd = sc.cd = R(0);
  return sc;
}

// NS = 64: the RK4 wave.  put(t, x): called with x_{t+1}.
template <class R, class Put>
__device__ void pipe_rk4(const DevModel<R>& M, State<R> x, int T, typename RolloutPipe<R, 64>::Lds& P, uint32_t* err,
                         Put put) {
  using RP = RolloutPipe<R, 64>;
  const int lane = threadIdx.x % WAVE;
  int seen = 0;
  wave_wait(&P.cnt[0], 0, seen, err);
  StepCtl<R> nx = pipe_ctl<R, 64>(P, 0, lane);
  for (int t = 0; t < T; ++t) {
    // the next step's controls are read before this step's chain
    const StepCtl<R> c = nx;
    if (t + 1 < T) {
      wave_wait(&P.cnt[0], t + 1, seen, err);
      nx = pipe_ctl<R, 64>(P, t + 1, lane);
    }
    rk4(M, c, x);
    R(*o)[64] = P.pos[t % RP::D];
    o[0][lane] = x.px;
    o[1][lane] = x.py;
    o[2][lane] = x.vx;
    wave_publish(&P.cnt[2], t + 1);
    put(t, x);
  }
}

// NS = 16: the velocity wave (lanes 0 .. 15) and the pose wave.
template <class R>
__device__ void pipe_vel(const DevModel<R>& M, State<R> x, int T, typename RolloutPipe<R, 16>::Lds& P, uint32_t* err) {
  using RP = RolloutPipe<R, 16>;
  const int s = threadIdx.x % WAVE;
  if (s >= 16) return;
  int seen = 0;
  wave_wait(&P.cnt[0], 0, seen, err);
  StepCtl<R> nx = pipe_ctl<R, 16>(P, 0, s);
  for (int t = 0; t < T; ++t) {
    // the next step's controls are read before this step's chain
    const StepCtl<R> c = nx;
    if (t + 1 < T) {
      wave_wait(&P.cnt[0], t + 1, seen, err);
      nx = pipe_ctl<R, 16>(P, t + 1, s);
    }
    VelStages<R> g;
    rk4_vel(M, c, x.vx, x.vy, x.om, g);
    R* o = static_cast<R*>(__builtin_assume_aligned(P.stg[t % RP::D][s], 16));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      o[q] = g.vx[q];
      o[4 + q] = g.vy[q];
      o[8 + q] = g.om[q];
    }
    P.pos[t % RP::D][2][s] = x.vx;
    wave_publish(&P.cnt[1], t + 1);
    // the next step's chain starts after the counter store
    asm volatile("" ::: "memory");
  }
}
template <class R>
__device__ void pipe_pose(const DevModel<R>& M, State<R> x, int T, typename RolloutPipe<R, 16>::Lds& P,
                          uint32_t* err) {
  using RP = RolloutPipe<R, 16>;
  const int lane = threadIdx.x % WAVE, s = lane >> 2, q = lane & 3;
  const R h = M.dt, h2 = R(0.5) * M.dt, h6 = M.dt * R(1.0 / 6.0);
  int seen = 0;
  for (int t = 0; t < T; ++t) {
    wave_wait(&P.cnt[1], t, seen, err);
    const R* g = static_cast<const R*>(__builtin_assume_aligned(P.stg[t % RP::D][s], 16));
    const R vq = g[q], wq = g[4 + q];
    const R o0 = g[8], o1 = g[9], o2 = g[10], o3 = g[11];
    // the heading of stage q, one sine and cosine per lane; every lane forms
    // the sums of rk4_pose in its order
    const R psq = q == 0 ? x.psi : fma_r(q == 3 ? h : h2, q == 1 ? o0 : (q == 2 ? o1 : o2), x.psi);
    R ex, ey;
    pose_deriv(psq, vq, wq, ex, ey);
    const R a0 = quad_get<0>(ex), b0 = quad_get<1>(ex), c0 = quad_get<2>(ex), d0 = quad_get<3>(ex);
    const R a1 = quad_get<0>(ey), b1 = quad_get<1>(ey), c1 = quad_get<2>(ey), d1 = quad_get<3>(ey);
    x.px = fma_r(h6, fma_r(R(2), b0 + c0, a0) + d0, x.px);
    x.py = fma_r(h6, fma_r(R(2), b1 + c1, a1) + d1, x.py);
    x.psi = fma_r(h6, fma_r(R(2), o1 + o2, o0) + o3, x.psi);
    R(*o)[16] = P.pos[t % RP::D];
    if (q < 2) o[q][s] = q ? x.py : x.px;
    wave_publish(&P.cnt[2], t + 1);
  }
}

// Sampled costs of NS samples per workgroup, grid (ceil(k_max / NS), B), no
// obstacles.
template <class R, int NS>
__global__ __launch_bounds__(RP_BLK) void k_rollout_pipe(RolloutArgs<R> a) {
  using RP = RolloutPipe<R, NS>;
  extern __shared__ __align__(16) unsigned char smem[];
  const int b = blockIdx.y;
  ProblemDims d;
  if (!load_dims(a.p, b, d)) return;
  const int m_base = blockIdx.x * NS;
  if (m_base >= d.K) return;
  R* Vs;
  const TrackView<R> tr = stage_problem(a.p, b, d, a.V, smem, &Vs);
  typename RP::Lds& P =
      *reinterpret_cast<typename RP::Lds*>(smem + stage_lds_bytes<R>(a.p.poly_max, a.p.t_max, a.p.obs_max));
  if (threadIdx.x < 8) P.cnt[threadIdx.x] = 0;
  __syncthreads();
  const int w = threadIdx.x / WAVE, lane = threadIdx.x % WAVE, T = d.T;
  const DevModel<R> M = model_in_vgprs(a.M);
  const DevCost<R> C = cost_in_vgprs(a.C);
  const State<R> x0 = load_state(a.p.x0 + 6 * (size_t)b);
  if (w == 0) {
    const int m = m_base + lane / RP::LN;
    R* eo = (a.eps_out && m < d.K) ? a.eps_out + (size_t)(d.k0 + m) * a.p.t_max * 2 : nullptr;
    pipe_noise<R, NS, RP::D, NS == 64 ? 2 : 1>(
        M, C, Vs, T, a.p.seed, (uint32_t)m, (uint32_t)(a.p.pid_base + b), a.p.iter[b], a.p.nominal != 0, P.cnt, a.p.err,
        [&](int t, int s, R v0, R v1, R, R, R u0, R u1) {
          pipe_put_ctl<R, NS>(P, M, C, t, s, v0, v1, u0, u1);
          if (eo) {
            eo[2 * t] = u0 - v0;
            eo[2 * t + 1] = u1 - v1;
          }
        });
  } else if (NS == 64 && w == 1) {
    if constexpr (NS == 64) pipe_rk4<R>(M, x0, T, P, a.p.err, [](int, const State<R>&) {});
  } else if (NS == 16 && w == 1) {
    if constexpr (NS == 16) pipe_vel<R>(M, x0, T, P, a.p.err);
  } else if (NS == 16 && w == 2) {
    if constexpr (NS == 16) pipe_pose<R>(M, x0, T, P, a.p.err);
  } else {
    constexpr int LT = RP::LT;
    const int tt = (int)threadIdx.x - (NS == 64 ? 2 : 3) * WAVE, j = tt / LT, part = tt % LT;
    int idx = tr.idx0, seen = 0;
    R ey2 = lateral_sq(tr, x0.px, x0.py, idx);
    R h0 = tr.w2 - ey2, vx = x0.vx;
    bool outside = h0 < R(0);
    R S = C.C_cbf * fmax((C.alpha - R(1)) * h0, R(0));
    const bool w4 = tr.n > 0 && tr.window == 4;
    WindowSlots<WindowRows<R, LT>::N> off;
#pragma unroll
    for (int k = 0; k < WindowRows<R, LT>::N; ++k) off.v[k] = window_slot<LT>(part, k);
    WindowRows<R, LT> rows;
    if (w4) rows = window_rows<R, LT>(tr, idx, off);
    for (int t = 0; t < T; ++t) {
      const R dv = vx - C.v_g;
      R q = fma_r(C.q_ey, ey2, C.q_v * dv * dv);
      if (outside) q += C.C_obs;
      wave_wait(&P.cnt[2], t, seen, a.p.err);
      const R(*qp)[NS] = P.pos[t % RP::D];
      const R px = qp[0][j], py = qp[1][j];
      vx = qp[2][j];
      const R ctl = P.ctl[t % RP::D][5][j];
      // counted as read once the reads are issued (the LDS performs this wave's
      // operations in order)
      wave_publish(&P.cnt[NS == 64 ? 2 + w : 4], t + 1);
      S += q + ctl;
      if (w4) {
        ey2 = window4_lanes<R, LT>(tr, rows, off, part, idx, px, py);
        rows = window_rows<R, LT>(tr, idx, off);  // the next step's window, read before its wait
      } else {
        ey2 = lateral_sq(tr, px, py, idx);
      }
      const R h1 = tr.w2 - ey2;
      const R pen = fmax(C.alpha * h0 - h1, R(0));
      h0 = h1;
      outside = h1 < R(0);
      S = fma_r(C.C_cbf, pen, S);
    }
    const R dv = vx - C.v_g;
    R q = fma_r(dv, C.q_v * dv, C.q_ey * ey2);
    if (outside) q += C.C_obs;
    S = fma_r(C.phi_w, q, S);
    if (part == 0 && m_base + j < d.K) a.S[d.k0 + m_base + j] = S;
  }
}

// FP32 rollouts with obstacles, 64 samples per workgroup: noise | RK4 | lateral offset
// | obstacles and cost, one lane per sample throughout (WaveObstacles needs whole
// waves: lanes past K run a copy of the last sample).  The last wave takes steps in
// pairs with one obstacle live set, as rollout_sample does, with the same operations in
// the same order (and the same multiply-adds, hence two forms of the speed term).  Bound
// by the RK4 wave up to one workgroup per compute unit, by issue beyond: K = 65536,
// T = 100, 64 obstacles 109 -> 85 us, K = 32768 108 -> 59 us.
struct ObsPipeLds {
  RolloutPipe<float, 64>::Lds p;  // cnt[3]: offsets written
  float ey2[RolloutPipe<float, 64>::D][64];
};

template <int NOBS>
__global__ __launch_bounds__(RP_BLK) void k_rollout_pipe_obs(RolloutArgs<float> a) {
  using RP = RolloutPipe<float, 64>;
  extern __shared__ __align__(16) unsigned char smem[];
  const int b = blockIdx.y;
  ProblemDims d;
  if (!load_dims(a.p, b, d)) return;
  const int m_base = blockIdx.x * WAVE;
  if (m_base >= d.K) return;
  float* Vs;
  const TrackView<float> tr = stage_problem(a.p, b, d, a.V, smem, &Vs);
  ObsPipeLds& L = *reinterpret_cast<ObsPipeLds*>(smem + stage_lds_bytes<float>(a.p.poly_max, a.p.t_max, a.p.obs_max));
  RP::Lds& P = L.p;
  if (threadIdx.x < 8) P.cnt[threadIdx.x] = 0;
  __syncthreads();
  const int w = threadIdx.x / WAVE, lane = threadIdx.x % WAVE, T = d.T;
  const DevModel<float> M = model_in_vgprs(a.M);
  const DevCost<float> C = cost_in_vgprs(a.C);
  const State<float> x0 = load_state(a.p.x0 + 6 * (size_t)b);
  const int m = m_base + lane;
  const bool own = m < d.K;
  if (w == 0) {
    float* eo = (a.eps_out && own) ? a.eps_out + (size_t)(d.k0 + m) * a.p.t_max * 2 : nullptr;
    pipe_noise<float, 64, RP::D, 2>(
        M, C, Vs, T, a.p.seed, (uint32_t)(own ? m : d.K - 1), (uint32_t)(a.p.pid_base + b), a.p.iter[b],
        a.p.nominal != 0, P.cnt, a.p.err, [&](int t, int s, float v0, float v1, float, float, float u0, float u1) {
          pipe_put_ctl<float, 64>(P, M, C, t, s, v0, v1, u0, u1);
          if (eo) {
            eo[2 * t] = u0 - v0;
            eo[2 * t + 1] = u1 - v1;
          }
        });
  } else if (w == 1) {
    pipe_rk4<float>(M, x0, T, P, a.p.err, [](int, const State<float>&) {});
  } else if (w == 2) {
    int idx = tr.idx0, seen = 0;
    for (int t = 0; t < T; ++t) {
      wave_wait(&P.cnt[2], t, seen, a.p.err);
      const float px = P.pos[t % RP::D][0][lane], py = P.pos[t % RP::D][1][lane];
      wave_publish(&P.cnt[4], t + 1);  // counted as read once the reads are issued
      L.ey2[t % RP::D][lane] = lateral_sq(tr, px, py, idx);
      wave_publish(&P.cnt[3], t + 1);
    }
  } else {
    const WaveObstacles os = wave_obstacles(a.p, b, a.C.alpha);
    int idx = tr.idx0, seen = 0;
    float ey2 = lateral_sq(tr, x0.px, x0.py, idx);
    float h0 = tr.w2 - ey2, vx = x0.vx, px = x0.px, py = x0.py;
    bool outside = h0 < 0.f;
    float S = C.C_cbf * fmaxf((C.alpha - 1.f) * h0, 0.f);
    float pz = 0.f;
    os.step(px, py, px, py, C.alpha, pz, outside);
    S = fma_r(C.C_cbf, pz, S);
    int t = 0;
    for (; t + 1 < T; t += 2) {
      wave_wait(&P.cnt[3], t + 1, seen, a.p.err);
      const float(*pa)[64] = P.pos[t % RP::D];
      const float(*pb)[64] = P.pos[(t + 1) % RP::D];
      const float ax = pa[0][lane], ay = pa[1][lane], av = pa[2][lane];
      const float bx = pb[0][lane], by = pb[1][lane], bv = pb[2][lane];
      const float ea = L.ey2[t % RP::D][lane], eb = L.ey2[(t + 1) % RP::D][lane];
      const float ca = P.ctl[t % RP::D][5][lane], cb = P.ctl[(t + 1) % RP::D][5][lane];
      wave_publish(&P.cnt[5], t + 2);
      const float dv = vx - C.v_g;
      float q = fma_r(C.q_ey, ey2, C.q_v * dv * dv);
      if (outside) q += C.C_obs;
      S += q + ca;
      float h1 = tr.w2 - ea;
      float pen0 = fmaxf(C.alpha * h0 - h1, 0.f);
      bool out1 = h1 < 0.f;
      h0 = h1;
      const float dv1 = av - C.v_g;
      float q1 = fma_r(dv1, C.q_v * dv1, C.q_ey * ea);
      h1 = tr.w2 - eb;
      float pen1 = fmaxf(C.alpha * h0 - h1, 0.f);
      h0 = h1;
      outside = h1 < 0.f;
      os.step2(px, py, ax, ay, bx, by, C.alpha, pen0, out1, pen1, outside);
      S = fma_r(C.C_cbf, pen0, S);
      if (out1) q1 += C.C_obs;
      S += q1 + cb;
      S = fma_r(C.C_cbf, pen1, S);
      px = bx;
      py = by;
      vx = bv;
      ey2 = eb;
    }
    if (t < T) {
      wave_wait(&P.cnt[3], t, seen, a.p.err);
      const float(*pa)[64] = P.pos[t % RP::D];
      const float ax = pa[0][lane], ay = pa[1][lane], av = pa[2][lane], ea = L.ey2[t % RP::D][lane];
      const float ca = P.ctl[t % RP::D][5][lane];
      const float dv = vx - C.v_g;
      float q = fma_r(C.q_ey, ey2, C.q_v * dv * dv);
      if (outside) q += C.C_obs;
      S += q + ca;
      const float h1 = tr.w2 - ea;
      float pen = fmaxf(C.alpha * h0 - h1, 0.f);
      outside = h1 < 0.f;
      os.step(px, py, ax, ay, C.alpha, pen, outside);
      S = fma_r(C.C_cbf, pen, S);
      vx = av;
      ey2 = ea;
    }
    const float dv = vx - C.v_g;
    float q = fma_r(dv, C.q_v * dv, C.q_ey * ey2);
    if (outside) q += C.C_obs;
    S = fma_r(C.phi_w, q, S);
    if (own) a.S[d.k0 + m] = S;
  }
}

}  // namespace smppi
