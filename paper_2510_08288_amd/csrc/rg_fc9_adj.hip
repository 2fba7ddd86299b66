// Weighted adjoint of the 9-state plant: one (scenario, upstream weight) entry
// per group of 9 lanes (layout of rg_fc9_lanes.hpp), lane i owning component i
// of the state, of the adjoint, and of the parameter sums.
#include <hip/hip_runtime.h>

#include "rg_adjoint.hpp"
#include "rg_fc9_lanes.hpp"

namespace rg {

// Forward pass with checkpoints every Kc steps and the first minimising step
// and row, then segment by segment back from it: recompute the segment's
// states, sweep them in reverse (the reverse RK4 step of rk4_vjp, a row per
// lane).
//
// The derivative of a scenario's margin is that at its first minimising step,
// and which step that is hangs, at a flat minimum, on the last bits of the
// trajectory; so the sweeps keep an arithmetic of their own (tanh itself in the
// coupling sum, the constant terms of phi_7 and phi_9 per evaluation, margin
// rows as g - F y), whatever the rollouts' becomes.
//
// A chain of dependent steps per entry: bound by latency.  One lane per entry
// took 1.9 us per forward step (the whole state on one lane) with 32 waves on
// 1024 SIMDs at N = 2048; a group takes 0.7 us.
template <int RNG, int INJ>
struct AdjLanes {
  using P = Plant<2, float>;
  const RollArgs<2, float>& a;
  const int i, k;
  const uint32_t t;
  float* const slot;
  // sampled factors of this lane's parameters: a_i; k_i (i < 6) or b_{i-5}; mu
  float fA, fK, fM;
  float A, K1, kin, b2v, mu, pm, pc, poff, q0, q6, qc, kq, v, xb, nkxb, axb, am, b;
  float wrow[9], wcol[9], wlo, wsp;
  int xw;
  const float* wb;
  // the evaluation point: activations, x_1, x_7, own orifice factor, the previous lane's
  float X0, X6, TZ[10], rl, rh, xn;

  __device__ __forceinline__ AdjLanes(const RollArgs<2, float>& a_, int i_, int k_, uint32_t t_,
                                      float v_, float* slot_)
      : a(a_), i(i_), k(k_), t(t_), slot(slot_), v(v_) {
    const float* tb = RNG == 0 ? step_th(a, t) : nullptr;
    auto factor = [&](int c) -> float {
      if (RNG == 0) return tb[(size_t)c * a.N + k];
      const Words r =
          philox10((uint32_t)k, 0u, t, (1u << 16) | (uint32_t)(c >> 2), a.seed, a.inst);
      const int q = c & 3;
      return box_draw(q == 0 ? r.v[0] : (q == 1 ? r.v[1] : (q == 2 ? r.v[2] : r.v[3])), a.thlo,
                      a.thspan);
    };
    auto theta = [&](int c, float f) { return a.pc.thnom[c] * f; };
    const int ck = 9 + i;  // k_i, or b_{i-5} for lanes 6..8 (coefficients 15..17)
    const int cm = i == 8 ? 19 : 18;
    fA = factor(i);
    fK = factor(ck);
    fM = factor(cm);
    A = theta(i, fA);
    const float kk = theta(ck, fK);
    mu = theta(cm, fM);
    kq = i < 6 ? kk : 0.f;
    b = i < 6 ? 0.f : kk;
    const int cin = 9 + (i >= 1 && i < 6 ? i - 1 : 0);
    kin = theta(cin, factor(cin));
    b2v = b * v;
    K1 = i < 6 ? -kk : (i == 7 ? 0.f : kk);
    pm = (i == 6 || i == 8) ? -mu : 0.f;
    poff = i == 8 ? 1.f : 0.f;
    pc = i == 0 ? a.pc.c_q0 : (i < 6 ? kin : (i == 7 ? b2v : 0.f));
    q0 = i == 6 ? 1.f : 0.f;
    q6 = (i == 0 || i == 7) ? 1.f : 0.f;
    qc = i == 6 ? -a.pc.p1ref : (i == 8 ? v : 0.f);
    xb = a.pc.xbar[i];
    nkxb = a.pc.nkxbar[i];
    axb = __fmul_rn(A, xb);
#pragma unroll
    for (int j = 0; j < 9; ++j) {
      wrow[j] = a.pc.W[9 * i + j];
      wcol[j] = a.pc.W[9 * j + i];
    }
    wlo = a.wlo[i];
    wsp = a.wspan[i];
    xw = i == 0 ? 9 : (i == 6 ? 10 : (i == 8 ? 11 : 12 + (i & 3)));
    wb = RNG == 0 ? step_w(a, t) + (size_t)i * a.N + k : nullptr;
  }
  __device__ __forceinline__ float draw(int j) const {
    if (RNG == 0) return wb[(size_t)j * P::nw * a.N];
    const Words r = philox10((uint32_t)k, (uint32_t)j, t, (uint32_t)(i >> 2), a.seed, a.inst);
    const int q = i & 3;
    return box_draw(q == 0 ? r.v[0] : (q == 1 ? r.v[1] : (q == 2 ? r.v[2] : r.v[3])), wlo, wsp);
  }
  // Exchange at the point whose component i is xv; returns this lane's tanh.
  __device__ __forceinline__ float exch(float xv) {
    const float tz = t_tanh_shift(xv, nkxb);
    slot[xw] = xv;
    slot[i] = tz;
    const float x1 = wave_shift<0x130>(xv);
    xn = i < 5 ? x1 : a.pc.p_amb;
    rh = P::orifice(xv, xn);
    rl = wave_shift<0x138>(rh);
    group_sync();
    read9(TZ);
    X0 = slot[9];
    X6 = slot[10];
    group_sync();
    return tz;
  }
  __device__ __forceinline__ void read9(float* d) const {
    typedef float V __attribute__((ext_vector_type(4)));
    const V* sv = reinterpret_cast<const V*>(slot);
    const V p = sv[0], q = sv[1];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      d[u] = p[u];
      d[4 + u] = q[u];
    }
    d[8] = slot[8];
  }
  // Row i of the derivative at the exchanged point.
  __device__ __forceinline__ float row(float s, float xv) const {
#pragma clang fp contract(off)
    float r = t_fma(K1, i < 6 ? rh : v, s);
    r = t_fma(-A, xv, r);
#pragma unroll
    for (int j = 0; j < 9; ++j) r = t_fma(wrow[j], TZ[j], r);
    const float Pq = t_fma(pm, xv - poff, pc);
    const float Q = (i >= 1 && i < 6) ? rl : t_fma(q0, X0, t_fma(q6, X6, qc));
    return t_fma(Pq, Q, r);
  }
  __device__ __forceinline__ float force(float w) const { return INJ == 0 ? w + axb : axb; }
  // One RK4 step from the exchanged state x; the new state is exchanged.
  __device__ __forceinline__ float step(float x, float w) {
    const float s = force(w);
    float kk = row(s, x), acc = kk;
    float xs = t_fma(a.hh, kk, x);
    exch(xs);
    kk = row(s, xs);
    acc = t_fma(2.f, kk, acc);
    xs = t_fma(a.hh, kk, x);
    exch(xs);
    kk = row(s, xs);
    acc = t_fma(2.f, kk, acc);
    xs = t_fma(a.h, kk, x);
    exch(xs);
    kk = row(s, xs);
    x = t_fma(a.h6, acc + kk, x);
    if (INJ == 1) x = x + w;
    exch(x);
    return x;
  }
  __device__ __forceinline__ float margin(int& r) const {
    float y[P::ny];
    y[0] = a.pc.c_q0 * X6 / t_fma(a.pc.d1, slot[11], a.pc.d0);
    y[1] = X0;
    y[2] = X6;
    float best = INFINITY;
    r = 0;
#pragma unroll
    for (int q = 0; q < kNC; ++q) {
      const float* F = a.F + q * P::ny;
      const float m = a.g[q] - t_fma(F[2], y[2], t_fma(F[1], y[1], F[0] * y[0]));
      if (m < best || m != m) {
        best = m;
        r = q;
      }
    }
    return best;
  }
  // What the reverse sweep keeps of one stage's point.
  struct Point {
    float x, tz, sq, dp, x0, x6;
  };
  __device__ __forceinline__ Point point(float x) {
    Point p;
    p.x = x;
    p.tz = exch(x);
    p.sq = rh;
    p.dp = x - xn;
    p.x0 = X0;
    p.x6 = X6;
    return p;
  }
  // Component i of J(x)^T al, with this lane's parameter sums (in FP64).
  __device__ __forceinline__ float vjp(const Point& p, float al, double& vb, double& tA, double& tK,
                                       double& tM) const {
    slot[i] = al;
    const float al1 = wave_shift<0x130>(al);
    group_sync();
    float g[10];
    read9(g);
    group_sync();
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < 9; ++j) acc = t_fma(wcol[j], g[j], acc);
    float u = t_fma(-A, al, acc * (1.f - p.tz * p.tz));
    tA += -(double)al * (double)(p.x - xb);
    // orifice flow q_{i+1} = k_i sqrt(max(dp, 0)): out of row i, into row i + 1
    const float d = (i < 6 && p.dp > 0.f) ? kq / (2.f * p.sq) : 0.f;
    const float beta = i < 5 ? al1 - al : -al;
    const float bd = beta * d;
    const float bp = wave_shift<0x138>(bd);  // row i - 1's flow, into this row
    u += bd - (i >= 1 && i < 6 ? bp : 0.f);
    const double dal = (double)al, dv = (double)v;
    if (i < 6) {
      tK += (double)beta * (double)p.sq;
      if (i == 0) u -= g[6] * mu * p.x6;  // phi_7 through x_1 (mu is mu_1 on this lane)
    } else if (i == 6) {
      u += g[0] * a.pc.c_q0 - al * mu * (p.x0 - a.pc.p1ref);
      vb += dal * (double)b;
      tK += dal * dv;
      tM += -dal * (double)p.x * ((double)p.x0 - (double)a.pc.p1ref);
    } else if (i == 7) {
      vb += dal * (double)b * (double)p.x6;
      tK += dal * dv * (double)p.x6;
    } else {
      u -= al * mu * v;
      vb += dal * ((double)b - (double)mu * ((double)p.x - 1.0));
      tK += dal * dv;
      tM += -dal * ((double)p.x - 1.0) * dv;
    }
    // phi_8 = b_2 v x_7: into x_7, from lane 7's coefficient
    const float b2v1 = wave_shift<0x130>(b2v);
    if (i == 6) u += g[7] * b2v1;
    return u;
  }
  // Reverse RK4 step at the state x under the draw w: lam <- (dPhi/dx)^T lam.
  __device__ __forceinline__ float step_vjp(float x, float w, float lam, double& vb, double& tA,
                                            double& tK, double& tM) {
    const float s = force(w);
    const Point p1 = point(x);
    const Point p2 = point(t_fma(a.hh, row(s, x), x));
    const Point p3 = point(t_fma(a.hh, row(s, p2.x), x));
    const Point p4 = point(t_fma(a.h, row(s, p3.x), x));
    const float h6 = a.h6, hh = a.hh, h = a.h;
    float u = vjp(p4, h6 * lam, vb, tA, tK, tM);
    float acc = u;
    u = vjp(p3, t_fma(h, u, 2.f * h6 * lam), vb, tA, tK, tM);
    acc += u;
    u = vjp(p2, t_fma(hh, u, 2.f * h6 * lam), vb, tA, tK, tM);
    acc += u;
    u = vjp(p1, t_fma(hh, u, h6 * lam), vb, tA, tK, tM);
    return lam + (acc + u);
  }
};

template <int RNG, int INJ>
__global__ void __launch_bounds__(64) k_adjoint_fc9(const RollArgs<2, float> a, const AdjArgs g) {
  __shared__ __align__(16) float xch[kWaveSlots<float>];
  const GroupLane gl;
  const int e = (int)blockIdx.x * kWaveGroups + gl.grp;
  if (gl.grp >= kWaveGroups || e >= g.grad->n_entries) return;  // whole groups
  const int cand = g.cand >= 0 ? g.cand : a.srch->nk_idx;
  if ((a.srch->done || cand < 0) && g.cand < 0) return;
  const int i = gl.li;
  const size_t L = (size_t)g.lmax;
  AdjLanes<RNG, INJ> M(a, i, g.k_list[e], a.st->t, (float)a.srch->v[cand],
                       xch + gl.grp * kGroupStride<float>);
  const float wgt = g.w_list[e];
  const int H = a.H, Kc = g.Kc;
  // forward: minimiser and checkpoints, draws four steps ahead
  float x = (float)a.st->x[i];
  M.exch(x);
  int rb = 0, jb = 0, left = Kc, seg = 0;
  float best = M.margin(rb), xbest = x;
  g.ckpt[(size_t)i * L + e] = x;
  constexpr int D = RNG == 0 ? 4 : 1;
  float wn[D];
  if (RNG == 0)
#pragma unroll
    for (int u = 0; u < D; ++u) wn[u] = M.draw(u < H ? u : H - 1);
  for (int j = 0; j < H;) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const float w = RNG == 0 ? wn[u] : M.draw(j);
      if (RNG == 0) wn[u] = M.draw(j + D < H ? j + D : H - 1);
      x = M.step(x, w);
      int r = 0;
      const float m = M.margin(r);
      ++j;
      if (m < best) {
        best = m;
        jb = j;
        rb = r;
        xbest = x;
      }
      if (--left == 0) {
        left = Kc;
        ++seg;
        if (j < H) g.ckpt[((size_t)seg * 9 + i) * L + e] = x;
      }
      if (j >= H) break;
    }
  }
  const bool finite =
      (__builtin_amdgcn_ballot_w64(!(x - x == 0.f) || best != best) & gl.mask) == 0;
  double vb = 0.0, tA = 0.0, tK = 0.0, tM = 0.0;
  if (finite) {
    // lam = dm/dx at the minimiser: rows of the output's gradient by lane
    M.exch(xbest);
    const float x8 = M.slot[11], x6 = M.X6;
    float xs9[9], lam9[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) xs9[c] = 0.f;
    xs9[6] = x6;
    xs9[8] = x8;
    Plant<2, float>::out_grad(a.pc, a.F + rb * Plant<2, float>::ny, xs9, lam9);
    float lam = i == 0 ? lam9[0] : (i == 6 ? lam9[6] : (i == 8 ? lam9[8] : 0.f));
    for (int sg = (jb - 1) / Kc; jb > 0 && sg >= 0; --sg) {
      const int j0 = sg * Kc, j1 = (j0 + Kc) < jb ? (j0 + Kc) : jb;
      float xs = g.ckpt[((size_t)sg * 9 + i) * L + e];
      float wf = M.draw(j0), w1 = j0 + 1 < j1 ? M.draw(j0 + 1) : 0.f;
      M.exch(xs);
      for (int j = j0; j < j1; ++j) {
        g.seg[((size_t)(j - j0) * 9 + i) * L + e] = xs;
        const float w2 = j + 2 < j1 ? M.draw(j + 2) : 0.f;
        if (j + 1 < j1) xs = M.step(xs, wf);  // the segment's end is not needed
        wf = w1;
        w1 = w2;
      }
      // states and draws of the reverse sweep two steps ahead
      auto sx = [&](int j) { return g.seg[((size_t)(j - j0) * 9 + i) * L + e]; };
      float xa = sx(j1 - 1), wa = M.draw(j1 - 1), xc = 0.f, wc = 0.f;
      if (j1 - 2 >= j0) {
        xc = sx(j1 - 2);
        wc = M.draw(j1 - 2);
      }
      for (int j = j1 - 1; j >= j0; --j) {
        float x2 = 0.f, w2 = 0.f;
        if (j - 2 >= j0) {
          x2 = sx(j - 2);
          w2 = M.draw(j - 2);
        }
        lam = M.step_vjp(xa, wa, lam, vb, tA, tK, tM);
        xa = xc;
        wa = wc;
        xc = x2;
        wc = w2;
      }
    }
  } else {
    best = -INFINITY;
  }
  // outputs: lanes 6, 7, 8 hold the set-point sums
  const double dw = (double)wgt;
  double* xd = reinterpret_cast<double*>(M.slot);
  group_sync();
  if (i >= 6) xd[i - 6] = vb;
  group_sync();
  if (i == 0) {
    g.out_m[e] = best;
    g.out_dv[e] = dw * ((xd[0] + xd[1]) + xd[2]);
    if (e == 0) {
      g.grad->j_star = jb;
      g.grad->r_star = rb;
    }
  }
  double* dth = g.out_dth + (size_t)e * kMaxTh;
  dth[i] = dw * tA * (double)M.fA;
  dth[9 + i] = dw * tK * (double)M.fK;
  if (i == 6) dth[18] = dw * tM * (double)M.fM;
  if (i == 8) dth[19] = dw * tM * (double)M.fM;
}

hipError_t launch_adjoint_fc9(const Problem& pr, const AdjArgs& g, int max_entries,
                              const DevBuffers& b, hipStream_t st) {
  auto a = make_args<2, float>(pr, 0.0, 0, 0, b);
  return by_bit(pr.s.rng_mode, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    return by_bit(pr.s.inject, [&](auto ic) {
      constexpr int I = decltype(ic)::value;
      hipLaunchKernelGGL((k_adjoint_fc9<R, I>), dim3(div_up(max_entries, kWaveGroups)), dim3(64), 0,
                         st, a, g);
      return hipGetLastError();
    });
  });
}

}  // namespace rg
