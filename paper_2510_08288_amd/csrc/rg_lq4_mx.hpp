// The 4-state plant in FP64 on the matrix cores: v_mfma_f64_4x4x4 multiplies a
// 4 x 4 matrix with 4 x 4 operands in four independent blocks, that is, with the
// states of 16 scenarios, and both its operand and its result layout put
// component (row) l >> 4 of scenario l & 15 on lane l.  So one wave runs 16
// scenarios, lane l owning state component l >> 4 of scenario l & 15, and a
// derivative s + A x + G (x.*x) is one multiplication and two matrix
// instructions with no exchange between lanes; the constraint rows g - (F C) x
// are one more, and the disturbance enters through another (its draws sit in
// the operand's component slots).  The instruction adds its four products in
// ascending order, one fused multiply-add each, so a derivative rounds as the
// one-lane FP64 derivative does.
//
// Matrix instructions ignore the lane mask and need whole waves: lanes without
// a scenario of their own repeat another one and their results are dropped.
#pragma once

#include "rg_roll.hpp"

namespace rg {

struct MxCoef {
  double a[16], g[16];  // A, G (row-major)
  double d[16];         // -(F C)
  double e[8], b[4];    // E, B
  double grow[4];       // g (+inf for padding rows)
};

inline MxCoef make_mx_coef(const Problem& pr) {
  MxCoef m;
  const double* c = pr.p.coeffs;
  for (int i = 0; i < 16; ++i) {
    m.a[i] = c[i];
    m.g[i] = c[20 + i];
  }
  for (int i = 0; i < 4; ++i) m.b[i] = c[16 + i];
  for (int i = 0; i < 8; ++i) m.e[i] = c[36 + i];
  for (int r = 0; r < 4; ++r) {
    for (int i = 0; i < 4; ++i) {
      double acc = 0.0;
      for (int y = 0; y < 2; ++y) acc += pr.c.F[r * 2 + y] * c[44 + 4 * y + i];
      m.d[4 * r + i] = -acc;
    }
    m.grow[r] = pr.c.g[r];
  }
  return m;
}

// D = A B + C over the wave (A: the 4 x 4 matrix, element [l & 3][l >> 4]).
__device__ __forceinline__ double mx_mul(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Or of a wave's ballot over the four lanes of each scenario: bit s for
// scenario s of the wave.
__device__ __forceinline__ uint32_t mx_scenarios(bool p) {
  const unsigned long long m = __builtin_amdgcn_ballot_w64(p);
  const uint32_t h = (uint32_t)m | (uint32_t)(m >> 32);
  return (h | (h >> 16)) & 0xffffu;
}

// Smallest value over the four lanes of each scenario.
__device__ __forceinline__ double mx_min(double v) {
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const double o = __shfl_xor(v, off);
    v = o < v ? o : v;
  }
  return v;
}

// A wave-uniform pointer in scalar registers.
__device__ __forceinline__ const char* uniform_ptr(const void* ptr) {
  const uint64_t p = (uint64_t)ptr;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
  return (const char*)(((uint64_t)hi << 32) | lo);
}

// One lane's share of the model.  RNG 0 (streamed draws): one value per lane
// holds the two disturbances of two steps, component l >> 4 being w0, w1 of the
// even step and w0, w1 of the odd one, and E selects a step's pair.  RNG 1: the
// lane draws both disturbances of step (l >> 4) of every four, and E selects
// that step's slot.  The other slots are multiplied by zero (draws are finite).
template <int RNG, int INJ>
struct MxLane {
  double A, G, D, grow, bv, h, hh, h6;
  double E0[RNG ? 4 : 2], E1[RNG ? 4 : 1];
  __device__ __forceinline__ void init(const MxCoef& m, double v, double h_, double hh_, double h6_) {
    const int l = threadIdx.x & 63, i = l & 3, q = l >> 4;
    A = m.a[4 * i + q];
    G = m.g[4 * i + q];
    D = m.d[4 * i + q];
    grow = m.grow[q];
    bv = m.b[q] * v;
    h = h_;
    hh = hh_;
    h6 = h6_;
    const double e0 = m.e[2 * i], e1 = m.e[2 * i + 1];
    if constexpr (RNG == 0) {
      const double e = (q & 1) ? e1 : e0;
      E0[0] = q < 2 ? e : 0.0;
      E0[1] = q < 2 ? 0.0 : e;
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        E0[u] = q == u ? e0 : 0.0;
        E1[u] = q == u ? e1 : 0.0;
      }
    }
  }
  __device__ __forceinline__ double margin(double x) const { return mx_mul(D, x, grow); }
  // c + E w of step u of a group (w: the group's draws of this lane)
  __device__ __forceinline__ double dist(const float* w, int u, double c) const {
    if constexpr (RNG == 0) return mx_mul(E0[u & 1], (double)w[u >> 1], c);
    const int b = u >> 2;
    return mx_mul(E1[RNG ? u & 3 : 0], (double)w[2 * b + 1],
                  mx_mul(E0[RNG ? u & 3 : 0], (double)w[2 * b], c));
  }
  __device__ __forceinline__ double deriv(double s, double x) const {
    return mx_mul(G, x * x, mx_mul(A, x, s));
  }
  __device__ __forceinline__ void step(const float* w, int u, double& x) const {
    const double s = INJ == 0 ? dist(w, u, bv) : bv;
    const double k1 = deriv(s, x);
    double acc = k1;
    double xs = __builtin_fma(hh, k1, x);
    const double k2 = deriv(s, xs);
    acc = __builtin_fma(2.0, k2, acc);
    xs = __builtin_fma(hh, k2, x);
    const double k3 = deriv(s, xs);
    acc = __builtin_fma(2.0, k3, acc);
    xs = __builtin_fma(h, k3, x);
    const double k4 = deriv(s, xs);
    x = __builtin_fma(h6, acc + k4, x);
    if (INJ == 1) x = x + dist(w, u, 0.0);
  }
};

// Rollout of the wave's 16 scenarios from x (this lane's component) over at
// most H steps: bm is this lane's constraint row's running minimum (RECORD: jq
// its first step).  k is the lane's scenario.  After every group of 16 steps
// stop.end(bm) may end the rollout (it must be uniform over the wave);
// stop.begin() runs at the group's start, so that a flag it reads is there by
// then.  Returns the steps run.
constexpr int kMxGroup = 16;

template <int RNG, int INJ, int RECORD, class Stop>
__device__ __forceinline__ int mx_rollout(const MxLane<RNG, INJ>& M, const RollArgs<1, double>& a,
                                          uint32_t t, int k, double& x, double& bm, int& jq,
                                          Stop& stop) {
  constexpr int U = kMxGroup;
  const int H = a.H, q = (threadIdx.x & 63) >> 4;
  bm = M.margin(x);
  jq = 0;
  // Streamed draws: buffer loads based at the group's first row, so the 32-bit
  // offsets (U rows of 8 N bytes) hold for every N the library takes; a row past
  // the horizon reads as zero.
  const uint32_t row = 8u * (uint32_t)a.N;
  const uint32_t off = 4u * (uint32_t)k + (q & 1) * 4u * (uint32_t)a.N + (q >> 1) * row;
  const char* wsrc = RNG == 0 ? uniform_ptr(step_w(a, t)) : nullptr;
  auto load = [&](int j, float* w) {
    if constexpr (RNG == 0) {
      const int rows = H - j < U ? (H - j > 0 ? H - j : 0) : U;
      const __amdgpu_buffer_rsrc_t res = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(wsrc + (uint64_t)j * row), (short)0, (int)(row * (uint32_t)rows), 0x00020000);
      // The range check compares the lane's offset with the record count minus
      // the scalar offset, unsigned: the scalar offset must not exceed the count.
#pragma unroll
      for (int u = 0; u < U / 2; ++u)
        w[u] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(
                       res, off, row * (uint32_t)(2 * u < rows ? 2 * u : rows), 0));
    } else {
#pragma unroll
      for (int u = 0; u < U / 4; ++u) {
        const Words r = philox10((uint32_t)k, (uint32_t)(j + 4 * u + q), t, 0u, a.seed, a.inst);
        w[2 * u] = box_draw(r.v[0], a.wlo[0], a.wspan[0]);
        w[2 * u + 1] = box_draw(r.v[1], a.wlo[1], a.wspan[1]);
      }
    }
  };
  auto one = [&](const float* w, int u, int j) {
    M.step(w, u, x);
    const double m = M.margin(x);
    if (RECORD) {
      const double mm = m == m ? m : -INFINITY;  // a state that left the range
      if (mm < bm) {
        bm = mm;
        jq = j + 1;
      }
    } else {
      bm = fmin(bm, m);
    }
  };
  float wa[U / 2], wb[U / 2];
  load(0, wa);
  const int full = H / U;
  int g = 0;
  auto group = [&](const float* wc, float* wn) -> bool {
    load((g + 1) * U, wn);
    stop.begin();
#pragma unroll
    for (int u = 0; u < U; ++u) one(wc, u, g * U + u);
    ++g;
    return stop.end(bm);
  };
  while (g < full) {  // two draw buffers in turn
    if (group(wa, wb)) return g * U;
    if (g == full) {
#pragma unroll
      for (int u = 0; u < U / 2; ++u) wa[u] = wb[u];
      break;
    }
    if (group(wb, wa)) return g * U;
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (full * U + u < H) one(wa, u, full * U + u);  // ragged tail of the horizon
  return H;
}

hipError_t launch_rollout_lq4_mx(const Problem& pr, double band, int early_exit, int record,
                                 const LaunchCfg& cfg, const DevBuffers& b, hipStream_t st,
                                 int gen_rows, float* gen_w, float* gen_th);

// FP32 set-point sweeps (full horizon, per-scenario margins recorded): how many
// candidates per lane the one-lane layout takes for M candidates, 0 where
// the quad layout is faster.
int sweep_candidates_per_lane(const Problem& pr, int M);
hipError_t launch_sweep_lq4(const Problem& pr, double band, int M, int cpl, const DevBuffers& b,
                            hipStream_t st);

}  // namespace rg
