// The 9-state plant with one scenario per group of 9 lanes, lane i owning state
// component i: seven scenarios per wave (lane 63 idles).  For the FP64 rollouts
// and rechecks, and for FP32 rounds with few scenarios: one lane per scenario
// would leave every serial RK4 step on one lane while most of the chip idles.
//
// At every derivative evaluation each lane computes its own activation and
// orifice factor; its neighbours' states and factors come by wave-wide DPP
// shifts (what crosses into another group is never used: a select drops it), and
// the group exchanges the nine activations and x_1, x_7, x_9 through its LDS
// slots.  Each lane then forms its row with coefficients of its own, so the rows
// differ by data, not by selects or branches; the row's operations and their
// order are those of the one-lane derivative (Plant<2>::row), and so the
// margins equal the one-lane rollout's bit for bit.  Control flow is uniform
// over the group (over the wave with WAVE): every branch depends on exchanged
// values or on a ballot.
#pragma once

#include "rg_roll.hpp"

namespace rg {

constexpr int kGroupLanes = 9;
constexpr int kWaveGroups = 7;

// LDS of one group, in values: the activations (16-byte reads), then x_1, x_7,
// x_9 and words that take the other lanes' writes; the stride keeps 16-byte
// alignment and sets the groups of a wave on different banks.
template <class T>
constexpr int kGroupStride = sizeof(T) == 4 ? 20 : 18;
template <class T>
constexpr int kWaveSlots = 8 * kGroupStride<T>;

__device__ __forceinline__ void group_sync() {
  // The group is part of one wave, whose LDS accesses complete in program
  // order; this only keeps the compiler from moving them across.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A value of the next (0x130) or previous (0x138) lane of the wave.
template <int CTRL>
__device__ __forceinline__ float wave_shift(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL,
                                                               0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double wave_shift(double x) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
}

// This lane's place: group 0..6 of its wave (7: lane 63, no group), component.
struct GroupLane {
  int grp, li;
  unsigned long long mask;  // the group's lanes
  __device__ __forceinline__ GroupLane() {
    const int lane = threadIdx.x & 63;
    grp = lane / kGroupLanes;
    li = lane - grp * kGroupLanes;
    mask = grp < kWaveGroups ? 0x1ffull << (kGroupLanes * grp) : 0ull;
  }
};

// Rollout of scenario k by its group.  WAVE (rollouts of one candidate): the
// whole wave stops at the first violation of any of its groups, and stop_flag is
// that candidate's dead flag; otherwise (rechecks, chance-constrained verdict)
// the group stops on its own and stop_flag (nullable) is only read.  CKPT with
// ck: adjoint checkpoints (lane i stores component i).  jbest: first step at the
// minimum; nsteps: steps run.
template <class T, int RNG, int INJ, bool WAVE = false, int CKPT = 0>
__device__ __forceinline__ T rollout_fc9_lanes(const RollArgs<2, T>& a, int early, T v, int k,
                                               uint32_t t, int32_t* stop_flag, T* slot,
                                               const GroupLane& gl, int& jbest, int& nsteps,
                                               bool ck = false, bool* stopped = nullptr) {
  using P = Plant<2, T>;
  const int i = gl.li;
  // sampled coefficient c of this scenario
  const float* tb = RNG == 0 ? step_th(a, t) : nullptr;
  auto theta = [&](int c) -> T {
    float f;
    if (RNG == 0) {
      f = tb[(size_t)c * a.N + k];
    } else {
      const Words r =
          philox10((uint32_t)k, 0u, t, (1u << 16) | (uint32_t)(c >> 2), a.seed, a.inst);
      const int q = c & 3;
      const uint32_t word = q == 0 ? r.v[0] : (q == 1 ? r.v[1] : (q == 2 ? r.v[2] : r.v[3]));
      f = box_draw(word, a.thlo, a.thspan);
    }
    return a.pc.thnom[c] * (T)f;
  };
  // this lane's row: coefficients of Plant<2>::row
  const T ai = theta(i), b1 = theta(15), b2 = theta(16), b3 = theta(17), mu1 = theta(18),
          mu2 = theta(19);
  const T kout = theta(9 + (i < 6 ? i : 0)), kin = theta(9 + (i >= 1 && i < 6 ? i - 1 : 0));
  const T xb = a.pc.xbar[i], nkxb = a.pc.nkxbar[i];
  T axb = t_fma(ai, xb, a.pc.csum[i]);
  if (i == 6) axb = t_fma(b1, v, axb);
  if (i == 8) axb = t_fma(b3 + mu2, v, axb);
  const T A = i == 8 ? t_fma(mu2, v, ai) : ai;
  const T K = i < 6 ? kout : (T)0;
  const T pm = i == 6 ? -mu1 : (T)0;  // P = pm x_i + pc
  const T pc = i == 0 ? a.pc.c_q0 : (i < 6 ? kin : (i == 7 ? b2 * v : (T)0));
  const T q0 = i == 6 ? (T)1 : (T)0;  // Q = q0 x_1 + q6 x_7 + qc, or the flow in
  const T q6 = (i == 0 || i == 7) ? (T)1 : (T)0;
  const T qc = i == 6 ? -a.pc.p1ref : (T)0;
  const bool inflow = i >= 1 && i < 6;
  T wrow[9];
#pragma unroll
  for (int j = 0; j < 9; ++j) wrow[j] = a.pc.W[9 * i + j];
  const float wlo = a.wlo[i], wsp = a.wspan[i];
  // where this lane writes its state: x_1, x_7, x_9, or a word nothing reads
  constexpr int kX = sizeof(T) == 4 ? 9 : 10;
  const int xw = i == 0 ? kX : (i == 6 ? kX + 1 : (i == 8 ? kX + 2 : kX + 3 + (i & 3)));
  // exchange of the evaluation point
  T X0, X6, TZ[10], rl, rh;
  auto exch = [&](T xv) {
    slot[xw] = xv;
    slot[i] = P::act(xv, xb, nkxb);
    const T xn = wave_shift<0x130>(xv);  // x_{i+1}
    rh = P::orifice(xv, i < 5 ? xn : a.pc.p_amb);
    rl = wave_shift<0x138>(rh);  // r_{i-1}
    group_sync();
    typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
    constexpr int n = 16 / sizeof(T);
    const V* sv = reinterpret_cast<const V*>(slot);
#pragma unroll
    for (int b = 0; b < 8 / n; ++b) {
      const V q = sv[b];
#pragma unroll
      for (int u = 0; u < n; ++u) TZ[n * b + u] = q[u];
    }
    TZ[8] = slot[8];
    X0 = slot[kX];
    X6 = slot[kX + 1];
    group_sync();
  };
  auto eval = [&](T xv, T si) {
    const T Q = inflow ? rl : t_fma(q0, X0, t_fma(q6, X6, qc));
    return P::row(si, K, rh, A, xv, wrow, TZ, t_fma(pm, xv, pc), Q);
  };
  auto margin = [&]() -> T {
    T y[P::ny];
    y[0] = t_quot(a.pc.c_q0 * X6, t_fma(a.pc.d1, slot[kX + 2], a.pc.d0));
    y[1] = X0;
    y[2] = X6;
    const T m = margin_rows<P::ny>(a.F, a.g, y);
    return (m == m) ? m : -t_inf<T>();
  };
  const float* wb = RNG == 0 ? step_w(a, t) + (size_t)i * a.N + k : nullptr;
  const size_t wstep = (size_t)P::nw * a.N;
  const int wq = i & 3;
  auto load = [&](int j) -> float {
    if (RNG == 0) return wb[(size_t)j * wstep];
    const Words r = philox10((uint32_t)k, (uint32_t)j, t, (uint32_t)(i >> 2), a.seed, a.inst);
    const uint32_t word = wq == 0 ? r.v[0] : (wq == 1 ? r.v[1] : (wq == 2 ? r.v[2] : r.v[3]));
    return box_draw(word, wlo, wsp);
  };
  T xv = (T)a.st->x[i];
  exch(xv);
  T best = margin();
  jbest = 0;
  int ck_left = 0, ck_seg = 0;  // steps to the next checkpoint, its index
  if constexpr (CKPT) {
    if (ck) {
      a.ckpt[(size_t)i * a.N + k] = (float)xv;
      ck_left = a.Kc;
    }
  }
  // Streamed draws are loaded four steps ahead (a step is shorter than the
  // latency of device memory); regenerated ones when the step needs them.
  constexpr int D = RNG == 0 ? 4 : 1;
  float wn[D];
  const int H = a.H;
  if (RNG == 0)
#pragma unroll
    for (int u = 0; u < D; ++u) wn[u] = load(u < H ? u : H - 1);
  bool stop_seen = false;  // dead flag read at the start of an 8-step block, tested at its end
  bool run = true;
  int j = 0;
  while (run && j < H) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const float wc = RNG == 0 ? wn[u] : load(j);
      if (RNG == 0) wn[u] = load(j + D < H ? j + D : H - 1);
      if (WAVE && early && (j & 7) == 0)
        stop_seen = __hip_atomic_load(stop_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
      const T si = INJ == 0 ? (T)wc + axb : axb;
      T kk = eval(xv, si);
      T acc = kk;
      T xs = t_fma(a.hh, kk, xv);
      exch(xs);
      kk = eval(xs, si);
      acc = t_fma((T)2, kk, acc);
      xs = t_fma(a.hh, kk, xv);
      exch(xs);
      kk = eval(xs, si);
      acc = t_fma((T)2, kk, acc);
      xs = t_fma(a.h, kk, xv);
      exch(xs);
      kk = eval(xs, si);
      xv = t_fma(a.h6, acc + kk, xv);
      if (INJ == 1) xv = xv + (T)wc;
      exch(xv);
      const T m = margin();
      if (m < best) {
        best = m;
        jbest = j + 1;
      }
      if constexpr (CKPT) {
        if (ck && --ck_left == 0) {
          ck_left = a.Kc;
          ++ck_seg;
          a.ckpt[((size_t)ck_seg * P::n + i) * a.N + k] = (float)xv;
        }
      }
      ++j;
      if (early) {
        if constexpr (WAVE) {
          // every group of the wave evaluates the same candidate
          const bool viol = best < -a.band;
          if (__builtin_amdgcn_ballot_w64(viol) != 0) {
            if (viol && i == 0) raise_dead(stop_flag);
            *stopped = true;
            run = false;
            break;
          }
          if ((j & 7) == 0 && __builtin_amdgcn_ballot_w64(stop_seen) != 0) {
            *stopped = true;
            run = false;
            break;
          }
        } else {
          if (best < -a.band) {
            run = false;
            break;
          }
          if ((j & 31) == 0 && stop_flag) {
            const bool f =
                __hip_atomic_load(stop_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
            if (__builtin_amdgcn_ballot_w64(f) & gl.mask) {
              run = false;
              break;
            }
          }
        }
      }
      if (j >= H) break;
    }
  }
  nsteps = j;
  if (__builtin_amdgcn_ballot_w64(!(xv - xv == (T)0)) & gl.mask) best = -t_inf<T>();
  return best;
}

hipError_t launch_rollout_fc9_lanes(const Problem& pr, double band, int precision, int early_exit,
                                    int record, const LaunchCfg& cfg, const DevBuffers& b,
                                    hipStream_t st, int ckpt_cand, int Kc, int gen_rows,
                                    float* gen_w, float* gen_th);
hipError_t launch_flat_rollout_fc9_lanes(int inject, int rng, const void* args_dev,
                                         const int* tile_inst, const int* tile_first, int tiles,
                                         int cmax, int block, hipStream_t st);
// Scenarios of one workgroup of `block` threads.
static inline int fc9_lanes_per_block(int block) { return block / 64 * kWaveGroups; }

}  // namespace rg
