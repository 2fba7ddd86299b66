// What the rollout kernels of both plants share: argument blocks and their
// host-side filling, scenario draws, the draw workgroups of a launch, workgroup
// reductions and the tests every rollout workgroup starts with.
#pragma once

#include <cstring>
#include <type_traits>

#include "rg_device.hpp"

namespace rg {

// ---------------------------------------------------------------------------
// Argument blocks
// ---------------------------------------------------------------------------
template <int KIND, class T>
struct RollArgs {
  using P = Plant<KIND, T>;
  typename P::Coef pc;
  T F[kNC * P::ny];
  T g[kNC];
  T h, hh, h6;
  T band;
  int H, N;
  int early, record, inject;
  uint32_t seed, inst;
  float wlo[P::nw], wspan[P::nw];
  float thlo, thspan;
  const float* wbuf;
  const float* thbuf;
  const DevState* st;
  DevSearch* srch;
  float* per_m;
  int32_t* per_j;
  unsigned long long* per_key;  // chance-constrained verdict: per-scenario margin keys
  int2* rlist;
  // checkpoints of one candidate's scenarios for the segment derivative:
  // ckpt[(s * n + i) * N + k] = state component i of scenario k at step s * Kc
  float* ckpt;
  int Kc;
  int ckpt_cand;  // that candidate (-1: the Newton iterate of the round)
  // gen_row0 > 0: rows blockIdx.y >= gen_row0 of the launch generate the
  // draws of step t + 1 into gen_w / gen_th instead of simulating
  int gen_row0;
  uint32_t gen_ofs;  // the draws generated are those of step t + gen_ofs
  float* gen_w;
  float* gen_th;
  // forward tangent (CKPT = 2): per scenario of the tangent candidate, dm/dv
  // (tan_dv[k]), the margin (per_m[k]) and its minimising step (per_j[k])
  float* tan_dv;
  // ring != 0 (closed loop): the draws of step s are in wring[s % kPairs],
  // selected from the step counter on the device (wbuf, gen_w and gen_th are
  // then unused; gen_w != nullptr only switches the draw workgroups on)
  int ring;
  float* wring[kPairs];
  float* thring[kPairs];
};

// Draws of step t (streamed mode).
template <class A>
__device__ __forceinline__ const float* step_w(const A& a, uint32_t t) {
  return a.ring ? a.wring[t % kPairs] : a.wbuf;
}
template <class A>
__device__ __forceinline__ const float* step_th(const A& a, uint32_t t) {
  return a.ring ? a.thring[t % kPairs] : a.thbuf;
}

template <int KIND>
struct CtlArgs {
  typename Plant<KIND, double>::Coef pc;
  DevState* st;
  DevSearch* srch;
  const double* r_seq;
  int closed_loop;
  DevGrad* grad;
};

// ---------------------------------------------------------------------------
// Draws
// ---------------------------------------------------------------------------
template <int NW>
__device__ __forceinline__ void draw_w(uint32_t seed, uint32_t inst, uint32_t t, uint32_t tag,
                                       uint32_t k, uint32_t j, const float* lo, const float* span,
                                       float* w) {
#pragma unroll
  for (int blk = 0; blk < (NW + 3) / 4; ++blk) {
    const Words r = philox10(k, j, t, (tag << 16) | (uint32_t)blk, seed, inst);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = 4 * blk + q;
      if (c < NW) w[c] = box_draw(r.v[q], lo[c], span[c]);
    }
  }
}

template <int NTH>
__device__ __forceinline__ void draw_theta_factor(uint32_t seed, uint32_t inst, uint32_t t,
                                                  uint32_t k, float lo, float span, float* f) {
#pragma unroll
  for (int blk = 0; blk < (NTH + 3) / 4; ++blk) {
    const Words r = philox10(k, 0u, t, (1u << 16) | (uint32_t)blk, seed, inst);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = 4 * blk + q;
      if (c < NTH) f[c] = box_draw(r.v[q], lo, span);
    }
  }
}

// Streamed draws: w[(j * nw + c) * N + k] (consecutive scenarios contiguous, so
// a wave's loads of one step coalesce), theta factors f[c * N + k].
template <int KIND, class A>
__device__ __forceinline__ void gen_body(const A& a, float* wbuf, float* thbuf, size_t gid,
                                         uint32_t t, bool streaming = false) {
  using P = Plant<KIND, float>;
  const size_t nwork = (size_t)a.H * a.N;
  if (gid < nwork) {
    const int j = (int)(gid / a.N);
    const int k = (int)(gid - (size_t)j * a.N);
    float w[P::nw];
    draw_w<P::nw>(a.seed, a.inst, t, 0u, (uint32_t)k, (uint32_t)j, a.wlo, a.wspan, w);
#pragma unroll
    for (int c = 0; c < P::nw; ++c) {
      float* dst = &wbuf[((size_t)j * P::nw + c) * a.N + k];
      if (streaming) __builtin_nontemporal_store(w[c], dst);
      else *dst = w[c];
    }
  } else if (P::nth > 0 && gid < nwork + (size_t)a.N) {
    const int k = (int)(gid - nwork);
    float f[P::nth > 0 ? P::nth : 1];
    draw_theta_factor<P::nth>(a.seed, a.inst, t, (uint32_t)k, a.thlo, a.thspan, f);
#pragma unroll
    for (int c = 0; c < P::nth; ++c) {
      float* dst = &thbuf[(size_t)c * a.N + k];
      if (streaming) __builtin_nontemporal_store(f[c], dst);
      else *dst = f[c];
    }
  }
}

// Draw rows of a rollout launch (grid-stride over the rows' threads): the
// draws of step t + gen_ofs, or in the closed loop (ring) those of the steps
// the step's setup chose (gen_lo .. gen_lo + gen_n - 1, in its first round
// only).  Returns true in those rows.
template <int KIND, class A>
__device__ __forceinline__ bool gen_rows(const A& a) {
  if (a.gen_row0 <= 0 || (int)blockIdx.y < a.gen_row0) return false;
  uint32_t t1 = a.st->t + a.gen_ofs;
  int nsteps = 1;
  if (a.ring) {  // while the chunk has steps left
    if (a.srch->round != 0 || a.st->cl_index >= a.st->cl_len) return true;
    t1 = a.st->gen_lo;
    nsteps = a.st->gen_n;
  }
  const size_t nth = (size_t)(gridDim.y - a.gen_row0) * gridDim.x * blockDim.x;
  const size_t work = (size_t)a.H * a.N + (Plant<KIND, float>::nth > 0 ? (size_t)a.N : 0);
  const size_t i0 =
      ((size_t)(blockIdx.y - a.gen_row0) * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x;
  for (int g = 0; g < nsteps; ++g, ++t1) {
    float* gw = a.ring ? a.wring[t1 % kPairs] : a.gen_w;
    float* gth = a.ring ? a.thring[t1 % kPairs] : a.gen_th;
    // streaming stores: these draws are read steps later, and lines left dirty
    // in L2 would have to be written back by the device-scope fences in between
    for (size_t i = i0; i < work; i += nth) gen_body<KIND>(a, gw, gth, i, t1, true);
  }
  return true;
}

// Wave64 + workgroup minimum of a 64-bit key; returns the minimum in thread 0.
__device__ __forceinline__ unsigned long long block_min_u64(unsigned long long v,
                                                             unsigned long long* sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t lo = __shfl_xor((uint32_t)v, off);
    const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), off);
    const unsigned long long o = ((unsigned long long)hi << 32) | lo;
    v = o < v ? o : v;
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[wave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int nw = (blockDim.x + 63) >> 6;
    for (int i = 1; i < nw; ++i) v = sh[i] < v ? sh[i] : v;
  }
  __syncthreads();
  return v;
}

// A candidate's dead flag, shared by all its waves: one that is set is not set
// again.  Stores and atomics on one line take their turn at the memory side,
// about 20 ns each, and where every scenario violates at once each wave has one.
__device__ __forceinline__ bool is_dead(const int32_t* flag) {
  return __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}
__device__ __forceinline__ void raise_dead(int32_t* flag) {
  if (!is_dead(flag)) __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over a workgroup's waves of a value uniform over each; in thread 0.
__device__ __forceinline__ unsigned long long block_sum_waves(unsigned long long v,
                                                               unsigned long long* sh) {
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int nw = (blockDim.x + 63) >> 6;
    for (int i = 1; i < nw; ++i) v += sh[i];
  }
  __syncthreads();
  return v;
}

// Step offset of candidate c: 0 for the step's own candidates, j for a
// speculative candidate of step t + j (closed loop, round 0).
__device__ __forceinline__ int cand_step(const DevSearch* S, int c) {
  const int r = c - S->spec_base;
  return (S->spec_n > 0 && r >= 0 && r < S->spec_n * S->spec_per) ? 1 + r / S->spec_per : 0;
}

// In decision mode a candidate whose FP64 steady-state test already fails is
// refused without simulating it (the verdict of Alg. 1 needs both tests).
// bx: the workgroup's scenario tile (tile 0 raises the flag).
__device__ __forceinline__ bool refused_by_steady_state(int early, DevSearch* S, int c,
                                                        int bx = -1) {
  if (!early || !(S->mss[c] < 0.0)) return false;
  if ((bx < 0 ? (int)blockIdx.x : bx) == 0 && threadIdx.x == 0)
    __hip_atomic_store(&S->dead[c], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// ---------------------------------------------------------------------------
// Host-side argument filling and dispatch helpers
// ---------------------------------------------------------------------------
template <int KIND, class T>
static RollArgs<KIND, T> make_args(const Problem& pr, double band, int early, int record,
                                   const DevBuffers& b) {
  using P = Plant<KIND, T>;
  RollArgs<KIND, T> a;
  memset(&a, 0, sizeof(a));
  P::load(a.pc, pr.p.coeffs);
  for (int r = 0; r < kNC; ++r) {
    for (int i = 0; i < P::ny; ++i) a.F[r * P::ny + i] = (T)pr.c.F[r * P::ny + i];
    a.g[r] = (T)pr.c.g[r];
  }
  a.h = (T)pr.dt;
  a.hh = (T)(pr.dt * 0.5);
  a.h6 = (T)(pr.dt / 6.0);
  a.band = (T)band;
  a.H = pr.H;
  a.N = pr.s.N;
  a.early = early;
  a.record = record;
  a.inject = pr.s.inject;
  a.seed = pr.s.seed;
  a.inst = pr.s.instance;
  for (int c = 0; c < P::nw; ++c) {
    a.wlo[c] = (float)pr.s.wlo[c];
    a.wspan[c] = (float)(pr.s.whi[c] - pr.s.wlo[c]);
  }
  a.thlo = (float)(1.0 - pr.s.theta_rel);
  a.thspan = (float)(2.0 * pr.s.theta_rel);
  a.wbuf = b.wbuf;
  a.thbuf = b.thbuf;
  a.ring = b.ring;
  for (int j = 0; j < kPairs; ++j) {
    a.wring[j] = b.wpair[j];
    a.thring[j] = b.thpair[j];
  }
  a.st = b.st;
  a.srch = b.srch;
  a.per_m = b.per_m;
  a.per_j = b.per_j;
  a.per_key = b.per_key;
  a.rlist = b.rlist;
  a.tan_dv = b.tan_dv;
  return a;
}

template <int V>
using IC = std::integral_constant<int, V>;

template <class F>
static inline hipError_t by_kind(int kind, F&& f) {
  if (kind == 1) return f(IC<1>{});
  if (kind == 2) return f(IC<2>{});
  return hipErrorInvalidValue;
}
template <class F>
static inline hipError_t by_bit(int v, F&& f) {
  return v ? f(IC<1>{}) : f(IC<0>{});
}

static inline int div_up(size_t a, size_t b) { return (int)((a + b - 1) / b); }

}  // namespace rg
