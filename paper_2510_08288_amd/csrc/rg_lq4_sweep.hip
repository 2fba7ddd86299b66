// FP32 set-point sweeps of the 4-state plant (rg_margin), one scenario per lane:
// the whole state in a lane's registers, no exchange between lanes, and draws
// that are loaded or regenerated once for every candidate the lane takes, where
// the quad layout regenerates them in all four lanes.
//
// A margin must not depend on which or how many other candidates are asked for,
// and the choice between the two layouts does; so every sum here has the order
// and the contractions of the quad rollout (quad_deriv and row_margin as
// compiled, the pairs its two butterflies form), and margins and minimising steps
// equal it bit for bit.
#include <hip/hip_runtime.h>

#include "rg_lq4_mx.hpp"

namespace rg {

// The model in vector registers, entry [r][s] the one of row r and column r ^ s
// (a scalar operand makes an FP32 instruction half as long again as a vector
// one, and two of them do not fit into one instruction).
struct SweepCoef {
  float a[4][4], g[4][4], d[4][4], e[4][2], grow[4];
  float b[4];
};

static SweepCoef make_sweep_coef(const Problem& pr) {
  const MxCoef m = make_mx_coef(pr);
  SweepCoef c;
  for (int r = 0; r < 4; ++r) {
    for (int s = 0; s < 4; ++s) {
      c.a[r][s] = (float)m.a[4 * r + (r ^ s)];
      c.g[r][s] = (float)m.g[4 * r + (r ^ s)];
      c.d[r][s] = (float)m.d[4 * r + (r ^ s)];
    }
    c.e[r][0] = (float)m.e[2 * r];
    c.e[r][1] = (float)m.e[2 * r + 1];
    c.b[r] = (float)m.b[r];
    c.grow[r] = (float)m.grow[r];
  }
  return c;
}

// A lane value equal to a uniform one (an identity DPP move).
__device__ __forceinline__ float lane_value(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xE4, 0xf, 0xf, true));
}
__device__ __forceinline__ float sweep_min2(float a, float b) { return b < a ? b : a; }

// Full-horizon rollouts of CPL candidates per lane (blockIdx.y: candidates CPL
// blockIdx.y ..), one wave per workgroup.  Bound by vector issue: about 230
// instructions per candidate-step of 64 scenarios, 250 ns with the SIMDs full
// (regenerated draws 290, 260 with three candidates sharing them), where the quad
// layout takes 4 x 98 ns (4 x 160).  Calls: 17 candidates at N = 16384 H = 1500 2.61
// -> 1.98 ms with streamed draws, 4.23 -> 2.22 with regenerated ones; 33 at N =
// 65536 H = 500 6.52 -> 4.23, 10.7 -> 4.32.  (FP32 matrix instructions take 265 and
// 325 ns, and add in an order of their own.)
template <int RNG, int INJ, int CPL>
__global__ void __launch_bounds__(64, 2) k_sweep_lq4(const RollArgs<1, float> a,
                                                     const SweepCoef sc) {
#pragma clang fp contract(off)
  constexpr int U = 8;  // steps per group of prefetched draws
  __shared__ unsigned long long sh[16];
  DevSearch* S = a.srch;
  const int c0 = (int)blockIdx.y * CPL;
  if (S->done || c0 >= S->n_cand) return;
  const int l = threadIdx.x;
  const int k = (int)blockIdx.x * 64 + l;
  const bool live = k < a.N;
  const int kk = live ? k : a.N - 1;  // lanes past N repeat the last scenario
  const uint32_t t = a.st->t;
  float A[4][4], G[4][4], D[4][4], E[4][2], grow[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      A[r][s] = lane_value(sc.a[r][s]);
      G[r][s] = lane_value(sc.g[r][s]);
      D[r][s] = lane_value(sc.d[r][s]);
    }
    E[r][0] = lane_value(sc.e[r][0]);
    E[r][1] = lane_value(sc.e[r][1]);
    grow[r] = lane_value(sc.grow[r]);
  }
  float x[CPL][4], bv[CPL][4], best[CPL];
  int jb[CPL];
  // smallest row margin, by the quad's lane 0
  auto row_min = [&](const float* y) {
#pragma clang fp contract(off)
    float m[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      m[r] = (__builtin_fmaf(D[r][0], y[r], grow[r]) + D[r][2] * y[r ^ 2]) +
             __builtin_fmaf(D[r][1], y[r ^ 1], D[r][3] * y[r ^ 3]);
    return sweep_min2(sweep_min2(m[0], m[1]), sweep_min2(m[2], m[3]));
  };
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int cc = c0 + c < S->n_cand ? c0 + c : c0;  // a short last group repeats
    const float v = (float)S->v[cc];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      bv[c][r] = sc.b[r] * v;
      x[c][r] = (float)a.st->x[r];
    }
    best[c] = row_min(x[c]);
    jb[c] = 0;
  }
  const float h = a.h, hh = a.hh, h6 = a.h6;
  // o = s + A y + G (y.*y)
  auto deriv = [&](const float* s, const float* y, float* o) {
#pragma clang fp contract(off)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float c0r = __builtin_fmaf(__builtin_fmaf(G[r][0], y[r], A[r][0]), y[r], s[r]);
      const float c2r = __builtin_fmaf(G[r][2], y[r ^ 2], A[r][2]) * y[r ^ 2];
      const float c3r = __builtin_fmaf(G[r][3], y[r ^ 3], A[r][3]) * y[r ^ 3];
      const float c1r = __builtin_fmaf(__builtin_fmaf(G[r][1], y[r ^ 1], A[r][1]), y[r ^ 1], c3r);
      o[r] = (c0r + c2r) + c1r;
    }
  };
  auto step = [&](float w0, float w1, int jnext) {
#pragma clang fp contract(off)
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      float s[4], kd[4], acc[4], xs[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        s[r] = INJ == 0 ? __builtin_fmaf(E[r][1], w1, __builtin_fmaf(E[r][0], w0, bv[c][r]))
                        : bv[c][r];
      deriv(s, x[c], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) xs[r] = __builtin_fmaf(hh, acc[r], x[c][r]);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        deriv(s, xs, kd);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[r] = __builtin_fmaf(2.f, kd[r], acc[r]);
          xs[r] = __builtin_fmaf(g == 0 ? hh : h, kd[r], x[c][r]);
        }
      }
      deriv(s, xs, kd);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[c][r] = __builtin_fmaf(h6, acc[r] + kd[r], x[c][r]);
        if (INJ == 1) x[c][r] = x[c][r] + __builtin_fmaf(E[r][0], w0, E[r][1] * w1);
      }
      const float m = row_min(x[c]);
      if (m < best[c]) {
        best[c] = m;
        jb[c] = jnext;
      }
    }
  };
  // draws, a group of U steps ahead: buffer loads based at the group's first row
  // (rows past the horizon read as zero)
  const uint32_t row = 8u * (uint32_t)a.N, vo0 = 4u * (uint32_t)kk, vo1 = vo0 + 4u * (uint32_t)a.N;
  const char* wsrc = RNG == 0 ? uniform_ptr(step_w(a, t)) : nullptr;
  const int H = a.H;
  auto load = [&](int j, float* w) {
    if (RNG == 0) {
      const int rows = H - j < U ? (H - j > 0 ? H - j : 0) : U;
      const __amdgpu_buffer_rsrc_t res = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(wsrc + (uint64_t)j * row), (short)0, (int)(row * (uint32_t)rows), 0x00020000);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t so = row * (uint32_t)(u < rows ? u : rows);  // see mx_rollout
        w[2 * u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(res, vo0, so, 0));
        w[2 * u + 1] =
            __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(res, vo1, so, 0));
      }
    }
  };
  float wa[2 * U], wb[2 * U];
  load(0, wa);
  for (int j = 0; j < H; j += U) {
    load(j + U, wb);
#pragma unroll 1
    for (int u = 0; u < U; u += 2) {
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        if (j + u + d >= H) break;
        float w0, w1;
        if (RNG == 0) {
          w0 = wa[2 * d];
          w1 = wa[2 * d + 1];
        } else {
          const Words r = philox10((uint32_t)kk, (uint32_t)(j + u + d), t, 0u, a.seed, a.inst);
          w0 = box_draw(r.v[0], a.wlo[0], a.wspan[0]);
          w1 = box_draw(r.v[1], a.wlo[1], a.wspan[1]);
        }
        step(w0, w1, j + u + d + 1);
      }
      if (RNG == 0)  // the group's draws move down two steps
#pragma unroll
        for (int q = 0; q < 2 * U - 4; ++q) wa[q] = wa[q + 4];
    }
    if (RNG == 0)
#pragma unroll
      for (int q = 0; q < 2 * U; ++q) wa[q] = wb[q];
  }
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int cc = c0 + c;
    if (cc >= S->n_cand) break;  // uniform
    float bad = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) bad += x[c][r] - x[c][r];
    float b = best[c];
    if (!(bad == 0.f) || b != b) b = -INFINITY;
    if (live) {
      a.per_m[(size_t)cc * a.N + k] = b;
      a.per_j[(size_t)cc * a.N + k] = jb[c];
      if (b < -a.band) {
        __hip_atomic_store(&S->dead[cc], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (b < a.band) {
        const int idx = atomicAdd(&S->n_recheck, 1);
        a.rlist[idx] = make_int2(cc, k);
      }
    }
    const unsigned long long key = live ? lane_key(b, k) : ~0ull;
    const unsigned long long kall = block_min_u64(key, sh);
    const unsigned long long kfar = block_min_u64(live && b >= a.band ? key : ~0ull, sh);
    const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(live));
    if (l == 0) {
      atomicMin(&S->key_all[cc], kall);
      if (kfar != ~0ull) atomicMin(&S->key_far[cc], kfar);
      atomicAdd(&S->lane_steps, (unsigned long long)n * (unsigned long long)H);
    }
  }
}

// Nanoseconds per step of a launch by layout, from the waves of the busiest SIMD:
// one wave alone pays its chain's latency, several share the issue slots.  Fitted
// to sweeps of 3 to 33 candidates at N = 1000 .. 65536 (mostly within 10 %),
// streamed / regenerated draws; two candidates per lane lie between one and three.
static double sweep_cost(int M, int N, int rng, int c) {
  const long long waves = (long long)div_up((size_t)M, (size_t)c) * div_up((size_t)N, 64);
  const double n = (double)((waves + 1023) / 1024);
  if (c == 1) return n == 1 ? (rng ? 545.0 : 480.0) : (rng ? 50.0 + 292.0 * n : 45.0 + 250.0 * n);
  if (n <= 2) return n == 1 ? (rng ? 1315.0 : 1240.0) : (rng ? 1450.0 : 1330.0);
  return n * (rng ? 790.0 : 770.0);
}
static double quad_cost(int M, int N, int rng) {
  const double n = (double)(((long long)M * div_up((size_t)N, 16) + 1023) / 1024);
  return rng ? 105.0 + 160.0 * n : 85.0 + 97.5 * n;
}

int sweep_candidates_per_lane(const Problem& pr, int M) {
  int best = 0;
  double cost = quad_cost(M, pr.s.N, pr.s.rng_mode);
  for (int c = 1; c <= 3; c += 2) {
    const double t = sweep_cost(M, pr.s.N, pr.s.rng_mode, c);
    if (t < cost) {
      cost = t;
      best = c;
    }
  }
  return best;
}

hipError_t launch_sweep_lq4(const Problem& pr, double band, int M, int cpl, const DevBuffers& b,
                            hipStream_t st) {
  const dim3 grid(div_up((size_t)pr.s.N, 64), div_up((size_t)M, (size_t)cpl));
  const SweepCoef sc = make_sweep_coef(pr);
  auto a = make_args<1, float>(pr, band, 0, 1, b);
  return by_bit(pr.s.rng_mode, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    return by_bit(pr.s.inject, [&](auto ic) {
      constexpr int I = decltype(ic)::value;
      switch (cpl) {
        case 1: hipLaunchKernelGGL((k_sweep_lq4<R, I, 1>), grid, dim3(64), 0, st, a, sc); break;
        case 3: hipLaunchKernelGGL((k_sweep_lq4<R, I, 3>), grid, dim3(64), 0, st, a, sc); break;
        default: return hipErrorInvalidValue;
      }
      return hipGetLastError();
    });
  });
}

}  // namespace rg
