// FP32 set-point sweeps of the 4-state plant (rg_margin) on the matrix cores:
// v_mfma_f32_4x4x1 multiplies, in sixteen blocks at once, a column of a 4 x 4
// matrix with one value per lane, and leaves the four rows of lane l's product in
// lane l's four result registers.  So a lane holds one scenario's whole state, a
// derivative s + A x + G (x.*x) is four squares and eight such instructions, and
// the one register of matrix columns (A, G, -(F C), E: block b of the register
// holds column b) serves every lane through the instruction's block broadcast.
// Each product is one fused multiply-add, added in the order of the other FP32
// rollouts of this plant.
#include <hip/hip_runtime.h>

#include "rg_lq4_mx.hpp"

namespace rg {

typedef float f4 __attribute__((ext_vector_type(4)));

// c + column `col` of the matrices times b.
template <int COL>
__device__ __forceinline__ f4 mf_col(float m, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(m, b, c, 4, COL, 0);
}
// out[c] += the four columns from COL0 times x[c], for every candidate c: column
// by column, so that dependent instructions are CPL apart.
template <int CPL, int COL0, int Q = 0>
__device__ __forceinline__ void mf_mat(float m, const f4 (&x)[CPL], f4 (&out)[CPL]) {
#pragma unroll
  for (int c = 0; c < CPL; ++c) out[c] = mf_col<COL0 + Q>(m, x[c][Q], out[c]);
  if constexpr (Q < 3) mf_mat<CPL, COL0, Q + 1>(m, x, out);
}

// Full-horizon rollouts of CPL candidates per lane (blockIdx.y: candidates CPL
// blockIdx.y ..), one wave per workgroup: the candidates share their scenario's
// draws, and their independent chains fill the matrix instructions' latency.
// Bound by issue (FP32 matrix instructions, 2.5 vector slots each, share the
// pipe with the vector ALU): 38 of them and about 50 vector instructions per
// candidate-step of 64 scenarios, 265 ns with the SIMDs full, where the quad
// layout takes 4 x 104 ns and regenerates the draws in every lane of a quad.
// 17 candidates at N = 16384 H = 1500: 2.65 -> 2.00 ms with streamed draws, 4.48
// -> 2.82 with regenerated ones; 33 at N = 65536 H = 500: 6.7 -> 4.2, 10.7 -> 4.6.
template <int RNG, int INJ, int CPL>
__global__ void __launch_bounds__(64, 2) k_sweep_lq4(const RollArgs<1, float> a, const MxCoef mc) {
  constexpr int U = 8;  // steps per group of prefetched draws
  __shared__ unsigned long long sh[16];
  DevSearch* S = a.srch;
  const int c0 = (int)blockIdx.y * CPL;
  if (S->done || c0 >= S->n_cand) return;
  const int l = threadIdx.x, blk = l >> 2, i4 = l & 3;
  const int k = (int)blockIdx.x * 64 + l;
  const bool live = k < a.N;
  const int kk = live ? k : a.N - 1;  // lanes past N repeat the last scenario
  const uint32_t t = a.st->t;
  // this lane's element of the matrix columns
  const float m = (float)(blk < 4    ? mc.a[4 * i4 + blk]
                          : blk < 8  ? mc.g[4 * i4 + blk - 4]
                          : blk < 12 ? mc.d[4 * i4 + blk - 8]
                          : blk < 14 ? mc.e[2 * i4 + blk - 12]
                                     : 0.0);
  f4 x[CPL], bv[CPL], grow;
  float best[CPL];
  int jb[CPL];
#pragma unroll
  for (int r = 0; r < 4; ++r) grow[r] = (float)mc.grow[r];
  float mr[CPL];
  auto row_min = [&]() {
    f4 y[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) y[c] = grow;
    mf_mat<CPL, 8>(m, x, y);
#pragma unroll
    for (int c = 0; c < CPL; ++c) mr[c] = fminf(fminf(y[c][0], y[c][1]), fminf(y[c][2], y[c][3]));
  };
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int cc = c0 + c < S->n_cand ? c0 + c : c0;  // a short last group repeats
    const float v = (float)S->v[cc];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      bv[c][r] = (float)mc.b[r] * v;
      x[c][r] = (float)a.st->x[r];
    }
    jb[c] = 0;
  }
  row_min();
#pragma unroll
  for (int c = 0; c < CPL; ++c) best[c] = mr[c];
  const float h = a.h, hh = a.hh, h6 = a.h6;
  f4 s[CPL], kd[CPL], acc[CPL], xs[CPL];
  // kd = s + A y + G (y.*y)
  auto deriv = [&](const f4(&y)[CPL]) {
    f4 q[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      kd[c] = s[c];
      q[c] = y[c] * y[c];
    }
    mf_mat<CPL, 0>(m, y, kd);
    mf_mat<CPL, 4>(m, q, kd);
  };
  auto axpy = [](float w, f4 p, f4 q) {
    f4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = __builtin_fmaf(w, p[r], q[r]);
    return o;
  };
  auto step = [&](float w0, float w1, int jnext) {
    f4 post = {0.f, 0.f, 0.f, 0.f};
    if (INJ == 1) post = mf_col<13>(m, w1, mf_col<12>(m, w0, post));
#pragma unroll
    for (int c = 0; c < CPL; ++c) s[c] = INJ == 0 ? mf_col<12>(m, w0, bv[c]) : bv[c];
    if (INJ == 0)
#pragma unroll
      for (int c = 0; c < CPL; ++c) s[c] = mf_col<13>(m, w1, s[c]);
    deriv(x);
#pragma unroll
    for (int g = 0; g < 3; ++g) {
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        acc[c] = g == 0 ? kd[c] : axpy(2.f, kd[c], acc[c]);
        xs[c] = axpy(g < 2 ? hh : h, kd[c], x[c]);
      }
      deriv(xs);
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      x[c] = axpy(h6, acc[c] + kd[c], x[c]);
      if (INJ == 1) x[c] = x[c] + post;
    }
    row_min();
#pragma unroll
    for (int c = 0; c < CPL; ++c)
      if (mr[c] < best[c]) {
        best[c] = mr[c];
        jb[c] = jnext;
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
    const f4 d = x[c] - x[c];
    float b = best[c];
    if (!((d[0] + d[1]) + (d[2] + d[3]) == 0.f) || b != b) b = -INFINITY;
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

// Nanoseconds per step of the busiest SIMD, by layout: a wave alone on its SIMD
// pays its chain's latency, several share the issue slots.  Measured on sweeps of
// 5 to 33 candidates at N = 1000 .. 65536 (within 10 %): c candidates per lane,
// streamed / regenerated draws, alone 470 / 555 (c = 1), 770 / 900 (2), 1080 /
// 1250 (3), else 265 / 380, 560 / 690, 830 / 970 per wave; the quad layout 185 /
// 290 alone, 104 / 176 per wave of 16 scenarios.
static double sweep_cost(int M, int N, int rng, int c) {
  const long long waves = (long long)div_up((size_t)M, (size_t)c) * div_up((size_t)N, 64);
  const double n = (double)((waves + 1023) / 1024);
  if (n == 1) return 155.0 + 310.0 * c + (rng ? 50.0 + 40.0 * c : 0.0);
  return n * (10.0 + 265.0 * c + (rng ? 105.0 + 10.0 * c : 0.0));
}
static double quad_cost(int M, int N, int rng) {
  const double n = (double)(((long long)M * div_up((size_t)N, 16) + 1023) / 1024);
  const double alone = rng ? 290.0 : 185.0, t = n * (rng ? 176.0 : 104.0);
  return t > alone ? t : alone;
}

int sweep_candidates_per_lane(const Problem& pr, int M) {
  int best = 0;
  double cost = quad_cost(M, pr.s.N, pr.s.rng_mode);
  for (int c = 1; c <= 3; ++c) {
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
  const MxCoef mc = make_mx_coef(pr);
  auto a = make_args<1, float>(pr, band, 0, 1, b);
  return by_bit(pr.s.rng_mode, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    return by_bit(pr.s.inject, [&](auto ic) {
      constexpr int I = decltype(ic)::value;
      switch (cpl) {
        case 1: hipLaunchKernelGGL((k_sweep_lq4<R, I, 1>), grid, dim3(64), 0, st, a, mc); break;
        case 2: hipLaunchKernelGGL((k_sweep_lq4<R, I, 2>), grid, dim3(64), 0, st, a, mc); break;
        case 3: hipLaunchKernelGGL((k_sweep_lq4<R, I, 3>), grid, dim3(64), 0, st, a, mc); break;
        default: return hipErrorInvalidValue;
      }
      return hipGetLastError();
    });
  });
}

}  // namespace rg
