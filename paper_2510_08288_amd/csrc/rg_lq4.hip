// FP64 rollouts of the 4-state plant on the matrix cores (layout and arithmetic
// in rg_lq4_mx.hpp).
#include <hip/hip_runtime.h>

#include "rg_lq4_mx.hpp"

namespace rg {

// blockIdx.y = candidate of the round; every wave takes 16 scenarios.  The
// bookkeeping (dead flags, margin keys, executed steps) is that of the other
// rollout kernels: the wave stops at the first violation of any of its
// scenarios and raises the candidate's dead flag for the others; CHANCE = 1
// counts each violating scenario once, and the candidate dies once more than q
// did.
//
// Bound by the latency of a wave's chain (per derivative two dependent matrix
// instructions and one multiply-add) up to about 1.5 waves per SIMD, then by
// issue: FP64 matrix and vector instructions share the pipe here.  Measured
// (H = 2000): 160 ns per step of one wave, 105 ns per wave-step with the SIMDs
// full, against 500 ns and 800 ns for 16 scenarios of the one-lane kernel this
// replaces.  Two waves per SIMD are asked for so that matrix results land in
// ordinary vector registers (with the whole register file one more move per
// result from the accumulation registers made a step 10 % longer).
template <int RNG, int INJ, int RECORD, int CHANCE>
__global__ void __launch_bounds__(256, 2) k_rollout_lq4_mx(const RollArgs<1, double> a,
                                                           const MxCoef mc) {
  if (gen_rows<1>(a)) return;
  DevSearch* S = a.srch;
  const int c = blockIdx.y;
  if (S->done || c >= S->n_cand) return;  // uniform over the workgroup
  const int early = a.early && !S->full[c];
  if (refused_by_steady_state(early, S, c)) return;
  __shared__ unsigned long long sh[16];
  const int lane = threadIdx.x & 63, q = lane >> 4;
  const int wave0 = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6) * 16;  // its scenarios
  const int k = wave0 + (lane & 15);
  // A wave that starts after its candidate died has nothing to decide, and a dead
  // candidate's margin keys are not read.  With every candidate refused at once (a
  // state outside Y) a round is its waves' start-up and what they write to shared
  // words, and there are four times as many waves as with one lane per scenario:
  // N = 16384, 13 candidates, 1.09 -> 0.22 ms per update (one lane: 0.32).
  const bool over = early && __builtin_amdgcn_readfirstlane(is_dead(&S->dead[c]));
  const bool live = !over && k < a.N;
  const uint32_t t = a.st->t;
  double best = INFINITY;
  int jb = 0, ns = 0;
  bool counted = false;        // CHANCE: this scenario's violation is counted in nviol
  if (!over && wave0 < a.N) {  // uniform over the wave
    struct Stop {
      DevSearch* S;
      int c, early, s;
      double band;
      bool live, lead;
      int seen;
      bool& counted;
      __device__ __forceinline__ void begin() {
        seen = early ? __hip_atomic_load(&S->dead[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                     : 0;
      }
      __device__ __forceinline__ bool end(double bm) {
        if (!early) return false;
        if constexpr (CHANCE) {
          const bool viol = (mx_scenarios(bm < -band) >> s) & 1u;
          if (viol && !counted) {
            counted = true;
            if (lead && live && atomicAdd(&S->nviol[c], 1) >= S->q) raise_dead(&S->dead[c]);
          }
          if (__builtin_amdgcn_ballot_w64(!viol) == 0) return true;  // every scenario violated
        } else {
          const bool viol = bm < -band;
          if (__builtin_amdgcn_ballot_w64(viol) != 0) {
            if (viol) raise_dead(&S->dead[c]);
            return true;
          }
        }
        // one load per wave address: every lane read the same flag
        return __builtin_amdgcn_readfirstlane(seen) != 0;
      }
    } stop{S, c, early, lane & 15, a.band, live, q == 0, 0, counted};
    MxLane<RNG, INJ> M;
    M.init(mc, S->v[c], a.h, a.hh, a.h6);
    double x = a.st->x[q], bm;
    const int kk = live ? k : a.N - 1;  // lanes past N repeat the last scenario
    ns = mx_rollout<RNG, INJ, RECORD>(M, a, t, kk, x, bm, jb, stop);
    best = mx_min(bm);
    if (RECORD) {  // the first step at which any row attains the minimum
      jb = bm == best ? jb : 0x7fffffff;
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const int j2 = __shfl_xor(jb, o);
        jb = j2 < jb ? j2 : jb;
      }
    }
    const bool bad = (mx_scenarios(!(x - x == 0.0)) >> (lane & 15)) & 1u;
    if (bad || best != best) best = -INFINITY;
  }
  const bool lead = q == 0 && live;
  if (lead) {
    if (RECORD) {
      a.per_m[(size_t)c * a.N + k] = (float)best;
      a.per_j[(size_t)c * a.N + k] = jb;
    }
    if (CHANCE) a.per_key[(size_t)c * a.N + k] = ord64(best);
    if (best < -a.band) {
      if (!CHANCE || (!counted && atomicAdd(&S->nviol[c], 1) >= S->q)) raise_dead(&S->dead[c]);
    }
  }
  const unsigned long long kall = block_min_u64(lead ? ord64(best) : ~0ull, sh);
  int wsum = lead ? ns : 0;
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) wsum += __shfl_xor(wsum, off);
  const unsigned long long steps = block_sum_waves((unsigned long long)wsum, sh);
  if (threadIdx.x == 0) {
    if (steps) atomicAdd(&S->lane_steps, steps);
    const bool fell = !CHANCE && early && kall != ~0ull && unord64(kall) < -a.band;
    if (kall != ~0ull && !fell) atomicMin(&S->key_all[c], kall);
  }
}

hipError_t launch_rollout_lq4_mx(const Problem& pr, double band, int early_exit, int record,
                                 const LaunchCfg& cfg, const DevBuffers& b, hipStream_t st,
                                 int gen_rows, float* gen_w, float* gen_th) {
  const int gx = div_up((size_t)pr.s.N * 4, (size_t)cfg.block);
  const dim3 grid(gx, cfg.cmax_round + gen_rows);
  const MxCoef mc = make_mx_coef(pr);
  auto a = make_args<1, double>(pr, band, early_exit, record, b);
  if (gen_rows > 0) {
    a.gen_row0 = cfg.cmax_round;
    a.gen_ofs = kSpecMax + 1;
    a.gen_w = gen_w;
    a.gen_th = gen_th;
  }
  return by_bit(pr.s.rng_mode, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    return by_bit(pr.s.inject, [&](auto ic) {
      constexpr int I = decltype(ic)::value;
      return by_bit(record, [&](auto dc) {
        constexpr int D = decltype(dc)::value;
        if (cfg.chance)
          hipLaunchKernelGGL((k_rollout_lq4_mx<R, I, D, 1>), grid, dim3(cfg.block), 0, st, a, mc);
        else
          hipLaunchKernelGGL((k_rollout_lq4_mx<R, I, D, 0>), grid, dim3(cfg.block), 0, st, a, mc);
        return hipGetLastError();
      });
    });
  });
}

}  // namespace rg
