// Rollouts of the 9-state plant by groups of 9 lanes (rg_fc9_lanes.hpp): FP64
// handles, and FP32 rounds with few scenario-candidate pairs.
#include <hip/hip_runtime.h>

#include "rg_fc9_lanes.hpp"

namespace rg {

// A candidate whose margin at the state itself is below -band is refused without
// simulating it: the outputs there depend on no draw, so every scenario violates.
// (What a round then costs is its waves' start-up, and there are nine times as
// many as with one lane per scenario.)
template <class T>
__device__ __forceinline__ bool refused_by_state(const RollArgs<2, T>& a, DevSearch* S, int c,
                                                 int bx) {
  const double* x = a.st->x;
  T y[3];
  y[0] = t_quot(a.pc.c_q0 * (T)x[6], t_fma(a.pc.d1, (T)x[8], a.pc.d0));
  y[1] = (T)x[0];
  y[2] = (T)x[6];
  if (!(margin_rows<3>(a.F, a.g, y) < -a.band)) return false;
  if (bx == 0 && threadIdx.x == 0) raise_dead(&S->dead[c]);
  return true;
}

// blockIdx.y = candidate, seven scenarios per wave.  The per-scenario
// bookkeeping is that of the one-lane kernel, made by the group's first lane;
// the margins equal that kernel's bit for bit.  CKPT = 1: the checkpoint
// candidate's groups store the adjoint's checkpoints.  CHANCE = 1: the
// chance-constrained verdict (groups stop on their own, every margin key kept).
// Body of one workgroup: candidate row c, scenario tile bx.
template <class T, int RNG, int INJ, int CKPT, int CHANCE>
__device__ __forceinline__ void fc9_lanes_block(const RollArgs<2, T>& a, int c, int bx) {
  __shared__ unsigned long long sh[16];
  __shared__ __align__(16) T xch[4 * kWaveSlots<T>];
  DevSearch* S = a.srch;
  if (S->done || c >= S->n_cand) return;  // uniform over the workgroup
  const bool ck = CKPT == 1 && c == (a.ckpt_cand >= 0 ? a.ckpt_cand : S->nk_idx);
  const int early = a.early && !S->full[c];
  if (refused_by_steady_state(early, S, c, bx)) return;
  if (!CHANCE && early && refused_by_state<T>(a, S, c, bx)) return;
  const GroupLane gl;
  const int wave = threadIdx.x >> 6;
  const int k = (int)(bx * (blockDim.x >> 6) + wave) * kWaveGroups + gl.grp;
  const uint32_t t = a.st->t;
  const int q = CHANCE ? S->q : 0;
  // A wave that starts after its candidate died has nothing to decide, and a dead
  // candidate's margin keys are not read.
  const bool over = early && __builtin_amdgcn_readfirstlane(is_dead(&S->dead[c]));
  const bool live = !over && gl.grp < kWaveGroups && k < a.N;
  T m = t_inf<T>();
  int jb = 0, ns = 0;
  if (live) {  // whole groups are active or inactive together
    T* slot = xch + wave * kWaveSlots<T> + gl.grp * kGroupStride<T>;
    bool stopped = false;  // the candidate died while this wave ran (no recheck needed)
    if constexpr (CHANCE)
      m = rollout_fc9_lanes<T, RNG, INJ, false, 0>(a, early, (T)S->v[c], k, t,
                                                   early ? &S->dead[c] : nullptr, slot, gl, jb, ns);
    else
      m = rollout_fc9_lanes<T, RNG, INJ, true, CKPT>(a, early, (T)S->v[c], k, t, &S->dead[c], slot,
                                                     gl, jb, ns, ck, &stopped);
    if (gl.li == 0) {
      if (CHANCE) a.per_key[(size_t)c * a.N + k] = ord64((double)m);
      if (a.record) {
        a.per_m[(size_t)c * a.N + k] = (float)m;
        a.per_j[(size_t)c * a.N + k] = jb;
      }
      if (m < -a.band) {
        if (q == 0 || atomicAdd(&S->nviol[c], 1) >= q) raise_dead(&S->dead[c]);
      } else if (m < a.band && !stopped) {
        const int idx = atomicAdd(&S->n_recheck, 1);
        a.rlist[idx] = make_int2(c, k);
      }
    }
  }
  const bool own = live && gl.li == 0;
  const unsigned long long key = own ? lane_key(m, k) : ~0ull;
  const unsigned long long kall = block_min_u64(key, sh);
  const unsigned long long kfar = block_min_u64((own && m >= a.band) ? key : ~0ull, sh);
  int wsum = own ? ns : 0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) wsum += __shfl_xor(wsum, off);
  const unsigned long long steps = block_sum_waves((unsigned long long)wsum, sh);
  if (threadIdx.x == 0) {
    if (steps) atomicAdd(&S->lane_steps, steps);
    const bool fell = !CHANCE && early && kall != ~0ull &&
                      key_margin(kall, sizeof(T) == 8) < -(double)a.band;
    if (kall != ~0ull && !fell) atomicMin(&S->key_all[c], kall);
    if (kfar != ~0ull && !fell) atomicMin(&S->key_far[c], kfar);
  }
}

template <class T, int RNG, int INJ, int CKPT, int CHANCE>
__global__ void __launch_bounds__(256) k_rollout_fc9_lanes(const RollArgs<2, T> a) {
  if (gen_rows<2>(a)) return;
  fc9_lanes_block<T, RNG, INJ, CKPT, CHANCE>(a, blockIdx.y, blockIdx.x);
}

// Batched serving: the FP32 form over every instance of a group (tables as
// k_flat_rollout's).
template <int RNG, int INJ>
__global__ void __launch_bounds__(256)
    k_flat_rollout_fc9_lanes(const RollArgs<2, float>* __restrict__ args,
                             const int* __restrict__ tile_inst,
                             const int* __restrict__ tile_first) {
  const int i = tile_inst[blockIdx.x];
  fc9_lanes_block<float, RNG, INJ, 0, 0>(args[i], blockIdx.y, (int)blockIdx.x - tile_first[i]);
}

hipError_t launch_flat_rollout_fc9_lanes(int inject, int rng, const void* args_dev,
                                         const int* tile_inst, const int* tile_first, int tiles,
                                         int cmax, int block, hipStream_t st) {
  return by_bit(rng, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    return by_bit(inject, [&](auto ic) {
      constexpr int I = decltype(ic)::value;
      hipLaunchKernelGGL((k_flat_rollout_fc9_lanes<R, I>), dim3(tiles, cmax), dim3(block), 0, st,
                         (const RollArgs<2, float>*)args_dev, tile_inst, tile_first);
      return hipGetLastError();
    });
  });
}

hipError_t launch_rollout_fc9_lanes(const Problem& pr, double band, int precision, int early_exit,
                                    int record, const LaunchCfg& cfg, const DevBuffers& b,
                                    hipStream_t st, int ckpt_cand, int Kc, int gen_rows,
                                    float* gen_w, float* gen_th) {
  const int gx = div_up((size_t)pr.s.N, (size_t)fc9_lanes_per_block(cfg.block));
  const dim3 grid(gx, cfg.cmax_round + gen_rows);
  auto fill = [&](auto& a) {
    a.ckpt = b.adj_ckpt;
    a.Kc = Kc;
    a.ckpt_cand = ckpt_cand;
    if (gen_rows > 0) {
      a.gen_row0 = cfg.cmax_round;
      a.gen_ofs = kSpecMax + 1;
      a.gen_w = gen_w;
      a.gen_th = gen_th;
    }
  };
  return by_bit(pr.s.rng_mode, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    return by_bit(pr.s.inject, [&](auto ic) {
      constexpr int I = decltype(ic)::value;
      if (precision == 0) {
        auto a = make_args<2, float>(pr, band, early_exit, record, b);
        fill(a);
        if (ckpt_cand >= -1)
          hipLaunchKernelGGL((k_rollout_fc9_lanes<float, R, I, 1, 0>), grid, dim3(cfg.block), 0, st,
                             a);
        else
          hipLaunchKernelGGL((k_rollout_fc9_lanes<float, R, I, 0, 0>), grid, dim3(cfg.block), 0, st,
                             a);
      } else {
        auto a = make_args<2, double>(pr, 0.0, early_exit, record, b);
        fill(a);
        if (cfg.chance)
          hipLaunchKernelGGL((k_rollout_fc9_lanes<double, R, I, 0, 1>), grid, dim3(cfg.block), 0,
                             st, a);
        else
          hipLaunchKernelGGL((k_rollout_fc9_lanes<double, R, I, 0, 0>), grid, dim3(cfg.block), 0,
                             st, a);
      }
      return hipGetLastError();
    });
  });
}

}  // namespace rg
