// jx_roll.h -- device code of the fused rollouts: one launch carries every env
// through all steps.
#pragma once
#include "jx_device.h"

namespace jx {

// Buffers of a fused rollout.
struct RollIo {
  const uint8_t* act;
  uint8_t* obs;
  int64_t obs_stride;
  float* rew;
  uint8_t* dn;
  uint8_t* prv;
  int T, store_mode;
};

// Kernels of jx_roll_narrow.hip, by map side and ASCII support: 2 or 4 waves per
// env (wpe), and 4 waves per SIMD of one-wave envs (byte frames of mazes).
int launch_roll_split(const DevState& s, int max_side, const RollIo& r, int groups, int wpe, int64_t frames_bytes, int n_cu,
                      hipStream_t st);
int launch_roll_dense(const DevState& s, int max_side, const RollIo& r, int wpb, int groups, hipStream_t st);

namespace {

// An env carried through a fused rollout: the state in registers (the pose and
// its sine and cosine in lane registers, the rest in scalar ones), the layout in
// the wave's LDS.
template <int MAXN>
struct Carried {
  EnvIn<MAXN> in;
  uint32_t n_invalid = 0, last_ev = 0;
  uint32_t a0 = 0, a1 = 0;  // lane l: the actions of steps t0 + l and t0 + 64 + l of a block of 128

  __device__ __forceinline__ void open(const DevState& S, int env, int lane, uint8_t* lmap) {
    load_env<MAXN>(S, nullptr, env, lane, in);
    sincos((double)in.th, &in.sn, &in.cs);
    stage_map<MAXN>(in, lane, lmap);
  }
  __device__ __forceinline__ void load_actions(int n, const RollIo& r, int t0, int lane) {
    const int s0 = t0 + lane, s1 = t0 + 64 + lane;
    a0 = s0 < r.T ? r.act[(int64_t)s0 * n + in.env] : 0u;
    a1 = s1 < r.T ? r.act[(int64_t)s1 * n + in.env] : 0u;
  }
  __device__ __forceinline__ int action(int k) const { return (int)lane_value(k < 64 ? a0 : a1, k); }
  // Step t's reward, done and previous action, and the state for the next step.
  __device__ __forceinline__ void take(int n, const RollIo& r, const EnvOut& o, int t, bool store) {
    if (store) {
      const int64_t at = (int64_t)t * n + in.env;
      r.rew[at] = o.reward;
      r.dn[at] = (uint8_t)o.done;
      if (r.prv) r.prv[at] = (uint8_t)o.prev;
    }
    n_invalid += (o.ev & EV_INVALID) ? 1u : 0u;
    last_ev = o.ev;
    in.x = o.x;
    in.y = o.y;
    in.th = o.th;
    in.t = o.t;
    in.ep = o.ep;
    in.fl = o.fl;
    in.nd = (int)o.nd;
    in.goal = o.goal;
    in.door = o.door;
    in.key = o.key;
    in.dec0 = o.dec0;
    in.dec1 = o.dec1;
    in.doors = o.doors;
    in.sn = o.sn;
    in.cs = o.cs;
  }
  // Lane 0 of the env's first wave, after the last step.
  __device__ __forceinline__ void close(const DevState& S) const {
    const int env = in.env;
    S.x[env] = in.x;
    S.y[env] = in.y;
    S.th[env] = in.th;
    S.t[env] = in.t;
    S.ep[env] = in.ep;
    S.goal[env] = in.goal;
    S.door[env] = in.door;
    S.key[env] = in.key;
    S.decor[2 * env] = in.dec0;
    S.decor[2 * env + 1] = in.dec1;
    S.flags[env] = (uint8_t)in.fl;
    S.ndecor[env] = (uint8_t)in.nd;
    S.events[env] = (uint8_t)last_ev;
    S.doors[env] = in.doors;
    if (n_invalid) S.invalid[env] += n_invalid;
  }
};

// The kernel's first argument, read anew from the argument segment.  A fused
// rollout needs the state's 25 addresses before and after its step loop only;
// held across the loop they would fill the scalar registers, and the loop would
// spend its time moving spilled ones in and out of lanes.
__device__ __forceinline__ const DevState& kernarg_state() {
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const DevState*)(const __attribute__((address_space(4))) DevState*)p;
}

__device__ __forceinline__ DevIo roll_step_io(const RollIo& r) {
  DevIo io{};
  io.obs = r.obs;
  io.mode = MODE_STEP;
  io.store_mode = r.store_mode;
  return io;
}

// One env's fused rollout: the wave carries the env through all T steps with
// the state in registers and its layout staged once in LDS, loading the env's
// actions 128 steps at a time.  Inside the step loop the wave issues no global
// loads, so its frame stores never stall it, and waves drift out of phase: one
// wave's casting overlaps another's stores.  Per step the results are those of
// a single-step launch; the state is written back once, after the last step.
template <int MAXN, bool ASC, int FMT>
__device__ __forceinline__ void roll_env(int n, int env, int lane, uint8_t* lmap, const uint32_t* lclr,
                                         const uint32_t* lcvt, uint32_t* lcol, const RollIo& r) {
  const DevIo io = roll_step_io(r);
  Carried<MAXN> c;
  int64_t obs_off;
  {
    const DevState& S = kernarg_state();
    c.open(S, env, lane, lmap);
    obs_off = obs_off_of(S, env);
  }
  for (int t0 = 0; t0 < r.T; t0 += 128) {
    c.load_actions(n, r, t0, lane);
    const int tend = r.T - t0 < 128 ? r.T - t0 : 128;
    for (int k = 0; k < tend; ++k) {
      // Wait for this wave's previous frame stores before the next step: a
      // wave then has at most one frame's stores in flight.  Measured on the
      // 4096-env workload this bound keeps the HBM write stream more
      // efficient than letting stores of many steps pile up (and the casting
      // of the other waves still overlaps them).  vmcnt 0, other counters
      // untouched.
      __builtin_amdgcn_s_waitcnt(0x0F70);
      // an opaque copy of the lane id keeps the per-column set-up inside the
      // loop instead of hoisted out of it and held live across all steps
      int ln = lane;
      asm volatile("" : "+v"(ln));
      EnvOut o;
      produce_env<MAXN, false, ASC>(c.in, io, c.action(k), ln, lmap, lclr, lcol, o);
      const int t = t0 + k;
      fill_frame<FMT, true>(lcol, lcvt, r.obs + (int64_t)t * r.obs_stride + obs_off, o.W, o.H, ln, r.store_mode);
      c.take(n, r, o, t, lane == 0);
    }
  }
  if (lane == 0 && r.T > 0) c.close(kernarg_state());
}

// Fused rollout: one launch for T steps of every env.  Waves take envs by a
// static stride over the work order (costliest first).
// OCC: waves per SIMD to build for (1: as many as its registers leave room for).
template <int MAXN, int WPB, bool ASC, int FMT, int OCC>
__global__ __launch_bounds__(64 * WPB, OCC) void k_roll(DevState S, RollIo r) {
  __shared__ __align__(16) uint8_t smap[WPB][map_slice(MAXN)];
  __shared__ __align__(16) uint32_t scol[WPB][2 * kMaxW];
  __shared__ uint32_t sclr[kColorWords];
  __shared__ uint32_t scvt[FMT % 3 ? 256 : 1];
  stage_tables<FMT>(sclr, scvt);
  const int w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  const int first = __builtin_amdgcn_readfirstlane((int)blockIdx.x * WPB + w);
  const int stride = (int)gridDim.x * WPB;
  for (int item = first; item < S.n; item += stride) {
    const int env = __builtin_amdgcn_readfirstlane(kernarg_state().order[item]);
    roll_env<MAXN, ASC, FMT>(S.n, env, lane, smap[w] + guard_bytes(MAXN), sclr, scvt, scol[w], r);
  }
}

// lds: bytes of LDS asked for beside the kernel's own, to bound the groups per CU
template <int MAXN, bool ASC, int FMT, int OCC>
int launch_roll_n(const DevState& s, const RollIo& r, int wpb, int groups, int lds, hipStream_t st) {
  if constexpr (FMT != 0) {
    hipLaunchKernelGGL((k_roll<MAXN, kFmtWaves, ASC, FMT, OCC>), dim3(groups), dim3(64 * kFmtWaves), lds, st, s, r);
  } else {
    switch (wpb) {
      case 1: hipLaunchKernelGGL((k_roll<MAXN, 1, ASC, 0, OCC>), dim3(groups), dim3(64), lds, st, s, r); break;
      case 2: hipLaunchKernelGGL((k_roll<MAXN, 2, ASC, 0, OCC>), dim3(groups), dim3(128), lds, st, s, r); break;
      case 4: hipLaunchKernelGGL((k_roll<MAXN, 4, ASC, 0, OCC>), dim3(groups), dim3(256), lds, st, s, r); break;
      case 8: hipLaunchKernelGGL((k_roll<MAXN, 8, ASC, 0, OCC>), dim3(groups), dim3(512), lds, st, s, r); break;
      default: return -1;
    }
  }
  return (int)hipGetLastError();
}

}  // namespace

}  // namespace jx
