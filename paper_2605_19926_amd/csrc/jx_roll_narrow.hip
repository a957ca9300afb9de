// jx_roll_narrow.hip -- fused rollout kernels built for few registers (gfx950):
// several waves per env, and 4 one-wave envs per SIMD.  Compiled without machine
// LICM (see build.py): hoisted, the constants of the double-precision sincos
// alone hold 30 lane registers across the step loop, and a wave less fits on
// each SIMD.
#include "jx_roll.h"

namespace jx {

namespace {

// Fused rollout with several waves per env (WPE 2 or 4, a workgroup each): one
// wave steps and casts step t (two waves do, half of the columns each, where four
// share an env whose rows have more than 64 columns) while the others write step
// t - 1's frame.  The records alternate between two LDS buffers, one workgroup
// barrier per step.  Workgroups take envs by a static stride over the work order.
// 64 steps of 512 envs (25-side, 64 x 64): 219 us with one wave per env, 161 with
// two and 169 with four (every wave stepping and casting for itself: 222, 223).
// THIRDS (WPE 2): the caster writes a third of a frame and the writer the rest.  A wave
// has no more than 63 stores under way, so where a frame is large and the chip has an
// env per CU or less, one writer falls behind the caster.  us for 8 steps of 64 envs
// without and with it: 128 x 128 float32 NCHW 116, 92, bfloat16 89, 73, 84 x 84 float32
// 79, 55, bfloat16 52, 47; 1000 envs of 100 x 100 float32 187, 267.
template <int MAXN, bool ASC, int FMT, int WPE, bool THIRDS>
__global__ __launch_bounds__(64 * WPE) void k_roll_split(DevState S, RollIo r) {
  __shared__ __align__(16) uint8_t smap[WPE / 2][map_slice(MAXN)];
  __shared__ __align__(16) uint32_t scol[2][2 * kMaxW];
  __shared__ uint32_t sclr[kColorWords];
  __shared__ uint32_t scvt[FMT % 3 ? 256 : 1];
  stage_tables<FMT>(sclr, scvt);
  const int part = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
  const DevIo io = roll_step_io(r);
  const int n = S.n;
  for (int item = (int)blockIdx.x; item < n; item += (int)gridDim.x) {
    int env, W, H;
    int64_t obs_off;
    {
      const DevState& Q = kernarg_state();
      env = __builtin_amdgcn_readfirstlane(Q.order[item]);
      const DevCfg& cf = Q.uniform ? Q.ucfg : Q.cfgs[Q.cfg_idx[env]];
      W = (int)uniform_u((uint32_t)cf.obs_w);
      H = (int)uniform_u((uint32_t)cf.obs_h);
      obs_off = obs_off_of(Q, env);
    }
    // two of four waves cast rows of more than 64 columns, unless float frames of many
    // envs wait for their writers (1000, 1500 envs for 8 steps with two and with one
    // casting: 100 x 100 float32 NCHW 240 and 229, 366 and 346 us, 84 x 84 NHWC 161 and
    // 156, 250 and 237; 600 of 84 x 84 bfloat16 41 and 45, 1500 of bytes 51 and 60)
    const int casters = WPE == 4 && W > 64 && (FMT % 3 == 0 || n <= 768) ? 2 : 1;
    uint8_t* at = r.obs + obs_off;
    if (part < casters) {
      uint8_t* lmap = smap[WPE == 4 ? part : 0] + guard_bytes(MAXN);
      Carried<MAXN> c;
      c.open(kernarg_state(), env, lane, lmap);
      const bool store = lane == 0 && part == 0;
      for (int t = 0; t < r.T; ++t) {
        if ((t & 127) == 0) c.load_actions(n, r, t, lane);
        int ln = lane;
        asm volatile("" : "+v"(ln));
        EnvOut o;
        produce_env<MAXN, false, ASC>(c.in, io, c.action(t & 127), ln, lmap, sclr, scol[t & 1], o, part, casters);
        c.take(n, r, o, t, store);
        __syncthreads();
        if (THIRDS) {
          fill_frame<FMT, false>(scol[t & 1], scvt, at, W, H, ln, r.store_mode, 2, 3, n);
          at += r.obs_stride;
        }
      }
      __syncthreads();  // the writers' last frame
      if (store) c.close(kernarg_state());
    } else {
      for (int t = 0; t < r.T; ++t) {
        __syncthreads();  // step t's records are in buffer t & 1
        int ln = lane;
        asm volatile("" : "+v"(ln));
        if (THIRDS) {
          for (int k = 0; k < 2; ++k)
            fill_frame<FMT, false>(scol[t & 1], scvt, at, W, H, ln, r.store_mode, k, 3, n);
        } else {
          fill_frame<FMT, false>(scol[t & 1], scvt, at, W, H, ln, r.store_mode, part - casters, WPE - casters, n);
        }
        at += r.obs_stride;
      }
      __syncthreads();
    }
  }
}

template <int MAXN, bool ASC, int FMT>
struct SplitL {
  static int run(const DevState& s, const RollIo& r, int groups, int wpe, bool thirds, hipStream_t st) {
    if constexpr (FMT % 3 != 0) {
      if (thirds) {
        hipLaunchKernelGGL((k_roll_split<MAXN, ASC, FMT, 2, true>), dim3(groups), dim3(128), 0, st, s, r);
        return (int)hipGetLastError();
      }
    }
    if (wpe == 2) hipLaunchKernelGGL((k_roll_split<MAXN, ASC, FMT, 2, false>), dim3(groups), dim3(128), 0, st, s, r);
    else hipLaunchKernelGGL((k_roll_split<MAXN, ASC, FMT, 4, false>), dim3(groups), dim3(256), 0, st, s, r);
    return (int)hipGetLastError();
  }
};

}  // namespace

int launch_roll_split(const DevState& s, int max_side, const RollIo& r, int groups, int wpe, int64_t frames_bytes, int n_cu,
                      hipStream_t st) {
  // (bytes have no frames that large, but for the largest, where it gives nothing)
  const bool thirds = wpe == 2 && s.obs_fmt % 3 != 0 && s.n <= n_cu && frames_bytes > (int64_t)s.n * (40 << 10);
  return by_shape<SplitL>(s, max_side, r, groups, wpe, thirds, st);
}

int launch_roll_dense(const DevState& s, int max_side, const RollIo& r, int wpb, int groups, hipStream_t st) {
  if (max_side <= 16) return launch_roll_n<16, false, 0, 4>(s, r, wpb, groups, 0, st);
  if (max_side <= 32) return launch_roll_n<32, false, 0, 4>(s, r, wpb, groups, 0, st);
  return launch_roll_n<64, false, 0, 4>(s, r, wpb, groups, 0, st);
}

}  // namespace jx
