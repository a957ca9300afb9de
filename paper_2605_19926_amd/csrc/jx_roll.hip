// jx_roll.hip -- fused rollout kernels of one wave per env for gfx950 (CDNA4) and
// the choice among all fused kernels.
#include "jx_roll.h"

namespace jx {

namespace {

// Persistent fused rollout: a grid sized to the chip's resident waves drains
// the work order (costliest first) one env per claim, each env carried
// through all T steps as in k_roll.  An env of a 128 x 128 frame costs 16
// times one of 32 x 32, so with uneven shapes dynamic claims keep every wave
// busy until the queue is empty (longest-first list scheduling) where a
// static stride leaves workgroups waiting on their slowest wave.  The queues
// and counter sets are those of k_persist (one claim per env: chunk 1).
template <int MAXN, int WPB, bool ASC>
__global__ __launch_bounds__(64 * WPB) void k_proll(DevState S, RollIo r, uint32_t seq) {
  __shared__ __align__(16) uint8_t smap[WPB][map_slice(MAXN)];
  __shared__ __align__(16) uint32_t scol[WPB][2 * kMaxW];
  __shared__ uint32_t sclr[kColorWords];
  stage_colors(sclr);
  const int w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  const QueueView v = queue_view<WPB>(S.queues, seq, S.n, w, lane, 1);
  queue_drain(v, lane, [&](int pos) {
    const int env = __builtin_amdgcn_readfirstlane(kernarg_state().order[pos]);
    roll_env<MAXN, ASC, 0>(S.n, env, lane, smap[w] + guard_bytes(MAXN), sclr, nullptr, scol[w], r);
  });
}

template <int MAXN, bool ASC, int FMT>
int launch_proll_n(const DevState& s, const RollIo& r, int wpb, int groups, uint32_t seq, hipStream_t st) {
  switch (wpb) {
    case 1: hipLaunchKernelGGL((k_proll<MAXN, 1, ASC>), dim3(groups), dim3(64), 0, st, s, r, seq); break;
    case 2: hipLaunchKernelGGL((k_proll<MAXN, 2, ASC>), dim3(groups), dim3(128), 0, st, s, r, seq); break;
    case 4: hipLaunchKernelGGL((k_proll<MAXN, 4, ASC>), dim3(groups), dim3(256), 0, st, s, r, seq); break;
    case 8: hipLaunchKernelGGL((k_proll<MAXN, 8, ASC>), dim3(groups), dim3(512), 0, st, s, r, seq); break;
    default: return -1;
  }
  return (int)hipGetLastError();
}

template <int MAXN, bool ASC, int FMT>
struct RollL {
  static int run(const DevState& s, const RollIo& r, int wpb, int groups, int lds, hipStream_t st) {
    return launch_roll_n<MAXN, ASC, FMT, 1>(s, r, wpb, groups, lds, st);
  }
};

template <int MAXN, bool ASC, int FMT>
struct PRollL {
  static int run(const DevState& s, const RollIo& r, int wpb, int groups, uint32_t seq, hipStream_t st) {
    return launch_proll_n<MAXN, ASC, FMT>(s, r, wpb, groups, seq, st);
  }
};

}  // namespace

int launch_rollout_fused(const DevState& s, const uint8_t* act, uint8_t* obs, int64_t obs_stride,
                         float* rew, uint8_t* dn, uint8_t* prev, int T, const LaunchCfg& lc, int max_side,
                         int n_cu, int64_t frames_bytes, uint32_t seq, void* stream) {
  if (s.n <= 0 || T <= 0) return 0;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const RollIo r{act, obs, obs_stride, rew, dn, prev, T, lc.store_mode};
  if (lc.form == 1 && s.obs_fmt == 0) {
    // persistent: the chip's share of resident workgroups, never more than needed
    const int wpb = lc.waves_per_group;
    int groups = n_cu * lc.groups_per_cu;
    const int need = (s.n + wpb - 1) / wpb;
    if (groups > need) groups = need;
    if (groups < 1) groups = 1;
    return by_shape_f<PRollL, 0>(s, max_side, r, wpb, groups, seq, st);
  }
  const int wpe = fused_waves_per_env(lc, s.n, n_cu);
  const int wpb = wpe > 1 ? wpe : s.obs_fmt != 0 ? kFmtWaves : lc.waves_per_group;
  // wpe waves per env while they fit on the chip, else a stride.
  int groups = (int)(((int64_t)s.n * wpe + wpb - 1) / wpb);
  const int per_cu = 16 / wpb;
  bool dense = false;
  if (wpe == 1 && s.obs_fmt == 0 && !s.any_ascii) {
    // Byte frames of generated mazes.  Frames below 8 KB wait for the casting:
    // where more than 3 waves per SIMD have work they run the kernel built for 4
    // (8192 envs of 32 x 32: 349 us for 32 steps without, 263 with it; 48 x 48:
    // 419 and 405).  Larger frames wait for the memory, which 2 waves per SIMD
    // fill, and more write less evenly (4096 envs of 64 x 64: 326 and 329 us, of
    // 84 x 84: 574 and 591).
    // (The other kernel lets in 12 waves per CU, or one 8-wave workgroup.)
    dense = frames_bytes < (int64_t)s.n * 8192 && s.n > (wpb == 8 ? 8 : 12) * n_cu;
  }
  int lds = 0;
  if (wpe == 1 && wpb == 4 && !s.any_ascii && max_side <= 32 && s.obs_fmt <= 3 && s.n > 12 * n_cu &&
      frames_bytes >= (int64_t)s.n * 8192) {
    // Groups of 4 waves whose registers (bytes, NHWC, sides to 32) let 12 waves onto
    // a CU, and frames that wait for the memory: 8 waves per CU write more evenly
    // than 12 and a rest.  LDS that nobody reads keeps the third group out (its own
    // is at most 10.4 KB of the 64 KB a group may ask for), so that a CU still takes
    // the next group when one ends.  us for 24 steps with 12 and 8 waves: 4096 envs of
    // 64 x 64 bytes 261 and 247, NCHW 271 and 254, bfloat16 475 and 467; 8192 of 84 x 84
    // bytes 892 and 846, NCHW 927 and 878, bfloat16 1720 and 1645.  Up to 12 per CU
    // all run at once (3072 of 64 x 64 bytes: 188 and 201).  Bytes in NHWC keep 12
    // where 8 fill their last round no better (5000 of 64 x 64: 305 and 314).
    const int64_t r8 = (s.n + 8 * n_cu - 1) / (8 * n_cu) * 8, r12 = (s.n + 12 * n_cu - 1) / (12 * n_cu) * 12;
    if (s.obs_fmt != 0 || r8 < r12) lds = 49 * 1024;
  }
  const int most = n_cu * (per_cu > 0 ? per_cu : 1);
  if (groups > most) groups = most;
  if (wpe > 1) return launch_roll_split(s, max_side, r, groups, wpe, frames_bytes, n_cu, st);
  if (dense) return launch_roll_dense(s, max_side, r, wpb, groups, st);
  return by_shape<RollL>(s, max_side, r, wpb, groups, lds, st);
}

}  // namespace jx
