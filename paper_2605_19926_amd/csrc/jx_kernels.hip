// jx_kernels.hip -- per-step and serving kernels of the fused step + raycast
// render for gfx950 (CDNA4); the device code they run is in jx_device.h.
#include <mutex>

#include "jx_device.h"

namespace jx {

namespace {

// wpe waves per env (1, 2 or 4): consecutive waves of a workgroup share an env.
template <int MAXN, int WPB, bool ASC, int FMT>
__global__ __launch_bounds__(64 * WPB) void k_plain(DevState S, DevIo io, int wpe) {
  __shared__ __align__(16) uint8_t smap[WPB][map_slice(MAXN)];
  __shared__ __align__(16) uint32_t scol[WPB][2 * kMaxW];
  __shared__ uint32_t sclr[kColorWords];
  __shared__ uint32_t scvt[FMT % 3 ? 256 : 1];
  stage_tables<FMT>(sclr, scvt);
  const int w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  const int gw = __builtin_amdgcn_readfirstlane((int)blockIdx.x * WPB + w);
  const int env = gw / wpe, part = gw - env * wpe;
  if (wpe == 1 && env >= S.n) return;
  process_env<MAXN, ASC, FMT>(S, io, env, lane, smap[w] + guard_bytes(MAXN), sclr, scvt, scol[w - part], part, wpe,
                              env < S.n);
}

template <int WPB, bool ASC>
__global__ __launch_bounds__(64 * WPB) void k_persist(DevState S, DevIo io, uint32_t seq) {
  __shared__ __align__(16) uint8_t smap[WPB][map_slice(kMaxSide)];
  __shared__ __align__(16) uint32_t scol[WPB][2 * kMaxW];
  __shared__ uint32_t sclr[kColorWords];
  stage_colors(sclr);
  const int w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  const QueueView v = queue_view<WPB>(S.queues, seq, S.n, w, lane);
  queue_drain(v, lane, [&](int pos) {
    const int env = __builtin_amdgcn_readfirstlane(S.order[pos]);
    process_env<kMaxSide, ASC, 0>(S, io, env, lane, smap[w] + guard_bytes(kMaxSide), sclr, nullptr, scol[w]);
  });
}

// Serving form: work items span several clients' batches.
template <int WPB>
__global__ __launch_bounds__(64 * WPB) void k_serve(const DevState* states, const DevIo* ios,
                                                    const ServeItem* items, int n_items,
                                                    uint32_t* queues, uint32_t seq) {
  __shared__ __align__(16) uint8_t smap[WPB][map_slice(kMaxSide)];
  __shared__ __align__(16) uint32_t scol[WPB][2 * kMaxW];
  __shared__ uint32_t sclr[kColorWords];
  stage_colors(sclr);
  const int w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  const QueueView v = queue_view<WPB>(queues, seq, n_items, w, lane);
  queue_drain(v, lane, [&](int pos) {
    const int d = __builtin_amdgcn_readfirstlane(items[pos].desc);
    const int env = __builtin_amdgcn_readfirstlane(items[pos].env);
    // fields are read from the descriptors where they are used (scalar loads)
    const DevState& S = states[d];
    const DevIo& io = ios[d];
    process_env<kMaxSide, true, 0>(S, io, env, lane, smap[w] + guard_bytes(kMaxSide), sclr, nullptr, scol[w]);
  });
}

// Pipelined form: a workgroup holds P wave pairs.  In each pair a producer
// wave loads, steps and casts envs (prefetching the next env's inputs while it
// computes the current one) and never stores to global memory; a writer wave
// expands the previous env's span records into its frame and stores frame and
// state.  The two alternate LDS buffers, one workgroup barrier per round, so
// producing env k+1 overlaps writing env k, and the writer's outstanding stores
// never stall a load.  Pairs walk the work order (costliest first) with a
// static stride of all pairs in the grid.
template <int MAXN, int P, bool ASC>
__global__ __launch_bounds__(128 * P) void k_pipe(DevState S, DevIo io) {
  __shared__ __align__(16) uint8_t smap[P][map_slice(MAXN)];
  __shared__ __align__(16) uint32_t scol[P][2][2 * kMaxW];
  __shared__ EnvOut sout[P][2];
  __shared__ uint32_t sclr[kColorWords];
  stage_colors(sclr);
  const int w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  const int pair = w >> 1;
  const bool writer = (w & 1) != 0;
  const int pairs = (int)gridDim.x * P;
  const int gp = (int)blockIdx.x * P + pair;
  const int lead = (int)blockIdx.x * P;  // the workgroup's pair with the most items
  const int rounds = S.n > lead ? (S.n - lead + pairs - 1) / pairs : 0;
  EnvIn<MAXN> cur, nxt;
  if (!writer && gp < S.n) load_env<MAXN>(S, io.act, __builtin_amdgcn_readfirstlane(S.order[gp]), lane, cur);
  for (int k = 0; k <= rounds; ++k) {
    const int b = k & 1;
    if (!writer) {
      const int item = gp + k * pairs;
      if (k < rounds && item < S.n) {
        const int nitem = item + pairs;
        if (nitem < S.n) load_env<MAXN>(S, io.act, __builtin_amdgcn_readfirstlane(S.order[nitem]), lane, nxt);
        EnvOut o;
        produce_env<MAXN, true, ASC>(cur, io, (int)cur.act, lane, smap[pair] + guard_bytes(MAXN), sclr, scol[pair][b], o);
        o.obs_off = obs_off_of(S, o.env);
        if (lane == 0) sout[pair][b] = o;
        cur = nxt;
      } else if (lane == 0) {
        sout[pair][b].env = -1;
      }
    } else if (k > 0) {
      const EnvOut o = sout[pair][b ^ 1];
      if (o.env >= 0) {
        fill_frame<0, true>(scol[pair][b ^ 1], nullptr, io.obs + o.obs_off, o.W, o.H, lane, io.store_mode);
        write_back(S, io, o, lane);
      }
    }
    __syncthreads();
  }
}

__global__ void k_clear_queues(uint32_t* q) {
  for (int i = (int)threadIdx.x; i < kQueueWords; i += (int)blockDim.x) q[i] = 0u;
}

template <int MAXN, bool ASC, int FMT>
int launch_plain_n(const DevState& s, const DevIo& io, int wpb, int wpe,
                   hipStream_t st) {
  if constexpr (FMT != 0) {
    const int grid = (int)(((int64_t)s.n * wpe + kFmtWaves - 1) / kFmtWaves);
    hipLaunchKernelGGL((k_plain<MAXN, kFmtWaves, ASC, FMT>), dim3(grid), dim3(64 * kFmtWaves), 0, st, s, io,
                       wpe);
    return (int)hipGetLastError();
  } else {
    const int grid = (int)(((int64_t)s.n * wpe + wpb - 1) / wpb);
    switch (wpb) {
      case 1: hipLaunchKernelGGL((k_plain<MAXN, 1, ASC, 0>), dim3(grid), dim3(64), 0, st, s, io, wpe); break;
      case 2: hipLaunchKernelGGL((k_plain<MAXN, 2, ASC, 0>), dim3(grid), dim3(128), 0, st, s, io, wpe); break;
      case 4: hipLaunchKernelGGL((k_plain<MAXN, 4, ASC, 0>), dim3(grid), dim3(256), 0, st, s, io, wpe); break;
      case 8: hipLaunchKernelGGL((k_plain<MAXN, 8, ASC, 0>), dim3(grid), dim3(512), 0, st, s, io, wpe); break;
      default: return -1;
    }
    return (int)hipGetLastError();
  }
}

}  // namespace

// Reset, render-only and debug launches always take the plain kernel.
inline bool mode_needs_plain(const DevIo& io) {
  return io.mode != MODE_STEP || io.dbg != nullptr || io.obs == nullptr;
}

template <int MAXN, bool ASC, int FMT>
int launch_pipe_n(const DevState& s, const DevIo& io, int p, int groups,
                  hipStream_t st) {
  switch (p) {
    case 1: hipLaunchKernelGGL((k_pipe<MAXN, 1, ASC>), dim3(groups), dim3(128), 0, st, s, io); break;
    case 2: hipLaunchKernelGGL((k_pipe<MAXN, 2, ASC>), dim3(groups), dim3(256), 0, st, s, io); break;
    case 4: hipLaunchKernelGGL((k_pipe<MAXN, 4, ASC>), dim3(groups), dim3(512), 0, st, s, io); break;
    default: return -1;
  }
  return (int)hipGetLastError();
}

template <bool ASC>
int launch_persist_n(const DevState& s, const DevIo& io, int wpb,
                     int groups, uint32_t seq, hipStream_t st) {
  switch (wpb) {
    case 1: hipLaunchKernelGGL((k_persist<1, ASC>), dim3(groups), dim3(64), 0, st, s, io, seq); break;
    case 2: hipLaunchKernelGGL((k_persist<2, ASC>), dim3(groups), dim3(128), 0, st, s, io, seq); break;
    case 4: hipLaunchKernelGGL((k_persist<4, ASC>), dim3(groups), dim3(256), 0, st, s, io, seq); break;
    case 8: hipLaunchKernelGGL((k_persist<8, ASC>), dim3(groups), dim3(512), 0, st, s, io, seq); break;
    default: return -1;
  }
  return (int)hipGetLastError();
}

template <int MAXN, bool ASC, int FMT>
struct PlainL {
  static int run(const DevState& s, const DevIo& io, int wpb, int wpe,
                 hipStream_t st) {
    return launch_plain_n<MAXN, ASC, FMT>(s, io, wpb, wpe, st);
  }
};
template <int MAXN, bool ASC, int FMT>
struct PipeL {
  static int run(const DevState& s, const DevIo& io, int p, int groups,
                 hipStream_t st) {
    return launch_pipe_n<MAXN, ASC, FMT>(s, io, p, groups, st);
  }
};
int launch_clear_queues(uint32_t* queues, void* stream) {
  hipLaunchKernelGGL(k_clear_queues, dim3(1), dim3(256), 0, reinterpret_cast<hipStream_t>(stream),
                     queues);
  return (int)hipGetLastError();
}

int launch_batch(const DevState& s, const DevIo& io,
                 const LaunchCfg& lc, int max_side, int max_w, int64_t frames_bytes, int n_cu, uint32_t seq,
                 void* stream) {
  if (s.n <= 0) return 0;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int wpb = lc.waves_per_group;
  // training-buffer formats: plain form only.  Several waves per env only for
  // steps and renders that write frames (resets and debug records take one).
  if (lc.form == 0 || s.obs_fmt != 0) {
    const bool frames = io.mode != MODE_RESET && io.obs != nullptr && io.dbg == nullptr;
    const int wpe = step_waves_per_env(lc, io.mode, frames, s.n, frames_bytes, max_w, n_cu);
    const int wpg = wpb < wpe ? wpe : wpb;
    return by_shape<PlainL>(s, max_side, io, wpg, wpe, st);
  }
  if (lc.form == 2) {
    // waves_per_group counts wave pairs (1, 2 or 4) in the pipelined form
    const int p = wpb > 4 ? 4 : wpb;
    int groups = n_cu * lc.groups_per_cu;
    const int need = (s.n + p - 1) / p;
    if (groups > need) groups = need;
    if (groups < 1) groups = 1;
    if (mode_needs_plain(io)) return by_shape<PlainL>(s, 64, io, 1, 1, st);
    return by_shape_f<PipeL, 0>(s, max_side, io, p, groups, st);
  }
  int groups = n_cu * lc.groups_per_cu;
  const int need = (s.n + wpb - 1) / wpb;
  if (groups > need) groups = need;
  if (groups < 1) groups = 1;
  return s.any_ascii ? launch_persist_n<true>(s, io, wpb, groups, seq, st)
                     : launch_persist_n<false>(s, io, wpb, groups, seq, st);
}

int launch_serve(const DevState* states_dev, const DevIo* ios_dev, const ServeItem* items_dev,
                 int n_items, uint32_t* queues_dev, uint32_t seq, int waves_per_group,
                 int n_groups, void* stream) {
  if (n_items <= 0) return 0;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  switch (waves_per_group) {
    case 1: hipLaunchKernelGGL((k_serve<1>), dim3(n_groups), dim3(64), 0, st, states_dev, ios_dev, items_dev, n_items, queues_dev, seq); break;
    case 2: hipLaunchKernelGGL((k_serve<2>), dim3(n_groups), dim3(128), 0, st, states_dev, ios_dev, items_dev, n_items, queues_dev, seq); break;
    case 4: hipLaunchKernelGGL((k_serve<4>), dim3(n_groups), dim3(256), 0, st, states_dev, ios_dev, items_dev, n_items, queues_dev, seq); break;
    default: return -1;
  }
  return (int)hipGetLastError();
}

const char* kernel_error_string(int code) { return hipGetErrorString((hipError_t)code); }

// Work-queue counters of the rollout entry point that allocates nothing: a
// file-scope device array, one copy per device, alive until the process ends.
// In host code `scratch` names a host-side stand-in, not a device address: the
// kernels receive the address looked up below, once per device.
static __device__ __align__(256) uint32_t scratch[kScratchWords];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint32_t* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

int scratch_device_address(int device, uint32_t** out) {
  *out = nullptr;
  if (device < 0 || device >= kMaxDevices) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    g_scratch_ptr[device] = static_cast<uint32_t*>(p);
  }
  *out = g_scratch_ptr[device];
  return 0;
}

}  // namespace jx
