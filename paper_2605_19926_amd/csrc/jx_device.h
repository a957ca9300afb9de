// jx_device.h -- device code shared by the per-step and the fused kernels:
// step, reset, column cast and frame fill of one env, and the work queues.
//
// One 64-lane wave owns one environment for the whole step (where a batch leaves the
// chip idle, 2 or 4 waves share one: one or two of them do 1 to 4, then all write):
//   1. stage the env's N x N tile map from HBM into the wave's LDS slice;
//   2. apply the action (turn / move / strafe, axis-separated collision), then
//      key, goal, reward, truncation (rules of the key-door and navigation tasks,
//      Table 1 and Table 2 of the paper);
//   3. on done, reset the episode in place: spawn, heading, goal by BFS, door on
//      a shortest path, key in the start region, decor.  BFS runs bit-parallel:
//      lane y holds map row y as a bit mask, one frontier expansion per level
//      (shift within the row, DPP move across rows);
//   4. cast one ray per screen column (lane c takes columns c, c+64, ...) with
//      DDA over tile boundaries (Sec. 2.1) through the LDS map, and reduce each
//      column to a span record: wall colour, wall half-height in rows, nearest
//      covering sprite's colour and half-height (billboard sprites, Fig. 1);
//   5. expand the span records straight into row-major uint8 RGB: each lane
//      emits 4 consecutive pixels (12 bytes) per iteration, so a wave writes 768
//      contiguous bytes per store instruction.  The training-buffer formats
//      (NCHW planes, byte / 255 as bfloat16 or float32) expand the same records
//      into converted elements.
// Nothing here is a dense contraction, so there is no MFMA; the bound is the
// HBM write of the frames and the vector ALU of the span expansion.
#pragma once
#include <hip/hip_runtime.h>

#include "jx_internal.h"

namespace jx {

namespace {

constexpr uint32_t rgb(uint32_t r, uint32_t g, uint32_t b) { return r | (g << 8) | (b << 16); }

// Colours of this library (the paper draws flat colours without assets).  The
// table is copied into each workgroup's LDS at kernel start: an indexed lookup
// in LDS costs no global load, and a global load inside a step loop would
// wait for every frame store the wave has in flight.
constexpr int kColorWords = 32;
constexpr int kClrPalette = 0;  // 8 wall colours, indexed by tile id mod K
constexpr int kClrWall9 = 8;    // ASCII maps: walls '1'..'9'
constexpr int kClrDoor = 17;    // ASCII maps: doors by type (8 slots; 5 types)
constexpr uint32_t kColorTable[kColorWords] = {
    rgb(180, 40, 40), rgb(40, 160, 40),  rgb(40, 60, 180),  rgb(190, 170, 40),
    rgb(150, 40, 170), rgb(40, 160, 170), rgb(200, 110, 30), rgb(150, 150, 150),
    rgb(180, 40, 40), rgb(40, 160, 40),  rgb(40, 60, 180),  rgb(190, 170, 40),
    rgb(150, 40, 170), rgb(40, 160, 170), rgb(200, 110, 30), rgb(150, 150, 150),
    rgb(230, 230, 230),
    rgb(120, 0, 0), rgb(0, 30, 130), rgb(140, 120, 0), rgb(70, 110, 230), rgb(230, 200, 60),
    rgb(120, 0, 0), rgb(120, 0, 0), rgb(120, 0, 0)};
// ASCII maps: key billboards by colour (red, blue, yellow)
constexpr uint32_t kAKeyRgb[3] = {rgb(255, 40, 40), rgb(40, 110, 255), rgb(255, 200, 40)};
// Tile bytes (layout sources): low nibble wall class (1 default, 2..10 '1'..'9'),
// bit 7 door (type in bits 4..6, index in 0..3), bits 5/6 spawn/goal candidates
// on floor tiles.
constexpr uint32_t kTileDoor = 0x80u, kTileSpawn = 0x20u, kTileGoal = 0x40u;
constexpr uint32_t kDoorBlueUnlocked = 3u, kDoorYellowUnlocked = 4u;

__device__ __forceinline__ void stage_colors(uint32_t* lclr) {
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < kColorWords; ++i) lclr[i] = kColorTable[i];
  }
  __syncthreads();
}

// Training-buffer formats (fmt = layout * 3 + dtype): the floating types hold
// byte / 255 rounded to nearest-even.  The quotient is an IEEE division in
// float (correctly rounded); bfloat16 rounds that float to nearest-even, which
// equals rounding the exact quotient directly because float carries more than
// twice bfloat16's 8 significant bits plus two.
template <int DT>
__device__ __forceinline__ uint32_t norm_entry(uint32_t b) {
  const uint32_t u = __float_as_uint((float)b / 255.0f);
  if (DT == 2) return u;
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// Colour table and, for the floating formats, the byte -> element table
// (256 words), both into the workgroup's LDS.
template <int FMT>
__device__ __forceinline__ void stage_tables(uint32_t* lclr, uint32_t* lcvt) {
  if (FMT % 3 != 0)
    for (int i = (int)threadIdx.x; i < 256; i += (int)blockDim.x) lcvt[i] = norm_entry<FMT % 3>((uint32_t)i);
  stage_colors(lclr);
}
constexpr uint32_t kCeil = rgb(50, 50, 60);
constexpr uint32_t kFloor = rgb(90, 80, 70);
constexpr uint32_t kDoor = rgb(120, 0, 0);
constexpr uint32_t kKeyRgb = rgb(255, 40, 40);
constexpr uint32_t kGoalRgb = rgb(255, 230, 0);
constexpr uint32_t kDecorRgb = rgb(0, 200, 120);

constexpr float kTwoPiF = 6.28318548202514648f;  // float nearest to 2*pi

// ---- wave primitives ---------------------------------------------------------
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Cross-lane moves by DPP: a lane shuffle through LDS (ds_bpermute) costs an LDS
// round trip, a DPP move one VALU instruction.  Lanes without a source read 0.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, ROWS == 0xF);
}
constexpr int kDppRowShr = 0x110, kDppWaveShl1 = 0x130, kDppWaveShr1 = 0x138, kDppBcast15 = 0x142,
              kDppBcast31 = 0x143;
// lane i takes lane i - 1's (prev) or lane i + 1's (next) value
__device__ __forceinline__ uint32_t lane_prev(uint32_t v) { return dpp<kDppWaveShr1>(v); }
__device__ __forceinline__ uint32_t lane_next(uint32_t v) { return dpp<kDppWaveShl1>(v); }
__device__ __forceinline__ uint64_t lane_prev(uint64_t v) {
  return ((uint64_t)lane_prev((uint32_t)(v >> 32)) << 32) | lane_prev((uint32_t)v);
}
__device__ __forceinline__ uint64_t lane_next(uint64_t v) {
  return ((uint64_t)lane_next((uint32_t)(v >> 32)) << 32) | lane_next((uint32_t)v);
}
// lane src's value (src uniform), in scalar registers
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int src) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, src & 63);
}
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int src) {
  return ((uint64_t)lane_value((uint32_t)(v >> 32), src) << 32) | lane_value((uint32_t)v, src);
}
// Inclusive prefix sum over the wave: within each row of 16 lanes, then row
// totals to the odd rows, then the lower half's total to the upper half.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += dpp<kDppRowShr + 1>(v);
  v += dpp<kDppRowShr + 2>(v);
  v += dpp<kDppRowShr + 4>(v);
  v += dpp<kDppRowShr + 8>(v);
  v += dpp<kDppBcast15, 0xA>(v);
  v += dpp<kDppBcast31, 0xC>(v);
  return v;
}
__device__ __forceinline__ bool wave_any(bool p) { return __ballot(p) != 0ull; }
__device__ __forceinline__ uint32_t uniform_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// ---- SplitMix64 (Steele, Lea & Flood 2014) --------------------------------------
__device__ __forceinline__ uint64_t sm_next(uint64_t& s) {
  s += 0x9E3779B97F4A7C15ull;
  uint64_t z = s;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ uint64_t sm_mix(uint64_t v) { return sm_next(v); }
__device__ __forceinline__ uint32_t sm_draw(uint64_t& s, uint32_t n) {
  return (uint32_t)(((sm_next(s) >> 32) * (uint64_t)n) >> 32);
}

// Row and column of a tile id (below 4096) on an N-wide map (N from 5 to 64) by
// one multiplication: m = floor(2^18 / N) + 1 exceeds 2^18 / N by at most 1, so
// id * m / 2^18 exceeds id / N by at most id / 2^18 < 1 / N (4095 * 64 < 2^18),
// which never reaches the next integer.  The quotient 2^18 / N itself comes from
// the hardware reciprocal: a quarter of its smallest fraction 1 / N is added, which
// is five times the error of the reciprocal (1 ulp) and the product.
struct TileDiv {
  int N;
  uint32_t m;
  __device__ __forceinline__ explicit TileDiv(int n)
      : N(n), m((uint32_t)(262144.25f * __builtin_amdgcn_rcpf((float)n)) + 1u) {}
  __device__ __forceinline__ int row(int id) const { return (int)(((uint32_t)id * m) >> 18); }
  __device__ __forceinline__ int col(int id) const { return id - row(id) * N; }
};

// ---- row-mask set operations (lane y < N holds row y; M has at least N bits) -----
__device__ __forceinline__ uint32_t bits_of(uint32_t m) { return (uint32_t)__popc(m); }
__device__ __forceinline__ uint32_t bits_of(uint64_t m) { return (uint32_t)__popcll(m); }
__device__ __forceinline__ int first_bit(uint32_t m) { return __ffs((int)m) - 1; }
__device__ __forceinline__ int first_bit(uint64_t m) { return __ffsll((unsigned long long)m) - 1; }

// Tile id of the r-th set bit in row-major order of the distributed mask.
template <typename M>
__device__ int mask_select(M m, uint32_t r, int N) {
  const uint32_t c = bits_of(m), incl = wave_incl_scan(c), excl = incl - c;
  const int L = first_bit((uint64_t)__ballot(r >= excl && r < incl));
  M mm = lane_value(m, L);
  const uint32_t k = r - lane_value(excl, L);
  for (uint32_t i = 0; i < k; ++i) mm &= mm - 1;
  return L * N + first_bit(mm);
}
template <typename M>
__device__ __forceinline__ uint32_t mask_count(M m) {
  return lane_value(wave_incl_scan(bits_of(m)), 63);
}
template <typename M>
__device__ __forceinline__ int mask_first(M m, int N) {
  const uint64_t own = __ballot(m != 0);
  if (own == 0ull) return -1;
  const int L = first_bit(own);
  return L * N + first_bit(lane_value(m, L));
}
template <typename M>
__device__ __forceinline__ M bit_of(int id, const TileDiv& td, int lane) {
  return (id >= 0 && lane == td.row(id)) ? ((M)1 << td.col(id)) : (M)0;
}

// One level of a level-synchronous search: the tiles of U (passable, not yet
// reached) beside the frontier F; they leave U.
template <typename M>
__device__ __forceinline__ M bfs_level(M F, M& U) {
  const M nf = ((F << 1) | (F >> 1) | lane_prev(F) | lane_next(F)) & U;
  U &= ~nf;
  return nf;
}

template <typename M>
struct Bfs {
  int level;    // of the farthest tiles
  M frontier;   // the farthest tiles
  M unreached;  // passable tiles the search did not reach
};
// Search over the passable mask until the frontier empties.  A reset's time is
// this serial chain (a loop-free 32-side maze has some 230 levels, a 64-side one
// 800, and a key-door reset searches three times), and one wave's chain
// makes a whole per-step launch end late.  So a level is 7 VALU instructions
// with 32-bit rows and 15 with 64-bit rows, and the wave asks only every fourth
// level whether the search has ended.  Against lane shuffles through LDS on
// 64-bit rows and a test per level, a step of 8192 32-side key-door envs with 8
// resets fell from 122 to 56 us (41 us without any reset), one of 4096 16-side
// mazes from 19.9 to 15.5 us.  Every wave reaches the exit: U shrinks with every
// level that is not empty.
template <typename M>
__device__ Bfs<M> bfs_all(M pass, int src, const TileDiv& td, int lane) {
  M f0, f1, f2, f3, f4 = bit_of<M>(src, td, lane);
  M U = pass & ~f4;
  int level = -4;
  do {
    f0 = f4;
    f1 = bfs_level(f0, U);
    f2 = bfs_level(f1, U);
    f3 = bfs_level(f2, U);
    f4 = bfs_level(f3, U);
    level += 4;
  } while (wave_any(f4 != 0));
  if (wave_any(f3 != 0)) return {level + 3, f3, U};
  if (wave_any(f2 != 0)) return {level + 2, f2, U};
  if (wave_any(f1 != 0)) return {level + 1, f1, U};
  return {level, f0, U};
}

// Tiles at distance h from a and at distance h + odd from b (both searches have
// that many levels); the two chains run side by side.
template <typename M>
__device__ M bfs_meet(M pass, int a, int b, int h, int odd, const TileDiv& td, int lane) {
  M Fa = bit_of<M>(a, td, lane), Fb = bit_of<M>(b, td, lane);
  M Ua = pass & ~Fa, Ub = pass & ~Fb;
  for (int i = 0; i < h; ++i) {
    Fa = bfs_level(Fa, Ua);
    Fb = bfs_level(Fb, Ub);
  }
  if (odd) Fb = bfs_level(Fb, Ub);
  return Fa & Fb;
}

// Row masks of the tiles that `test` marks (bit 7 of each byte of a dword of 4
// tiles): each lane turns 8 tiles into one byte of a row-major bit string in
// LDS, then lane y takes its N bits from it.  `lbits` holds 512 bytes.
template <typename M, typename T>
__device__ __forceinline__ M row_masks(const uint8_t* lmap, uint32_t* lbits, int N, int lane, T&& test) {
  const int NN = N * N;
  const u32x2* l2 = reinterpret_cast<const u32x2*>(lmap);
  auto four = [](uint32_t b7) { return ((b7 >> 7) * 0x01020408u >> 24) & 15u; };  // byte k's bit 7 -> bit k
  for (int k = lane; 8 * k < NN; k += 64) {
    const u32x2 v = l2[k];
    reinterpret_cast<uint8_t*>(lbits)[k] = (uint8_t)(four(test(v.x)) | (four(test(v.y)) << 4));
  }
  wave_sync();
  M m = 0;
  if (lane < N) {
    const uint32_t at = (uint32_t)(lane * N), sh = at & 31u;
    const uint32_t* w = lbits + (at >> 5);
    // (a row that fills its last word takes no bit from the one after it)
    const bool more = sh + (uint32_t)N > (sizeof(M) == 8 ? 64u : 32u);
    uint64_t v = __builtin_amdgcn_alignbit(sizeof(M) == 8 || more ? w[1] : 0u, w[0], sh);
    if (sizeof(M) == 8) v |= (uint64_t)__builtin_amdgcn_alignbit(more ? w[2] : 0u, w[1], sh) << 32;
    m = (M)(v & (~0ull >> (64 - N)));
  }
  wave_sync();
  return m;
}

// ---- the lattice of a maze -------------------------------------------------------
// A maze's floor lies on rooms (odd row, odd column) and separators between two of
// them; its pillars (even, even) are walls.  Sets of such tiles take 32-bit words
// where tile rows take 64: lane k holds rooms r of row 2k + 1 (bit c: column 2c +
// 1), separators e right of them and s below them.  Levels alternate between rooms
// and separators, so a search takes two at a time: 11 VALU instructions where two
// levels of 64-bit rows take 30.
struct Lattice {
  uint32_t r, e, s;
};
__device__ __forceinline__ bool lattice_any(const Lattice& a) { return wave_any((a.r | a.e | a.s) != 0u); }
__device__ __forceinline__ Lattice lattice_tile(int id, const TileDiv& td, int lane) {
  const int y = td.row(id), x = td.col(id);
  const uint32_t b = lane == ((y - 1) >> 1) ? 1u << (((x - 1) >> 1) & 31) : 0u;
  return {(y & 1) && (x & 1) ? b : 0u, (y & 1) && !(x & 1) ? b : 0u, !(y & 1) && (x & 1) ? b : 0u};
}
// Bits 0, 2, 4, ... of v packed, and the reverse.
__device__ __forceinline__ uint32_t even_bits(uint64_t v) {
  v &= 0x5555555555555555ull;
  v = (v | (v >> 1)) & 0x3333333333333333ull;
  v = (v | (v >> 2)) & 0x0F0F0F0F0F0F0F0Full;
  v = (v | (v >> 4)) & 0x00FF00FF00FF00FFull;
  v = (v | (v >> 8)) & 0x0000FFFF0000FFFFull;
  return (uint32_t)(v | (v >> 16));
}
__device__ __forceinline__ uint64_t spread_bits(uint32_t w) {
  uint64_t v = w;
  v = (v | (v << 16)) & 0x0000FFFF0000FFFFull;
  v = (v | (v << 8)) & 0x00FF00FF00FF00FFull;
  v = (v | (v << 4)) & 0x0F0F0F0F0F0F0F0Full;
  v = (v | (v << 2)) & 0x3333333333333333ull;
  return (v | (v << 1)) & 0x5555555555555555ull;
}
__device__ __forceinline__ uint64_t lane_of(uint64_t v, int src) {
  return ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(v >> 32), src, 64) << 32) | (uint32_t)__shfl((int)(uint32_t)v, src, 64);
}
// The lattice of row masks m (lane y: row y); false if some pillar is floor.
__device__ __forceinline__ bool to_lattice(uint64_t m, int lane, Lattice* out) {
  const int k = lane & 31;
  const uint64_t a = lane_of(m, 2 * k + 1), b = k < 31 ? lane_of(m, 2 * k + 2) : 0ull;
  const bool own = lane < 32;
  *out = {own ? even_bits(a >> 1) : 0u, own ? even_bits(a >> 2) : 0u, own ? even_bits(b >> 1) : 0u};
  return !wave_any(own && even_bits(b >> 2) != 0u);
}
__device__ __forceinline__ uint64_t from_lattice(const Lattice& a, int lane) {
  const int k = (lane - 1) >> 1;
  const uint32_t r = (uint32_t)__shfl((int)a.r, k & 63, 64), e = (uint32_t)__shfl((int)a.e, k & 63, 64),
                 s = (uint32_t)__shfl((int)a.s, k & 63, 64);
  if (lane == 0) return 0ull;
  return (lane & 1) ? (spread_bits(r) << 1) | (spread_bits(e) << 2) : spread_bits(s) << 1;
}
// Smallest tile id of the set, -1 if it is empty.
__device__ __forceinline__ int lattice_first(const Lattice& a, int N) {
  const uint64_t own = __ballot((a.r | a.e | a.s) != 0u);
  if (own == 0ull) return -1;
  const int k = first_bit(own);
  const uint32_t r = lane_value(a.r, k), e = lane_value(a.e, k), s = lane_value(a.s, k);
  if ((r | e) == 0u) return (2 * k + 2) * N + 2 * first_bit(s) + 1;
  const int xr = r ? 2 * first_bit(r) + 1 : 64, xe = e ? 2 * first_bit(e) + 2 : 64;
  return (2 * k + 1) * N + min(xr, xe);
}
// Separators of `in` beside the rooms F, and rooms of `in` beside the separators.
__device__ __forceinline__ void beside_rooms(uint32_t F, const Lattice& in, uint32_t* e, uint32_t* s) {
  *e = (F | (F >> 1)) & in.e;
  *s = (F | lane_next(F)) & in.s;
}
__device__ __forceinline__ uint32_t beside_separators(uint32_t e, uint32_t s, const Lattice& in) {
  return (e | (e << 1) | s | lane_prev(s)) & in.r;
}

struct LatticeSearch {
  int level;          // of the farthest tiles
  int rooms0;         // the first level that holds rooms (0 or 1)
  Lattice farthest;
  Lattice unreached;
  // reached tiles whose level is 2 or 3 more than rooms0, modulo 4: with a tile's
  // kind, which says its level modulo 2, this tells the levels before and after a
  // tile's own apart
  Lattice upper;
};
// Search over the passable tiles until nothing is left to reach; every wave
// reaches the exit, since `unreached` shrinks in every round.
__device__ LatticeSearch lattice_search(const Lattice& pass, int src, const TileDiv& td, int lane) {
  const Lattice at = lattice_tile(src, td, lane);
  LatticeSearch q;
  Lattice U{pass.r & ~at.r, pass.e & ~at.e, pass.s & ~at.s};
  Lattice up{0u, 0u, 0u};
  uint32_t F = at.r;
  q.rooms0 = 0;
  if (!wave_any(F != 0u)) {  // from a separator: its rooms come first
    F = beside_separators(at.e, at.s, U);
    U.r &= ~F;
    q.rooms0 = 1;
    if (!wave_any(F != 0u)) {
      q.level = 0;
      q.farthest = at;
      q.unreached = U;
      q.upper = up;
      return q;
    }
  }
  uint32_t F0, e1, s1, F1, e2, s2, F2 = F;
  int level = q.rooms0 - 4;
  do {
    F0 = F2;
    beside_rooms(F0, U, &e1, &s1);
    U.e &= ~e1;
    U.s &= ~s1;
    F1 = beside_separators(e1, s1, U);
    U.r &= ~F1;
    beside_rooms(F1, U, &e2, &s2);
    U.e &= ~e2;
    U.s &= ~s2;
    F2 = beside_separators(e2, s2, U);
    U.r &= ~F2;
    up.r |= F1;
    up.e |= e2;
    up.s |= s2;
    level += 4;
  } while (wave_any(F2 != 0u));
  if (wave_any((e2 | s2) != 0u)) {
    level += 3;
    q.farthest = {0u, e2, s2};
  } else if (wave_any(F1 != 0u)) {
    level += 2;
    q.farthest = {F1, 0u, 0u};
  } else if (wave_any((e1 | s1) != 0u)) {
    level += 1;
    q.farthest = {0u, e1, s1};
  } else {
    q.farthest = {F0, 0u, 0u};
  }
  q.level = level;
  q.unreached = U;
  q.upper = up;
  return q;
}

// Tiles at level h of search q on a shortest path from its source to `to`, a tile
// of its last level (h >= 1): level by level back from `to`.
__device__ Lattice lattice_back(const LatticeSearch& q, const Lattice& pass, int to, int h, const TileDiv& td, int lane) {
  Lattice B = lattice_tile(to, td, lane);
  const Lattice lo{pass.r & ~q.upper.r, pass.e & ~q.upper.e, pass.s & ~q.upper.s};
  const Lattice hi{pass.r & q.upper.r, pass.e & q.upper.e, pass.s & q.upper.s};
  // one level down, to the level that is j more than rooms0 modulo 4
  auto back = [&](int j) {
    const Lattice& in = j < 2 ? lo : hi;
    if (j & 1) {
      uint32_t e, s;
      beside_rooms(B.r, in, &e, &s);
      B = {0u, e, s};
    } else {
      B = {beside_separators(B.e, B.s, in), 0u, 0u};
    }
  };
  auto any_level = [&](int k) {
    switch ((k - q.rooms0) & 3) {
      case 0: back(0); break;
      case 1: back(1); break;
      case 2: back(2); break;
      default: back(3); break;
    }
  };
  int k = q.level;
  while (k > h && ((k - q.rooms0) & 3)) any_level(--k);
  for (; k - 4 >= h; k -= 4) {
    back(3);
    back(2);
    back(1);
    back(0);
  }
  while (k > h) any_level(--k);
  return B;
}

struct Episode {
  float x, y, th;
  int goal, door, key, nd, dec0, dec1;
};

// Episode reset for episode `e` of the env with layout in `lmap` (0 floor).
// M: row masks (32 bits where the map is at most 32 wide).
// ASC: the batch may hold ASCII maps, LATTICE: maps wider than 16 (else that code
// is compiled out).
template <bool ASC, bool LATTICE, typename M>
__device__ Episode episode_reset(const DevCfg& cf, const TileDiv& td, const uint8_t* lmap, uint32_t* lbits, uint64_t seed,
                                 uint32_t e, int lane) {
  const int N = cf.side;
  uint64_t s = seed ^ sm_mix((uint64_t)e + 1ull);
  // floor tiles: no wall class and no door
  auto is_free = [](uint32_t v) {
    const uint32_t t = v & 0x8F8F8F8Fu;
    return ~(((t & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | t) & 0x80808080u;
  };
  const M freem = row_masks<M>(lmap, lbits, N, lane, is_free);
  const uint32_t n_free = mask_count(freem);
  Episode ep;
  if (ASC && cf.ascii) {
    // ASCII maps: spawn among the spawn candidates (every floor tile if none),
    // heading, goal among the goal candidates (else the farthest tile from the
    // spawn with doors passable, smallest id); keys and doors come from the map
    const M spawnm = row_masks<M>(lmap, lbits, N, lane, [&](uint32_t v) { return is_free(v) & (v << 2); });
    const M goalm = row_masks<M>(lmap, lbits, N, lane, [&](uint32_t v) { return is_free(v) & (v << 1); });
    const uint32_t n_s = mask_count(spawnm);
    const int spawn = n_s ? mask_select(spawnm, sm_draw(s, n_s), N) : mask_select(freem, sm_draw(s, n_free), N);
    const uint32_t k24 = (uint32_t)(sm_next(s) >> 40);
    ep.th = (float)k24 * (kTwoPiF * 0x1p-24f);
    ep.x = (float)td.col(spawn) + 0.5f;
    ep.y = (float)td.row(spawn) + 0.5f;
    const uint32_t n_g = mask_count(goalm);
    if (n_g) {
      ep.goal = mask_select(goalm, sm_draw(s, n_g), N);
    } else {
      const M doorm = row_masks<M>(lmap, lbits, N, lane, [](uint32_t v) { return v & 0x80808080u; });
      ep.goal = mask_first(bfs_all<M>(freem | doorm, spawn, td, lane).frontier, N);
    }
    ep.door = ep.key = -1;
    ep.nd = 0;
    ep.dec0 = ep.dec1 = -1;
    return ep;
  }
  const int spawn = mask_select(freem, sm_draw(s, n_free), N);
  const uint32_t k24 = (uint32_t)(sm_next(s) >> 40);
  ep.th = (float)k24 * (kTwoPiF * 0x1p-24f);
  ep.x = (float)td.col(spawn) + 0.5f;
  ep.y = (float)td.row(spawn) + 0.5f;

  // goal: the first of the farthest tiles; door: the first tile halfway on a
  // shortest path to it; key: in the region that the shut door leaves to the spawn
  ep.door = -1;
  ep.key = -1;
  const M spawnb = bit_of<M>(spawn, td, lane);
  M region = 0;
  bool keyed = false;
  Lattice floor_;
  // 64-bit rows search on the lattice where the map is a maze's; 32-bit rows where
  // a door asks for two more searches (one is over before the lattice is laid out).
  // A step of 1000 key-door envs of 64 x 64, with one reset: 64-side 72 -> 38 us
  // (11.5 without it), 33-side 28.7 -> 19.2, 32-side 21.0 -> 18.3; 16-side 16.3 ->
  // 16.7.
  if (LATTICE && (sizeof(M) == 8 || (cf.key_door && N > 16)) && to_lattice((uint64_t)freem, lane, &floor_)) {
    const LatticeSearch q = lattice_search(floor_, spawn, td, lane);
    ep.goal = lattice_first(q.farthest, N);
    keyed = cf.key_door && q.level >= 2;
    if (keyed) {
      ep.door = lattice_first(lattice_back(q, floor_, ep.goal, q.level / 2, td, lane), N);
      const Lattice d = lattice_tile(ep.door, td, lane);
      const Lattice pass2{floor_.r & ~d.r, floor_.e & ~d.e, floor_.s & ~d.s};
      const Lattice u = lattice_search(pass2, spawn, td, lane).unreached;
      region = (M)from_lattice({pass2.r & ~u.r, pass2.e & ~u.e, pass2.s & ~u.s}, lane) & ~spawnb;
    }
  } else {
    const Bfs<M> b = bfs_all<M>(freem, spawn, td, lane);
    const int L = b.level;
    ep.goal = mask_first(b.frontier, N);
    keyed = cf.key_door && L >= 2;
    if (keyed) {
      ep.door = mask_first(bfs_meet<M>(freem, spawn, ep.goal, L / 2, L & 1, td, lane), N);
      const M pass2 = freem & ~bit_of<M>(ep.door, td, lane);
      region = pass2 & ~bfs_all<M>(pass2, spawn, td, lane).unreached & ~spawnb;
    }
  }
  if (keyed) {
    const uint32_t c = mask_count(region);
    ep.key = (c == 0) ? spawn : mask_select(region, sm_draw(s, c), N);
  }
  ep.nd = 0;
  ep.dec0 = -1;
  ep.dec1 = -1;
  if (cf.max_decor > 0) {
    M cand = freem & ~spawnb & ~bit_of<M>(ep.goal, td, lane) & ~bit_of<M>(ep.key, td, lane) &
             ~bit_of<M>(ep.door, td, lane);
    const uint32_t C = mask_count(cand);
    const int md = cf.max_decor > kMaxDecor ? kMaxDecor : cf.max_decor;
    int nd = (int)sm_draw(s, (uint32_t)(md + 1));
    if (nd > (int)C) nd = (int)C;
    for (int j = 0; j < nd; ++j) {
      const int id = mask_select(cand, sm_draw(s, C - (uint32_t)j), N);
      cand &= ~bit_of<M>(id, td, lane);
      if (j == 0) ep.dec0 = id;
      else ep.dec1 = id;
    }
    ep.nd = nd;
  }
  return ep;
}

typedef __attribute__((address_space(1))) uint32_t GlobalU32;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x2 GlobalU32x2;
typedef __attribute__((address_space(1))) u32x4 GlobalU32x4;

// 12 bytes (4 RGB pixels) to global memory; non-temporal on request.
__device__ __forceinline__ void store12(uint8_t* p, uint32_t a, uint32_t b, uint32_t c, int nt) {
  if (nt) {
    GlobalU32* q = (GlobalU32*)p;
    __builtin_nontemporal_store(a, q);
    __builtin_nontemporal_store(b, q + 1);
    __builtin_nontemporal_store(c, q + 2);
  } else {
    GlobalU32* q = (GlobalU32*)p;
    q[0] = a;
    q[1] = b;
    q[2] = c;
  }
}

// Pixel colours of one column group (4 columns), byte-parallel.  A column's
// span record is (wall rgb | cov << 24, sprite rgb | sc << 24), where rows at
// distance i < sc from the horizon show the sprite, sc <= i < cov the wall and
// the rest ceiling (above) or floor (below).  The group keeps:
//   pw, ps  the 4 wall / sprite colours packed as 12 frame bytes (3 dwords);
//   cova/covb, sca/scb  cov and sc of pixels (0,1) / (2,3) in bytes 1 and 3,
//           biased by 0x7F, so that subtracting i from both bytes at once
//           leaves the byte's sign bit set exactly when i < count (0x7F + count
//           - i stays in [0x40, 0xBF] for counts and i up to 64: no carries);
//   any     the largest cov: rows at i >= any are background in this group.
struct ColGroup {
  uint32_t pw[3], ps[3];
  uint32_t cova, covb, sca, scb;
  uint32_t any;
};

// v_perm_b32 selectors: bytes 0-3 of {hi, lo} come from lo, 4-7 from hi;
// 8..11 replicate the sign bit of bytes 1, 3, 5, 7; 12 gives 0x00.
constexpr uint32_t kSelPack0 = 0x04020100u;  // lo.b0 lo.b1 lo.b2 hi.b0
constexpr uint32_t kSelPack1 = 0x05040201u;  // lo.b1 lo.b2 hi.b0 hi.b1
constexpr uint32_t kSelPack2 = 0x06050402u;  // lo.b2 hi.b0 hi.b1 hi.b2
constexpr uint32_t kSelCount = 0x070C030Cu;  // 0, lo.b3, 0, hi.b3
constexpr uint32_t kSelMask0 = 0x09080808u;  // pixel 0 x3, pixel 1
constexpr uint32_t kSelMask1 = 0x0A0A0909u;  // pixel 1 x2, pixel 2 x2
constexpr uint32_t kSelMask2 = 0x0B0B0B0Au;  // pixel 2, pixel 3 x3
constexpr uint32_t kCountBias = 0x7F007F00u;
constexpr uint32_t kRowStep = 0x01000100u;    // i in bytes 1 and 3

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}
__device__ __forceinline__ uint32_t bitsel(uint32_t m, uint32_t a, uint32_t b) {
  return (m & a) | (~m & b);
}

__device__ __forceinline__ ColGroup col_group(const uint32_t* lcol, int cq) {
  const uint4* l4 = reinterpret_cast<const uint4*>(lcol);
  const uint4 A = l4[2 * cq], B = l4[2 * cq + 1];
  // A = (w0, s0, w1, s1), B = (w2, s2, w3, s3)
  ColGroup g;
  g.pw[0] = perm(A.z, A.x, kSelPack0);
  g.pw[1] = perm(B.x, A.z, kSelPack1);
  g.pw[2] = perm(B.z, B.x, kSelPack2);
  g.ps[0] = perm(A.w, A.y, kSelPack0);
  g.ps[1] = perm(B.y, A.w, kSelPack1);
  g.ps[2] = perm(B.w, B.y, kSelPack2);
  g.cova = perm(A.z, A.x, kSelCount) + kCountBias;
  g.covb = perm(B.z, B.x, kSelCount) + kCountBias;
  g.sca = perm(A.w, A.y, kSelCount) + kCountBias;
  g.scb = perm(B.w, B.y, kSelCount) + kCountBias;
  const uint32_t a = max(A.x >> 24, A.z >> 24), b = max(B.x >> 24, B.z >> 24);
  g.any = max(a, b);
  return g;
}

// Crossings per batch of the DDA walk (one LDS round trip each).
constexpr int kDdaBatch = 4;
// A wave's map in LDS lies between two guards of blocking bytes, each as long as
// the farthest a batch can step past a map of side MAXN: walks read without a
// bounds check, and one that leaves the map stops on a guard.
constexpr int guard_bytes(int maxn) { return kDdaBatch * maxn; }
constexpr int map_slice(int maxn) { return maxn * maxn + 2 * guard_bytes(maxn); }
typedef const __attribute__((address_space(3))) uint8_t* LdsBytes;

constexpr uint32_t kCeil3[3] = {kCeil | (kCeil << 24), (kCeil >> 8) | (kCeil << 16),
                                (kCeil >> 16) | (kCeil << 8)};
constexpr uint32_t kFloor3[3] = {kFloor | (kFloor << 24), (kFloor >> 8) | (kFloor << 16),
                                 (kFloor >> 16) | (kFloor << 8)};

// Writes the mirrored row pair at distance i (row H/2-1-i above, H/2+i below);
// ii = i * kRowStep.  When no lane of the wave has a wall or sprite pixel at
// its distance, the whole wave stores the constant ceiling and floor patterns.
__device__ __forceinline__ void emit_pair(const ColGroup& g, uint32_t i, uint32_t ii, uint8_t* up,
                                          uint8_t* dn, int nt) {
  if (__ballot(i < g.any) == 0ull) {
    store12(up, kCeil3[0], kCeil3[1], kCeil3[2], nt);
    store12(dn, kFloor3[0], kFloor3[1], kFloor3[2], nt);
    return;
  }
  const uint32_t ca = g.cova - ii, cb = g.covb - ii;  // sign bits: i < cov
  const uint32_t sa = g.sca - ii, sb = g.scb - ii;    // sign bits: i < sc
  const uint32_t m0 = perm(cb, ca, kSelMask0), m1 = perm(cb, ca, kSelMask1), m2 = perm(cb, ca, kSelMask2);
  const uint32_t x0 = bitsel(perm(sb, sa, kSelMask0), g.ps[0], g.pw[0]);
  const uint32_t x1 = bitsel(perm(sb, sa, kSelMask1), g.ps[1], g.pw[1]);
  const uint32_t x2 = bitsel(perm(sb, sa, kSelMask2), g.ps[2], g.pw[2]);
  store12(up, bitsel(m0, x0, kCeil3[0]), bitsel(m1, x1, kCeil3[1]), bitsel(m2, x2, kCeil3[2]), nt);
  store12(dn, bitsel(m0, x0, kFloor3[0]), bitsel(m1, x1, kFloor3[1]), bitsel(m2, x2, kFloor3[2]), nt);
}

// ---- training-buffer formats --------------------------------------------------
// Each lane covers a group of kCols columns and one mirrored row pair per
// iteration.  NHWC ([row][col][ch]): the columns that fill 12 bytes (4 of uint8,
// 2 of bfloat16, 1 of float32), one 12-byte store per row, so that a wave's store
// is one run of memory.  With 4 columns of every type a lane's 24 or 48 bytes went
// out in stores that each touched every line of the run and wrote part of it:
// 2048 envs of 60x60 bfloat16 stepped in 17.5 us, now 15.8 (1500 of float32 24.5,
// now 17.6; 1500 of 128x128 float32 78, now 62).  NCHW: 4 columns, kElem dwords
// into each of the 3 channel planes.  Colour
// words hold converted elements; per-pixel masks come from the same biased
// counts as the byte format (v_perm sign-bit replication, selector 8 + pixel).
template <int FMT>
struct ObsFmt {
  static constexpr bool kPlanar = FMT >= 3;
  static constexpr int kDtype = FMT % 3;
  static constexpr int kElem = kDtype == 0 ? 1 : (kDtype == 1 ? 2 : 4);
  static constexpr int kCols = kPlanar ? 4 : 4 / kElem;           // columns per lane
  static constexpr int kWords = kPlanar ? 3 * kElem : 3;          // dwords per lane and row
  static constexpr int kPer = 4 / kElem;    // elements per dword
  // pixel (0..kCols - 1 in the group) and channel of element j of dword k
  static constexpr int pixel(int k, int j) { return kPlanar ? (k % kElem) * kPer + j : (k * kPer + j) / 3; }
  static constexpr int channel(int k, int j) { return kPlanar ? k / kElem : (k * kPer + j) % 3; }
  static constexpr uint32_t mask_sel(int k) {
    uint32_t v = 0;
    for (int b = 0; b < 4; ++b) v |= (uint32_t)(8 + pixel(k, b / kElem)) << (8 * b);
    return v;
  }
  // byte strides of a frame row, a lane's column group and a channel plane
  __device__ static int64_t row_bytes(int W) { return (int64_t)(kPlanar ? W : 3 * W) * kElem; }
  static constexpr int kGroupBytes = kPlanar ? 4 * kElem : 12;
};
static_assert(ObsFmt<0>::mask_sel(0) == kSelMask0 && ObsFmt<0>::mask_sel(1) == kSelMask1 &&
                  ObsFmt<0>::mask_sel(2) == kSelMask2, "byte format masks");

template <int FMT>
struct ColGroupF {
  uint32_t pw[ObsFmt<FMT>::kWords], ps[ObsFmt<FMT>::kWords];
  uint32_t cova, covb, sca, scb;
  uint32_t any;
};

template <int DT>
__device__ __forceinline__ uint32_t elem_of(const uint32_t* lcvt, uint32_t b) {
  return DT == 0 ? b : lcvt[b];
}

// The kWords dwords of 4 pixels with colours c[0..3] (rgb words).
template <int FMT>
__device__ __forceinline__ void pack_words(const uint32_t* lcvt, const uint32_t (&c)[4],
                                           uint32_t (&out)[ObsFmt<FMT>::kWords]) {
  using F = ObsFmt<FMT>;
#pragma unroll
  for (int k = 0; k < F::kWords; ++k) {
    uint32_t v = 0;
#pragma unroll
    for (int j = 0; j < F::kPer; ++j)
      v |= elem_of<F::kDtype>(lcvt, (c[F::pixel(k, j)] >> (8 * F::channel(k, j))) & 0xFFu) << (8 * F::kElem * j);
    out[k] = v;
  }
}

// The same words for one colour on all 4 pixels, at compile time (the
// constant evaluator divides with IEEE round-to-nearest-even, as the device
// does): the ceiling and floor then live in scalar registers.
template <int DT>
constexpr uint32_t norm_const(uint32_t b) {
  const uint32_t u = __builtin_bit_cast(uint32_t, (float)b / 255.0f);
  return DT == 0 ? b : (DT == 2 ? u : (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
template <int FMT>
struct BgWords {
  uint32_t w[ObsFmt<FMT>::kWords];
};
template <int FMT>
constexpr BgWords<FMT> bg_words(uint32_t rgb) {
  using F = ObsFmt<FMT>;
  BgWords<FMT> r{};
  for (int k = 0; k < F::kWords; ++k)
    for (int j = 0; j < F::kPer; ++j)
      r.w[k] |= norm_const<F::kDtype>((rgb >> (8 * F::channel(k, j))) & 0xFFu) << (8 * F::kElem * j);
  return r;
}

template <int FMT>
__device__ __forceinline__ ColGroupF<FMT> col_group_f(const uint32_t* lcol, const uint32_t* lcvt, int cq) {
  constexpr int n = ObsFmt<FMT>::kCols;
  const u32x2* rec = reinterpret_cast<const u32x2*>(lcol) + n * cq;
  ColGroupF<FMT> g;
  uint32_t w[4] = {0u, 0u, 0u, 0u}, sp[4] = {0u, 0u, 0u, 0u};  // (no pixel: counts 0)
#pragma unroll
  for (int k = 0; k < n; ++k) {
    const u32x2 r = rec[k];
    w[k] = r.x;
    sp[k] = r.y;
  }
  pack_words<FMT>(lcvt, w, g.pw);
  pack_words<FMT>(lcvt, sp, g.ps);
  g.cova = perm(w[1], w[0], kSelCount) + kCountBias;
  g.covb = perm(w[3], w[2], kSelCount) + kCountBias;
  g.sca = perm(sp[1], sp[0], kSelCount) + kCountBias;
  g.scb = perm(sp[3], sp[2], kSelCount) + kCountBias;
  g.any = max(max(w[0] >> 24, w[1] >> 24), max(w[2] >> 24, w[3] >> 24));
  return g;
}

// One vector per lane, past the caches on request.  The branches hold something that
// tells them apart, else the compiler makes one store of them and drops the request.
template <typename V>
__device__ __forceinline__ void store_vector(GlobalU32* q, V v, int nt) {
  typedef __attribute__((address_space(1))) V G;
  if (nt) {
    asm volatile("; past the caches");
    __builtin_nontemporal_store(v, (G*)q);
    asm volatile("; past the caches");
  } else {
    *(G*)q = v;
  }
}

// Stores one row's dwords of a lane: p is the lane's place in plane 0.  Planes take
// one vector per lane: left to the compiler, which cannot know the alignment, the
// fused kernels' non-temporal stores were single dwords and triples.
template <int FMT>
__device__ __forceinline__ void store_words(uint8_t* p, int64_t plane, const uint32_t (&v)[ObsFmt<FMT>::kWords],
                                            int nt) {
  using F = ObsFmt<FMT>;
  constexpr int runs = F::kPlanar ? 3 : 1, per = F::kPlanar ? F::kElem : F::kWords;
#pragma unroll
  for (int r = 0; r < runs; ++r) {
    GlobalU32* q = (GlobalU32*)(p + r * plane);
    const uint32_t* w = v + r * per;
    if constexpr (per == 4) {
      store_vector(q, u32x4{w[0], w[1], w[2], w[3]}, nt);
    } else if constexpr (per == 2) {
      store_vector(q, u32x2{w[0], w[1]}, nt);
    } else if (nt) {
#pragma unroll
      for (int k = 0; k < per; ++k) __builtin_nontemporal_store(w[k], q + k);
    } else {
#pragma unroll
      for (int k = 0; k < per; ++k) q[k] = w[k];
    }
  }
}

// Mirrored row pair at distance i (as emit_pair) in format FMT; cw / fw are
// the ceiling / floor dwords.
template <int FMT>
__device__ __forceinline__ void emit_pair_f(const ColGroupF<FMT>& g, uint32_t i, uint32_t ii, uint8_t* up,
                                            uint8_t* dn, int64_t plane, int nt) {
  using F = ObsFmt<FMT>;
  constexpr BgWords<FMT> cb_ = bg_words<FMT>(kCeil), fb_ = bg_words<FMT>(kFloor);
  const uint32_t(&cw)[F::kWords] = cb_.w;
  const uint32_t(&fw)[F::kWords] = fb_.w;
  if (__ballot(i < g.any) == 0ull) {
    store_words<FMT>(up, plane, cw, nt);
    store_words<FMT>(dn, plane, fw, nt);
    return;
  }
  const uint32_t ca = g.cova - ii, cb = g.covb - ii;
  const uint32_t sa = g.sca - ii, sb = g.scb - ii;
  uint32_t u[F::kWords], d[F::kWords];
#pragma unroll
  for (int k = 0; k < F::kWords; ++k) {
    const uint32_t m = perm(cb, ca, F::mask_sel(k));
    const uint32_t x = bitsel(perm(sb, sa, F::mask_sel(k)), g.ps[k], g.pw[k]);
    u[k] = bitsel(m, x, cw[k]);
    d[k] = bitsel(m, x, fw[k]);
  }
  store_words<FMT>(up, plane, u, nt);
  store_words<FMT>(dn, plane, d, nt);
}

struct ColDbg {
  int32_t hit, side;
  float t;
  int32_t cell;
};

// Casts the env's columns and reduces each to a span record in lcol (and
// writes debug records when asked).
// dsn, dcs: sine and cosine of the heading in double.
// col0, hop: this lane casts columns col0, col0 + hop, ...
// The pose, the tiles and the flags are uniform across the wave.
// A wave's time here is latency as much as issue (1,300 of a step's 5,500 cycles
// in the walk of a 25-side map, 600 in the sprites, 800 in the rest): so guards
// stand in for bounds checks, tile coordinates and palette indices come from one
// multiplication each, and slots that hold nothing in front of the camera are
// passed over.  With the same for the step, a fused step of 64 such envs fell
// from 3.45 to 3.13 us, one of 8192 32 x 32 frames from 12.3 to 10.4 us.
template <bool ASC>
__device__ void render_columns(const DevCfg& cf, const TileDiv& td, const DevIo& io, int env, int col0, int hop,
                               const uint8_t* lmap, const uint32_t* lclr, uint32_t* lcol, float x, float y, double dsn,
                               double dcs, int goal, int door, int key, uint32_t fl, int nd, int dec0, int dec1,
                               uint32_t doors, int ak0, int ak1, int ak2) {
  // every rounding is spelled out: products meet sums in fmaf where one rounding is meant
#pragma clang fp contract(off)
  const int N = cf.side, H = cf.obs_h, W = cf.obs_w, K = cf.n_colors, S_lv = cf.shade_levels;
  // the shut locked door blocks rays like a wall (tile id `shut`, -1 if none)
  const int shut = (door >= 0 && !(fl & FL_DOOR_OPEN)) ? door : -1;
  const float sn = (float)dsn, cs = (float)dcs;
  // column c's ray offset along `right` is (2c + 1 - W) * q, q = tanH / W
  const double rq = (double)cf.ray_q_hi + (double)cf.ray_q_lo;

  // Sprites in fixed slots, in painting-index order: key, goal, decor 0, decor 1
  // (ASCII maps: red, blue, yellow key, goal).  Empty slots are skipped, which
  // keeps the relative order of the active ones.
  const bool asc = ASC && cf.ascii != 0;
  const int gsp = (cf.goal_sprite && goal >= 0) ? goal : -1;
  const int sid[4] = {asc ? ((ak0 >= 0 && !(fl & FL_AKEY0)) ? ak0 : -1) : ((key >= 0 && !(fl & FL_KEY)) ? key : -1),
                      asc ? ((ak1 >= 0 && !(fl & (FL_AKEY0 << 1))) ? ak1 : -1) : gsp,
                      asc ? ((ak2 >= 0 && !(fl & (FL_AKEY0 << 2))) ? ak2 : -1) : (nd > 0 ? dec0 : -1),
                      asc ? gsp : (nd > 1 ? dec1 : -1)};
  const uint32_t srgb[4] = {asc ? kAKeyRgb[0] : kKeyRgb, asc ? kAKeyRgb[1] : kGoalRgb,
                            asc ? kAKeyRgb[2] : kDecorRgb, asc ? kGoalRgb : kDecorRgb};
  float sY[4], sU[4], sHW[4], sHS[4];
  uint32_t seen = 0u;  // bit j: slot j is in front of the camera
  const float halfW = 0.5f * (float)W;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    sY[j] = sU[j] = sHW[j] = sHS[j] = 0.f;
    if (sid[j] < 0) continue;  // uniform across the wave
    const float dx = ((float)td.col(sid[j]) + 0.5f) - x;
    const float dy = ((float)td.row(sid[j]) + 0.5f) - y;
    const float tY = fmaf(dx, cs, dy * sn);
    if (!wave_any(tY > 0.05f)) continue;     // (every lane holds the same)
    const float tX = fmaf(dy, cs, -(dx * sn));
    const float inv = 1.0f / tY;             // one division per sprite
    const float q = inv * cf.inv_tanH;       // 1 / (tanH tY)
    seen |= 1u << j;
    sY[j] = tY;
    sU[j] = halfW * fmaf(tX, q, 1.0f);
    sHW[j] = halfW * 0.25f * q;
    sHS[j] = (float)H * 0.25f * inv;
  }

  seen = uniform_u(seen);
  const int ix0 = (int)floorf(x), iy0 = (int)floorf(y);
  const float halfH = (float)(H >> 1);
  const float INF = __builtin_huge_valf();
  const LdsBytes map0 = (LdsBytes)lmap;
  const LdsBytes shutq = map0 + shut;
  const uint32_t last = (uint32_t)(N * N - 1);
  // hit / K by one multiplication (hit below 4096, K at most 8: hit times the
  // excess of km over 2^16 / K stays below 2^16); km = floor(65535 / K) + 1, half of
  // the smallest fraction added as in TileDiv
  const uint32_t km = (uint32_t)(65535.5f * __builtin_amdgcn_rcpf((float)K)) + 1u;
  for (int col = col0; col < W; col += hop) {
    // The ray components are formed in double and rounded once: dir and the
    // column's offset along `right` can nearly cancel, and a float sum would
    // then lose most of the component's digits.  Each float component is
    // within half an ulp of the exact one.
    const double k = (double)(2 * col + 1 - W) * rq;
    const float rx = (float)fma(k, -dsn, dcs);
    const float ry = (float)fma(k, dcs, dsn);
    const int stx = rx > 0.f ? 1 : -1, sty = ry > 0.f ? N : -N;
    const float Xn = (float)(rx > 0.f ? ix0 + 1 : ix0);
    const float Yn = (float)(ry > 0.f ? iy0 + 1 : iy0);
    const float ivx = __builtin_amdgcn_rcpf(rx), ivy = __builtin_amdgcn_rcpf(ry);
    // Ray parameter of the k-th x / y grid line ahead: t0 + k |1/r|, one fused
    // multiply-add from the crossing count (Xn - x is exact, 1/r within an
    // ulp), so every crossing parameter is within a few float ulps of the
    // exact one whatever the walk's length.
    const float t0x = rx != 0.f ? (Xn - x) * ivx : INF;
    const float t0y = ry != 0.f ? (Yn - y) * ivy : INF;
    const float dtx = rx != 0.f ? fabsf(ivx) : 0.f, dty = ry != 0.f ? fabsf(ivy) : 0.f;
    float kx = 0.f, ky = 0.f;
    float tx = t0x, ty = t0y;
    float tst = INF;
    bool xface = true;
    // Branch-free walk in batches: the sequence of tiles a ray crosses does
    // not depend on the map, only where it stops does.  Each batch computes
    // the next kDdaBatch crossings (one grid line each: the tile moves by +-1
    // on an x crossing, +-N on a y crossing, and that axis's crossing count by
    // one), issues their LDS reads together and keeps the first blocking one,
    // so a lane waits for one LDS round trip per batch instead of one per
    // crossing.  The border of blocking tiles (checked on the host) stops every
    // walk inside the map, and the guards one that starts in the border;
    // crossings past the stop are discarded.
    LdsBytes q = map0 + (iy0 * N + ix0), hitq = map0 - 1;
    bool found = false;
    for (int it = 0; it < 4 * N + 8 && !found; it += kDdaBatch) {
      LdsBytes qs[kDdaBatch];
      float ts[kDdaBatch];
      bool sd[kDdaBatch], stop[kDdaBatch];
#pragma unroll
      for (int u = 0; u < kDdaBatch; ++u) {
        const bool sx = tx < ty;
        ts[u] = sx ? tx : ty;
        sd[u] = sx;
        q += sx ? stx : sty;
        kx = sx ? kx + 1.f : kx;
        ky = sx ? ky : ky + 1.f;
        tx = fmaf(kx, dtx, t0x);
        ty = fmaf(ky, dty, t0y);
        qs[u] = q;
      }
      uint32_t vs[kDdaBatch];
#pragma unroll
      for (int u = 0; u < kDdaBatch; ++u) vs[u] = *qs[u];
      if (asc) {
        // map doors block while their bit in `doors` is clear
#pragma unroll
        for (int u = 0; u < kDdaBatch; ++u) {
          const uint32_t v = vs[u];
          const bool open = (v & kTileDoor) && ((doors >> (v & 15u)) & 1u);
          stop[u] = ((v & 0x8Fu) != 0u) && !open;
        }
      } else {
#pragma unroll
        for (int u = 0; u < kDdaBatch; ++u) stop[u] = vs[u] != 0u;
        if (shut >= 0) {  // uniform
#pragma unroll
          for (int u = 0; u < kDdaBatch; ++u) stop[u] |= qs[u] == shutq;
        }
      }
#pragma unroll
      for (int u = kDdaBatch - 1; u >= 0; --u) {  // the earliest stop wins
        tst = stop[u] ? ts[u] : tst;
        xface = stop[u] ? sd[u] : xface;
        hitq = stop[u] ? qs[u] : hitq;
        found |= stop[u];
      }
    }
    const uint32_t hv = *hitq;  // the hit's tile byte (1 on a guard)
    const uint32_t hid = (uint32_t)(hitq - map0);
    const int hit = hid > last ? -1 : (int)hid;
    const int cell = (hit >= 0 && (hit == shut || (hv & kTileDoor))) ? 2 : 1;
    const uint32_t h = hit < 0 ? 0u : (uint32_t)hit;
    uint32_t wc = lclr[kClrPalette + h - __umul24(__umul24(h, km) >> 16, (uint32_t)K)];
    if (asc) {
      const uint32_t wcls = hv & 15u;
      if (hv & kTileDoor) wc = lclr[kClrDoor + ((hv >> 4) & 7u)];
      else if (wcls >= 2u && wcls <= 10u) wc = lclr[kClrWall9 + wcls - 2u];
    } else if (cell == 2) {
      wc = kDoor;
    }
    if (!xface) wc = (wc >> 1) & 0x7F7F7Fu;
    if (S_lv > 0) {
      // distance shading: level l = min(floor(t* S / D), S - 1), each channel
      // scaled by (S - l) / S and rounded down; the division by S (numerators
      // below 4096) is a multiply by ceil(2^16 / S) and a shift
      const int lv = min((int)floorf(tst * cf.shade_scale), S_lv - 1);
      const uint32_t f = (uint32_t)(S_lv - lv), m = cf.shade_mul;
      const uint32_t r = __umul24(__umul24(wc & 0xFFu, f), m) >> 16;
      const uint32_t g = __umul24(__umul24((wc >> 8) & 0xFFu, f), m) >> 16;
      const uint32_t b = __umul24(__umul24((wc >> 16) & 0xFFu, f), m) >> 16;
      wc = r | (g << 8) | (b << 16);
    }
    // rows at i + 0.5 < H / (2 t*): ceil(H / (2 t*) - 0.5) of them, at most H / 2
    const float wrows = ceilf(fmaf(halfH, __builtin_amdgcn_rcpf(tst), -0.5f));
    const uint32_t wcount = (uint32_t)__builtin_amdgcn_fmed3f(wrows, 0.f, halfH);
    // nearest covering sprite; on equal depth the later slot wins (painted last)
    float bestY = INF, bestHS = 0.f;
    uint32_t bestRgb = 0u;
    bool any = false;
    if (seen) {  // uniform
      const float cc = (float)col + 0.5f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (!((seen >> j) & 1u)) continue;
        if (fabsf(cc - sU[j]) < sHW[j] && sY[j] < tst && sY[j] <= bestY) {
          bestY = sY[j];
          bestHS = sHS[j];
          bestRgb = srgb[j];
          any = true;
        }
      }
    }
    uint32_t srec = 0u, scount = 0u;
    if (any) {
      scount = (uint32_t)__builtin_amdgcn_fmed3f(ceilf(bestHS - 0.5f), 0.f, halfH);
      srec = bestRgb | (scount << 24);
    }
    // span record: wall colour with the covered half-height (wall or sprite),
    // sprite colour with the sprite's half-height
    *reinterpret_cast<u32x2*>(lcol + 2 * col) = u32x2{wc | ((wcount > scount ? wcount : scount) << 24), srec};
    if (io.dbg) {
      ColDbg* d = reinterpret_cast<ColDbg*>(io.dbg) + (int64_t)env * io.dbg_stride + col;
      *d = ColDbg{hit, xface ? 0 : 1, tst, cell};
    }
  }
  wave_sync();
}

// s_waitcnt immediate: vector-memory count 4, the other counters untouched.
// After each row pair a wave waits until at most 4 of its stores (two row
// pairs) are in flight: on the 4096-env rollout the HBM write stream measured
// about 1% faster with this bound than with the step-level bound alone (and
// 2% slower with 8 or 12 in flight at the step level).
constexpr int kWaitTwoPairs = 0x0F74;

// Expands the span records into the frame, one mirrored row pair per lane and
// iteration: lane -> (column group cq, distance i from the horizon).  The
// wave's di * Q lanes cover di row pairs of every column group per iteration
// (Q = W / 4 groups, di = 64 / Q), so each lane's group is fixed.
template <int FMT>
__device__ void fill_frame_f(const uint32_t* lcol, const uint32_t* lcvt, uint8_t* base, int W, int H, int lane,
                             int nt, int part, int parts, int n) {
  using F = ObsFmt<FMT>;
  const int H2 = H >> 1;
  const int64_t rowb = F::row_bytes(W), plane = (int64_t)H * W * F::kElem;
  // float32 rows longer than the wave: each lane takes two pixels of a row, so that
  // its cache lines are written together, or the first 64 columns are written in
  // one pass and the rest, several rows at a time, in a second one.  The second
  // pass is fewer instructions while the rest is short, but its lines are gone
  // from the L2 when it comes unless few waves write: with one wave per frame
  // 1500 fused envs of 84x84 take 212 us against 347 (8 steps).  Where waves share a
  // frame 200 of 68x68 take 41 against 32, of 84x84 47.4 against 39.5, of 100x100 53.7
  // against 57.3; 700 of 68x68 63 against 58, of 76x76 89 against 110, of 84x84 111
  // against 147; 1000 of 68x68 103 against 126, of 84x84 161 against 219.
  const int two_pass_n = W <= 72 ? 768 : 512;
  if (F::kCols == 1 && W > 64 && (parts == 1 || W > 84 || n > two_pass_n)) {
    const int l2 = lane + 64;
    const bool two = l2 < W;
    const ColGroupF<FMT> g = col_group_f<FMT>(lcol, lcvt, lane), g2 = col_group_f<FMT>(lcol, lcvt, two ? l2 : lane);
    for (int i = part; i < H2; i += parts) {
      uint8_t* up = base + (int64_t)(H2 - 1 - i) * rowb + F::kGroupBytes * lane;
      uint8_t* dn = base + (int64_t)(H2 + i) * rowb + F::kGroupBytes * lane;
      const uint32_t ii = (uint32_t)i * kRowStep;
      emit_pair_f<FMT>(g, (uint32_t)i, ii, up, dn, plane, nt);
      if (two) emit_pair_f<FMT>(g2, (uint32_t)i, ii, up + F::kGroupBytes * 64, dn + F::kGroupBytes * 64, plane, nt);
    }
    return;
  }
  int c0 = 0;
  do {
    const int Q = min(W / F::kCols - c0, 64);
    const int di = 64 / Q;
    const int cq = c0 + lane % Q;
    if (lane < di * Q) {
      const ColGroupF<FMT> g = col_group_f<FMT>(lcol, lcvt, cq);
      int i = lane / Q + part * di;
      uint8_t* up = base + (int64_t)(H2 - 1 - i) * rowb + F::kGroupBytes * cq;
      uint8_t* dn = base + (int64_t)(H2 + i) * rowb + F::kGroupBytes * cq;
      const int pdi = parts * di;
      const int64_t step = (int64_t)pdi * rowb;
      uint32_t ii = (uint32_t)i * kRowStep;
      const uint32_t dii = (uint32_t)pdi * kRowStep;
      for (; i < H2; i += pdi) {
        emit_pair_f<FMT>(g, (uint32_t)i, ii, up, dn, plane, nt);
        ii += dii;
        up -= step;
        dn += step;
      }
    }
    c0 += 64;
  } while (F::kCols == 1 && c0 < W);
}

// BOUND: keep at most two row pairs of the wave's stores in flight (see kWaitTwoPairs).
// n: envs of the batch.
template <int FMT, bool BOUND>
__device__ void fill_frame(const uint32_t* lcol, const uint32_t* lcvt, uint8_t* base, int W, int H, int lane,
                           int nt, int part = 0, int parts = 1, int n = 1) {
  if constexpr (FMT != 0) {
    fill_frame_f<FMT>(lcol, lcvt, base, W, H, lane, nt, part, parts, n);
    return;
  }
  // lane -> (column group cq, first distance i); the wave's di * Q lanes
  // (all 64 when Q divides 64, 63 of them at W = 84) cover di row pairs of
  // every column group per iteration, so each lane's column group is fixed and
  // its records stay in registers.  When `parts` waves share the env, wave
  // `part` takes every parts-th block of di row pairs.
  const int Q = W >> 2, H2 = H >> 1;
  const int rowb = 3 * W;
  const int di = 64 / Q;
  const int cq = lane % Q;
  int i = lane / Q + part * di;
  if (lane < di * Q) {
    const ColGroup g = col_group(lcol, cq);
    uint8_t* up = base + (int64_t)(H2 - 1 - i) * rowb + 12 * cq;
    uint8_t* dn = base + (int64_t)(H2 + i) * rowb + 12 * cq;
    const int pdi = parts * di;
    const int64_t step = (int64_t)pdi * rowb;
    uint32_t ii = (uint32_t)i * kRowStep;
    const uint32_t dii = (uint32_t)pdi * kRowStep;
    for (; i < H2; i += pdi) {
      emit_pair(g, (uint32_t)i, ii, up, dn, nt);
      if (BOUND) __builtin_amdgcn_s_waitcnt(kWaitTwoPairs);
      ii += dii;
      up -= step;
      dn += step;
    }
  }
}

// Everything one env-step produces, handed from the computing wave to the
// wave that writes it back (or kept by the same wave in the plain form).
struct EnvOut {
  int64_t obs_off;
  int env, W, H, mode;
  float x, y, th, reward;
  uint32_t t, ep, fl, nd, ev, done, doors;
  uint32_t prev;  // previous action beside the frame (n_actions: none)
  int goal, door, key, dec0, dec1;
  double sn, cs;  // sine and cosine of th, in double
};

// Inputs of one env-step, loaded ahead of use: the configuration and state
// (uniform, scalar loads) and this lane's share of the map's dwords.
template <int MAXN>
struct EnvIn {
  static constexpr int kMapWords = (MAXN * MAXN + 255) / 256;  // dwords per lane
  DevCfg cf;
  int env;
  float x, y, th;
  uint32_t t, ep, fl, doors;
  int goal, door, key, dec0, dec1, nd;
  int ak0, ak1, ak2;  // ASCII maps: key tiles (constant per env)
  uint64_t seed;
  uint32_t act;       // per-step forms: this step's action
  double sn, cs;      // fused form: sine and cosine of th, in double
  uint32_t map[kMapWords];
};

// act: the step's actions, loaded beside the state (nullable).
template <int MAXN>
__device__ __forceinline__ void load_env(const DevState& S, const uint8_t* act, int env, int lane, EnvIn<MAXN>& in) {
  in.env = env;
  in.act = act ? act[env] : 0u;
  in.cf = S.uniform ? S.ucfg : S.cfgs[S.cfg_idx[env]];
  const int NN = in.cf.side * in.cf.side;
  const uint8_t* mp = S.uniform ? S.maps + (int64_t)env * S.map_stride : S.maps + S.map_off[env];
  const uint32_t* gm = reinterpret_cast<const uint32_t*>(mp);
#pragma unroll
  for (int k = 0; k < EnvIn<MAXN>::kMapWords; ++k) {
    const int i = lane + 64 * k;
    in.map[k] = (i < ((NN + 3) >> 2)) ? gm[i] : 0u;
  }
  in.x = S.x[env];
  in.y = S.y[env];
  in.th = S.th[env];
  in.t = S.t[env];
  in.ep = S.ep[env];
  in.goal = S.goal[env];
  in.door = S.door[env];
  in.key = S.key[env];
  in.dec0 = S.decor[2 * env];
  in.dec1 = S.decor[2 * env + 1];
  in.fl = S.flags[env];
  in.nd = S.ndecor[env];
  in.seed = S.seed[env];
  in.doors = S.doors[env];
  in.ak0 = S.akey[3 * env];
  in.ak1 = S.akey[3 * env + 1];
  in.ak2 = S.akey[3 * env + 2];
}

// Bit mask of the map's locked doors of colour c (door type c), gathered by
// the whole wave from its LDS map.
__device__ uint32_t locked_doors_of(const uint8_t* lmap, int NN, uint32_t c, int lane) {
  uint32_t m = 0u;
  for (int i = lane; i < NN; i += 64) {
    const uint32_t v = lmap[i];
    if ((v & kTileDoor) && ((v >> 4) & 7u) == c) m |= 1u << (v & 15u);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m |= (uint32_t)__shfl_xor((int)m, off, 64);
  return uniform_u(m);
}

// Copies the env's layout words from registers into the wave's LDS map and puts
// the guards around it.  The LDS map is read-only afterwards (the shut door is
// tested separately), so a wave that keeps one env for several steps stages it
// once.
template <int MAXN>
__device__ __forceinline__ void stage_map(const EnvIn<MAXN>& in, int lane, uint8_t* lmap) {
  constexpr uint32_t kBlock = 0x01010101u;
  constexpr int kGuard = guard_bytes(MAXN) / 4;  // words
  const int NN = in.cf.side * in.cf.side, part = NN & 3;
  uint32_t* lm32 = reinterpret_cast<uint32_t*>(lmap);
#pragma unroll
  for (int k = 0; k < EnvIn<MAXN>::kMapWords; ++k) {
    const int i = lane + 64 * k;
    // the word that the map ends in, if any, ends with the guard
    if (i < ((NN + 3) >> 2)) {
      const uint32_t tail = part && i == (NN >> 2) ? ~0u << (8 * part) : 0u;
      lm32[i] = (in.map[k] & ~tail) | (kBlock & tail);
    }
  }
  if (lane < kGuard) {
    lm32[lane - kGuard] = kBlock;
    lm32[((NN + 3) >> 2) + lane] = kBlock;
  }
}

// Step, reset and column cast of one env from its loaded inputs: LDS and
// registers only, no global stores (so a wave doing only this never waits on
// outstanding stores).  All lanes run the uniform parts redundantly.
// STAGE: a per-step form, which copies the layout into LDS and computes the
// heading's sine and cosine (the fused form has staged the layout and carries
// both in its inputs).
// part, casters: `casters` waves run the same step, each on its own LDS map, and
// cast every casters-th block of 64 columns into the shared records.
template <int MAXN, bool STAGE, bool ASC>
__device__ void produce_env(const EnvIn<MAXN>& in, const DevIo& io, int a,
                            int lane, uint8_t* lmap, const uint32_t* lclr, uint32_t* lcol, EnvOut& o,
                            int part = 0, int casters = 1) {
#pragma clang fp contract(off)
  const DevCfg& cf = in.cf;
  const int env = in.env;
  const int N = cf.side;
  const TileDiv td(N);
  float x = in.x, y = in.y, th = in.th;
  uint32_t t = in.t, ep = in.ep;
  int goal = in.goal, door = in.door, key = in.key;
  int dec0 = in.dec0, dec1 = in.dec1;
  uint32_t doors = in.doors;
  a = (int)uniform_u((uint32_t)a);
  const uint64_t seed = in.seed;

  // Every value here is uniform across the wave.  The branches ask ballots, so
  // they stay scalar.  (Moving the state itself into scalar registers as well
  // took 40 lane registers off, but made a step of the fused rollout 3% and a
  // reset of the 32-side key-door envs 20% slower: the scalar registers spill.)
  const int mode = io.mode;
  float reward = 0.f;
  uint32_t ev = 0;
  bool done = false;
  // Sine and cosine of the heading in double, once per heading: an action
  // either turns (nothing moves, and only the new heading's are needed) or
  // keeps the heading.
  double dsn = in.sn, dcs = in.cs;
  bool heading_changed = false;
  uint32_t prev = (uint32_t)cf.n_actions;
  const int turn_l = cf.n_actions == 4 ? 2 : 4;
  const bool turns = mode == MODE_STEP && a >= turn_l && a < cf.n_actions && cf.turn != 0.f;
  if (turns) {
    float t2 = th + (a == turn_l ? -cf.turn : cf.turn);
    if (t2 < 0.f) t2 += kTwoPiF;
    else if (t2 >= kTwoPiF) t2 -= kTwoPiF;
    th = t2;
    heading_changed = true;
  } else if (STAGE && mode != MODE_RESET) {
    sincos((double)th, &dsn, &dcs);
  }
  // (the map's loads are still under way during the sincos)
  if (STAGE) stage_map<MAXN>(in, lane, lmap);
  uint32_t fl = uniform_u(in.fl);
  int nd = (int)uniform_u((uint32_t)in.nd);
  wave_sync();
  if (mode == MODE_STEP) {
    if (a >= cf.n_actions) ev |= EV_INVALID;
    else prev = (uint32_t)a;
    if (a < turn_l) {
      const float sn = (float)dsn, cs = (float)dcs;
      const float vx = a < 2 ? cs : sn, vy = a < 2 ? sn : cs;
      const bool negx = a == 1 || a == 3, negy = a == 1 || a == 2;
      const float mx = cf.move * (negx ? -vx : vx), my = cf.move * (negy ? -vy : vy);
      const bool dclosed = door >= 0 && !(fl & FL_DOOR_OPEN);
      // x first, then y from the new x: the three tiles either test can ask for
      // are read together
      const float nx = x + mx, ny = y + my;
      const int tx0 = (int)floorf(x), ty0 = (int)floorf(y), tx1 = (int)floorf(nx), ty1 = (int)floorf(ny);
      auto tile = [&](int tx, int ty) -> uint32_t {
        const bool in_map = (unsigned)tx < (unsigned)N && (unsigned)ty < (unsigned)N;
        return lmap[in_map ? ty * N + tx : -1];  // off the map: a guard
      };
      const uint32_t v10 = tile(tx1, ty0), v01 = tile(tx0, ty1), v11 = tile(tx1, ty1);
      auto blocks = [&](uint32_t v, int tx, int ty) -> bool {
        if (ASC && (v & kTileDoor)) return !((doors >> (v & 15u)) & 1u);  // map door: shut unless open
        return (v & 0x0Fu) != 0u || (dclosed && ty * N + tx == door);
      };
      // ASCII maps: walking into a shut unlocked door opens it (the move is refused)
      auto bump = [&](uint32_t v) {
        v = uniform_u(v);
        const uint32_t type = (v >> 4) & 7u;
        if ((v & kTileDoor) && (type == kDoorBlueUnlocked || type == kDoorYellowUnlocked) &&
            !((doors >> (v & 15u)) & 1u)) {
          doors |= 1u << (v & 15u);
          ev |= EV_DOOR;
        }
      };
      bool moved = false;
      if (wave_any(mx != 0.f)) {
        if (!wave_any(blocks(v10, tx1, ty0))) {
          x = nx;
          moved = true;
        } else {
          ev |= EV_BLOCKED_X;
          if (ASC) bump(v10);
        }
      }
      if (wave_any(my != 0.f)) {
        const uint32_t v = moved ? v11 : v01;
        if (!wave_any(blocks(v, moved ? tx1 : tx0, ty1))) {
          y = ny;
        } else {
          ev |= EV_BLOCKED_Y;
          if (ASC) bump(v);
        }
      }
    }
    auto near_tile = [&](int id) -> bool {
      const float dx = x - ((float)td.col(id) + 0.5f);
      const float dy = y - ((float)td.row(id) + 0.5f);
      return wave_any(fmaf(dx, dx, dy * dy) < cf.pr2);
    };
    if (key >= 0 && !(fl & FL_KEY) && near_tile(key)) {
      fl |= FL_KEY | FL_DOOR_OPEN;
      reward += cf.r_key;
      ev |= EV_KEY;
    }
    if (ASC && cf.ascii) {
      // ASCII maps: picking up the key of colour c opens every locked door of colour c
      const int ak[3] = {in.ak0, in.ak1, in.ak2};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (ak[c] < 0 || (fl & (FL_AKEY0 << c))) continue;
        if (near_tile(ak[c])) {
          fl |= FL_AKEY0 << c;
          reward += cf.r_key;
          ev |= EV_KEY;
          const uint32_t m = locked_doors_of(lmap, N * N, (uint32_t)c, lane);
          if (m & ~doors) ev |= EV_DOOR;
          doors |= m;
        }
      }
    }
    bool term = false;
    if (goal >= 0 && wave_any((int)floorf(x) == td.col(goal) && (int)floorf(y) == td.row(goal))) {
      reward += cf.r_goal;
      term = true;
      ev |= EV_GOAL;
    }
    t += 1;
    const bool trunc = t >= (uint32_t)cf.cap;
    if (trunc) ev |= EV_TRUNC;
    done = term || trunc;
    if (done) prev = (uint32_t)cf.n_actions;
  }
  if (mode == MODE_RESET || done) {
    const uint32_t e = (mode == MODE_RESET) ? 0u : ep + 1u;
    // the LDS of the records that this wave is about to write is scratch here
    // (where two waves cast, each has the half of its own 64 columns)
    uint32_t* lbits = lcol + 128 * part;
    const Episode n = MAXN <= 32 || N <= 32 ? episode_reset<ASC, (MAXN > 16), uint32_t>(cf, td, lmap, lbits, seed, e, lane)
                                            : episode_reset<ASC, (MAXN > 16), uint64_t>(cf, td, lmap, lbits, seed, e, lane);
    // (no goal: a map without floor, which only a loaded state can hold; the draws
    // found no tile, and the agent stands off the map)
    x = n.goal < 0 ? -0.5f : n.x;
    y = n.goal < 0 ? -0.5f : n.y;
    th = n.th;
    goal = n.goal;
    door = n.door;
    key = n.key;
    nd = n.nd;
    dec0 = n.dec0;
    dec1 = n.dec1;
    t = 0;
    ep = e;
    fl = 0;
    doors = 0u;
    if (done) ev |= EV_RESET;
    heading_changed = true;
  }
  if (heading_changed) sincos((double)th, &dsn, &dcs);
  if (io.obs || io.dbg)
    render_columns<ASC>(cf, td, io, env, lane + 64 * part, 64 * casters, lmap, lclr, lcol, x, y, dsn, dcs, goal, door,
                        key, fl, nd, dec0, dec1, doors, in.ak0, in.ak1, in.ak2);
  o.obs_off = 0;  // set by the caller (obs_off_of), outside any step loop
  o.env = env;
  o.W = cf.obs_w;
  o.H = cf.obs_h;
  o.mode = mode;
  o.x = x;
  o.y = y;
  o.th = th;
  o.reward = reward;
  o.t = t;
  o.ep = ep;
  o.fl = fl;
  o.nd = (uint32_t)nd;
  o.ev = ev;
  o.done = done ? 1u : 0u;
  o.goal = goal;
  o.door = door;
  o.key = key;
  o.dec0 = dec0;
  o.dec1 = dec1;
  o.doors = doors;
  o.prev = prev;
  o.sn = dsn;
  o.cs = dcs;
}

// Scalar results of one env-step, stored by lane 0 with vector stores.
__device__ void write_back(const DevState& S, const DevIo& io, const EnvOut& o, int lane) {
  if (lane != 0 || o.mode == MODE_RENDER) return;
  const int env = o.env;
  S.x[env] = o.x;
  S.y[env] = o.y;
  S.th[env] = o.th;
  S.t[env] = o.t;
  S.ep[env] = o.ep;
  S.goal[env] = o.goal;
  S.door[env] = o.door;
  S.key[env] = o.key;
  S.decor[2 * env] = o.dec0;
  S.decor[2 * env + 1] = o.dec1;
  S.flags[env] = (uint8_t)o.fl;
  S.ndecor[env] = (uint8_t)o.nd;
  S.events[env] = (uint8_t)o.ev;
  S.doors[env] = o.doors;
  if (o.ev & EV_INVALID) S.invalid[env] += 1u;
  if (o.mode == MODE_STEP) {
    io.rew[env] = o.reward;
    io.done[env] = (uint8_t)o.done;
    if (io.prev) io.prev[env] = (uint8_t)o.prev;
  }
}

// Byte offset of env's frame in a step's observation buffer.
__device__ __forceinline__ int64_t obs_off_of(const DevState& S, int env) {
  return S.uniform ? (int64_t)env * S.obs_stride : S.obs_off[env];
}

// The whole per-env pipeline.
// part / parts: this wave is one of `parts` waves of a workgroup that share the
// env and its records `lcol`.  Wave 0 steps and casts (two waves do, half of the
// columns each, where a row has more than one wave's 64), the others wait for
// the records; then each fills its share of the frame's row pairs.  live: the
// wave has an env (all waves meet at the barrier).  One wave writes a frame at
// about 20 bytes a cycle, so a large frame is most of a small batch's step: 100
// envs of 128 x 128 float32 frames take 23.3 us with one wave each and 12.7 us
// with four, 256 of 64 x 64 12.0 and 10.4 us.
template <int MAXN, bool ASC, int FMT>
__device__ __forceinline__ void process_env(const DevState& S, const DevIo& io, int env, int lane, uint8_t* lmap,
                            const uint32_t* lclr, const uint32_t* lcvt, uint32_t* lcol, int part = 0,
                            int parts = 1, bool live = true) {
  EnvOut o{};
  int casters = 1;
  if (parts > 1 && live) {  // (one wave per env does not wait for this)
    const DevCfg& cf = S.uniform ? S.ucfg : S.cfgs[S.cfg_idx[env]];
    casters = cf.obs_w > 64 ? 2 : 1;
    o.W = cf.obs_w;
    o.H = cf.obs_h;
  }
  if (live && part < casters) {
    EnvIn<MAXN> in;
    load_env<MAXN>(S, io.mode == MODE_STEP ? io.act : nullptr, env, lane, in);
    produce_env<MAXN, true, ASC>(in, io, (int)in.act, lane, lmap, lclr, lcol, o, part, casters);
  }
  if (parts > 1) __syncthreads();
  if (!live) return;
  o.obs_off = obs_off_of(S, env);
  if (io.obs) fill_frame<FMT, false>(lcol, lcvt, io.obs + o.obs_off, o.W, o.H, lane, io.store_mode, part, parts, S.n);
  if (part == 0) write_back(S, io, o, lane);
}

// Work distribution of the persistent forms (word 0 of a queue's line counts
// claims, word 1 the waves that left it).  Items (positions in a work
// order) are split over up to 32 queues by position modulo the queue count; a
// workgroup serves queue blockIdx % nq (so each queue is served from one XCD),
// and the queues (one 128-byte line each) sit in different L2 channels: their
// atomics do not serialize on one address.  Each wave first takes one chunk statically, then claims further
// chunks with one atomic each.  Launch `seq` counts in counter set seq % 4 and
// clears set (seq + 1) % 4 for the next launch on the same stream.
struct QueueView {
  uint32_t* ctr;      // this queue's counter
  int q, nq;          // queue index and count
  int items;          // items in this queue
  int waves, wave;    // waves serving it and this wave's rank among them
  int chunk;
};

template <int WPB>
__device__ __forceinline__ QueueView queue_view(uint32_t* queues, uint32_t seq, int n_items, int w,
                                                int lane, int max_chunk = 1 << 30) {
  QueueView v;
  const int grid = (int)gridDim.x;
  v.nq = grid < kQueues ? grid : kQueues;
  v.q = (int)blockIdx.x % v.nq;
  const int slot = (int)(seq % kQueueSlots);
  v.ctr = queues + (slot * kQueues + v.q) * kQueueStride;
  v.items = n_items > v.q ? (n_items - v.q + v.nq - 1) / v.nq : 0;
  v.waves = ((grid - v.q + v.nq - 1) / v.nq) * WPB;
  v.wave = ((int)blockIdx.x / v.nq) * WPB + w;
  const int c = v.items / (2 * v.waves);
  v.chunk = c < 1 ? 1 : (c > max_chunk ? max_chunk : c);
  if (blockIdx.x == 0 && w == 0 && lane < kQueues) {
    const int nxt = (int)((seq + 1) % kQueueSlots);
    queues[(nxt * kQueues + lane) * kQueueStride] = 0u;       // claims
    queues[(nxt * kQueues + lane) * kQueueStride + 1] = 0u;   // exits
  }
  return v;
}

// Calls f(position) for every item position this wave owns or claims.  Every
// wave leaves once its claim passes the end of its queue.
template <typename F>
__device__ __forceinline__ void queue_drain(const QueueView& v, int lane, F&& f) {
  const int dyn0 = v.waves * v.chunk;  // first position handed out by the counter
  int first = v.wave * v.chunk;        // static first chunk
  while (first < v.items) {
    const int end = min(first + v.chunk, v.items);
    for (int j = first; j < end; ++j) f(v.q + j * v.nq);
    if (dyn0 >= v.items) break;        // the static chunks cover the queue
    // a plain read first: a drained queue costs no atomic
    uint32_t cur = 0;
    if (lane == 0) cur = __hip_atomic_load(v.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (dyn0 + __builtin_amdgcn_readfirstlane((int)cur) >= v.items) break;
    uint32_t got = 0;
    if (lane == 0) got = atomicAdd(v.ctr, (uint32_t)v.chunk);
    first = dyn0 + __builtin_amdgcn_readfirstlane((int)got);
  }
  // The last wave to leave the queue returns its claim and exit counters to
  // zero, so every launch leaves its counter set clean and a launch captured
  // once replays correctly.  A wave counts its exit only after its last claim
  // has returned, so no claim can follow the reset.
  if (lane == 0) {
    const uint32_t left = atomicAdd(v.ctr + 1, 1u);
    if (left == (uint32_t)v.waves - 1u) {
      __hip_atomic_store(v.ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(v.ctr + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// The training-buffer formats (FMT != 0) are built for 4 waves per workgroup
// only: the host maps every launch of such a batch to that shape.
constexpr int kFmtWaves = 4;

// Picks the kernel variant by the largest map side and by whether the batch
// holds ASCII maps (frame format FMT fixed).
template <template <int, bool, int> class L, int FMT, typename... A>
int by_shape_f(const DevState& s, int max_side, A&&... a) {
  if (s.any_ascii) {
    if (max_side <= 16) return L<16, true, FMT>::run(s, a...);
    if (max_side <= 32) return L<32, true, FMT>::run(s, a...);
    return L<64, true, FMT>::run(s, a...);
  }
  if (max_side <= 16) return L<16, false, FMT>::run(s, a...);
  if (max_side <= 32) return L<32, false, FMT>::run(s, a...);
  return L<64, false, FMT>::run(s, a...);
}
// ... and by the batch's frame format
template <template <int, bool, int> class L, typename... A>
int by_shape(const DevState& s, int max_side, A&&... a) {
  switch (s.obs_fmt) {
    case 0: return by_shape_f<L, 0>(s, max_side, a...);
    case 1: return by_shape_f<L, 1>(s, max_side, a...);
    case 2: return by_shape_f<L, 2>(s, max_side, a...);
    case 3: return by_shape_f<L, 3>(s, max_side, a...);
    case 4: return by_shape_f<L, 4>(s, max_side, a...);
    case 5: return by_shape_f<L, 5>(s, max_side, a...);
    default: return -1;
  }
}

}  // namespace

}  // namespace jx
