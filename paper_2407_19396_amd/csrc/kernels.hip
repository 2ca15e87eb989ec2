// kernels.hip -- gfx950 kernels of the batched gridworld environment step.
//
// The step is NAVIX's interaction protocol (arXiv 2407.19396, Sec. 3.2.2:
// step(timestep, action) with autoreset; reset pads action -1, reward 0)
// applied to MiniGrid's dynamics, which the paper reproduces exactly
// (Sec. 3.2.1): the intervention / transition / observation / reward /
// termination systems of Table "systems" and App. A over the entities of
// Table "entities", for every family of Table "envs".
//
// Three kernels share the device functions below:
//   k_plain  -- one launch per step; one env per lane; state, grid and
//               outputs in HBM; the view's rows read straight from the grid,
//               and moving balls' surroundings too.
//   k_fused  -- each workgroup takes tiles of up to 64 envs of any mix of
//               sizes, stages their grids in LDS as one code byte per cell,
//               runs K steps with the pose in registers, writes one
//               trajectory record per env-step, then writes the state back;
//               with few tiles a second wave writes the records.  Its serving
//               variant also admits and resets new requests.
//   k_reset  -- episode 0 of every env, laid out in LDS as in k_fused.
// First-person observations are staged in LDS as one code per cell, so that
// a wave's records leave as one contiguous block, decoded on the way out, in
// 12-byte stores.  Whole-grid observations leave the same way, packed like
// the grids.
//
// All arithmetic is integer except the reward, which is three separately
// rounded fp32 operations (built with -ffp-contract=off).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.h"

namespace gx {
namespace {

constexpr int kWave = 64;
constexpr int kView = 7;
constexpr int kObsBytes = kView * kView * 3;        // 147
constexpr int kCatBytes = kView * kView;            // categorical record: 49

// Cell triples are packed as type | colour << 8 | state << 16 (MiniGrid's
// object, colour and state indices).
constexpr uint32_t kEmpty = 1, kWall = 2, kDoor = 4, kKey = 5, kBall = 6, kBox = 7, kGoal = 8,
                   kLava = 9;
constexpr uint32_t kGreen = 1, kGrey = 5;
constexpr uint32_t kOpen = 0, kClosed = 1, kLocked = 2;
constexpr uint32_t kCellEmpty = kEmpty;

constexpr uint32_t kFlagTerminated = 1, kFlagTruncated = 2, kFlagFirst = 4;
constexpr uint32_t kActionNone = 0xFF;

enum : uint32_t { kLeft = 0, kRight = 1, kForward = 2, kPickup = 3, kDrop = 4, kToggle = 5 };
enum : uint32_t {
  kFamEmpty = 0, kFamTwoRoom = 1, kFamFourRooms = 2,
  kFamLavaGap = 3, kFamCrossings = 4, kFamDistShift = 5, kFamDynObs = 6, kFamGoToDoor = 7,
  kFamKeyCorridor = 8
};
constexpr int kMaxObst = 8;
constexpr uint32_t kBlue = 2;

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): counter-based, so every draw is a
// pure function of (key, counter) and needs no stored generator state.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return (uint32_t)__builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox_round(uint4 c, uint2 k) {
  const uint32_t lo0 = 0xD2511F53u * c.x, hi0 = __umulhi(0xD2511F53u, c.x);
  const uint32_t lo1 = 0xCD9E8D57u * c.z, hi1 = __umulhi(0xCD9E8D57u, c.z);
  return make_uint4(xor3(hi1, c.y, k.x), lo1, xor3(hi0, c.w, k.y), lo0);
}

// N blocks of one key, round by round beside each other: one alone is a chain
// of dependent operations (8 cycles each against 5).  With this, one
// exclusive or of three and the balls' straight line (move_balls): 30 011
// envs of all families, 64 steps 316 -> 301 us, 65 536 Dynamic-Obstacles 293 ->
// 275, KeyCorridor 221 -> 213.
template <int N>
__device__ __forceinline__ void philox10(uint4 (&c)[N], uint2 k) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k.x += 0x9E3779B9u;
      k.y += 0xBB67AE85u;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) c[i] = philox_round(c[i], k);
  }
}

__device__ __forceinline__ uint4 philox10(uint4 c, uint2 k) {
  uint4 one[1] = {c};
  philox10<1>(one, k);
  return one[0];
}

// A value the compiler knows nothing about from here on, so that what is
// derived from it is not computed ahead of the step loop and held in
// registers: a draw's and a ball move's many constants per lane would
// otherwise cost a wave per SIMD.
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ uint2 opaque(uint2 v) { return make_uint2(opaque(v.x), opaque(v.y)); }

// uniform integer in [0, n)
__device__ __forceinline__ uint32_t bounded(uint32_t word, uint32_t n) { return __umulhi(word, n); }

__device__ __forceinline__ uint32_t pick4(uint4 v, uint32_t lane) {
  uint32_t r = v.x;
  r = lane == 1 ? v.y : r;
  r = lane == 2 ? v.z : r;
  r = lane == 3 ? v.w : r;
  return r;
}

// Random-policy words of an env's call block `call >> 2`: counter (id,
// block, 0, 1); call = the env's step calls since its reset.
__device__ __forceinline__ uint4 policy_block(uint2 seed, uint32_t rng_id, uint32_t call) {
  return philox10(make_uint4(rng_id, call >> 2, 0u, 1u), seed);
}

// ---------------------------------------------------------------------------
// Start states (reset(key) of Sec. 3.2.2; the families of Table "envs").
// Layout parameters come from the layout stream, counter (id, episode,
// block, 0), in draw order; "uniform placement" picks the k-th free cell
// in row-major order, which every family below reaches in closed form.
// ---------------------------------------------------------------------------
struct Layout {
  int fam, S;
  int a, b, c, d;      // TwoRoom: a = wall column, b = door row; FourRooms: the 4 openings;
                       // LavaGap: a = lava column, b = gap row; DistShift: a = second lava row;
                       // GoToDoor: the doors' positions along the top, right, bottom, left walls
  int colour;          // TwoRoom, KeyCorridor: locked door / key colour; GoToDoor: door i's
                       // colour at bits 4i..4i+3
  int kx, ky;          // TwoRoom, KeyCorridor: key; GoToDoor: the room's width and height
  int gx, gy;          // goal
  int ax, ay, dir;     // agent
  uint32_t vmask, hmask;   // Crossings: river columns / rows (bit = coordinate)
  uint64_t vopen, hopen;   // Crossings: opening row of each river column, opening column
                           // of each river row, 5 bits each in ascending river order
  uint32_t ob[4];          // Dynamic-Obstacles: ball b at bytes 2b (x), 2b + 1 (y); 0xFF unused
  uint32_t kd[3];          // KeyCorridor: the doors between rooms, one byte each (see below)
};

// (x, y) of ball b from a packed obstacle list
__device__ __forceinline__ uint32_t obst_at(const uint32_t (&ob)[4], int b) {
  return (ob[b >> 1] >> (16 * (b & 1))) & 0xFFFFu;
}

__device__ __forceinline__ void obst_set(uint32_t (&ob)[4], int b, uint32_t x, uint32_t y) {
  const int sh = 16 * (b & 1);
  ob[b >> 1] = (ob[b >> 1] & ~(0xFFFFu << sh)) | ((x | (y << 8)) << sh);
}

// The layout stream for the two generators whose number of draws varies: a
// window of kDrawWords words per lane in LDS (word i of lane l at [64 i + l]).
// Drawn word by word from registers, some lane would need a new Philox block
// at nearly every draw, and the whole wave would compute it.  Twelve words
// fit the fused kernel's stage; a larger window would cost it a workgroup per
// compute unit on the mixed batch (20 steps 184 -> 211 us at 24 words).
constexpr int kDrawBlocks = 3;
constexpr int kDrawWords = 4 * kDrawBlocks;
constexpr int kDrawBytes = kDrawWords * kWave * 4;

struct DrawWindow {
  uint32_t* words;    // the lane's column
  uint2 seed;
  uint32_t id, episode;
  uint32_t block, w;  // the window's first block; the next word, from there

  __device__ __forceinline__ void fill() {
    block += w >> 2;
    w &= 3u;
    uint4 v[kDrawBlocks];
#pragma unroll
    for (int b = 0; b < kDrawBlocks; ++b) v[b] = make_uint4(id, episode, block + (uint32_t)b, 0u);
    philox10<kDrawBlocks>(v, opaque(seed));
#pragma unroll
    for (int b = 0; b < kDrawBlocks; ++b) {
      uint32_t* p = words + 4 * kWave * b;
      p[0] = v[b].x;
      p[kWave] = v[b].y;
      p[2 * kWave] = v[b].z;
      p[3 * kWave] = v[b].w;
    }
  }
  // refills every lane's window if some lane's holds fewer than n <= 9 words
  __device__ __forceinline__ void need(uint32_t n) {
    if (__ballot(w + n > kDrawWords)) fill();
  }
  __device__ __forceinline__ uint32_t next(uint32_t n) { return bounded(words[kWave * w++], n); }
};

// position of the k-th (0-based) set bit of m
__device__ __forceinline__ int kth_bit(uint32_t m, int k) {
  for (int i = 0; i < k; ++i) m &= m - 1u;
  return __builtin_ctz(m);
}

// Crossings(S, N): N of the M = S - 3 candidate rivers (columns 2, 4, ..,
// S - 3, then rows 2, 4, .., S - 3) by a partial Fisher-Yates shuffle, then
// a monotone path of room moves, each opening one cell of the river it
// crosses (Table "envs", Crossings; lava of Table "entities").  The shuffle
// keeps only the positions it touched: entry k records that position
// mkey[k] now holds candidate mval[k].
constexpr int kMaxRivers = 8;

struct Rivers {
  uint32_t vmask, hmask;
  uint64_t vopen, hopen;
};

__device__ __forceinline__ Rivers crossings_layout(int S, int N, uint2 seed, uint32_t rng_id,
                                                   uint32_t episode, uint32_t* words) {
  static_assert(kMaxRivers <= kDrawWords, "the rivers' draws fit the window");
  DrawWindow d{words, seed, rng_id, episode, 0u, 0u};
  d.fill();
  const int M = S - 3, h = M / 2;
  int mkey[kMaxRivers], mval[kMaxRivers];
  Rivers R{0u, 0u, 0ull, 0ull};
#pragma unroll
  for (int k = 0; k < kMaxRivers; ++k) {
    if (k < N) {
      const int r = k + (int)d.next((uint32_t)(M - k));
      int vk = k, vr = r;
#pragma unroll
      for (int j = 0; j < k; ++j) {
        vk = mkey[j] == k ? mval[j] : vk;
        vr = mkey[j] == r ? mval[j] : vr;
      }
      mkey[k] = r;
      mval[k] = vk;
      if (vr < h) R.vmask |= 1u << (2 + 2 * vr);
      else R.hmask |= 1u << (2 + 2 * (vr - h));
    }
  }
  const int nv = __builtin_popcount(R.vmask), nh = __builtin_popcount(R.hmask);
  int ci = 0, rj = 0;
  for (int q = 0; q < N; ++q) {
    d.need(2u);
    const int rv = nv - ci, rh = nh - rj;
    if ((int)d.next((uint32_t)(rv + rh)) < rv) {
      const int lo = rj == 0 ? 0 : kth_bit(R.hmask, rj - 1);
      const int hi = rj == nh ? S - 1 : kth_bit(R.hmask, rj);
      const uint64_t y = (uint64_t)(lo + 1 + (int)d.next((uint32_t)(hi - lo - 1)));
      R.vopen |= y << (5 * ci);
      ++ci;
    } else {
      const int lo = ci == 0 ? 0 : kth_bit(R.vmask, ci - 1);
      const int hi = ci == nv ? S - 1 : kth_bit(R.vmask, ci);
      const uint64_t x = (uint64_t)(lo + 1 + (int)d.next((uint32_t)(hi - lo - 1)));
      R.hopen |= x << (5 * rj);
      ++rj;
    }
  }
  return R;
}

// q = k / w, r = k % w for k < 2^16 and 1 <= w <= 32.  The single-precision
// quotient is within a few ulp of k / w, far less than the 1 / w distance
// between its fractional part and the next integer when k % w != 0; when
// k % w == 0 it may fall just short of q, which the correction repairs.
__device__ __forceinline__ void small_divmod(uint32_t k, uint32_t w, uint32_t& q, uint32_t& r) {
  q = (uint32_t)((float)k * __builtin_amdgcn_rcpf((float)w));
  r = k - q * w;
  const bool under = r >= w;
  q += under ? 1u : 0u;
  r -= under ? w : 0u;
}

// KeyCorridor(S = 3s - 2, R rows of rooms): walls between two rooms, one
// byte each in L.kd (byte e of word e / 4): bit 7 set when the wall has a
// door, bits 4-6 its colour, bits 0-3 its position along the wall.  Walls
// between columns i and i + 1 in row j: e = 2j + i; walls between rows jw
// and jw + 1 in column 0 or 2: e = 6 + 2 jw + i / 2 (column 1 is the open
// hallway).  The locked door is the wall e = 2 rl + 1 of the locked row rl.
__device__ __forceinline__ uint32_t kc_byte(const uint32_t (&kd)[3], int e) {
  const uint64_t lo = (uint64_t)kd[0] | ((uint64_t)kd[1] << 32);
  return e < 8 ? (uint32_t)(lo >> (8 * e)) & 0xFFu : (kd[2] >> (8 * (e - 8))) & 0xFFu;
}

struct KcLayout {
  int rl, colour, gx, gy, kx, ky, ax, ay, dir;
  uint32_t kd[3];
};

// What connects a layout's rooms so far, for the lanes that keycorridor_layout
// leaves to connect_few: the doors as bits of the room on their west or north
// side, the door positions, the next word of the stream, the attempts made.
struct KcRest {
  uint32_t todo, right, down;
  uint64_t pos;
  uint32_t word, tries;
};
constexpr uint32_t kKcTries = 1024;
constexpr int kKcFew = 8;

// From the hallway any room is at most one wall across and two along.
__device__ __forceinline__ bool kc_connected(uint32_t R, uint32_t right, uint32_t down) {
  const uint32_t all = (1u << (3u * R)) - 1u;
  uint32_t reached = 0x92u & all;
#pragma unroll
  for (int hop = 0; hop < 3; ++hop)
    reached |= ((reached & right) << 1) | ((reached >> 1) & right) | ((reached & down) << 3) | ((reached >> 3) & down);
  return reached == all;
}

// An attempt picks a room and a wall of it, three words, and takes a fourth for
// the colour if it adds a door: 0, or 1 | room << 1 | across << 6 | wall << 7 |
// the door's table entry << 11.
__device__ __forceinline__ uint32_t kc_attempt(const uint32_t (&w)[4], uint32_t R, uint32_t rl, uint32_t right,
                                               uint32_t down, uint64_t pos) {
  const int i = (int)bounded(w[0], 3u), j = (int)bounded(w[1], R);
  const uint32_t k = bounded(w[2], 4u), c = bounded(w[3], 6u);
  // k: east, south, west, north
  const int i2 = i + (k == 0u ? 1 : 0) - (k == 2u ? 1 : 0), j2 = j + (k == 1u ? 1 : 0) - (k == 3u ? 1 : 0);
  const uint32_t across = (k & 1u) ^ 1u;
  const int il = min(i, i2), jl = min(j, j2);
  const uint32_t room = (uint32_t)(3 * jl + il) & 31u;
  const uint32_t known = ((across ? right : down) >> room) & 1u;
  const uint32_t inside = ((unsigned)i2 < 3u ? 1u : 0u) & ((unsigned)j2 < R ? 1u : 0u);
  // a cell (room) number 3 j + i tells the locked room apart
  const int lock = (int)(3u * rl + 2u);
  const uint32_t locked = (3 * j + i == lock ? 1u : 0u) | (3 * j2 + i2 == lock ? 1u : 0u);
  const uint32_t e = (uint32_t)(across ? 2 * jl + il : 6 + 2 * jl + (i >> 1)) & 15u;
  const uint32_t entry = 0x80u | (c << 4) | (uint32_t)((pos >> (4u * e)) & 15u);
  return inside & ~(known | locked) ? 1u | (room << 1) | (across << 6) | (e << 7) | (entry << 11) : 0u;
}

__device__ __forceinline__ void kc_add(uint32_t door, uint32_t& right, uint32_t& down, uint32_t (&kd)[3]) {
  const uint32_t bit = (door & 1u) << ((door >> 1) & 31u);
  const bool across = (door >> 6) & 1u;
  right |= across ? bit : 0u;
  down |= across ? 0u : bit;
  const uint32_t e = (door >> 7) & 15u, v = (door >> 11) << (8u * (e & 3u));
  kd[0] |= e < 4u ? v : 0u;
  kd[1] |= (e >> 2) == 1u ? v : 0u;
  kd[2] |= (e >> 2) == 2u ? v : 0u;
}

template <bool kTogether>
__device__ __forceinline__ KcLayout keycorridor_layout(int S, int R, uint2 seed, uint32_t rng_id,
                                                       uint32_t episode, uint32_t* words, KcRest& rest) {
  DrawWindow d{words, seed, rng_id, episode, 0u, 0u};
  d.fill();   // the walls take at most 12 draws
  const int st = (S - 1) / 3, inner = st - 1;
  // door positions of walls e = 0..9 (the table's numbering), 4 bits each
  uint64_t pos = 0;
  for (int j = 0; j < R; ++j)
    for (int i = 0; i < 3; ++i) {
      if (i < 2) pos |= (uint64_t)d.next((uint32_t)inner) << (4 * (2 * j + i));
      if (j < R - 1) {
        const uint64_t p = d.next((uint32_t)inner);   // the hallway's wall draws one too
        if (i != 1) pos |= p << (4 * (6 + 2 * j + (i >> 1)));
      }
    }
  KcLayout K;
  d.need(7u);
  K.rl = (int)d.next((uint32_t)R);
  K.colour = (int)d.next(6u);
  const int el = 2 * K.rl + 1;   // < 8
  const uint32_t locked_door = 0x80u | ((uint32_t)K.colour << 4) | (uint32_t)((pos >> (4 * el)) & 15u);
  K.kd[0] = el < 4 ? locked_door << (8 * el) : 0u;
  K.kd[1] = el < 4 ? 0u : locked_door << (8 * (el - 4));
  K.kd[2] = 0u;
  uint32_t q, r;
  small_divmod(d.next((uint32_t)(inner * inner)), (uint32_t)inner, q, r);
  K.gx = 2 * st + 1 + (int)r;
  K.gy = K.rl * st + 1 + (int)q;
  const int rk = (int)d.next((uint32_t)R);
  small_divmod(d.next((uint32_t)(inner * inner)), (uint32_t)inner, q, r);
  K.kx = 1 + (int)r;
  K.ky = rk * st + 1 + (int)q;
  const int ra = R / 2;
  small_divmod(d.next((uint32_t)(inner * inner)), (uint32_t)inner, q, r);
  K.ax = st + 1 + (int)r;
  K.ay = ra * st + 1 + (int)q;
  K.dir = (int)d.next(4u);
  // connect every room (MiniGrid's connect_all), the locked room excepted
  uint32_t right = 1u << (3 * K.rl + 1), down = 0u;   // the locked door
  for (int j = 0; j + 1 < R; ++j) down |= 1u << (3 * j + 1);   // the hallway
  // The wave runs attempts until its last lanes are left (55 and more for the
  // longest of 64 layouts), so an attempt is selects without branches.
  bool todo = true;
  uint32_t it = 0;
  for (; it < kKcTries; ++it) {
    todo = !kc_connected((uint32_t)R, right, down);
    if (__popcll(__ballot(todo)) <= (kTogether ? kKcFew : 0)) break;
    d.need(4u);
    const uint32_t* at = d.words + kWave * d.w;
    const uint32_t w[4] = {at[0], at[kWave], at[2 * kWave], at[3 * kWave]};
    const uint32_t door = todo ? kc_attempt(w, (uint32_t)R, (uint32_t)K.rl, right, down, pos) : 0u;
    d.w += todo ? 3u + (door & 1u) : 0u;
    kc_add(door, right, down, K.kd);
  }
  if (kTogether) rest = KcRest{todo && it < kKcTries ? 1u : 0u, right, down, pos, 4u * d.block + d.w, it};
  return K;
}

// Finishes the at most kKcFew layouts of the wave with rest.todo set, doors
// into kd: each has a group of 8 lanes, and lane t of a group tries the t-th
// next attempt.  As long as none adds a door every attempt takes three words, so
// the first that does is the one a serial run would come to.  All lanes
// call this.  A layout may take over a hundred attempts one after another, and
// 65 536 envs always hold such a one: a reset of 65 536 envs of all families 109 ->
// 55 us, of KeyCorridor alone 111 -> 61; 64 steps of 30 011 envs of all families
// 301 -> 281, of 65 536 KeyCorridor envs 213 -> 173.  Step kernels for batches
// without KeyCorridor leave it out: the code would cost each of their steps
// 1-3 % (4096 Empty 8x8 240 -> 247 us for 256 steps).
__device__ __forceinline__ void connect_few(uint32_t (&kd)[3], uint32_t rl, const KcRest& rest, uint32_t meta,
                                            uint2 seed, uint32_t rng_id, uint32_t episode) {
  const uint64_t few = __ballot(rest.todo != 0u);
  if (!few) return;
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int group = lane >> 3;
  const uint32_t t = (uint32_t)lane & 7u;
  int owner = 0, groups = 0;
  for (uint64_t m = few; m; m &= m - 1, ++groups) owner = group == groups ? __ffsll((unsigned long long)m) - 1 : owner;
  auto of = [&](uint32_t v) { return (uint32_t)__shfl((int)v, owner, kWave); };
  const uint32_t R = (of(meta) >> 16) & 255u, lock = of(rl), id = of(rng_id), ep = of(episode);
  const uint2 key = make_uint2(of(seed.x), of(seed.y));
  const uint64_t pos = (uint64_t)of((uint32_t)rest.pos) | ((uint64_t)of((uint32_t)(rest.pos >> 32)) << 32);
  uint32_t right = of(rest.right), down = of(rest.down), word = of(rest.word), tries = of(rest.tries);
  uint32_t doors[3] = {of(kd[0]), of(kd[1]), of(kd[2])};
  while (true) {
    const bool todo = group < groups && tries < kKcTries && !kc_connected(R, right, down);
    if (!__ballot(todo)) break;
    const uint32_t at = word + 3u * t, sh = at & 3u;
    uint4 b[2] = {make_uint4(id, ep, at >> 2, 0u), make_uint4(id, ep, (at >> 2) + 1u, 0u)};
    philox10<2>(b, key);
    const uint32_t v[7] = {b[0].x, b[0].y, b[0].z, b[0].w, b[1].x, b[1].y, b[1].z};
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t lo = (sh & 1u) ? v[q + 1] : v[q], hi = q + 3 < 7 ? ((sh & 1u) ? v[q + 3] : v[q + 2]) : v[q + 2];
      w[q] = (sh & 2u) ? hi : lo;
    }
    const uint32_t door = todo && tries + t < kKcTries ? kc_attempt(w, R, lock, right, down, pos) : 0u;
    const uint64_t hits = __ballot(door != 0u);
    const uint32_t mine = (uint32_t)(hits >> (8 * group)) & 255u;
    const uint32_t first = mine ? (uint32_t)__builtin_ctz(mine) : 0u;
    const uint32_t added = (uint32_t)__shfl((int)door, 8 * group + (int)first, kWave);
    kc_add(mine ? added : 0u, right, down, doors);
    word += mine ? 3u * first + 4u : 24u;
    tries += mine ? first + 1u : 8u;
  }
  const int rank = (int)__popcll(few & ((1ull << lane) - 1ull));
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const uint32_t v = (uint32_t)__shfl((int)doors[q], (8 * rank) & 63, kWave);
    kd[q] = rest.todo ? v : kd[q];
  }
}

// idx-th free cell, row-major, of a four-room grid of side S = 2m + 1 with
// openings (m, g1), (m, g2) in the vertical wall (g1 < m < g2) and
// (g3, m), (g4, m) in the horizontal one.  Rows other than m hold S - 3 free
// cells (the wall column removed), S - 2 in the opening rows g1 and g2; row
// m holds the two openings.
__device__ __forceinline__ void fourrooms_cell(int S, int m, int g1, int g2, int g3, int g4,
                                               uint32_t idx, int& x, int& y) {
  const uint32_t W = (uint32_t)(S - 3);
  const uint32_t top = (uint32_t)(m - 1) * W + 1u;   // free cells in rows 1 .. m-1
  if (idx - top < 2u) {                              // row m
    y = m;
    x = idx == top ? g3 : g4;
    return;
  }
  const bool low = idx >= top;
  const int row0 = low ? m + 1 : 1, gap = low ? g2 : g1;
  const uint32_t k = low ? idx - top - 2u : idx;
  const uint32_t before = (uint32_t)(gap - row0) * W;   // cells in the rows above the gap row
  if (k - before <= W) {                                // the gap row: every interior cell
    y = gap;
    x = 1 + (int)(k - before);
    return;
  }
  uint32_t q, r;
  small_divmod(k < before ? k : k - 1u, W, q, r);
  y = row0 + (int)q;
  x = 1 + (int)r;
  x += x >= m ? 1 : 0;
}

// meta = family | side << 8 | parameter << 16 (Crossings: rivers; DistShift:
// variant; Dynamic-Obstacles: balls; KeyCorridor: rows of rooms).  The lava
// families and Dynamic-Obstacles start at (1, 1) facing east.
// words: the lane's column of the draw window.
template <bool kTogether>
__device__ __forceinline__ Layout make_layout(uint32_t meta, uint2 seed, uint32_t rng_id, uint32_t episode, uint32_t* words,
                              KcRest& rest) {
  const uint32_t fam = meta & 0xFF;
  const int S = (int)((meta >> 8) & 0xFF), param = (int)((meta >> 16) & 0xFF);
  Layout L;
  L.fam = (int)fam;
  L.S = S;
  L.a = L.b = L.c = L.d = -1;
  L.colour = 0;
  L.kx = L.ky = -1;
  L.gx = S - 2;
  L.gy = S - 2;
  L.vmask = L.hmask = 0;
  L.vopen = L.hopen = 0;
  L.ob[0] = L.ob[1] = L.ob[2] = L.ob[3] = 0xFFFFFFFFu;
  L.kd[0] = L.kd[1] = L.kd[2] = 0u;
  if (fam == kFamKeyCorridor) {
    const KcLayout K = keycorridor_layout<kTogether>(S, param, seed, rng_id, episode, words, rest);
    L.a = K.rl;
    L.b = param;   // rows of rooms
    L.colour = K.colour;
    L.gx = K.gx;
    L.gy = K.gy;
    L.kx = K.kx;
    L.ky = K.ky;
    L.ax = K.ax;
    L.ay = K.ay;
    L.dir = K.dir;
    L.kd[0] = K.kd[0];
    L.kd[1] = K.kd[1];
    L.kd[2] = K.kd[2];
    return L;
  }
  if (fam == kFamDynObs) {
    // balls in order, ball b at the draw-b-th free interior cell other than
    // the agent's (1, 1): linear interior index c = draw + 1, moved past every
    // earlier ball at or before it, in ascending order of the balls
    L.ax = L.ay = 1;
    L.dir = 0;
    const uint32_t w = (uint32_t)(S - 2);
    uint4 blk[2] = {make_uint4(rng_id, episode, 0u, 0u), make_uint4(rng_id, episode, 1u, 0u)};
    philox10<2>(blk, seed);
    const uint4 w0 = blk[0], w1 = blk[1];
    uint32_t sorted[kMaxObst];
#pragma unroll
    for (int b = 0; b < kMaxObst; ++b) {
      sorted[b] = 0xFFFFu;
      if (b < param) {
        const uint32_t word = pick4(b < 4 ? w0 : w1, (uint32_t)(b & 3));
        uint32_t c = bounded(word, w * w - 2u - (uint32_t)b) + 1u;
#pragma unroll
        for (int j = 0; j < b; ++j) c += sorted[j] <= c ? 1u : 0u;
        uint32_t q, r;
        small_divmod(c, w, q, r);
        obst_set(L.ob, b, 1u + r, 1u + q);
#pragma unroll
        for (int j = 0; j < b; ++j) {   // insert c
          const uint32_t lo = min(sorted[j], c);
          c = max(sorted[j], c);
          sorted[j] = lo;
        }
        sorted[b] = c;
      }
    }
    return L;
  }
  if (fam == kFamGoToDoor) {
    // room w x h in the top-left corner, one closed door per wall (top x,
    // right y, bottom x, left y), four distinct colours by a partial
    // Fisher-Yates shuffle of the six, the mission the colour of door u(4),
    // the agent uniform over the room's interior; 13 words in draw order
    uint4 w[4];
#pragma unroll
    for (uint32_t b = 0; b < 4; ++b) w[b] = make_uint4(rng_id, episode, b, 0u);
    philox10<4>(w, seed);
    const uint4 w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
    const int rw = 5 + (int)bounded(w0.x, (uint32_t)(S - 4));
    const int rh = 5 + (int)bounded(w0.y, (uint32_t)(S - 4));
    L.kx = rw;
    L.ky = rh;
    L.gx = L.gy = -1;   // no goal square
    L.a = 1 + (int)bounded(w0.z, (uint32_t)(rw - 2));
    L.b = 1 + (int)bounded(w0.w, (uint32_t)(rh - 2));
    L.c = 1 + (int)bounded(w1.x, (uint32_t)(rw - 2));
    L.d = 1 + (int)bounded(w1.y, (uint32_t)(rh - 2));
    uint32_t col = 0x543210u;   // colour k at bits 4k..4k+3
    const uint32_t sw[4] = {w1.z, w1.w, w2.x, w2.y};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t r = (uint32_t)k + bounded(sw[k], (uint32_t)(6 - k));
      const uint32_t ck = (col >> (4 * k)) & 15u, cr = (col >> (4 * r)) & 15u;
      col = (col & ~((15u << (4 * k)) | (15u << (4 * r)))) | (cr << (4 * k)) | (ck << (4 * r));
    }
    L.colour = (int)(col & 0xFFFFu);
    const uint32_t target = bounded(w2.z, 4u);
    L.ob[0] = 0xFFFFFF00u | ((col >> (4 * target)) & 15u);
    uint32_t q, r;
    small_divmod(bounded(w2.w, (uint32_t)((rw - 2) * (rh - 2))), (uint32_t)(rw - 2), q, r);
    L.ax = 1 + (int)r;
    L.ay = 1 + (int)q;
    L.dir = (int)bounded(w3.x, 4u);
    return L;
  }
  if (fam >= kFamLavaGap) {
    L.ax = L.ay = 1;
    L.dir = 0;
    if (fam == kFamLavaGap) {
      const uint4 w0 = philox10(make_uint4(rng_id, episode, 0u, 0u), seed);
      L.a = 2 + (int)bounded(w0.x, (uint32_t)(S - 4));
      L.b = 1 + (int)bounded(w0.y, (uint32_t)(S - 2));
    } else if (fam == kFamCrossings) {
      const Rivers R = crossings_layout(S, param, seed, rng_id, episode, words);
      L.vmask = R.vmask;
      L.hmask = R.hmask;
      L.vopen = R.vopen;
      L.hopen = R.hopen;
    } else {
      L.gy = 1;
      L.a = param == 1 ? 2 : S - 2;
    }
    return L;
  }
  uint4 w[2] = {make_uint4(rng_id, episode, 0u, 0u), make_uint4(rng_id, episode, 1u, 0u)};
  philox10<2>(w, seed);
  const uint4 w0 = w[0], w1 = w[1];
  if (fam == kFamEmpty) {
    const int w = S - 2;
    const uint32_t k = bounded(w0.x, (uint32_t)(w * w - 1));   // interior minus the last (goal) cell
    uint32_t q, r;
    small_divmod(k, (uint32_t)w, q, r);
    L.ax = 1 + (int)r;
    L.ay = 1 + (int)q;
    L.dir = (int)bounded(w0.y, 4u);
  } else if (fam == kFamTwoRoom) {
    L.a = 2 + (int)bounded(w0.x, (uint32_t)(S - 4));
    L.b = 1 + (int)bounded(w0.y, (uint32_t)(S - 3));
    L.colour = (int)bounded(w0.z, 6u);
    const uint32_t lw = (uint32_t)(L.a - 1), n = lw * (uint32_t)(S - 2);
    const uint32_t kk = bounded(w0.w, n);
    uint32_t q, r;
    small_divmod(kk, lw, q, r);
    L.kx = 1 + (int)r;
    L.ky = 1 + (int)q;
    uint32_t ka = bounded(w1.x, n - 1u);
    ka += ka >= kk ? 1u : 0u;
    small_divmod(ka, lw, q, r);
    L.ax = 1 + (int)r;
    L.ay = 1 + (int)q;
    L.dir = (int)bounded(w1.y, 4u);
  } else {
    const int m = S / 2;
    L.a = 1 + (int)bounded(w0.x, (uint32_t)(m - 1));
    L.b = m + 1 + (int)bounded(w0.y, (uint32_t)(m - 1));
    L.c = 1 + (int)bounded(w0.z, (uint32_t)(m - 1));
    L.d = m + 1 + (int)bounded(w0.w, (uint32_t)(m - 1));
    const uint32_t nfree = (uint32_t)((S - 2) * (S - 2)) - (uint32_t)(2 * (S - 2) - 1) + 4u;
    const uint32_t kg = bounded(w1.x, nfree);
    fourrooms_cell(S, m, L.a, L.b, L.c, L.d, kg, L.gx, L.gy);
    uint32_t ka = bounded(w1.y, nfree - 1u);
    ka += ka >= kg ? 1u : 0u;
    fourrooms_cell(S, m, L.a, L.b, L.c, L.d, ka, L.ax, L.ay);
    L.dir = (int)bounded(w1.z, 4u);
  }
  return L;
}

__device__ __forceinline__ int bcast(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

__device__ __forceinline__ uint64_t bcast64(uint64_t v, int lane) {
  return (uint64_t)(uint32_t)bcast((int)(uint32_t)v, lane) | ((uint64_t)(uint32_t)bcast((int)(v >> 32), lane) << 32);
}

// Reward of Eq. (1) in the time-discounted form 1 - 0.9 * (t / T), t after
// the step, as three IEEE fp32 operations; reward_mode 1: unit reward.
__device__ __forceinline__ float goal_reward(int32_t t, int32_t T, int32_t mode) {
  if (mode == 1) return 1.0f;
  const float q = __fdiv_rn((float)t, (float)T);
  const float p = __fmul_rn(0.9f, q);
  return __fsub_rn(1.0f, p);
}

// the mission reported with every record: GoToDoor's target colour, else 0xFF
__device__ __forceinline__ uint32_t mission_of(uint32_t fam, uint32_t ob0) {
  return fam == kFamGoToDoor ? (ob0 & 0xFFu) : 0xFFu;
}

// All the data that the lanes of one wave exchange lives in LDS, whose
// operations a wave performs in issue order: a wavefront-scope fence (no wait
// instruction) plus a compiler barrier is enough to make one lane's LDS writes
// visible to the others' later reads.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The barrier of a workgroup of two waves that share LDS only: outstanding
// loads and stores of device memory are not waited for.
__device__ __forceinline__ void pair_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kAgent = 10;

// ---------------------------------------------------------------------------
// Cells as codes
// ---------------------------------------------------------------------------
// One byte per cell in LDS.  Bits 0-3 hold the type, bits 4-6 the colour and
// bit 7 is set on cells that block sight.  A door's state is in bits 7 and 0:
// open 0x04, closed 0x84, locked 0x85 (a key, type 5, never blocks sight);
// only doors have a state.  A word of four codes turns into the four cells'
// types, colours and states with byte-parallel integer operations
// (decode_cells), so neither the view nor the records need a table read per
// cell.  Whole-grid records draw the agent as type 10 with its heading in the
// colour bits.
constexpr uint32_t kCodeEmpty = kEmpty;
constexpr uint32_t kCodeWall = 0x80u | (kGrey << 4) | kWall;
constexpr uint32_t kCodeGoal = (kGreen << 4) | kGoal;
constexpr uint32_t kCodeLava = kLava;
constexpr uint32_t kCodeBall = (kBlue << 4) | kBall;
constexpr uint32_t kCodeWall4 = kCodeWall * 0x01010101u;

__device__ __forceinline__ uint32_t key_code(uint32_t colour) { return (colour << 4) | kKey; }
__device__ __forceinline__ uint32_t door_code(uint32_t colour, uint32_t state) {
  return (colour << 4) | kDoor | (state != kOpen ? 0x80u : 0u) | (state == kLocked ? 1u : 0u);
}

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}

// The cells of four codes: types, colours and states, one byte each.
// kAgents: type 10 carries its state (the heading) in the colour bits.
struct Cells4 {
  uint32_t type, colour, state;
};

__device__ __forceinline__ uint32_t types4(uint32_t w) {
  // bit 2 set where a door is closed or locked (blocks sight, type bit 2)
  const uint32_t shut = (w >> 5) & w & 0x04040404u;
  return w & 0x0F0F0F0Fu & ~(shut >> 2);
}

template <bool kAgents>
__device__ __forceinline__ Cells4 decode_cells(uint32_t w) {
  const uint32_t shut = ((w >> 5) & w & 0x04040404u) >> 2;
  Cells4 c;
  c.type = w & 0x0F0F0F0Fu & ~shut;
  c.colour = (w >> 4) & 0x07070707u;
  c.state = shut + (w & shut);
  if (kAgents) {
    const uint32_t a8 = (w << 2) & w & 0x08080808u;   // only type 10 has bits 3 and 1
    const uint32_t m = a8 - (a8 >> 3);
    c.state |= c.colour & m;
    c.colour &= ~m;
  }
  return c;
}

// the 12 triple bytes of four cells
__device__ __forceinline__ void interleave(const Cells4& c, uint32_t (&w)[3]) {
  const uint32_t a = perm(c.state, c.colour, 0x05010400u);   // C0 S0 C1 S1
  const uint32_t b = perm(c.colour, c.type, 0x07030602u);    // T2 C2 T3 C3
  w[0] = perm(a, c.type, 0x01050400u);
  w[1] = perm(b, a, 0x05040302u);
  w[2] = perm(b, c.state, 0x03070602u);
}

// codes of the four cells whose 12 triple bytes are w0, w1, w2; a state
// counts on doors only
__device__ __forceinline__ uint32_t encode_cells(uint32_t w0, uint32_t w1, uint32_t w2) {
  const uint32_t t = perm(w2, perm(w1, w0, 0x0C060300u), 0x05020100u) & 0x0F0F0F0Fu;
  const uint32_t c = perm(w2, perm(w1, w0, 0x0C070401u), 0x06020100u) & 0x07070707u;
  const uint32_t s = perm(w2, perm(w1, w0, 0x0C0C0502u), 0x07040100u);
  const uint32_t t1 = t >> 1, t2 = t >> 2;
  const uint32_t door = t2 & ~t & ~t1 & 0x01010101u;   // type 4
  const uint32_t wall = t1 & ~t2 & 0x01010101u;       // type 2
  const uint32_t s1 = s >> 1;
  const uint32_t shut = (s | s1) & door, locked = s1 & door;
  return t | (c << 4) | ((shut | wall) << 7) | locked;
}

// code of one triple (the carried object)
__device__ __forceinline__ uint32_t code_of(uint32_t tri) {
  return encode_cells(tri & 0xFFFFFFu, 0u, 0u) & 0xFFu;
}

// A view reaches at most 6 cells ahead and 3 to the side of an interior
// agent, i.e. at most 5 rows and 5 columns outside an S <= 32 grid: with
// row-major indexing that is within 5 * 32 + 5 = 165 bytes before or after
// the grid, read in whole words (8 bytes further at most).  Such cells are
// never visible (the wall border blocks sight), so only their addresses must
// stay inside the allocation; what they hold does not matter.
constexpr int kMargin = 192;

// dynamic LDS of a fused workgroup: the largest tile's grids plus both margins
__host__ __device__ inline size_t tile_lds_bytes(int32_t max_tile_cells) {
  const size_t b = 2 * (size_t)kMargin + (size_t)max_tile_cells;
  return (b + 15) & ~(size_t)15;
}

// The intervention of `intervene` on codes, as integer selects: every lane
// holds its own action, and comparisons combined as booleans would go through
// the scalar unit.  front is the code ahead, carry_code the held object's
// (kCodeEmpty: an empty hand); act >= 6 changes nothing.
struct CodeAction {
  uint32_t new_front;
  uint32_t ok;        // ~0 if the action succeeded (a walk, pickup, drop, toggle), else 0
  uint32_t goal;      // 1: walked onto the goal
  uint32_t lava;      // 1: walked into lava
};

__device__ __forceinline__ CodeAction act_on_code(uint32_t act, uint32_t carry_code, uint32_t front) {
  // kind of the cell: its type, + 16 if it blocks sight
  const uint32_t kind = (front & 15u) | ((front >> 3) & 16u);
  constexpr uint32_t kOpenKinds = (1u << kEmpty) | (1u << kDoor) | (1u << kGoal) | (1u << kLava);
  constexpr uint32_t kThings = (1u << kKey) | (1u << kBall) | (1u << kBox);
  constexpr uint32_t kFlips = (1u << kDoor) | (1u << (16 + kDoor)), kLockedKind = 1u << (16 + kKey);
  // a locked door's code less bit 7 is the code of its colour's key
  const uint32_t toggles = kFlips | (carry_code == (front & 0x7Fu) ? kLockedKind : 0u);
  const uint32_t things = carry_code == kCodeEmpty ? kThings : 0u;
  const uint32_t empties = carry_code == kCodeEmpty ? 0u : 1u << kEmpty;
  uint32_t kinds = act == kForward ? kOpenKinds : 0u;   // the kinds the action works on
  kinds = act == kPickup ? things : kinds;
  kinds = act == kDrop ? empties : kinds;
  kinds = act == kToggle ? toggles : kinds;
  CodeAction r;
  r.ok = (uint32_t)((int32_t)(kinds << (31u - kind)) >> 31);
  const uint32_t walked = act == kForward ? r.ok : 0u;
  r.goal = walked & (kind == kGoal ? 1u : 0u);
  r.lava = walked & (kind == kLava ? 1u : 0u);
  r.new_front = (front ^ 0x80u) & ~1u;   // open <-> closed, locked -> open
  r.new_front = act == kDrop ? carry_code : r.new_front;
  r.new_front = act == kPickup ? kCodeEmpty : r.new_front;
  return r;
}

// triple of a carried object's code (objects have no state)
__device__ __forceinline__ uint32_t carry_triple(uint32_t code) { return (code & 15u) | ((code << 4) & 0x700u); }

// whether the code is a door's (any state)
__device__ __forceinline__ bool is_door_code(uint32_t code) {
  return (code & 15u) == kDoor || (code & 0x8Fu) == (0x80u | kKey);
}

// The transition system of Dynamic-Obstacles (Table "systems"; Fig. 1) on codes:
// every ball, in list order, moves to a uniformly drawn empty cell of the 8
// around it that the agent does not occupy, or stays if there is none.  A
// ball's 3x3 block is three rows of two aligned words; an exact-match mask of
// the rows' bytes and three dot products give its 8 neighbours as bits (7-14,
// row-major, the ball's own cell skipped), and a table (kth_cell, by mask)
// the k-th free one.  The agent's cell is marked taken for the while.
// Entries off the interior (only a malformed state has them) do not move.
// One ball is a chain of some 25 dependent operations and two LDS round trips,
// and a wave runs it for its lane with the most balls: 65 536 envs of the four
// obstacle tasks 7.4 -> 6.5 us a step against eight byte reads and a search,
// 4.6 -> 4.3 without a branch for each of a ball's conditions (lanes whose ball
// is none of theirs look at the interior's first cell and move nothing).
constexpr int kMaskPatterns = 256;

// entry m: nibble k is the place of the k-th set bit of m among the 8
// neighbours, as (dx + 1) | (dy + 1) << 2
__device__ __forceinline__ void build_kth_table(uint32_t* table, int lane) {
#pragma unroll
  for (int j = 0; j < kMaskPatterns / kWave; ++j) {
    const uint32_t m = (uint32_t)(lane + j * kWave);
    uint32_t v = 0, k = 0;
#pragma unroll
    for (uint32_t i = 0; i < 8; ++i) {
      const uint32_t cell = i + (i >= 4u ? 1u : 0u);
      const bool set = (m >> i) & 1u;
      v |= set ? (cell % 3u | (cell / 3u) << 2) << (4u * k) : 0u;
      k += set ? 1u : 0u;
    }
    table[m] = v;
  }
}

// Bits of a ball's 8 neighbours among the mask of a 3x3 block (7-14), taken a
// row at a time: row r's three codes are the low bytes of w, empty cells'
// bits are added to mask.
template <int r>
__device__ __forceinline__ uint32_t empty_neighbours(uint32_t w, uint32_t mask) {
  // bytes equal to kCodeEmpty: zero after the exclusive or; bit 7 of each byte
  // of ((v & 0x7F) + 0x7F) | v is clear exactly there
  const uint32_t v = w ^ (kCodeEmpty * 0x01010101u);
  const uint32_t empty = ~(((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v) & 0x80808080u;
  constexpr uint32_t kPlaces[3] = {0x00040201u, 0x00100008u, 0x00804020u};
  return __builtin_amdgcn_udot4(empty, kPlaces[r], mask, false);
}

// The cell a ball at (bx, by) moves to: the free neighbour that `word` picks.
__device__ __forceinline__ void ball_target(uint32_t mask, uint32_t word, const uint32_t* kth, uint32_t bx,
                                            uint32_t by, uint32_t& nx, uint32_t& ny) {
  const uint32_t k = bounded(word, (uint32_t)__builtin_popcount(mask));
  const uint32_t v = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(kth) + (mask >> 5)) >> (4u * k);
  nx = bx + (v & 3u) - 1u;
  ny = by + ((v >> 2) & 3u) - 1u;
}

// at: byte offset of the env's grid in `lds`, pos: the agent's cell in it,
// most: the largest n of the wave
__device__ __forceinline__ void move_balls(uint8_t* lds, int at, int S, int n, int most, int pos, uint32_t (&ob)[4],
                                           uint2 seed, uint32_t rng_id, uint32_t call, const uint32_t* kth) {
  uint8_t under = lds[at + pos];
  lds[at + pos] = 0;
  const uint32_t inner = (uint32_t)(S - 2);
  uint4 blk[2] = {make_uint4(rng_id, call, 0u, 2u), make_uint4(rng_id, call, 1u, 2u)};
  philox10<2>(blk, seed);
#pragma unroll
  for (int b = 0; b < kMaxObst; ++b) {
    if (b < most) {
      const uint32_t word = pick4(blk[b >> 2], (uint32_t)(b & 3));
      const uint32_t xy = obst_at(ob, b);
      const uint32_t bx = xy & 0xFFu, by = xy >> 8;
      const bool ok = b < n && max(bx - 1u, by - 1u) < inner;
      const int cell = at + (ok ? (int)(by * (uint32_t)S + bx) : S + 1);
      auto row = [&](int r) {
        const int o = cell + (r - 1) * S - 1;
        const uint32_t* p = reinterpret_cast<const uint32_t*>(lds + (o & ~3));
        return __builtin_amdgcn_alignbyte(p[1], p[0], (uint32_t)o & 3u);
      };
      uint32_t mask = empty_neighbours<0>(row(0), 0u);
      mask = empty_neighbours<1>(row(1), mask);
      mask = empty_neighbours<2>(row(2), mask);
      mask = ok ? mask : 0u;
      uint32_t nx, ny;
      ball_target(mask, word, kth, bx, by, nx, ny);
      const bool from_agent = cell == at + pos;   // a malformed state's ball under the agent
      if (mask) {
        under = from_agent ? (uint8_t)kCodeEmpty : under;
        lds[cell] = from_agent ? (uint8_t)0 : (uint8_t)kCodeEmpty;
        lds[at + (int)(ny * (uint32_t)S + nx)] = (uint8_t)kCodeBall;
        obst_set(ob, b, nx, ny);
      }
    }
  }
  lds[at + pos] = under;
}

// ---------------------------------------------------------------------------
// The first-person view from the LDS codes.
//
// Whatever the heading, the view is a 7x7 square of the world, i.e. 7 grid
// rows of 7 consecutive bytes: three aligned words a row instead of 49 byte
// reads, which at random banks cost 14-20 cycles each.  The rows are loaded in
// the order of the view's rows (north, south) or columns (east, west); south
// and east views run backwards along a grid row, so their bytes are reversed
// by one permute a word; east and west views are then transposed (26
// permutes) and every lane picks its form.
//
// Sight blocked by a row's cells is bit 7 of their codes, gathered by dot
// products with powers of two.  Row masks are kept in a dual form: the 7
// column bits in bits 7-13 and the same bits reversed in bits 18-24.  One add
// then fills runs towards higher columns in the low field and towards lower
// columns in the high field (a carry out of either lands in an unused bit),
// and one bit reversal merges the two.  Per view row the visible cells are
// the seeds plus the see-through runs that touch a see-through seed, widened
// by one cell on each side; the next row's seeds are the three cells ahead of
// every visible see-through cell.  A row's 7 visibility bits become byte
// masks through a 128-entry table.
// ---------------------------------------------------------------------------
constexpr uint32_t kDual = 0x01FC3F80u;
constexpr uint32_t kDualCentre = (1u << 10) | (1u << 21);   // column 3
constexpr int kMaskEntries = 128;

// entry v: bytes 0-6 are 0xFF where bit 0-6 of v is set, byte 7 is 0
__device__ __forceinline__ void build_mask_table(uint2* table, int lane) {
#pragma unroll
  for (int k = 0; k < kMaskEntries / kWave; ++k) {
    const uint32_t v = (uint32_t)(lane + k * kWave);
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      lo |= ((v >> b) & 1u) ? 0xFFu << (8 * b) : 0u;
      hi |= (b < 3 && ((v >> (4 + b)) & 1u)) ? 0xFFu << (8 * b) : 0u;
    }
    table[v] = make_uint2(lo, hi);
  }
}

// transposes the 4x4 bytes of a, b, c, d (rows) into columns
__device__ __forceinline__ void transpose4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&t)[4]) {
  const uint32_t ab0 = perm(b, a, 0x05010400u), ab1 = perm(b, a, 0x07030602u);
  const uint32_t cd0 = perm(d, c, 0x05010400u), cd1 = perm(d, c, 0x07030602u);
  t[0] = perm(cd0, ab0, 0x05040100u);
  t[1] = perm(cd0, ab0, 0x07060302u);
  t[2] = perm(cd1, ab1, 0x05040100u);
  t[3] = perm(cd1, ab1, 0x07060302u);
}

// the first three bytes of each column of a, b, c (rows); byte 3 is c's next
__device__ __forceinline__ void transpose3(uint32_t a, uint32_t b, uint32_t c, uint32_t (&t)[4]) {
  const uint32_t ab0 = perm(b, a, 0x05010400u), ab1 = perm(b, a, 0x07030602u);
  t[0] = perm(c, ab0, 0x0C040100u);
  t[1] = perm(c, ab0, 0x0C050302u);
  t[2] = perm(c, ab1, 0x0C060100u);
  t[3] = perm(c, ab1, 0x0C070302u);
}

// See-through cells of a row (codes 0-3 and 4-6), dual form.
__device__ __forceinline__ uint32_t see_through(uint32_t lo, uint32_t hi) {
  const uint32_t o = __builtin_amdgcn_udot4(lo & 0x80808080u, 0x08040201u,
                                            __builtin_amdgcn_udot4(hi & 0x80808080u, 0x00402010u, 0u, false), false);
  return ~(o | __builtin_bitreverse32(o)) & kDual;
}

// One row of the flood, nearest first: from the row's lit cells on through the
// see-through ones, then to the cells around them and the next row's.  Bits
// beside the fields may be set in both results.
__device__ __forceinline__ uint32_t see_row(uint32_t p, uint32_t& seeds) {
  const uint32_t g = seeds & p;
  const uint32_t fill = (((p + g) ^ p) | g) & p;
  const uint32_t wide = fill | (fill << 1) | (fill >> 1);
  const uint32_t next = wide | __builtin_bitreverse32(wide);
  const uint32_t vis = seeds | next;
  seeds = next;
  return vis;
}

// Columns inside the grid, for a view from (x, y), and in `ahead` its rows
// beyond the agent's.
__device__ __forceinline__ uint32_t columns_inside(int S, int x, int y, int dir, int& ahead) {
  const int e = S - 1 - x, s = S - 1 - y;   // cells to the east and south
  ahead = dir == 0 ? e : (dir == 1 ? s : (dir == 2 ? x : y));
  const int left = dir == 0 ? y : (dir == 1 ? e : (dir == 2 ? s : x));
  const int right = dir == 0 ? s : (dir == 1 ? x : (dir == 2 ? y : e));
  return (0x7Fu << max(3 - left, 0)) & (0x7Fu >> max(3 - right, 0)) & 0x7Fu;
}

// The lane's view as 13 words of codes f[0..12], cell j * 7 + i (view row j,
// column i) at byte j * 7 + i, unseen cells and the bytes past the 49th 0.
// at: the agent's cell's byte offset in `lds` (its grid's rows are S bytes
// apart).  check (wave-uniform): cells outside the grid are taken as walls on
// lanes with `edge` set, for the rare step whose view can leave the grid,
// through a door on the outer ring that the step itself opened (GoToDoor
// rooms use the grid's border as walls).
//
// view_from_rows: the same from the rows' codes, row r's cells 0-3 and 4-6 in
// lo[r] and hi[r], rows in the order described above, bytes ascending.
// patch: ~0 where the cell ahead of the agent shows `front` instead.
__device__ __forceinline__ void view_from_rows(uint32_t (&lo)[7], uint32_t (&hi)[7], int S, int x, int y, int dir,
                                               uint32_t carry_code, uint32_t patch, uint32_t front,
                                               const uint2* masks, bool check, bool edge, uint32_t (&f)[13]);

template <class Loaded>
__device__ __forceinline__ void view_codes(const uint8_t* lds, int at, int S, int x, int y, int dir,
                                           uint32_t carry_code, const uint2* masks, bool check, bool edge,
                                           uint32_t (&f)[13], Loaded loaded) {
  const bool vert = (dir & 1) != 0;            // south, north
  const int step = (dir == 1 || dir == 2) ? -S : S;   // south, west: rows loaded bottom up
  int idx = at - (vert ? 3 : (dir == 0 ? 0 : 6)) - (vert ? 6 : 3) * step;
  uint32_t lo[kView], hi[kView], raw[kView][3];
  int at_row = idx;
#pragma unroll
  for (int r = 0; r < kView; ++r) {
    const uint32_t* p = reinterpret_cast<const uint32_t*>(lds + (at_row & ~3));
#pragma unroll
    for (int k = 0; k < 3; ++k) raw[r][k] = p[k];
    at_row += step;
  }
  __builtin_amdgcn_sched_barrier(0);   // all reads in flight before the first is used
  loaded();
#pragma unroll
  for (int r = 0; r < kView; ++r) {
    const uint32_t sh = (uint32_t)idx & 3u;
    lo[r] = __builtin_amdgcn_alignbyte(raw[r][1], raw[r][0], sh);
    hi[r] = __builtin_amdgcn_alignbyte(raw[r][2], raw[r][1], sh);
    idx += step;
  }
  view_from_rows(lo, hi, S, x, y, dir, carry_code, 0u, 0u, masks, check, edge, f);
}

__device__ __forceinline__ void view_from_rows(uint32_t (&lo)[7], uint32_t (&hi)[7], int S, int x, int y, int dir,
                                               uint32_t carry_code, uint32_t patch, uint32_t front,
                                               const uint2* masks, bool check, bool edge, uint32_t (&f)[13]) {
  const bool vert = (dir & 1) != 0;
  const bool flip = dir < 2;                   // south, east: the view runs backwards along a row
  const uint32_t sel_lo = flip ? 0x03040506u : 0x03020100u;
  const uint32_t sel_hi = flip ? 0x0C000102u : 0x0C060504u;
#pragma unroll
  for (int r = 0; r < kView; ++r) {
    const uint32_t l = lo[r], h = hi[r];
    lo[r] = perm(h, l, sel_lo);
    hi[r] = perm(h, l, sel_hi);
  }
  {
    uint32_t a[4], b[4], c[4], d[4];
    transpose4(lo[0], lo[1], lo[2], lo[3], a);
    transpose4(hi[0], hi[1], hi[2], hi[3], b);
    transpose3(lo[4], lo[5], lo[6], c);
    transpose3(hi[4], hi[5], hi[6], d);
#pragma unroll
    for (int r = 0; r < kView; ++r) {
      lo[r] = vert ? lo[r] : (r < 4 ? a[r & 3] : b[r & 3]);
      hi[r] = vert ? hi[r] : (r < 4 ? c[r & 3] : d[r & 3]);
    }
  }
  lo[5] = (lo[5] & ~(patch & 0xFF000000u)) | (patch & (front << 24));
  if (check) {
    int ahead;
    const uint2 m = masks[columns_inside(S, x, y, dir, ahead)];
#pragma unroll
    for (int r = 0; r < kView; ++r) {
      const bool in = 6 - r <= ahead;
      const uint32_t ml = edge ? (in ? m.x : 0u) : ~0u, mh = edge ? (in ? m.y : 0u) : ~0u;
      lo[r] = (lo[r] & ml) | (kCodeWall4 & ~ml);
      hi[r] = (hi[r] & mh) | (kCodeWall4 & ~mh);
    }
  }
  uint32_t seeds = kDualCentre;
#pragma unroll
  for (int j = kView - 1; j >= 0; --j) {
    const uint32_t vis = see_row(see_through(lo[j], hi[j]), seeds);
    const uint2 m = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint8_t*>(masks) + ((vis >> 4) & 0x3F8u));
    lo[j] &= m.x;
    hi[j] &= m.y;
  }
  lo[6] = (lo[6] & 0x00FFFFFFu) | (carry_code << 24);   // the agent's cell shows what it carries
  f[0] = lo[0];
  f[1] = perm(lo[1], hi[0], 0x04020100u);
  f[2] = perm(hi[1], lo[1], 0x04030201u);
  f[3] = perm(lo[2], hi[1], 0x05040201u);
  f[4] = perm(hi[2], lo[2], 0x05040302u);
  f[5] = perm(lo[3], hi[2], 0x06050402u);
  f[6] = perm(hi[3], lo[3], 0x06050403u);
  f[7] = lo[4];
  f[8] = perm(lo[5], hi[4], 0x04020100u);
  f[9] = perm(hi[5], lo[5], 0x04030201u);
  f[10] = perm(lo[6], hi[5], 0x05040201u);
  f[11] = perm(hi[6], lo[6], 0x05040302u);
  f[12] = (hi[6] >> 16) & 0xFFu;
}

// The views of the first n <= 8 lanes' envs, one after another at `stage`: lane
// 8 i + r computes row r of env i (r = 7: row 6 again, not stored).  A view of
// its own per lane costs some 250 instructions however few lanes have one;
// here each handles seven cells, and the flood, which needs the see-through
// cells of all rows, receives them from the lanes of its group.
template <class Loaded>
__device__ __forceinline__ void views_of_few(const uint8_t* lds, uint32_t* stage, uint2 pose, int lane, int n,
                                             const uint2* masks, bool check, Loaded loaded) {
  const uint32_t r = min((uint32_t)lane & 7u, 6u);
  const int S = (int)((pose.y >> 16) & 255u), dir = (int)((pose.x >> 18) & 3u);
  const bool vert = (dir & 1) != 0;
  const int fwd = vert ? S : 1, side = vert ? 1 : S;
  const int ahead_by = dir >= 2 ? -fwd : fwd;                // one cell ahead
  const int step = dir == 1 || dir == 2 ? -side : side;      // one cell to the right
  const uint8_t* p = lds + ((int)(pose.x & 0x3FFFFu) + (6 - (int)r) * ahead_by - 3 * step);
  uint32_t c[kView];
#pragma unroll
  for (int k = 0; k < kView; ++k) {
    c[k] = *p;
    p += step;
  }
  __builtin_amdgcn_sched_barrier(0);
  loaded();
  uint32_t lo = c[0] | (c[1] << 8) | (c[2] << 16) | (c[3] << 24), hi = c[4] | (c[5] << 8) | (c[6] << 16);
  if (check) {
    int ahead;
    const uint2 m = masks[columns_inside(S, (int)(pose.y & 255u), (int)((pose.y >> 8) & 255u), dir, ahead)];
    const bool edge = ((pose.x >> 20) & 1u) != 0u, in = 6 - (int)r <= ahead;
    const uint32_t ml = edge ? (in ? m.x : 0u) : ~0u, mh = edge ? (in ? m.y : 0u) : ~0u;
    lo = (lo & ml) | (kCodeWall4 & ~ml);
    hi = (hi & mh) | (kCodeWall4 & ~mh);
  }
  const int see = (int)see_through(lo, hi);
  uint32_t rows[kView];
  rows[0] = (uint32_t)__builtin_amdgcn_ds_swizzle(see, 0x18 | 0 << 5);
  rows[1] = (uint32_t)__builtin_amdgcn_ds_swizzle(see, 0x18 | 1 << 5);
  rows[2] = (uint32_t)__builtin_amdgcn_ds_swizzle(see, 0x18 | 2 << 5);
  rows[3] = (uint32_t)__builtin_amdgcn_ds_swizzle(see, 0x18 | 3 << 5);
  rows[4] = (uint32_t)__builtin_amdgcn_ds_swizzle(see, 0x18 | 4 << 5);
  rows[5] = (uint32_t)__builtin_amdgcn_ds_swizzle(see, 0x18 | 5 << 5);
  rows[6] = (uint32_t)__builtin_amdgcn_ds_swizzle(see, 0x18 | 6 << 5);
  uint32_t seeds = kDualCentre, vis = 0;
#pragma unroll
  for (int j = kView - 1; j >= 0; --j) {
    const uint32_t v = see_row(rows[j], seeds);
    vis = r == (uint32_t)j ? v : vis;
  }
  const uint2 m = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint8_t*>(masks) + ((vis >> 4) & 0x3F8u));
  lo &= m.x;
  hi &= m.y;
  lo = r == 6 ? (lo & 0x00FFFFFFu) | (pose.y & 0xFF000000u) : lo;   // the agent's cell shows what it carries
  if ((lane & 7) < kView && (lane >> 3) < n) {
    uint8_t* q = reinterpret_cast<uint8_t*>(stage) + kCatBytes * (lane >> 3) + kView * (lane & 7);
#pragma unroll
    for (int k = 0; k < kView; ++k) q[k] = (uint8_t)(k < 4 ? lo >> (8 * k) : hi >> (8 * (k - 4)));
  }
}

// Writes the first n lanes' views (49 codes each) one after another at
// `stage`.  Lane l's start 49 l mod 4 = l mod 4 bytes into a word, which then
// holds the last cells of lane l - 1 as well: that word is the higher lane's,
// with the lower one's last word received by a lane shift.
__device__ __forceinline__ void store_view(uint32_t* stage, const uint32_t (&f)[13], int lane, int n) {
  const uint32_t k = (uint32_t)lane & 3u;
  const uint32_t sel = 0x07060504u - k * 0x01010101u;
  uint32_t g[13];
  g[0] = perm(f[0], 0u, sel);
#pragma unroll
  for (int q = 1; q < 13; ++q) g[q] = perm(f[q], f[q - 1], sel);
  const uint32_t tail = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)g[12], 0x138, 0xF, 0xF, true);   // lane - 1's
  g[0] |= k != 0 ? tail : 0u;
  if (lane < n) {
    uint32_t* p = stage + ((uint32_t)(kCatBytes * lane) >> 2);
#pragma unroll
    for (int q = 0; q < 12; ++q) p[q] = g[q];
    if (k == 3 || lane == n - 1) p[12] = g[12];
  }
}

// ---------------------------------------------------------------------------
// Records and grids from codes.
//
// n consecutive cells at `cells` (LDS) leave as 3 n triple bytes (or n type
// bytes, kCat) at dst, any alignment.  A wave pass takes 256 cells, four a
// lane: one word read, a dozen byte-parallel operations and one 12-byte store,
// 768 contiguous bytes a pass.  Passes start c0 cells in, where 3 c0 bytes
// reach dst's next 64-byte boundary (3 * 43 = 1 mod 64), so every pass covers
// whole 64-byte units of HBM (which writes a partial one as a
// read-modify-write); the c0 cells before are the last of an extra first
// pass.  Stores of a constant in this pattern reach 5.2 TB/s, 16-byte stores
// of the same bytes 5.1, and passes off the boundary 3.9-4.7, at 262 144
// tiles' rows of 9408 bytes.
// Groups cut by either end store their bytes one by one.  Reads reach at
// most 4 bytes before the cells and 8 past them.
// ---------------------------------------------------------------------------
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef u32x3 u32x3_any __attribute__((aligned(1)));
typedef u32x4 u32x4_any __attribute__((aligned(1)));

// first cell of pass 0 (in (-64, 0]) for an output at dst
template <bool kCat>
__device__ __forceinline__ int first_cell(const uint8_t* dst) {
  const uint32_t d = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)reinterpret_cast<uintptr_t>(dst));
  const int c0 = (int)((0u - d) * (kCat ? 1u : 43u)) & 63;
  return c0 ? c0 - 64 : 0;
}

// word of codes at cell c (kShift: c is not a multiple of 4, c mod 4 = sh)
template <bool kShift>
__device__ __forceinline__ uint32_t load_cells(const uint8_t* cells, int c, uint32_t sh) {
  const uint32_t* p = reinterpret_cast<const uint32_t*>(cells + (c & ~3));
  return kShift ? __builtin_amdgcn_alignbyte(p[1], p[0], sh) : p[0];
}

template <bool kAgents, bool kNT>
__device__ __forceinline__ void store_cells(uint8_t* dst, uint32_t w) {
  uint32_t o[3];
  interleave(decode_cells<kAgents>(w), o);
  const u32x3 v = {o[0], o[1], o[2]};
  if (kNT) __builtin_nontemporal_store(v, reinterpret_cast<u32x3_any*>(dst));
  else *reinterpret_cast<u32x3_any*>(dst) = v;
}

// the whole groups of the pass from cell p on that lie inside [0, n)
template <bool kAgents, bool kShift, bool kNT>
__device__ __forceinline__ void emit_some(uint8_t* dst, const uint8_t* cells, int n, int p, uint32_t sh, int lane,
                                          bool keep = true) {
  const int c = p + 4 * lane;
  const uint32_t w = load_cells<kShift>(cells, min(max(c, 0), n), sh);
  if (keep && c >= 0 && c + 4 <= n) store_cells<kAgents, kNT>(dst + 3 * c, w);
}

// the triples (kCat: types) of the first `head` and the last `tail` cells, at
// most 15 each, a byte per lane
template <bool kAgents, bool kCat>
__device__ __forceinline__ void emit_ends(uint8_t* dst, const uint8_t* cells, int n, int head, int tail, int lane) {
  constexpr int kPer = kCat ? 1 : 3;
  const int half = lane >> 5, b = lane & 31, cell = kCat ? b : b / 3;
  const int at = half ? n - tail + cell : cell;
  if (b < kPer * (half ? tail : head) && at < n) {
    const Cells4 v = decode_cells<kAgents>(cells[at]);
    const int ch = kCat ? 0 : b - 3 * cell;
    dst[kPer * at + ch] = (uint8_t)(ch == 0 ? v.type : (ch == 1 ? v.colour : v.state));
  }
}

// kDepth passes from cell p on, their LDS reads issued together.  kWhole: all
// inside [0, n), so that no group needs a bounds test.
template <bool kAgents, bool kShift, int kDepth, bool kWhole>
__device__ __forceinline__ void emit_block(uint8_t* dst, const uint8_t* cells, int n, int p, uint32_t sh, int lane) {
  constexpr int kPass = 4 * kWave;
  uint32_t w[kDepth], o[kDepth][3];
  const int c0 = p + 4 * lane;
#pragma unroll
  for (int u = 0; u < kDepth; ++u) {
    const int c = c0 + u * kPass;
    w[u] = load_cells<kShift>(cells, kWhole ? c : min(max(c, 0), n), sh);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < kDepth; ++u) {
    interleave(decode_cells<kAgents>(w[u]), o[u]);
    // not to be moved under the store's bounds test
    if (!kWhole) asm volatile("" : "+v"(o[u][0]), "+v"(o[u][1]), "+v"(o[u][2]));
  }
#pragma unroll
  for (int u = 0; u < kDepth; ++u) {
    const int c = c0 + u * kPass;
    const u32x3 q = {o[u][0], o[u][1], o[u][2]};
    if (kWhole || (c >= 0 && c + 4 <= n))
      __builtin_nontemporal_store(q, reinterpret_cast<u32x3_any*>(dst + 3 * c));
  }
}

template <bool kAgents, bool kShift>
__device__ __forceinline__ void emit_passes(uint8_t* dst, const uint8_t* cells, int n, int start, int lane) {
  constexpr int kPass = 4 * kWave;
  constexpr int kDeep = 4;
  const uint32_t sh = (uint32_t)start & 3u;
  int p = start;
  if (p < 0 && n > kDeep * kPass) {
    emit_block<kAgents, kShift, 1, false>(dst, cells, n, p, sh, lane);
    p += kPass;
  }
  for (; p + kPass < n; p += kDeep * kPass) {
    if (p >= 0 && p + kDeep * kPass <= n) emit_block<kAgents, kShift, kDeep, true>(dst, cells, n, p, sh, lane);
    else emit_block<kAgents, kShift, kDeep, false>(dst, cells, n, p, sh, lane);
  }
  if (p < n) emit_block<kAgents, kShift, 1, false>(dst, cells, n, p, sh, lane);
  const int head = start & 3, tail = (n - start) & 3;
  if (head | tail) emit_ends<kAgents, false>(dst, cells, n, min(head, n), tail, lane);
}

template <bool kAgents>
__device__ __forceinline__ void emit_triples(uint8_t* dst, const uint8_t* cells, int n, int lane) {
  const int start = first_cell<false>(dst);
  if (start & 3) emit_passes<kAgents, true>(dst, cells, n, start, lane);
  else emit_passes<kAgents, false>(dst, cells, n, start, lane);
}

// emit_triples for the 3136 cells of 64 views at a 64-byte boundary, every pass
// on a 128-byte one, so that no line is shared by two passes: three whole blocks,
// and the 64 cells ahead of them or behind.  For single waves whose rows all
// start so: 262 144 mixed envs in single-wave workgroups, 1024 steps 8.69 -> 8.30
// ms, all families 256 steps 3.69 -> 3.52.  Pairs of waves lose by it (65 536
// TwoRoom 8x8, 128 steps 241 -> 254 us), and so does a batch of which only some
// rows do (100 000 Empty 8x8, 64 steps 214 -> 220: the step loop then runs through
// both forms).
__device__ __forceinline__ void emit_64_views(uint8_t* dst, const uint8_t* cells, int lane) {
  constexpr int kPass = 4 * kWave, kDeep = 4, kWhole = 3 * kDeep * kPass, kCells = kWave * kCatBytes;
  static_assert(kCells == kWhole + 64, "three whole blocks and 64 cells");
  const int first = __builtin_amdgcn_readfirstlane((int)(uint32_t)reinterpret_cast<uintptr_t>(dst)) & 64;
  if (first) emit_block<false, false, 1, false>(dst, cells, kCells, first - kPass, 0u, lane);
#pragma unroll
  for (int p = 0; p < kWhole; p += kDeep * kPass)
    emit_block<false, false, kDeep, true>(dst, cells, kCells, first + p, 0u, lane);
  if (!first) emit_block<false, false, 1, false>(dst, cells, kCells, kWhole, 0u, lane);
}

// types alone: 16 cells a lane and store
__device__ __forceinline__ void emit_types(uint8_t* dst, const uint8_t* cells, int n, int lane) {
  const int start = first_cell<true>(dst);
  const uint32_t sh = (uint32_t)start & 3u;
  for (int p = start; p < n; p += 16 * kWave) {
    const int c = p + 16 * lane;
    const uint32_t* q = reinterpret_cast<const uint32_t*>(cells + (min(max(c, 0), n) & ~3));
    uint32_t w[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) w[k] = q[k];
    u32x4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = types4(__builtin_amdgcn_alignbyte(w[k + 1], w[k], sh));
    if (c >= 0 && c + 16 <= n) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_any*>(dst + c));
  }
  const int head = start & 15, tail = (n - start) & 15;
  if (head | tail) emit_ends<true, true>(dst, cells, n, min(head, n), tail, lane);
}

// Write-back of the grids that changed in a launch (the lanes with `dirty`
// set; every other env's grid in HBM still holds the bytes staged in, so
// writing it again would change nothing).  The dirty lanes mark the blocks
// of 64 cells (192 bytes, on 64-byte boundaries of the output) that their
// grids touch, in a bitmap in `marks` (LDS), and the passes of emit_triples
// store the marked blocks only: a block's other cells belong to neighbouring
// envs and are rewritten with their current values, which equal what HBM
// holds.  Ordinary stores, since the next launch reads the grids again.
__device__ __forceinline__ void emit_dirty_grids(uint8_t* dst, int n_cells, bool dirty, int my_off, int my_cells,
                                                 const uint8_t* codes, uint32_t* marks, int lane) {
  if (!__ballot(dirty)) return;
  const int start = first_cell<false>(dst);
  const int blocks = (n_cells - start + 63) >> 6;
  for (int w = lane; w < (blocks + 31) >> 5; w += kWave) marks[w] = 0u;
  wave_sync();
  if (dirty && my_cells > 0) {
    const int b0 = (my_off - start) >> 6, b1 = (my_off + my_cells - 1 - start) >> 6;   // at most 17 blocks
    for (int w = b0 >> 5; w <= b1 >> 5; ++w) {
      const int lo = max(b0 - 32 * w, 0), hi = min(b1 - 32 * w, 31);
      atomicOr(&marks[w], (~0u >> (31 - (hi - lo))) << lo);
    }
  }
  wave_sync();
  const uint32_t sh = (uint32_t)start & 3u;
  for (int p = 0; 4 * p < blocks; ++p) {   // a pass: four blocks
    const uint32_t m = (marks[p >> 3] >> (4 * (p & 7))) & 15u;
    if (__builtin_amdgcn_readfirstlane((int)m))
      emit_some<false, true, false>(dst, codes, n_cells, start + 4 * kWave * p, sh, lane, (m >> (lane >> 4)) & 1u);
  }
  const int head = start & 3, tail = (n_cells - start) & 3;
  if (head | tail) emit_ends<false, false>(dst, codes, n_cells, min(head, n_cells), tail, lane);
}

// Stages a tile's grids, the 3 * n_cells bytes at src (any alignment), into
// LDS as codes.  Lane u converts cells [16u, 16u + 16), i.e. the 48 bytes
// at src + 48u; 48 being a multiple of 16, every such run starts at the
// same offset r = src mod 16 in its first aligned 16-byte chunk, so a run is
// four aligned chunk loads and one realignment by the wave-uniform r (the
// conversion is instantiated per r / 4, so the realignment needs no
// selects).  A chunk past the block's last one is read as that last chunk
// (so every load lies in the block's own memory pages); the codes of the at
// most 15 cells past n_cells land in the trailing LDS margin.  The lane's
// next run is loaded before its current run is converted, so the wave's
// reads stay in flight while it converts.
struct GridRun {
  u32x4 q[4];
};

__device__ __forceinline__ GridRun load_run(uintptr_t a, uintptr_t last) {
  GridRun g;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uintptr_t c = a + 16 * (uintptr_t)k;
    g.q[k] = *(const __attribute__((address_space(1))) u32x4*)(c < last ? c : last);
  }
  return g;
}

template <int kRW>
__device__ __forceinline__ void convert_run(const GridRun& g, uint32_t rb, uint8_t* dst) {
  uint32_t w[16];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int c = 0; c < 4; ++c) w[4 * k + c] = g.q[k][c];
  // bytes r .. r + 47 of the chunks as 12 words (r = 4 kRW + rb)
  uint32_t b[12];
#pragma unroll
  for (int i = 0; i < 12; ++i)
    b[i] = i + kRW + 1 < 16 ? __builtin_amdgcn_alignbyte(w[i + kRW + 1], w[i + kRW], rb) : w[i + kRW] >> (8 * rb);
  u32x4 out;
#pragma unroll
  for (int k = 0; k < 4; ++k) out[k] = encode_cells(b[3 * k], b[3 * k + 1], b[3 * k + 2]);
  *reinterpret_cast<u32x4*>(dst) = out;
}

template <int kRW>
__device__ __forceinline__ void stage_in_runs(uintptr_t a0, uintptr_t last, uint32_t rb, int units,
                                              uint8_t* codes, int lane) {
  int u = lane;
  if (u >= units) return;
  GridRun cur = load_run(a0 + 48 * (uintptr_t)u, last);
  while (true) {
    const int nu = u + kWave;
    const bool more = nu < units;
    GridRun nxt;
    if (more) nxt = load_run(a0 + 48 * (uintptr_t)nu, last);
    convert_run<kRW>(cur, rb, codes + 16 * u);
    if (!more) break;
    cur = nxt;
    u = nu;
  }
}

__device__ __forceinline__ void stage_in_codes(const uint8_t* src, int n_cells, uint8_t* codes, int lane) {
  const uintptr_t s0 = reinterpret_cast<uintptr_t>(src);
  const uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane((int)(s0 & 15u));
  const uintptr_t end = s0 + 3 * (uintptr_t)(uint32_t)n_cells;
  const uintptr_t a0 = s0 - r, last = (end - 1) & ~(uintptr_t)15;
  const int units = (n_cells + 15) >> 4;
  switch (r >> 2) {
    case 0: stage_in_runs<0>(a0, last, r & 3u, units, codes, lane); break;
    case 1: stage_in_runs<1>(a0, last, r & 3u, units, codes, lane); break;
    case 2: stage_in_runs<2>(a0, last, r & 3u, units, codes, lane); break;
    default: stage_in_runs<3>(a0, last, r & 3u, units, codes, lane); break;
  }
}

// ---------------------------------------------------------------------------
// Resets.
//
// A lane keeps the layout of its next episode (Next), which depends on its
// seed, id and episode counter alone.  When a lane resets that has used its
// Next up, the layouts of all the wave's lanes of that family without one
// are drawn together: drawing one costs as much as drawing 64, so a draw
// serves about ten resets of a wave of one family, instead of one step's.
// The grid is then filled in two parts: a base of walls, lines of walls or
// lava, and empty cells, described by a few bit masks that the whole wave
// broadcasts and fills, 64 cells a pass; and the few single cells (goal,
// doors, key, openings, balls), which every resetting lane writes itself,
// all at once.  Per step of 64 steps a launch, 65 536 envs: GoToDoor 7.6 -> 5.1
// us, Dynamic-Obstacles (types alone) 9.3 -> 7.3, lava 5.0 -> 3.9.
// ---------------------------------------------------------------------------
struct Next {
  uint32_t pose;     // ax, ay (5 bits each), dir (2), gx, gy, kx, ky (5 each)
  uint32_t shape;    // xl, yl (bytes): cells at x >= xl or y >= yl are wall; colour(s) << 16
  uint32_t cols, rows, span;   // line cells: x in cols, or y in rows and x in span (bit masks)
  uint32_t u[4];     // openings, doors, balls: see fill_grids
};

__device__ __forceinline__ Next pack_layout(const Layout& L) {
  const uint32_t S = (uint32_t)L.S;
  Next n;
  n.pose = (uint32_t)L.ax | ((uint32_t)L.ay << 5) | ((uint32_t)L.dir << 10) | (((uint32_t)L.gx & 31u) << 12) |
           (((uint32_t)L.gy & 31u) << 17) | (((uint32_t)L.kx & 31u) << 22) | ((uint32_t)L.ky << 27);
  uint32_t xl = S - 1u, yl = S - 1u;
  n.cols = n.rows = 0u;
  n.span = ~0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) n.u[i] = 0u;
  const uint32_t abcd = ((uint32_t)L.a & 255u) | (((uint32_t)L.b & 255u) << 8) | (((uint32_t)L.c & 255u) << 16) |
                        ((uint32_t)L.d << 24);
  if (L.fam == kFamTwoRoom || L.fam == kFamLavaGap) {
    n.cols = 1u << L.a;
    n.u[0] = abcd;
  } else if (L.fam == kFamFourRooms) {
    n.cols = n.rows = 1u << (S >> 1);
    n.u[0] = abcd;
  } else if (L.fam == kFamCrossings) {
    n.cols = L.vmask;
    n.rows = L.hmask;
    n.u[0] = (uint32_t)L.vopen;
    n.u[1] = (uint32_t)(L.vopen >> 32);
    n.u[2] = (uint32_t)L.hopen;
    n.u[3] = (uint32_t)(L.hopen >> 32);
  } else if (L.fam == kFamDistShift) {
    n.rows = 2u | (1u << L.a);
    n.span = (~0u << 3) & (~0u >> (34u - S));   // x = 3 .. S - 3
  } else if (L.fam == kFamDynObs) {
#pragma unroll
    for (int i = 0; i < 4; ++i) n.u[i] = L.ob[i];
  } else if (L.fam == kFamGoToDoor) {
    xl = (uint32_t)L.kx - 1u;
    yl = (uint32_t)L.ky - 1u;
    n.u[0] = abcd;
    n.u[1] = L.ob[0];
  } else if (L.fam == kFamKeyCorridor) {
    const uint32_t st = (S - 1u) / 3u;
    n.cols = (1u << st) | (1u << (2u * st));
    n.rows = (1u << st) | (1u << (2u * st));
    n.span = ~(((1u << (st - 1u)) - 1u) << (st + 1u));   // all but the hallway
    yl = (uint32_t)L.b * st;
#pragma unroll
    for (int i = 0; i < 3; ++i) n.u[i] = L.kd[i];
    n.u[3] = (uint32_t)L.a;
  }
  n.shape = xl | (yl << 8) | ((uint32_t)L.colour << 16);
  return n;
}

// The layout of (seed, id, episode) of every active lane of family f, which
// is uniform across the wave.
template <uint32_t F, bool kTogether>
__device__ __forceinline__ Next draw_family(uint32_t meta, uint2 seed, uint32_t rng_id, uint32_t episode,
                                            uint32_t* words, KcRest& rest) {
  return pack_layout(make_layout<kTogether>((meta & ~255u) | F, seed, rng_id, episode, words, rest));
}

template <bool kTogether>
__device__ __forceinline__ Next draw_layout(uint32_t f, uint32_t meta, uint2 seed, uint32_t rng_id,
                                            uint32_t episode, uint32_t* words, KcRest& rest) {
  switch (f) {
    case kFamEmpty: return draw_family<kFamEmpty, kTogether>(meta, seed, rng_id, episode, words, rest);
    case kFamTwoRoom: return draw_family<kFamTwoRoom, kTogether>(meta, seed, rng_id, episode, words, rest);
    case kFamFourRooms: return draw_family<kFamFourRooms, kTogether>(meta, seed, rng_id, episode, words, rest);
    case kFamLavaGap: return draw_family<kFamLavaGap, kTogether>(meta, seed, rng_id, episode, words, rest);
    case kFamCrossings: return draw_family<kFamCrossings, kTogether>(meta, seed, rng_id, episode, words, rest);
    case kFamDistShift: return draw_family<kFamDistShift, kTogether>(meta, seed, rng_id, episode, words, rest);
    case kFamDynObs: return draw_family<kFamDynObs, kTogether>(meta, seed, rng_id, episode, words, rest);
    case kFamGoToDoor: return draw_family<kFamGoToDoor, kTogether>(meta, seed, rng_id, episode, words, rest);
    default: return draw_family<kFamKeyCorridor, kTogether>(meta, seed, rng_id, episode, words, rest);
  }
}

// Steps a launch must have left for KeyCorridor layouts to be drawn ahead, for
// all of a wave's lanes instead of those that reset.  A KeyCorridor resets
// every few hundred steps and its draws vary, so that a wave waits for the
// longest of up to 64: drawn ahead they pay from 16 steps on.  us, ahead from 2 / 8
// / 16 / 32 steps, KeyCorridor: 65 536 envs, 2 steps 43.7 / 22.9 / 19.6 / 21.7, 8
// steps 61.8 / 58.7 / 42.8 / 42.5, 64 steps 174 / 173 / 172 / 173 (never: 202);
// 262 144 envs, 2 steps 70 / 49 / 47 / 48.  The other families draw ahead from two
// steps on (Crossings, 65 536 envs, 8 steps 40.6 / 45.4 / 50.5 / 51.0; GoToDoor 41.5
// / 43.5 / 44.7 / 44.7), and kernels for batches without KeyCorridor leave the
// rule out: in their step loops it costs 1-4 %.
constexpr int kCorridorsAhead = 16;

// Gives every lane with `need` set a Next for `episode`, drawing with it those
// of the `active` lanes of its family that have none (have == false).
// kTogether: see connect_few.
template <bool kTogether = false>
__device__ __forceinline__ void draw_missing(Next& n, bool& have, bool need, bool active, uint32_t meta, uint2 seed,
                                             uint32_t rng_id, uint32_t episode, uint32_t* words) {
  while (true) {
    const uint64_t missing = __ballot(need && !have);
    if (!missing) return;
    const uint32_t f =
        (uint32_t)bcast((int)meta, __ffsll((unsigned long long)missing) - 1) & 255u;
    KcRest rest{};
    if (active && !have && (meta & 255u) == f) {
      n = draw_layout<kTogether>(f, opaque(meta), opaque(seed), opaque(rng_id), episode, words, rest);
      have = true;
    }
    if (kTogether && f == kFamKeyCorridor) {
      uint32_t kd[3] = {n.u[0], n.u[1], n.u[2]};   // (see pack_layout)
      connect_few(kd, n.u[3], rest, opaque(meta), opaque(seed), opaque(rng_id), episode);
#pragma unroll
      for (int q = 0; q < 3; ++q) n.u[q] = rest.todo ? kd[q] : n.u[q];
    }
  }
}

// The agent's pose and the family state (balls, mission) at the start of n.
__device__ __forceinline__ void start_episode(const Next& n, uint32_t fam, int& x, int& y, int& dir,
                                              uint32_t (&ob)[4]) {
  x = (int)(n.pose & 31u);
  y = (int)((n.pose >> 5) & 31u);
  dir = (int)((n.pose >> 10) & 3u);
  ob[0] = fam == kFamGoToDoor ? n.u[1] : ~0u;
  ob[1] = ob[2] = ob[3] = ~0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) ob[i] = fam == kFamDynObs ? n.u[i] : ob[i];
}

// Whether a grid of family f, once filled, keeps its base: nothing in it can
// be picked up or opened, so only the agent and the balls ever move.
__device__ __forceinline__ bool keeps_base(uint32_t f) {
  return f == kFamEmpty || f == kFamDistShift || f == kFamDynObs;
}

// The single cells of the lane's grid (family F, compile-time).
template <uint32_t F>
__device__ __forceinline__ void fill_cells(const Next& n, uint32_t S, uint32_t param, uint8_t* g) {
  auto put = [&](uint32_t x, uint32_t y, uint32_t code) { g[y * S + x] = (uint8_t)code; };
  const uint32_t colour = n.shape >> 16;
  const uint32_t a = n.u[0] & 255u, b = (n.u[0] >> 8) & 255u, c = (n.u[0] >> 16) & 255u, d = n.u[0] >> 24;
  if (F == kFamTwoRoom || F == kFamKeyCorridor) put((n.pose >> 22) & 31u, n.pose >> 27, key_code(colour));
  if (F == kFamTwoRoom) put(a, b, door_code(colour, kLocked));
  if (F == kFamLavaGap) put(a, b, kCodeEmpty);
  if (F == kFamFourRooms) {
    const uint32_t m = S >> 1;
    put(m, a, kCodeEmpty);
    put(m, b, kCodeEmpty);
    put(c, m, kCodeEmpty);
    put(d, m, kCodeEmpty);
  }
  if (F == kFamCrossings) {
    uint64_t open = (uint64_t)n.u[0] | ((uint64_t)n.u[1] << 32);
    for (uint32_t m = n.cols; m; m &= m - 1u, open >>= 5)
      put((uint32_t)__builtin_ctz(m), (uint32_t)open & 31u, kCodeEmpty);
    open = (uint64_t)n.u[2] | ((uint64_t)n.u[3] << 32);
    for (uint32_t m = n.rows; m; m &= m - 1u, open >>= 5)
      put((uint32_t)open & 31u, (uint32_t)__builtin_ctz(m), kCodeEmpty);
  }
  if (F == kFamDynObs) {
#pragma unroll
    for (int i = 0; i < kMaxObst; ++i) {
      const uint32_t xy = (uint32_t)i < param ? obst_at(n.u, i) : obst_at(n.u, 0);
      put(xy & 255u, xy >> 8, kCodeBall);
    }
  }
  if (F == kFamGoToDoor) {
    const uint32_t xl = n.shape & 255u, yl = (n.shape >> 8) & 255u;
    put(a, 0u, door_code(colour & 15u, kClosed));
    put(xl, b, door_code((colour >> 4) & 15u, kClosed));
    put(c, yl, door_code((colour >> 8) & 15u, kClosed));
    put(0u, d, door_code(colour >> 12, kClosed));
  }
  if (F == kFamKeyCorridor) {
    const uint32_t st = (S - 1u) / 3u;
    const uint32_t kd[3] = {n.u[0], n.u[1], n.u[2]};
#pragma unroll
    for (int e = 0; e < 10; ++e) {
      const uint32_t v = kc_byte(kd, e), p = (v & 15u) + 1u;
      const uint32_t state = (uint32_t)e == 2u * n.u[3] + 1u ? kLocked : kClosed;
      const uint32_t x = e < 6 ? (uint32_t)((e & 1) + 1) * st : (uint32_t)(e & 1) * 2u * st + p;
      const uint32_t y = e < 6 ? (uint32_t)(e >> 1) * st + p : (uint32_t)((e - 6) / 2 + 1) * st;
      if (v & 0x80u) put(x, y, door_code((v >> 4) & 7u, state));
    }
  }
  // last: FourRooms may have its goal in an opening
  if (F != kFamGoToDoor) put((n.pose >> 12) & 31u, (n.pose >> 17) & 31u, kCodeGoal);
}

// Fills the grids of the lanes in `pending` from their Next: the bases one
// env at a time (those not kept, see keeps_base), then the single cells.
__device__ __forceinline__ void fill_grids(uint64_t pending, bool kept, const Next& n, uint32_t meta, uint8_t* codes,
                                           int my_off, int lane) {
  meta = opaque(meta);
  const bool mine = (pending >> lane) & 1u;
  const uint32_t my_S = (meta >> 8) & 255u;
  // v / S = v * recip >> 16 for v <= 64 and S <= 32
  const uint32_t recip = (uint32_t)(65536.0f * __builtin_amdgcn_rcpf((float)my_S)) + 1u;
  const uint32_t code = (meta & 255u) >= kFamLavaGap && (meta & 255u) <= kFamDistShift ? kCodeLava : kCodeWall;
  const uint32_t packed = recip | (my_S << 16) | (code << 24);
  for (uint64_t todo = __ballot(mine && !kept); todo; todo &= todo - 1) {
    const int r = __ffsll((unsigned long long)todo) - 1;
    const uint32_t pk = (uint32_t)bcast((int)packed, r), shape = (uint32_t)bcast((int)n.shape, r);
    const uint32_t cols = (uint32_t)bcast((int)n.cols, r), rows = (uint32_t)bcast((int)n.rows, r);
    const uint32_t span = (uint32_t)bcast((int)n.span, r);
    uint8_t* gp = codes + bcast(my_off, r) + lane;
    const uint32_t S = (pk >> 16) & 255u, inv = pk & 0xFFFFu, line = pk >> 24, cells = S * S;
    // wall columns and rows: 0, and from xl / yl on
    const uint32_t wall_x = 1u | (~0u << (shape & 31u)), wall_y = 1u | (~0u << ((shape >> 8) & 31u));
    const uint32_t dy = ((uint32_t)kWave * inv) >> 16, dx = (uint32_t)kWave - dy * S;
    uint32_t y = ((uint32_t)lane * inv) >> 16, x = (uint32_t)lane - y * S;
    uint32_t c0 = 0;
    do {
      const uint32_t on_line = (cols >> x) | ((rows >> y) & (span >> x));
      const uint32_t on_wall = (wall_x >> x) | (wall_y >> y);
      uint32_t code_here = (on_line & 1u) ? line : kCodeEmpty;
      code_here = (on_wall & 1u) ? kCodeWall : code_here;
      if (c0 + (uint32_t)lane < cells) gp[c0] = (uint8_t)code_here;
      x += dx;
      y += dy;
      const bool wrap = x >= S;
      x -= wrap ? S : 0u;
      y += wrap ? 1u : 0u;
      c0 += kWave;
    } while (c0 < cells);
  }
  wave_sync();
  if (mine) {
    uint8_t* g = codes + my_off;
    const uint32_t param = (meta >> 16) & 255u, f = meta & 255u;
    if (f == kFamEmpty) fill_cells<kFamEmpty>(n, my_S, param, g);
    if (f == kFamTwoRoom) fill_cells<kFamTwoRoom>(n, my_S, param, g);
    if (f == kFamFourRooms) fill_cells<kFamFourRooms>(n, my_S, param, g);
    if (f == kFamLavaGap) fill_cells<kFamLavaGap>(n, my_S, param, g);
    if (f == kFamCrossings) fill_cells<kFamCrossings>(n, my_S, param, g);
    if (f == kFamDistShift) fill_cells<kFamDistShift>(n, my_S, param, g);
    if (f == kFamDynObs) fill_cells<kFamDynObs>(n, my_S, param, g);
    if (f == kFamGoToDoor) fill_cells<kFamGoToDoor>(n, my_S, param, g);
    if (f == kFamKeyCorridor) fill_cells<kFamKeyCorridor>(n, my_S, param, g);
  }
}

// the stage of a wave's views: 64 of 49 codes, and what emit_* may read
// before and past them
constexpr int kStageMargin = 16;
// envs of a tile up to which the renderer computes the views together
// (views_of_few takes 8): Empty 8x8, us a step, 4096 envs in tiles of 4 1.21 ->
// 0.98, 8192 in tiles of 8 1.40 -> 1.22.
constexpr int kFewEnvs = 8;
constexpr int kViewStageBytes = kStageMargin + kWave * kCatBytes + 32;
// words of emit_dirty_grids's bitmap: one bit per 64 cells of at most 64
// grids of side 32, starting up to 63 cells before the first
constexpr int kMarkWords = ((kWave * 32 * 32 + 63 + 63) / 64 + 31) / 32;
static_assert(kDrawBytes <= kViewStageBytes && kMarkWords * 4 <= kViewStageBytes, "the stage holds each of its uses");

__device__ __forceinline__ int wave_excl_scan(int v, int lane, int& total) {
  int incl = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int n = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += n;
  }
  total = bcast(incl, kWave - 1);
  return incl - v;
}

// ---------------------------------------------------------------------------
// Plain kernel: one step of every env per launch, state and grids in HBM, the
// first-person record modes or none.  Whole-grid records, and moving balls
// where reading every grid costs less than their trips to HBM (step_in_hbm),
// run k_fused for one step.
//
// The view is read as soon as the action is known, before it is applied: a
// step ends in one of at most two 7x7 squares (a turn: the new heading's;
// forward: the current one or the one a cell ahead; anything else, and a
// reset: the current one), whose union is the final heading's square extended
// by one cell along it, 8 grid rows of 8 cells at most, and holds the cell
// ahead as well.  So the cell ahead and the view come in one round trip to
// HBM.  A row is 24 bytes at any alignment, converted to eight codes; from
// there on the step is k_fused's.  Rows outside the grid are read as its first
// or last row: no cell outside the grid is visible (see kMargin).
//
// Bound by HBM: the grids' lines that the views touch (2.9 of 128 bytes each
// on the mixed batch), the state and the records, 145 MB a launch for 262 144
// mixed envs; with few envs by its chain of two round trips and one wave's
// instructions, so small batches run in small tiles (launch_tile_envs).
// ---------------------------------------------------------------------------
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(1)));

// Codes of eight rows of eight cells: row q starts at cell (x0, y0 + q step),
// y clamped to the grid.  first / last: the env's grid is the first / last of
// the buffer, whose bytes beyond are not to be read: such rows are read from
// the buffer's edge and shifted into place by whole cells.
__device__ __forceinline__ void load_rows(const uint8_t* g, int S, int x0, int y0, int step, bool first, bool last,
                                          uint32_t (&lo)[8], uint32_t (&hi)[8]) {
  const int least = first ? 0 : -21, most = last ? 3 * S * S - 24 : 3 * S * S;
  x0 = min(max(x0, -7), S - 1);
  u32x4 w4[8];
  u32x2_any w2[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int y = min(max(y0 + q * step, 0), S - 1);
    const uint8_t* p = g + min(max(3 * (y * S + x0), least), most);
    w4[q] = *reinterpret_cast<const u32x4_any*>(p);
    w2[q] = *reinterpret_cast<const u32x2_any*>(p + 16);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    lo[q] = encode_cells(w4[q].x, w4[q].y, w4[q].z);
    hi[q] = encode_cells(w4[q].w, w2[q].x, w2[q].y);
  }
  if (__ballot(first || last)) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int o = 3 * (min(max(y0 + q * step, 0), S - 1) * S + x0);
      const int cells = (min(max(o, least), most) - o) / 3;   // -8 .. 7
      const uint64_t v = (uint64_t)lo[q] | ((uint64_t)hi[q] << 32);
      const uint64_t s = cells >= 0 ? v << (8 * cells) : (cells > -8 ? v >> (-8 * cells) : 0ull);
      lo[q] = (uint32_t)s;
      hi[q] = (uint32_t)(s >> 32);
    }
  }
}

__device__ __forceinline__ void store_code(uint8_t* p, uint32_t code) {
  const Cells4 c = decode_cells<false>(code);
  p[0] = (uint8_t)c.type;
  p[1] = (uint8_t)c.colour;
  p[2] = (uint8_t)c.state;
}

__device__ __forceinline__ uint32_t load_code(const uint8_t* p) {
  return code_of((uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16));
}

// move_balls on a grid in HBM (at g, the agent at (x, y)): bound by latency, one
// trip per ball for the three rows of nine bytes around it, but no byte of any
// other env's grid.  One step of Empty 31x31 with 1 % Dynamic-Obstacles, 262 144
// envs: 44 us, without records 15 (464 and 447 with every grid staged in LDS);
// 65 536 FourRooms 19x19 with 1 %: 13.6 (27).
__device__ __forceinline__ void move_balls_hbm(uint8_t* g, int S, int n, int x, int y, uint32_t (&ob)[4], uint2 seed,
                                               uint32_t rng_id, uint32_t call, const uint32_t* kth) {
  const uint32_t inner = (uint32_t)(S - 2);
  uint4 blk[2] = {make_uint4(rng_id, call, 0u, 2u), make_uint4(rng_id, call, 1u, 2u)};
  philox10<2>(blk, seed);
#pragma unroll
  for (int b = 0; b < kMaxObst; ++b) {
    const uint32_t xy = obst_at(ob, b);
    const uint32_t bx = xy & 0xFFu, by = xy >> 8;
    if (b >= n || max(bx - 1u, by - 1u) >= inner) continue;
    uint8_t* cell = g + 3u * (by * (uint32_t)S + bx);
    u32x2_any lo[3];
    uint32_t hi[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const uint8_t* p = cell + 3 * ((r - 1) * S - 1);
      lo[r] = *reinterpret_cast<const u32x2_any*>(p);
      hi[r] = p[8];
    }
    uint32_t mask = empty_neighbours<0>(encode_cells(lo[0].x, lo[0].y, hi[0]), 0u);
    mask = empty_neighbours<1>(encode_cells(lo[1].x, lo[1].y, hi[1]), mask);
    mask = empty_neighbours<2>(encode_cells(lo[2].x, lo[2].y, hi[2]), mask);
    // the agent's cell, if it is one of the eight, is taken
    const uint32_t ax = (uint32_t)x - bx + 1u, ay = (uint32_t)y - by + 1u, at = 3u * ay + ax;
    mask &= max(ax, ay) < 3u && at != 4u ? ~(1u << (7u + at - (at > 4u ? 1u : 0u))) : ~0u;
    if (!mask) continue;
    uint32_t nx, ny;
    ball_target(mask, pick4(blk[b >> 2], (uint32_t)(b & 3)), kth, bx, by, nx, ny);
    store_code(cell, kCodeEmpty);
    store_code(g + 3u * (ny * (uint32_t)S + nx), kCodeBall);
    obst_set(ob, b, nx, ny);
  }
}

// Lays out the grids of the lanes in `pending` (a lane's grid at g in HBM) by
// way of `buf`, as many at a time as it holds.
constexpr int kNewGridBytes = 4096;   // at least one grid of side 32

__device__ __forceinline__ void write_new_grids(uint64_t pending, const Next& n, uint32_t meta, uint8_t* g,
                                                uint8_t* buf, int lane) {
  const int S = (int)((meta >> 8) & 255u), cells = S * S;
  while (pending) {
    const bool mine = (pending >> lane) & 1u;
    int total;
    const int off = wave_excl_scan(mine ? (cells + 3) & ~3 : 0, lane, total);
    const uint64_t now = __ballot(mine && off + cells <= kNewGridBytes);
    fill_grids(now, false, n, meta, buf, off, lane);
    wave_sync();
    for (uint64_t todo = now; todo; todo &= todo - 1) {
      const int r = __ffsll((unsigned long long)todo) - 1;
      uint8_t* dst = reinterpret_cast<uint8_t*>(bcast64(reinterpret_cast<uint64_t>(g), r));
      const uint8_t* src = buf + bcast(off, r);
      const int c = bcast(cells, r);
      for (int p = 0; p < c; p += 4 * kWave) emit_some<false, false, false>(dst, src, c, p, 0u, lane);
      if (c & 3) emit_ends<false, false>(dst, src, c, 0, c & 3, lane);
    }
    wave_sync();
    pending &= ~now;
  }
}

struct PlainArgs {
  EnvTables env;
  StateBufs st;
  const uint8_t* actions;
  TrajBufs out;
  int32_t row;
  int32_t tile_envs;   // envs per workgroup
};

// kObs: 0 symbolic, 1 categorical first person, 2 no observations
// kBalls: some env is a Dynamic-Obstacles; its balls move in HBM before the
// view is read
template <int kObs, bool kBalls>
__global__ __launch_bounds__(kWave) void k_plain(PlainArgs a) {
  __shared__ __align__(16) uint2 masks[kObs == 2 ? 1 : kMaskEntries];
  __shared__ __align__(16) uint32_t stage_words[kViewStageBytes / 4];   // and the draw window, before
  __shared__ __align__(16) uint8_t new_grids[kNewGridBytes + 16];
  __shared__ __align__(16) uint32_t kth_cell[kBalls ? kMaskPatterns : 1];
  const int lane = threadIdx.x;
  const int N = a.env.n;
  const int e0 = (int)blockIdx.x * a.tile_envs, e = e0 + lane;
  const int n_here = min(a.tile_envs, N - e0);
  const bool active = lane < n_here;

  // a lane without an env reads the first bytes of the buffer (48 at least)
  uint32_t fam = 0, meta = 0;
  int S = 4, T = 1, x = 1, y = 1, dir = 0, t = 0;
  uint32_t carry = kCellEmpty, episode = 0, rid = 0, calls = 0, act = 6u;
  bool done_prev = false;
  uint2 seed = make_uint2(0, 0);
  uint8_t* g = a.st.grid;
  uint32_t ob[4] = {~0u, ~0u, ~0u, ~0u};
  if (active) {
    meta = a.env.meta[e];
    T = a.env.max_steps[e];
    seed = a.env.seed[e];
    rid = a.env.rng_id[e];
    g = a.st.grid + a.env.grid_off[e];
    x = a.st.x[e];
    y = a.st.y[e];
    dir = a.st.dir[e];
    t = a.st.t[e];
    carry = (uint32_t)a.st.carry[e];
    episode = a.st.episode[e];
    done_prev = a.st.done_prev[e] != 0;
    calls = a.st.calls[e];
    if (a.actions) act = a.actions[e];
    fam = meta & 0xFF;
    S = (int)((meta >> 8) & 0xFF);
    if (fam == kFamGoToDoor) ob[0] = *reinterpret_cast<const uint32_t*>(a.st.obst + 16 * (size_t)e);   // the mission
    if (kBalls && fam == kFamDynObs) {
      const uint4 o4 = *reinterpret_cast<const uint4*>(a.st.obst + 16 * (size_t)e);
      ob[0] = o4.x; ob[1] = o4.y; ob[2] = o4.z; ob[3] = o4.w;
    }
  }
  if (kObs != 2) build_mask_table(masks, lane);
  const bool do_reset = active && done_prev;
  const uint64_t pending = __ballot(do_reset);
  uint32_t carry_code = code_of(carry);
  bool carry_changed = do_reset;
  if (pending) {
    Next next{};
    bool have = false;
    draw_missing(next, have, do_reset, do_reset, meta, seed, rid, episode + 1u, stage_words + lane);
    if (do_reset) {
      episode += 1u;
      start_episode(next, fam, x, y, dir, ob);
      t = 0;
      carry_code = kCodeEmpty;
    }
    write_new_grids(pending, next, meta, g, new_grids, lane);
    __threadfence_block();
    __syncthreads();
  }
  const bool live = active && !do_reset;
  if (!a.actions) act = bounded(pick4(policy_block(seed, rid, calls), calls & 3u), 7u);
  act = live ? act : 6u;
  const uint32_t dir2 = 2u * (uint32_t)dir;
  const int dx = (int)((0x46u >> dir2) & 3u) - 1, dy = (int)((0x19u >> dir2) & 3u) - 1;
  const bool balls = kBalls && fam == kFamDynObs && live;
  uint32_t penalty = 0;
  if (kBalls && __ballot(balls)) {
    build_kth_table(kth_cell, lane);
    wave_sync();
    if (balls) {
      // three actions; the cell ahead is judged before the balls move
      act = act > kForward ? kLeft : act;
      const uint32_t before = load_code(g + 3 * (min(max(y + dy, 0), S - 1) * S + min(max(x + dx, 0), S - 1)));
      penalty = (act == kForward && before != kCodeEmpty && (before & 0x8Fu) != kGoal) ? 1u : 0u;
      move_balls_hbm(g, S, (int)((meta >> 16) & 255u), x, y, ob, seed, rid, calls, kth_cell);
    }
  }
  const uint32_t a6 = min(act, 6u);

  // the cell ahead, and the rows of the view
  const int dir_f = (dir + (int)((7u >> (2u * a6)) & 3u)) & 3;   // left 3, right 1
  const bool vert = (dir_f & 1) != 0;
  uint32_t rlo[8], rhi[8], front;
  if (kObs != 2) {
    const bool back = dir_f == 1 || dir_f == 2;   // rows bottom up
    load_rows(g, S, x - (vert ? 3 : (dir_f == 0 ? 0 : 7)), back ? y + (vert ? 7 : 3) : y - (vert ? 7 : 3),
              back ? -1 : 1, e == 0 || !active, e == N - 1 || !active, rlo, rhi);
    front = vert ? rlo[6] >> 24 : ((dir_f == 0 ? rlo[3] >> 8 : rhi[3] >> 16) & 255u);
  } else {
    front = load_code(g + 3 * (min(max(y + dy, 0), S - 1) * S + min(max(x + dx, 0), S - 1)));
  }

  const CodeAction r = act_on_code(a6, carry_code, front);
  dir = dir_f;
  const uint32_t walked = a6 == kForward ? r.ok : 0u;
  const int ahead = (y + dy) * S + x + dx;
  x += (int)(walked & (uint32_t)dx);
  y += (int)(walked & (uint32_t)dy);
  penalty |= r.lava;
  uint32_t goal = r.goal, ended = goal | penalty;
  const uint32_t patch = a6 > kForward ? r.ok : 0u;   // a pickup, drop or toggle changed the cell ahead
  bool edge_view = false;
  if (fam == kFamGoToDoor && live) {
    // on_door_done of Tables "rewards" and "terminations": the done action
    // (any value >= 6) with the mission's door directly ahead achieves the
    // task; toggling ends the episode with reward 0
    const bool done_at = act >= 6u && is_door_code(front) && ((front >> 4) & 7u) == (ob[0] & 0xFFu);
    goal |= done_at ? 1u : 0u;
    ended |= (done_at || act == kToggle) ? 1u : 0u;
    edge_view = patch != 0u;   // a door toggled, possibly on the outer ring
  }
  if (patch) {
    store_code(g + 3 * ahead, r.new_front);
    const bool held = a6 != kToggle;
    carry_code = held ? (a6 == kPickup ? front : kCodeEmpty) : carry_code;
    carry_changed = carry_changed || held;
  }
  t += live ? 1 : 0;
  const uint32_t trunc = (live && t >= T) ? 1u : 0u;
  float reward = 0.0f;
  if (__ballot(ended != 0u)) reward = penalty ? -1.0f : (goal ? goal_reward(t, T, a.env.reward_mode) : 0.0f);
  const uint32_t flags = do_reset ? kFlagFirst : ended * kFlagTerminated | trunc * kFlagTruncated;
  const size_t row0 = (size_t)a.row * (size_t)N + (size_t)e0;

  if (kObs != 2) {
    // the final square among the rows read: one row or one column of the eight
    // falls away
    const bool down = vert && !walked;
    const uint32_t right = (!vert && (dir == 0) == (walked != 0u)) ? 1u : 0u;
    uint32_t lo[kView], hi[kView], f[13];
#pragma unroll
    for (int q = 0; q < kView; ++q) {
      const uint32_t l = down ? rlo[q + 1] : rlo[q], h = down ? rhi[q + 1] : rhi[q];
      lo[q] = __builtin_amdgcn_alignbyte(h, l, right);
      hi[q] = __builtin_amdgcn_alignbyte(0u, h, right);
    }
    view_from_rows(lo, hi, S, x, y, dir, carry_code, patch, r.new_front, masks, __ballot(edge_view) != 0, edge_view,
                   f);
    uint32_t* const stage = stage_words + kStageMargin / 4;
    store_view(stage, f, lane, n_here);
    wave_sync();
    const uint8_t* cells = reinterpret_cast<const uint8_t*>(stage);
    if (kObs == 1) emit_types(a.out.obs + row0 * kCatBytes, cells, n_here * kCatBytes, lane);
    else emit_triples<false>(a.out.obs + row0 * kObsBytes, cells, n_here * kCatBytes, lane);
  }
  if (active) {
    a.out.reward[row0 + lane] = reward;
    a.out.flags[row0 + lane] = (uint8_t)flags;
    a.out.action[row0 + lane] = (uint8_t)(live ? act : kActionNone);
    if (a.out.mission) a.out.mission[row0 + lane] = (uint8_t)mission_of(fam, ob[0]);
    a.st.x[e] = x;
    a.st.y[e] = y;
    a.st.dir[e] = dir;
    a.st.t[e] = t;
    if (carry_changed) a.st.carry[e] = (int32_t)carry_triple(carry_code);
    a.st.episode[e] = episode;
    a.st.done_prev[e] = (ended | trunc) != 0u ? 1 : 0;
    a.st.calls[e] = calls + 1u;
    if (do_reset || balls)
      *reinterpret_cast<uint4*>(a.st.obst + 16 * (size_t)e) = make_uint4(ob[0], ob[1], ob[2], ob[3]);
  }
}

// Which wave of a workgroup of two is the renderer (kSplit).  A SIMD with a
// renderer and a stepper keeps pace; one with two renderers does not, and the
// whole launch waits for it.  Which SIMDs a workgroup's waves land on depends on
// where the kernel before left off: by the wave's number alone every SIMD has one
// of each after a launch of the same shape, but after a kernel of larger
// workgroups a tenth of the compute units has two renderers on two SIMDs and two
// steppers on the others.  So where pairs take many tiles in turn (kLong), the
// workgroups of a compute unit count their renderers by SIMD, in a byte each, and
// a workgroup takes the SIMD with fewer: 262 144 Empty 8x8, 1024 steps after a
// fill of 256 MB 9.39 -> 7.28 ms (single waves 8.14), 128 steps 1.19 -> 0.97, as
// without the fill.  The claim takes some two microseconds a launch.  The counts
// steer speed alone and are back to what they were when a launch ends.
__device__ uint32_t renderers_on[16 * 256];   // by XCC and compute unit

// what a workgroup has counted, kept in LDS: a wave may end on another compute
// unit than it began on (it is saved and restored when processes take turns)
struct Claim {
  uint32_t shifts[2];   // the waves' SIMDs as shifts of the count
  uint32_t unit, second;
};

// 0 or 1: the wave of the workgroup that is to render, from now on counted
__device__ __forceinline__ int claim_renderer(Claim& c, int wave, int lane) {
  constexpr int kHwId = 4 | (15 << 11), kXccId = 20 | (3 << 11);   // s_getreg operands: bits 0-15, 0-3
  const uint32_t hw = (uint32_t)__builtin_amdgcn_s_getreg(kHwId), xcc = (uint32_t)__builtin_amdgcn_s_getreg(kXccId);
  if (lane == 0) c.shifts[wave] = 8u * ((hw >> 4) & 3u);
  pair_barrier();
  if (wave == 0 && lane == 0) {
    const uint32_t s0 = c.shifts[0], s1 = c.shifts[1];
    c.unit = ((xcc & 15u) << 8) | ((hw >> 8) & 255u);
    uint32_t* const count = renderers_on + c.unit;
    uint32_t seen = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), second;
    do {   // fails only when another workgroup's claim or end came between
      second = ((seen >> s1) & 255u) < ((seen >> s0) & 255u) ? 1u : 0u;
    } while (!__hip_atomic_compare_exchange_strong(count, &seen, seen + (1u << (second ? s1 : s0)), __ATOMIC_RELAXED,
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    c.second = second;
  }
  pair_barrier();
  return __builtin_amdgcn_readfirstlane((int)c.second);
}

__device__ __forceinline__ void give_back(const Claim& c) {
  __hip_atomic_fetch_sub(renderers_on + c.unit, 1u << c.shifts[c.second], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct FusedArgs {
  EnvTables env;
  TileTables tiles;
  StateBufs st;
  const uint8_t* actions;   // [k_steps][N] or nullptr
  int32_t k_steps;
  TrajBufs out;
  int32_t row0;
  ServeTile* serve;               // per-tile requests (serving), else nullptr
  const ServeTile* host_tiles;    // serving: staging of newly admitted tiles (pinned host memory)
  const SlotConfig* host_slots;   // serving: their slot configurations
};

// What bounds a step: with few tiles (up to one wave per SIMD, 65 536 envs)
// one wave's own instruction stream, 5 cycles per independent vector
// instruction and 8 per dependent one, 14-20 per LDS read; with many, the
// record stores.  Views and records computed on bytes (four cells a word)
// instead of a table read per cell took the LDS instructions of a step from
// 153 to about 60: 65 536 TwoRoom 8x8 envs 3.2 -> 2.6 us a step, 30 011 envs of
// the uneven mix (rows off every alignment) 5.9 -> 3.5 us, 65 536 mixed
// envs' whole grids 10.0 -> 7.7 us, 262 144 mixed envs' 20 steps 242 -> 222 us.
//
// kActions: actions come from a.actions; otherwise from the random policy.
// kServe: tiles belong to requests described by a.serve (serving): each runs
// min(K, steps it has left) steps from the count the host lists it with and
// writes to its own output rows.
// kObs: the observation records written, 0 symbolic first person, 1
// categorical first person, 2 whole grid (a.env.obs_mode 2 or 3); each
// variant carries only its own record code.
// kLong: launches of several steps that keep one of two more rules, see
// claim_renderer (kSplit) and emit_64_views.
// kSplit: a workgroup of two waves.  The second takes the steps (policy,
// actions, resets, balls, the step's scalars), the first writes the records:
// it is handed each lane's pose in LDS, reads the views' rows out of the
// grids, lets the second go on, and computes and stores the records meanwhile.
// Two barriers a step, one after the step is taken and one after the rows are
// read; both waves pass each `steps` times per tile.  Only LDS is shared, so
// neither wave waits for device memory at them.  Which wave is the longer one
// changes from step to step: the renderer runs at priority 1, the other at 0,
// and at 2 while layouts are drawn and filled or balls move.  65 536 TwoRoom
// 8x8 envs: 2.45 -> 1.92 us a step, 5.3 TB/s of records; 4096 Empty 8x8
// 1.61 -> 1.16 (0.95 with views_of_few), 30 011 envs of all families
// 6.4 -> 4.95, 65 536 Dynamic-Obstacles envs as type ids 5.7 -> 4.6.  Without
// the priorities 2.0 / 1.24 / 5.3 / 4.95.
// On this GPU one counter tracks both outstanding loads and stores, so a
// load consumed in the same step would also wait for every earlier record
// store: the action of step s + 1 is therefore fetched during step s, and
// the policy variant has no loads in its step loop at all.
template <bool kActions, bool kServe, int kObs, bool kSplit, bool kTogether = false, bool kLong = false>
__global__ __launch_bounds__(kSplit ? 2 * kWave : kWave) void k_fused(FusedArgs a) {
  // first-person variants: the byte masks of a row's visibility bits.  The
  // stage holds, one after another, the words of layouts being drawn, the
  // wave's views, and after the last step the bitmap of emit_dirty_grids.
  __shared__ __align__(16) uint2 masks[kObs == 2 ? 1 : kMaskEntries];
  __shared__ __align__(16) uint32_t stage_words[kViewStageBytes / 4];
  __shared__ __align__(16) uint32_t kth_cell[kMaskPatterns];
  // per lane: whether a pickup, drop or toggle changed a cell of its grid
  __shared__ uint8_t cell_changed[kWave];
  // kSplit: the renderer's own stage, and the poses it is handed (x: the agent's
  // byte of LDS, heading << 18, toggled << 20; y: x, y, side, carried code)
  __shared__ __align__(16) uint32_t view_words[kSplit ? kViewStageBytes / 4 : 1];
  __shared__ uint2 poses[kSplit ? kWave : 1];
  extern __shared__ __align__(16) uint8_t grids[];
  uint8_t* codes = grids + kMargin;
  const int lane = kSplit ? threadIdx.x & (kWave - 1) : threadIdx.x;
  __shared__ Claim claim;
  const int wave = kSplit ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
  const bool renders = kSplit && wave == (kLong ? claim_renderer(claim, wave, lane) : 0);
  const int N = a.env.n;
  if (renders) __builtin_amdgcn_s_setprio(1);

  // a view's first cell lies kStageMargin bytes in (emit_* read a little
  // before and past their cells)
  uint32_t* const stage = (kSplit ? view_words : stage_words) + kStageMargin / 4;
  if (kObs != 2 && (!kSplit || renders)) {
    build_mask_table(masks, lane);
    wave_sync();
  }

  for (int it = blockIdx.x; it < a.tiles.n_tiles; it += gridDim.x) {
    // serving lists mark a newly admitted tile with the top bit: its
    // descriptor and slot configurations are still in host staging and its
    // envs are reset here (episode 0) before its first step
    const int part = kServe ? it & ((1 << a.tiles.parts_log2) - 1) : 0;
    const uint2 entry = kServe ? a.tiles.list[it >> a.tiles.parts_log2] : make_uint2((uint32_t)it, 0u);
    const int tile = (int)(entry.x & 0x7FFFFFFFu);
    const bool fresh = kServe && (entry.x >> 31) != 0;
    // where this tile's envs live and where their records go: record of
    // step s, lane l is at index rec_base + s * rec_step (+ l) of the outputs
    const int tile_envs = a.tiles.tile_envs;
    const int first = part * tile_envs;   // of the listed tile's envs
    const int e0 = kServe ? tile * kWave + first : tile * tile_envs;
    int n_here, steps;
    uint64_t g0 = 0;
    uint8_t *o_obs, *o_flags, *o_action, *o_mission = nullptr;
    float* o_reward;
    uint32_t step0 = 0;
    size_t rec_stride;
    if (kServe) {
      const ServeTile d = fresh ? a.host_tiles[tile] : a.serve[tile];
      if (fresh && part == 0 && lane == 0 && !renders) a.serve[tile] = d;   // the device copy later launches read
      step0 = entry.y;
      n_here = min(tile_envs, (int)d.n_envs - first);
      if (!d.active || step0 >= d.n_steps || n_here <= 0) continue;
      steps = min(a.k_steps, (int)(d.n_steps - step0));
      o_obs = d.obs;
      o_reward = d.reward;
      o_flags = d.flags;
      o_action = d.action;
      rec_stride = d.stride;
      const size_t local = (size_t)d.local0 + (size_t)first;
      o_obs = o_obs ? o_obs + local * kObsBytes : nullptr;
      o_reward += local;
      o_flags += local;
      o_action += local;
    } else {
      n_here = min(tile_envs, N - e0);
      steps = a.k_steps;
      o_obs = a.out.obs ? a.out.obs + (size_t)e0 * (kObs == 1 ? kCatBytes : kObsBytes) : nullptr;
      o_reward = a.out.reward + e0;
      o_flags = a.out.flags + e0;
      o_action = a.out.action + e0;
      o_mission = a.out.mission ? a.out.mission + e0 : nullptr;
      rec_stride = (size_t)N;
    }
    // the staged views as the first-person records from index rec on
    const auto write_views = [&](size_t rec) {
      wave_sync();
      const uint8_t* cells = reinterpret_cast<const uint8_t*>(stage);
      if (kObs == 1) emit_types(o_obs + rec * kCatBytes, cells, n_here * kCatBytes, lane);
      else if (kLong && !kSplit) emit_64_views(o_obs + rec * kObsBytes, cells, lane);
      else emit_triples<false>(o_obs + rec * kObsBytes, cells, n_here * kCatBytes, lane);
    };
    int ring_row = kServe ? 0 : a.row0;   // output row of the next step
    if (renders) {
      for (int s = 0; s < steps; ++s) {
        const size_t row = kServe ? (size_t)(step0 + s) : (size_t)ring_row;
        if (!kServe) ring_row = ring_row + 1 == a.out.rows ? 0 : ring_row + 1;
        pair_barrier();   // the step is taken
        if (o_obs) {
          // the rows are read: grids may change
          const auto rows_read = [] { pair_barrier(); };
          if (tile_envs <= kFewEnvs) {
            const uint2 p = poses[lane >> 3];
            views_of_few(grids, stage, p, lane, n_here, masks, __ballot((p.x >> 20) & 1u) != 0, rows_read);
          } else {
            const uint2 p = poses[lane];
            const bool edge_view = ((p.x >> 20) & 1u) != 0u;
            uint32_t f[13];
            view_codes(grids, (int)(p.x & 0x3FFFFu), (int)((p.y >> 16) & 255u), (int)(p.y & 255u),
                       (int)((p.y >> 8) & 255u), (int)((p.x >> 18) & 3u), p.y >> 24, masks, __ballot(edge_view) != 0,
                       edge_view, f, rows_read);
            __builtin_amdgcn_sched_barrier(0);
            store_view(stage, f, lane, n_here);
          }
          write_views(row * rec_stride);
          wave_sync();
        } else {
          pair_barrier();
        }
      }
      continue;
    }
    const int e = e0 + lane;
    const bool active = lane < n_here;

    uint32_t fam = 0, meta = 0;
    int S = 0, T = 1, x = 1, y = 1, dir = 0, t = 0;
    uint32_t carry = kCellEmpty, episode = 0, rid = 0, calls = 0;
    bool done_prev = false;
    uint2 seed = make_uint2(0, 0);
    uint64_t goff = 0;
    uint32_t ob[4] = {~0u, ~0u, ~0u, ~0u};
    Next next{};
    bool have_next = false;   // next holds the layout of episode + 1
    if (active && fresh) {
      const SlotConfig c = a.host_slots[e];
      meta = c.meta;
      T = c.max_steps;
      seed = c.seed;
      rid = c.rng_id;
      a.env.meta[e] = c.meta;
      a.env.max_steps[e] = c.max_steps;
      a.env.seed[e] = c.seed;
      a.env.rng_id[e] = c.rng_id;
      a.env.grid_off[e] = c.grid_off;
      goff = c.grid_off;
      fam = meta & 0xFF;
      S = (int)((meta >> 8) & 0xFF);
    } else if (active) {
      meta = a.env.meta[e];
      fam = meta & 0xFF;
      S = (int)((meta >> 8) & 0xFF);
      T = a.env.max_steps[e];
      seed = a.env.seed[e];
      rid = a.env.rng_id[e];
      goff = a.env.grid_off[e];
      x = a.st.x[e];
      y = a.st.y[e];
      dir = a.st.dir[e];
      t = a.st.t[e];
      carry = (uint32_t)a.st.carry[e];
      episode = a.st.episode[e];
      done_prev = a.st.done_prev[e] != 0;
      calls = a.st.calls[e];
      const uint4 o4 = *reinterpret_cast<const uint4*>(a.st.obst + 16 * (size_t)e);
      ob[0] = o4.x; ob[1] = o4.y; ob[2] = o4.z; ob[3] = o4.w;
    }
    int tile_cells;
    const int my_off = wave_excl_scan(S * S, lane, tile_cells);
    cell_changed[lane] = 0;
    uint8_t* my_codes = codes + my_off;
    // the tile's grids are contiguous in HBM: stage them as codes (a fresh
    // tile's are laid out here instead)
    g0 = bcast64(goff, 0);
    if (fresh) {
      draw_missing<kTogether>(next, have_next, active, active, meta, seed, rid, 0u, stage_words + lane);
      if (active) start_episode(next, fam, x, y, dir, ob);
      fill_grids(__ballot(active), false, next, meta, codes, my_off, lane);
      have_next = false;
    } else {
      stage_in_codes(a.st.grid + g0, tile_cells, codes, lane);
    }
    uint32_t carry_code = code_of(carry);
    bool carry_changed = fresh;   // until then the state's own triple stays
    const bool any_missions = __ballot(fam == kFamGoToDoor) != 0;
    int pos = y * S + x;          // the agent's cell in its grid
    bool filled = fresh;          // the grid was laid out in this launch
    int most_balls = 0;           // of an env of this tile
    while (most_balls < kMaxObst && __ballot(fam == kFamDynObs && ((meta >> 16) & 255u) > (uint32_t)most_balls))
      ++most_balls;
    if (most_balls) build_kth_table(kth_cell, lane);
    wave_sync();

    uint4 pol = make_uint4(0, 0, 0, 0);
    uint32_t act_next = 0;
    if (kActions && active) act_next = a.actions[e];
    for (int s = 0; s < steps; ++s) {
      // the env's call count; envs stepped together share it, so the policy
      // block refresh every 4 calls is uniform across the wave in practice
      const uint32_t call = calls + (uint32_t)s;
      uint32_t act_now = 0;
      if (kActions) {
        act_now = act_next;
        if (active && s + 1 < steps) act_next = a.actions[(size_t)(s + 1) * N + e];
      } else if (s == 0 || (call & 3) == 0) {
        pol = policy_block(opaque(seed), rid, call);
      }

      if (kSplit && s > 0) pair_barrier();   // the rows of step s - 1 are read
      const bool do_reset = active && done_prev;
      const uint64_t pending = __ballot(do_reset);
      if (kSplit && (pending || most_balls != 0)) __builtin_amdgcn_s_setprio(2);
      if (pending) {
        // in the launch's last step only for the lanes that reset: nothing is
        // kept for the next launch (and see kCorridorsAhead)
        bool ahead = s + 1 < steps;
        if (kTogether || kServe) ahead = ahead && (fam != kFamKeyCorridor || steps - s >= kCorridorsAhead);
        draw_missing<kTogether>(next, have_next, do_reset, ahead ? active : do_reset, meta, seed, rid, episode + 1u,
                                stage_words + lane);
        const bool kept = filled && keeps_base(fam);
        if (most_balls != 0 && do_reset && kept && fam == kFamDynObs) {   // the old balls leave
          const uint32_t balls = (opaque(meta) >> 16) & 255u;
#pragma unroll
          for (int i = 0; i < kMaxObst; ++i) {
            const uint32_t xy = (uint32_t)i < balls ? obst_at(ob, i) : obst_at(ob, 0);
            my_codes[(xy >> 8) * (uint32_t)S + (xy & 255u)] = (uint8_t)kCodeEmpty;
          }
        }
        if (do_reset) {
          episode += 1u;
          start_episode(next, fam, x, y, dir, ob);
          pos = y * S + x;
          t = 0;
          carry_code = kCodeEmpty;
          carry_changed = true;
        }
        fill_grids(pending, kept, next, meta, codes, my_off, lane);
        have_next = have_next && !do_reset;
        filled = filled || do_reset;
        wave_sync();
      }

      // lanes that reset, and lanes without an env, act as 6 (no effect)
      const bool live = active && !do_reset;
      float reward = 0.0f;
      bool edge_view = false;
      uint32_t act = live ? (kActions ? act_now : bounded(pick4(pol, call & 3u), 7u)) : 6u;
      // one cell ahead: (dx, dy) by heading from two-bit fields (dx + 1, dy + 1)
      const uint32_t dir2 = 2u * (uint32_t)dir;
      const int dx = (int)((0x46u >> dir2) & 3u) - 1, dy = (int)((0x19u >> dir2) & 3u) - 1;
      const int ahead = pos + dy * S + dx;
      uint32_t front = my_codes[ahead];
      uint32_t penalty = 0;
      if (most_balls != 0 && fam == kFamDynObs && live) {
        // three actions; the cell ahead is judged before the balls move
        act = act > kForward ? kLeft : act;
        penalty = (act == kForward && front != kCodeEmpty && (front & 0x8Fu) != kGoal) ? 1u : 0u;
        move_balls(grids, kMargin + my_off, S, (int)((opaque(meta) >> 16) & 0xFF), most_balls, pos, ob,
                   opaque(seed), opaque(rid), call, kth_cell);
        front = my_codes[ahead];
      }
      const uint32_t a6 = min(act, 6u);
      const CodeAction r = act_on_code(a6, carry_code, front);
      dir = (dir + (int)((7u >> (2u * a6)) & 3u)) & 3;   // left 3, right 1
      {
        const uint32_t step = a6 == kForward ? r.ok : 0u;
        x += (int)(step & (uint32_t)dx);
        y += (int)(step & (uint32_t)dy);
        pos = step ? ahead : pos;
      }
      penalty |= r.lava;
      uint32_t goal = r.goal, ended = goal | penalty;
      if (any_missions && fam == kFamGoToDoor && live) {
        // as in k_plain
        const bool done_at = act >= 6u && is_door_code(front) && ((front >> 4) & 7u) == (ob[0] & 0xFFu);
        goal |= done_at ? 1u : 0u;
        ended |= (done_at || act == kToggle) ? 1u : 0u;
        edge_view = a6 > kForward && r.ok != 0u;   // a door toggled, possibly on the outer ring
      }
      if (a6 > kForward && r.ok) {
        my_codes[ahead] = (uint8_t)r.new_front;
        cell_changed[lane] = 1;
        const bool held = a6 != kToggle;
        carry_code = held ? (a6 == kPickup ? front : kCodeEmpty) : carry_code;
        carry_changed = carry_changed || held;
      }
      t += live ? 1 : 0;
      const uint32_t trunc = (live && t >= T) ? 1u : 0u;
      if (__ballot((goal | penalty) != 0u))
        reward = penalty ? -1.0f : (goal ? goal_reward(t, T, a.env.reward_mode) : 0.0f);
      const uint32_t flags = do_reset ? kFlagFirst : ended * kFlagTerminated | trunc * kFlagTruncated;
      const uint32_t act_rec = live ? act : kActionNone;
      done_prev = (ended | trunc) != 0u;

      const size_t row = kServe ? (size_t)(step0 + s) : (size_t)ring_row;
      if (!kServe) ring_row = ring_row + 1 == a.out.rows ? 0 : ring_row + 1;
      const size_t rec = row * rec_stride;   // index of lane 0's record
      if (kObs == 2 && o_obs && !kServe) {
        // whole-grid records, packed like the tile's grids (from g0): the
        // agents are drawn into the codes for the copy and then removed
        uint8_t* at = my_codes + pos;
        uint8_t under = 0;
        if (active) {
          under = *at;
          *at = (uint8_t)(kAgent | ((uint32_t)dir << 4));
        }
        wave_sync();   // every lane's grid writes of this step, and the agents
        uint8_t* dst = a.out.obs + row * a.out.obs_row;
        if (a.env.obs_mode == 3) emit_types(dst + g0 / 3, codes, tile_cells, lane);
        else emit_triples<true>(dst + g0, codes, tile_cells, lane);
        wave_sync();
        if (active) *at = under;
      } else if (kObs != 2 && o_obs) {
        // inactive lanes (S = 0, pose (1, 1)) read inside the guard margin
        const int at = kMargin + my_off + pos;
        if (kSplit) {
          poses[lane] = make_uint2((uint32_t)at | ((uint32_t)dir << 18) | (edge_view ? 1u << 20 : 0u),
                                   (uint32_t)x | ((uint32_t)y << 8) | ((uint32_t)S << 16) | (carry_code << 24));
        } else {
          uint32_t f[13];
          view_codes(grids, at, S, x, y, dir, carry_code, masks, __ballot(edge_view) != 0, edge_view, f, [] {});
          __builtin_amdgcn_sched_barrier(0);   // no step of the view is put off into the stores
          store_view(stage, f, lane, n_here);
          write_views(rec);
        }
      }
      if (kSplit) pair_barrier();   // grids and poses are step s's
      if (kSplit) __builtin_amdgcn_s_setprio(0);
      if (active) {
        o_reward[rec + lane] = reward;
        o_flags[rec + lane] = (uint8_t)flags;
        o_action[rec + lane] = (uint8_t)act_rec;
        if (o_mission) o_mission[rec + lane] = (uint8_t)mission_of(fam, ob[0]);
      }
      wave_sync();
    }

    if (kSplit && steps > 0) pair_barrier();   // the rows of the last step are read

    // write the chunk's final state back: the grids that changed (laid out
    // afresh, by a reset (the episode counter moved on from the one still
    // in HBM) or at admission, written by a pickup, drop or toggle, or
    // holding balls, which move every step)
    const bool dirty = active && (fresh || fam == kFamDynObs || cell_changed[lane] != 0 ||
                                  episode != a.st.episode[e]);
    emit_dirty_grids(a.st.grid + g0, tile_cells, dirty, my_off, S * S, codes, stage_words, lane);
    if (active) {
      a.st.x[e] = x;
      a.st.y[e] = y;
      a.st.dir[e] = dir;
      a.st.t[e] = t;
      if (carry_changed) a.st.carry[e] = (int32_t)carry_triple(carry_code);
      a.st.episode[e] = episode;
      a.st.done_prev[e] = done_prev ? 1 : 0;
      a.st.calls[e] = calls + (uint32_t)steps;
      *reinterpret_cast<uint4*>(a.st.obst + 16 * (size_t)e) = make_uint4(ob[0], ob[1], ob[2], ob[3]);
    }
    wave_sync();
  }
  if (kSplit && kLong && renders && lane == 0) give_back(claim);
}

// Every env's episode 0 (env_reset), tile by tile as k_fused runs them: the
// layouts are drawn a family at a time, the grids laid out in LDS and written
// as one block, the first timestep's record taken from them.  Bound by the
// fill, one env of the tile after another (hence its smaller tiles,
// reset_tile_envs), and the draws; the plain kernel,
// which did this before, wrote the grids cell by cell as three bytes each.
template <int kObs>
__global__ __launch_bounds__(kWave) void k_reset(FusedArgs a) {
  __shared__ __align__(16) uint2 masks[kObs == 2 ? 1 : kMaskEntries];
  __shared__ __align__(16) uint32_t stage_words[kViewStageBytes / 4];
  extern __shared__ __align__(16) uint8_t grids[];
  uint8_t* codes = grids + kMargin;
  const int lane = threadIdx.x;
  const int N = a.env.n;
  const int e0 = (int)blockIdx.x * a.tiles.tile_envs, e = e0 + lane;
  const int n_here = min(a.tiles.tile_envs, N - e0);
  const bool active = lane < n_here;
  if (kObs != 2) build_mask_table(masks, lane);

  uint32_t meta = 0, rid = 0;
  uint2 seed = make_uint2(0, 0);
  uint64_t goff = 0;
  if (active) {
    meta = a.env.meta[e];
    seed = a.env.seed[e];
    rid = a.env.rng_id[e];
    goff = a.env.grid_off[e];
  }
  const uint32_t fam = meta & 0xFF;
  const int S = (int)((meta >> 8) & 0xFF);
  int tile_cells;
  const int my_off = wave_excl_scan(S * S, lane, tile_cells);
  const uint64_t g0 = bcast64(goff, 0);
  Next next{};
  bool have = false;
  draw_missing<true>(next, have, active, active, meta, seed, rid, 0u, stage_words + lane);
  int x = 1, y = 1, dir = 0;
  uint32_t ob[4] = {~0u, ~0u, ~0u, ~0u};
  if (active) start_episode(next, fam, x, y, dir, ob);
  fill_grids(__ballot(active), false, next, meta, codes, my_off, lane);
  wave_sync();

  uint32_t* const stage = stage_words + kStageMargin / 4;
  if (a.out.obs && kObs == 2) {
    uint8_t* at = codes + my_off + y * S + x;
    uint8_t under = 0;
    if (active) {
      under = *at;
      *at = (uint8_t)(kAgent | ((uint32_t)dir << 4));
    }
    wave_sync();
    if (a.env.obs_mode == 3) emit_types(a.out.obs + g0 / 3, codes, tile_cells, lane);
    else emit_triples<true>(a.out.obs + g0, codes, tile_cells, lane);
    wave_sync();
    if (active) *at = under;
    wave_sync();
  } else if (a.out.obs && kObs != 2) {
    uint32_t f[13];
    view_codes(grids, kMargin + my_off + y * S + x, S, x, y, dir, kCodeEmpty, masks, false, false, f, [] {});
    store_view(stage, f, lane, n_here);
    wave_sync();
    const uint8_t* cells = reinterpret_cast<const uint8_t*>(stage);
    if (kObs == 1) emit_types(a.out.obs + (size_t)e0 * kCatBytes, cells, n_here * kCatBytes, lane);
    else emit_triples<false>(a.out.obs + (size_t)e0 * kObsBytes, cells, n_here * kCatBytes, lane);
    wave_sync();
  }
  emit_dirty_grids(a.st.grid + g0, tile_cells, active, my_off, S * S, codes, stage_words, lane);
  if (active) {
    if (a.out.reward) {
      a.out.reward[e] = 0.0f;
      a.out.flags[e] = (uint8_t)kFlagFirst;
      a.out.action[e] = (uint8_t)kActionNone;
      if (a.out.mission) a.out.mission[e] = (uint8_t)mission_of(fam, ob[0]);
    }
    a.st.x[e] = x;
    a.st.y[e] = y;
    a.st.dir[e] = dir;
    a.st.t[e] = 0;
    a.st.carry[e] = (int32_t)kCellEmpty;
    a.st.episode[e] = 0u;
    a.st.done_prev[e] = 0;
    a.st.calls[e] = 0u;
    *reinterpret_cast<uint4*>(a.st.obst + 16 * (size_t)e) = make_uint4(ob[0], ob[1], ob[2], ob[3]);
  }
}

}  // namespace

size_t fused_dynamic_lds_bytes(int32_t max_tile_cells) { return tile_lds_bytes(max_tile_cells); }

// LDS that a pair of waves needs besides: the renderer's stage and the poses
constexpr size_t kSplitLds = kViewStageBytes + kWave * sizeof(uint2);
constexpr size_t kFixedLds = kMaskEntries * sizeof(uint2) + kViewStageBytes + kMaskPatterns * sizeof(uint32_t) + kWave;
static_assert(kFixedLds + kSplitLds + sizeof(Claim) + 2 * kMargin + kWave * 32 * 32 <= 160 * 1024,
              "the largest tile fits the LDS of a compute unit");

size_t fused_lds_bytes(int32_t max_tile_cells, bool pairs) {
  return kFixedLds + (pairs ? kSplitLds : 0) + fused_dynamic_lds_bytes(max_tile_cells);
}

hipError_t launch_plain(const EnvTables& env, const StateBufs& st, const uint8_t* actions,
                        const TrajBufs& out, int32_t row, bool balls, hipStream_t stream) {
  using PlainKernel = void (*)(PlainArgs);
  static const PlainKernel kernels[2][3] = {{&k_plain<0, false>, &k_plain<1, false>, &k_plain<2, false>},
                                            {&k_plain<0, true>, &k_plain<1, true>, &k_plain<2, true>}};
  const int32_t tile_envs = launch_tile_envs(env.n);
  const PlainArgs a{env, st, actions, out, row, tile_envs};
  const int blocks = (env.n + tile_envs - 1) / tile_envs;
  hipLaunchKernelGGL(kernels[balls ? 1 : 0][out.obs ? env.obs_mode : 2], dim3(blocks), dim3(kWave), 0, stream, a);
  return hipGetLastError();
}

namespace {

using FusedKernel = void (*)(FusedArgs);

hipError_t launch_tiles(FusedKernel fn, const FusedArgs& a, int32_t blocks, int32_t threads, hipStream_t stream) {
  const size_t lds = fused_dynamic_lds_bytes(a.tiles.max_tile_cells);
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(fn, dim3(blocks), dim3(threads), lds, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fused(const EnvTables& env, const TileTables& tiles, const StateBufs& st,
                        const uint8_t* actions, int32_t k_steps,
                        const TrajBufs& out, int32_t row0, int32_t grid_blocks,
                        hipStream_t stream, ServeTile* serve, const ServeTile* host_tiles,
                        const SlotConfig* host_slots) {
  const FusedArgs a{env, tiles, st, actions, k_steps, out, row0, serve, host_tiles, host_slots};
  // serving requests record symbolic first-person observations
  const int obs = serve ? 0 : (env.obs_mode >= 2 ? 2 : env.obs_mode);
  static const FusedKernel kernels[2][3] = {
      {&k_fused<false, false, 0, false>, &k_fused<false, false, 1, false>, &k_fused<false, false, 2, false>},
      {&k_fused<true, false, 0, false>, &k_fused<true, false, 1, false>, &k_fused<true, false, 2, false>}};
  static const FusedKernel split[2][2] = {{&k_fused<false, false, 0, true>, &k_fused<false, false, 1, true>},
                                          {&k_fused<true, false, 0, true>, &k_fused<true, false, 1, true>}};
  // batches with KeyCorridor envs: connect_few (see there)
  static const FusedKernel together[2][3] = {{&k_fused<false, false, 0, false, true>, &k_fused<false, false, 1, false, true>,
                                              &k_fused<false, false, 2, false, true>},
                                             {&k_fused<true, false, 0, false, true>, &k_fused<true, false, 1, false, true>,
                                              &k_fused<true, false, 2, false, true>}};
  static const FusedKernel split_together[2][2] = {{&k_fused<false, false, 0, true, true>, &k_fused<false, false, 1, true, true>},
                                                   {&k_fused<true, false, 0, true, true>, &k_fused<true, false, 1, true, true>}};
  const int with = actions ? 1 : 0;
  const bool pair = in_pairs(grid_blocks, obs) && (serve || out.obs);
  FusedKernel fn = pair ? split[with][obs & 1] : kernels[with][obs];
  if (tiles.corridors) fn = pair ? split_together[with][obs & 1] : together[with][obs];
  if (!actions && !serve && obs == 0) {
    // pairs that take many tiles in turn: renderers counted by SIMD (claim_renderer)
    if (pair && !tiles.corridors && k_steps >= 128 && tiles.n_tiles > grid_blocks)
      fn = &k_fused<false, false, 0, true, false, true>;
    // single waves, every row of every tile 64 records from a 64-byte boundary on (emit_64_views)
    if (!pair && out.obs && k_steps > 1 && tiles.tile_envs == kWave && env.n % kWave == 0 &&
        (reinterpret_cast<uintptr_t>(out.obs) & 63u) == 0)
      fn = tiles.corridors ? &k_fused<false, false, 0, false, true, true> : &k_fused<false, false, 0, false, false, true>;
  }
  if (serve) fn = pair ? &k_fused<false, true, 0, true> : &k_fused<false, true, 0, false>;
  return launch_tiles(fn, a, grid_blocks, pair ? 2 * kWave : kWave, stream);
}

hipError_t launch_reset(const EnvTables& env, const TileTables& tiles, const StateBufs& st, const TrajBufs& out,
                        hipStream_t stream) {
  const FusedArgs a{env, tiles, st, nullptr, 0, out, 0, nullptr, nullptr, nullptr};
  static const FusedKernel kernels[3] = {&k_reset<0>, &k_reset<1>, &k_reset<2>};
  return launch_tiles(kernels[env.obs_mode >= 2 ? 2 : env.obs_mode], a, tiles.n_tiles, kWave, stream);
}

}  // namespace gx
