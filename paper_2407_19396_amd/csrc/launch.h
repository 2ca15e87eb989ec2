// launch.h -- internal interface between the host runtime (runtime.cpp) and
// the gfx950 kernels (kernels.hip).  Not part of the public C-ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <initializer_list>

namespace gx {

// Per-env static tables in device memory (structure of arrays).
struct EnvTables {
  int32_t n;
  uint32_t* meta;             // family | side << 8 | family parameter << 16
  int32_t* max_steps;         // truncation limit T >= 1
  uint2* seed;                // Philox key (lo, hi)
  uint32_t* rng_id;           // Philox counter word 0
  uint64_t* grid_off;         // byte offset of the env's [S][S][3] grid
  int32_t reward_mode;        // 0: 1 - 0.9 t/T, 1: unit reward
  int32_t obs_mode;           // 0: symbolic first person (147 B), 1: categorical first
                              // person (49 B), 2: symbolic whole grid, 3: categorical whole grid
};

// Caller-owned state (device pointers).
struct StateBufs {
  uint8_t* grid;
  int32_t *x, *y, *dir, *t, *carry;
  uint32_t* episode;
  uint8_t* done_prev;
  uint32_t* calls;     // step calls since reset: the random policy's counter
  uint8_t* obst;       // [N][16] obstacle positions (x, y per ball, 0xFF unused)
};

// Per-step outputs: row r of each buffer holds N entries.
struct TrajBufs {
  uint8_t* obs;     // [rows][N][147], [rows][N][49], or whole-grid rows of obs_row bytes; or nullptr
  float* reward;    // [rows][N]
  uint8_t* flags;   // [rows][N]
  uint8_t* action;  // [rows][N]
  int32_t rows;
  uint64_t obs_row = 0;        // bytes of one whole-grid observation row (sum 3 S^2 or sum S^2)
  uint8_t* mission = nullptr;  // [rows][N] the episode's mission (GoToDoor colour, else 0xFF), or nullptr
};

// Fused rollout tiling: tile i covers envs [i*E, i*E+E) (the last is
// ragged), E = tile_envs envs on the first E lanes of a wave (serving: 64).
struct TileTables {
  int32_t n_tiles;
  int32_t max_tile_cells;     // LDS bytes of the largest tile's code grids (sum of S^2)
  const uint2* list;          // serving: the tiles to run, else nullptr (tiles 0..n_tiles-1).  x: tile
                              // id, top bit set when admitted since the last launch; y: the steps its
                              // request has run
  int32_t tile_envs = 64;     // E, 1..64
  int32_t parts_log2 = 0;     // serving: a listed tile of 64 slots is run as 64 / E tiles; n_tiles counts
                              // these
  bool corridors = false;     // some env is a KeyCorridor
};

// Envs per tile of a launch whose caller has not chosen (env_set_tiling,
// env_set_launch): the smallest of 4, 8, 16, 32 that leaves at most one tile per
// SIMD (1024 of them), else 64.  A wave's step costs the same for one env as
// for 64 except for its records and its resets, so spare SIMDs are best given
// fewer envs each; beyond one tile per SIMD the waves share the vector unit.
// Empty 8x8, us a step in tiles of 4 / 8 / 16 / 32 / 64: 4096 envs 0.98 / 1.19 /
// 1.34 / 1.64 / 1.84, 8192 envs 2.04 / 1.20 / 1.38 / 1.64 / 1.84, 16 384 envs
// 3.9 / 2.37 / 1.41 / 1.70 / 1.87, 30 011 envs 7.7 / 4.7 / 2.54 / 1.81 / 2.10,
// 65 536 envs - / 8.8 / 4.6 / 2.90 / 1.98.
inline int32_t launch_tile_envs(int64_t n_envs) {
  for (const int32_t e : {4, 8, 16, 32})
    if ((n_envs + e - 1) / e <= 1024) return e;
  return 64;
}

// The same for resets (k_reset): at most 32.  An env's grid is laid out by its
// whole wave, one env after another, and a tile of half the size leaves LDS for
// twice the waves: 65 536 envs in tiles of 64 / 32 / 16, Empty 8x8 22.9 / 17.2 /
// 16.2 us, the uneven mix 43 / 31 / 29, FourRooms 19x19 68 / 42 / 47, all
// families 63 / 55 / 62 (most of it draws of a varying number, where a wave
// waits for its longest), 262 144 envs of the mix 102 / 89 / 83.
inline int32_t reset_tile_envs(int64_t n_envs) {
  const int32_t e = launch_tile_envs(n_envs);
  return e < 32 ? e : 32;
}

// Cells of the largest tile of a batch, for each number of envs a tile can be
// given by the rules above: add() every env's in order, then finish().
struct TileCells {
  static constexpr int32_t kSizes[5] = {4, 8, 16, 32, 64};
  int32_t sum[5] = {}, most[5] = {};
  void add(int32_t env, int32_t cells) {
    sum[0] += cells;
    for (int i = 0; i < 5 && (env & (kSizes[i] - 1)) == kSizes[i] - 1; ++i) close(i);
  }
  void finish() {
    for (int i = 0; i < 5; ++i) close(i);
  }
  int32_t of(int32_t envs) const {
    for (int i = 0; i < 5; ++i)
      if (kSizes[i] == envs) return most[i];
    return 0;
  }

 private:
  void close(int i) {   // a tile of size i ends and counts for the next size
    most[i] = sum[i] > most[i] ? sum[i] : most[i];
    if (i < 4) sum[i + 1] += sum[i];
    sum[i] = 0;
  }
};

// Envs per tile of a launch that reads or lays out every grid once (a reset, one
// step of the fused kernel): e, or less while a tile holds more than 16 384
// cells, whose LDS leaves a compute unit only a few single-wave workgroups.  us in
// tiles of 64 / 32 / 16 / 8, 262 144 envs: resets of Empty 31x31 1159 / 644 / 372
// / 291, 24x24 532 / 259 / 192 / 161, 16x16 148 / 100 / 84 / 100; one step with
// grids as types, 31x31 441 / 278 / 207 / 236, 24x24 208 / 140 / 131 / 154, 19x19
// 107 / 85 / 94 / 131, 16x16 55 / 51 / 61 / 88.
inline int32_t one_pass_tile_envs(int32_t e, const TileCells& cells) {
  while (e > TileCells::kSizes[0] && cells.of(e) > 16384) e /= 2;
  return e;
}

// Whether a launch of the fused kernel that writes records runs in pairs of waves
// (k_fused, kSplit): first-person records (obs_mode 0, 1) in up to 1024
// workgroups, one pair per SIMD at most.  With more workgroups a SIMD has its two
// waves without pairs, and a pair's second wave would only take their place:
// 262 144 mixed envs (4096 workgroups), 20 steps 190 us, in pairs 250; 90 000
// (1407) 167 against 204; 131 072 TwoRoom 8x8 envs (2048) 275 against 302.
inline bool in_pairs(int32_t blocks, int32_t obs_mode) { return blocks <= 1024 && obs_mode < 2; }

// Workgroups of a launch of k steps under the random policy, writing symbolic
// first-person records of a batch of Empty, DoorKey and FourRooms, whose caller
// has chosen none.  Long launches of many tiles drift apart and are bound by
// their record stores, which 1024 workgroups of two waves that take the tiles in
// turn write in better step.
// That holds from 128 steps on, where the turns come out even and where resets
// are rare; steps that lay out grids or move balls want the more tiles in
// flight.  ms, one workgroup per tile / 1024 in turn: 262 144 mixed envs, 128 steps
// 1.08 / 1.05, 256 steps 2.19 / 2.03, 1024 steps 8.30 / 7.47 (64 steps 0.52 /
// 0.56); Empty 8x8, 256 steps 2.13 / 1.94; 131 072 mixed, 128 steps 0.55 / 0.51;
// 90 000 mixed (1407 tiles), 256 steps 0.85 / 0.99; GoToDoor 2.85 / 3.38, lava
// 2.19 / 2.34, all families 3.52 / 4.50; mixed under given actions, whose loads
// wait for the wave's stores, 2.11 / 2.73.
inline int32_t rollout_blocks(const TileTables& tiles, int32_t k) {
  if (tiles.tile_envs != 64 || k < 128 || tiles.n_tiles <= 1024) return tiles.n_tiles;
  const int32_t turns = (tiles.n_tiles + 1023) / 1024;
  return tiles.n_tiles >= turns * 960 ? 1024 : tiles.n_tiles;
}

// Steps per launch of a rollout of n_steps of such a batch, when the caller leaves
// them to the library: 64, or up to 1024 where rollout_blocks has the tiles taken
// in turn.  256 steps in launches of 64 / in one, ms: 262 144 mixed envs 2.21 / 2.03,
// Empty 8x8 2.15 / 1.94.
inline int32_t rollout_steps(const TileTables& tiles, int32_t n_steps) {
  const int32_t k = n_steps < 1024 ? n_steps : 1024;
  return rollout_blocks(tiles, k) < tiles.n_tiles ? k : 64;
}

// Whether one step of a batch with Dynamic-Obstacles envs moves its balls in HBM
// (k_plain) rather than in the LDS of a one-step fused launch, which reads
// every grid of the batch whole.  A ball in HBM is a trip of its own, about
// what staging 40 cells costs; a step that writes records gains from LDS up to
// 4096 cells a tile.  us, fused / plain, 1 % of the envs with 4 balls: side 8,
// 262 144 envs without records 24.6 / 14.0, with 29.7 / 24.2, 4096 envs 8.1 /
// 8.7; side 16, 65 536 envs 21.4 / 12.2; side 31, 262 144 envs 472 / 44, 4096
// envs 11.6 / 9.3.  Every env with 8 balls: side 8, 262 144 envs 45 / 83, side 16
// 108 / 125, side 24 396 / 232.  All families: 262 144 envs 50 / 38, 4096 envs
// 11.9 / 12.9, without records 45 / 31 and 11.2 / 10.8.
inline bool step_in_hbm(int32_t n_envs, int64_t cells, int64_t balls, bool records) {
  const int64_t tile = launch_tile_envs(n_envs) < n_envs ? launch_tile_envs(n_envs) : n_envs;
  return tile * (cells - 40 * balls) > (records ? 4096 * (int64_t)n_envs : 0);
}

// A tile of 64 slots serving one request (device memory, 64 bytes).  The
// tile's envs are slots [tile * 64, tile * 64 + n_envs); their grids are
// contiguous from the first slot's on.  The record of the request's step r for its
// env l goes to index r * stride + l of its output buffers.
struct alignas(64) ServeTile {
  uint32_t active;     // 0: the tile is free
  uint32_t n_envs;     // 1..64
  uint8_t* obs;        // [n_steps][stride][147] or nullptr
  float* reward;       // [n_steps][stride]
  uint8_t* flags;
  uint8_t* action;
  uint32_t stride;     // envs per output row of the request
  uint32_t local0;     // request-local index of the tile's first env
  uint32_t n_steps;    // steps the request asked for
};

// Configuration of one server slot, staged in pinned host memory until the
// first launch that runs its tile copies it to the device tables.
struct SlotConfig {
  uint32_t meta;       // family | side << 8
  int32_t max_steps;
  uint2 seed;
  uint32_t rng_id;     // request-local env index
  uint32_t pad;
  uint64_t grid_off;   // byte offset of the slot's grid in the pool
};


// Whether (family, side, param) describes a valid env with side <= max_side
// (the families of Table "envs"; param: Crossings rivers, DistShift variant,
// Dynamic-Obstacles balls, KeyCorridor rows of rooms).
inline bool family_ok(int family, int side, int param, int max_side) {
  if (side > max_side || side > 32) return false;
  switch (family) {
    case 0: return side >= 4;                                  // Empty
    case 1: return side >= 5;                                  // DoorKey
    case 2: return side >= 7 && (side & 1) == 1;               // FourRooms
    case 3: return side >= 5;                                  // LavaGap
    case 4: return side >= 5 && (side & 1) == 1 && param >= 1 && param <= 8 &&
                   param <= side - 3;                          // Crossings
    case 5: return side >= 6 && (param == 1 || param == 2);    // DistShift
    case 6: return side >= 5 && param >= 1 && param <= 8 &&
                   param <= (side - 2) * (side - 2) - 2;       // Dynamic-Obstacles
    case 7: return side >= 5;                                  // GoToDoor
    case 8: return side >= 7 && (side + 2) % 3 == 0 && param >= 1 &&
                   param <= 3;                                 // KeyCorridor: side 3s - 2, R rows
    default: return false;
  }
}

// One launch of the plain kernel: one step of every env, records first person
// (obs_mode 0, 1) or none (out.obs nullptr).  balls: some env is a
// Dynamic-Obstacles.  Writes output row `row`.
hipError_t launch_plain(const EnvTables& env, const StateBufs& st, const uint8_t* actions,
                        const TrajBufs& out, int32_t row, bool balls, hipStream_t stream);

// One launch of the reset kernel: the start of episode 0 of every env, its
// first timestep in row 0 of `out` (obs may be nullptr; reward nullptr: no
// outputs at all).
hipError_t launch_reset(const EnvTables& env, const TileTables& tiles, const StateBufs& st, const TrajBufs& out,
                        hipStream_t stream);

// One launch of the fused kernel: k_steps steps of every env, state staged
// in LDS for the whole chunk; step s (0-based within the chunk) writes row
// (row0 + s) % rows.  actions: [k_steps][N] for this chunk, or nullptr.
// With serve != nullptr the tiles are requests instead (see ServeTile):
// random policy, each tile runs min(k_steps, its steps left).
hipError_t launch_fused(const EnvTables& env, const TileTables& tiles, const StateBufs& st,
                        const uint8_t* actions, int32_t k_steps,
                        const TrajBufs& out, int32_t row0, int32_t grid_blocks,
                        hipStream_t stream, ServeTile* serve = nullptr,
                        const ServeTile* host_tiles = nullptr, const SlotConfig* host_slots = nullptr);

// LDS bytes one workgroup of the fused kernel needs for a tile size (static
// tables and record stages plus the dynamic tile grids), in pairs of waves or not.
size_t fused_lds_bytes(int32_t max_tile_cells, bool pairs);

}  // namespace gx
