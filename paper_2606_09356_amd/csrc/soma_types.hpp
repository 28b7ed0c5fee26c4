// soma_types.hpp -- device-side tables of the SCMF sweep library.
//
// Shared by the kernels and the host runtime of libsoma_mi355x only.
#pragma once
#include <stdint.h>

namespace soma {

constexpr int kWave = 64;              // CDNA wavefront width
constexpr int kMaxN = 128;             // beads per chain handled by one wave (2 beads per lane)
constexpr int kPatternWords = kMaxN / 32;

// Accepted-move counters: each system owns kAcceptSlots 64-bit counters one
// cache line apart; wave w of a launch adds to slot (w mod kAcceptSlots), so
// no single address takes more than 1/kAcceptSlots of the updates.
constexpr int kAcceptSlots = 128;
constexpr int kAcceptStride = 8;          // uint64 words between slots (64 B)

enum Repr : int { REPR_F32 = 0, REPR_CELL = 1 };
enum CountW : int { COUNT_U16 = 0, COUNT_U32 = 1 };

// Device status bits, latched by the kernels and read at synchronising calls.
// (Fields are never non-finite on the device: they are affine in integer
// counts, and a frozen field array is checked on the host when it is set.)
enum StatusBits : uint32_t {
    ST_COUNT_OVERFLOW = 1u,
    ST_CELL_OVERFLOW = 4u,
    ST_INTERNAL = 8u,
    ST_PLACEMENT = 16u,     // a chain did not fit between the walls (initial walks, placement)
};

// What the check of a state set from the host finds.
enum StateBits : uint32_t { ST_BAD_VALUE = 1u, ST_BAD_OFFSET = 2u, ST_BAD_CELL = 4u, ST_BAD_WALL = 8u };
constexpr int kStateCellLimit = 1 << 22;   // |cell| of a state set from the host stays below this

// The reorder sorts chains by the block of kSortBlock^3 cells of their middle
// bead.
constexpr int kSortBlock = 4;
__host__ __device__ inline int64_t sort_blocks(int n) { return (n + kSortBlock - 1) / kSortBlock; }

// Attempts of the initial walks and of the placement to draw a chain that
// fits between walls.
constexpr int kMaxAttempts = 64;

// One system, as the kernels see it.  Offsets are in elements of the flat
// arrays shared by all systems of a context.
struct alignas(16) DevSys {
    int64_t slot_off;      // first bead slot (chains stored with an even stride 2P)
    int64_t cell_off;      // first cell of the count / field arrays
    int64_t chain_off;     // first chain of the context-wide chain arrays
    int32_t n_chains;
    int32_t N;             // beads per chain
    int32_t P;             // bead pairs per chain = ceil(N/2); lane p holds beads 2p, 2p+1
    int32_t G;             // chains per wave tile = 64 / P
    int32_t n_chains_a;    // chains [0, n_chains_a) use pat_a
    uint32_t sys_id;       // Philox counter word 3
    int32_t n[3];          // grid
    int32_t frozen;        // 1: fields come from the frozen array, else from the counts
    int32_t edge_dyadic;   // 1: every cell edge is a power of two (x * (1/edge) is exact)
    float inv_n[3];        // 1 / n, for the periodic wrap
    float edge[3];         // cell edge (FP32)
    float inv_edge[3];     // 1 / edge (FP32)
    float k_half;          // k/2 = 3(N-1)/(2 Re^2)
    float delta;           // move half-width
    float inv_P;           // 1 / P
    // omega_A = c_same nA + c_other nB + c0, omega_B = c_other nA + c_same nB + c0
    float c_same, c_other, c0;
    int64_t n_cells;
    // Storage order of the cells (counts, fluxes, frozen fields, targets):
    // bricks of 4 x 4 cells in y and z, a brick's 16 cells consecutive (one
    // 64-byte line of packed counts), bricks in the linear order of their
    // grid, whose ragged edges are padded; or, with brick_shift 0, the linear
    // order (x * ny + y) * nz + z itself.
    int32_t brick_shift;   // 2 or 0
    int32_t brick_mask;    // (1 << brick_shift) - 1
    int32_t B1, B2;        // bricks (cells) along y and z
    int64_t n_store;       // stored cells, padding included
    double r_n1, r_n2, r_B1, r_B2;   // reciprocals of n[1], n[2], B1, B2
    // chain reorder: blocks of kSortBlock^3 cells
    int64_t blk_off;       // first block of the system (context-wide)
    int32_t nb1, nb2;      // blocks along y and z
    // bond-force-biased moves (smc != 0): displacement A F + sqrt(2A) xi in
    // FP64, rejected at 0.99 cell edges; the acceptance ratio in FP32
    int32_t smc;
    float smc_Af;          // A
    float smc_inv4A;       // 1 / (4 A)
    float k_f;             // k = 3(N-1)/Re^2
    float dmax[3];         // 0.99 cell edge
    double smc_A;          // A
    double smc_s2A;        // sqrt(2 A)
    double k_spring;       // k in FP64 (the force of the proposal)
    // Coupling (Sec. 3.2): umbrella potential toward target concentration
    // fields, hard walls at z-cell faces, molecular-type conversion zones.
    int32_t umb;           // 1: omega_t gains -umb_coef * target_t(c) (the lambda phi_t/N part is in the cXX)
    float umb_coef;        // lambda / N
    int32_t walls;         // 1: trial positions outside z cells [wall_lo, wall_hi) are rejected
    int32_t wall_lo, wall_hi;
    int32_t zones;         // 1: conversion zones at the walls
    int32_t cls_array;     // 1: chain classes come from the class array (zones, or classes set by
                           //    the caller); 0: chains [0, n_chains_a) are class a
    int32_t zone_a, zone_b;            // lower / upper zone present
    int32_t zone_a_lim, zone_b_lim;    // N (wall_lo + lower width), N (wall_hi - upper width)
    alignas(16) uint32_t pat_a[kPatternWords];   // bit i: type of bead i (0 = A, 1 = B)
    alignas(16) uint32_t pat_b[kPatternWords];
};

// Stored index of cell (x, y, z).
__host__ __device__ inline int64_t stored_cell(const DevSys &S, int x, int y, int z)
{
    const int64_t b = ((int64_t)x * S.B1 + (y >> S.brick_shift)) * S.B2 + (z >> S.brick_shift);
    return (b << 2 * S.brick_shift) + ((y & S.brick_mask) << S.brick_shift) + (z & S.brick_mask);
}

// One tile of the sweep (wave, block or stream tile): everything a wave needs
// to address its beads, so that the position loads go out one scalar load
// after the kernel's arguments (they do not wait for the system table).
// Consecutive lanes of a tile hold consecutive bead pairs.
struct alignas(32) Tile {
    uint32_t sys;          // index into the system table (not the Philox system id)
    int32_t chain0;        // chain (within its system) of lane 0; stream tiles: one before that of lane 1
    int64_t slot;          // bead slot of lane 0's pair (lane l: 2 l further)
    int64_t chain;         // context-wide chain slot of chain0
    uint32_t lanes;        // see tile_word
    float inv_P;           // 1 / P
};
// lanes word: bits 0..10 number of lanes with a bead pair (stream tiles: end
// of the valid lanes), 11..17 P, 18 lane 0 is valid, 24..31 pair index of
// lane 0 within chain0 (stream tiles: plus P, counted from chain0)
__host__ __device__ inline uint32_t tile_word(uint32_t n, uint32_t P, bool first, uint32_t q)
{
    return n | P << 11 | (first ? 1u << 18 : 0u) | q << 24;
}

}  // namespace soma
