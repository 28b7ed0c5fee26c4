// soma_kernels.hip -- HIP kernels of the SCMF Monte-Carlo sweep for gfx950.
//
// The method (Sec. 2, SOMA paragraph, and Sec. 2.2 of the paper): chains
// move independently under frozen quasi-instantaneous fields; each sweep
// performs biased/Metropolis trial moves with energy evaluations, then
// rebuilds the particle density fields, then refreshes the fields.
//
// Mapping onto CDNA4
//   * One wavefront owns a tile of whole chains: lane p of a chain holds the
//     bead pair (2p, 2p+1), so a chain of N <= 128 beads fits one wave and
//     the bond neighbours of a bead sit in the same lane or the adjacent
//     lane (a whole-wave DPP shift; no barrier).
//   * Positions are SoA with chains stored at an even stride, so each lane
//     reads and writes one 8-byte pair per coordinate: fully coalesced.
//   * The even pass moves bead 2p of every lane, the odd pass bead 2p+1;
//     beads of one parity share no bond, so all lanes move at once.
//   * The fields are never stored: omega of a cell is an affine function of
//     its two counts, evaluated where a moved bead needs it (only when the
//     trial move leaves the bead's cell).
//   * The density is updated, not rebuilt: a sweep reads frozen counts (for
//     the fields) and adds -1/+1 atomically only for accepted moves that
//     change cell (about a fifth of the beads), not one atomic per bead; a
//     wave first merges its updates in LDS.  Four placements of those
//     atomics (density modes): a delta folded by a streaming kernel after
//     the sweep (0); a delta folded by the next sweep's own threads, which
//     read B[s-1] + D[s-1] (1); face fluxes, folded as their divergence
//     (2); or the second of two identical count buffers, which no gather of
//     the sweep reads, copied back afterwards (3).
//   * Tilings: wave tiles (whole chains on the lanes of one wave), block
//     tiles (whole chains packed over the waves of a workgroup) and stream
//     tiles (a system's lanes in chain order, 62 owned lanes per wave plus
//     two overlap lanes whose pairs come from a halo copy).
//   * Accepted moves are counted per tile by the wave- and stream-tile
//     kernels (a plain load and store per wave), per system with one atomic
//     per wave by the others.
//   * Philox4x32-10 is counter based: one 128-bit block per (bead, logical
//     chain, sweep, system); no RNG state lives in memory.
//   * Per system, the trial move is uniform in a cube or bond-force biased
//     ("smart", SOMA's move): the biased move draws FP64 Box-Muller normals
//     and needs the moved even beads before the odd proposals.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "soma_boxmuller.hpp"
#include "soma_launch.hpp"
#include "soma_types.hpp"

namespace soma {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64-bit
// multiplies with the key bumped by the Weyl constants between rounds.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t m0 = (uint64_t)0xD2511F53u * c.x;
        const uint64_t m1 = (uint64_t)0xCD9E8D57u * c.z;
        // three-input XOR in one instruction (truth table 0x96)
        const uint32_t nx = __builtin_amdgcn_bitop3_b32((uint32_t)(m1 >> 32), c.y, k0, 0x96);
        const uint32_t nz = __builtin_amdgcn_bitop3_b32((uint32_t)(m0 >> 32), c.w, k1, 0x96);
        c.y = (uint32_t)m1;
        c.w = (uint32_t)m0;
        c.x = nx;
        c.z = nz;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

struct Draw {
    float dx, dy, dz, u;
};

// Top 24 bits of each word: displacement = delta * ((w >> 8) - 2^23) * 2^-23
// (one FP32 multiply of exact operands), acceptance variate u = (w >> 8) 2^-24.
// delta_s = delta * 2^-23 (exact), so delta_s * m rounds exactly like
// delta * (m * 2^-23): one FP32 rounding of the same real product.
__device__ __forceinline__ Draw move_draw(uint32_t bead, uint32_t chain, uint32_t sweep,
                                          uint32_t sys, uint32_t k0, uint32_t k1, float delta_s)
{
    const uint4 w = philox4x32_10(make_uint4(bead, chain, sweep, sys), k0, k1);
    Draw d;
    d.dx = delta_s * (float)((int)(w.x >> 8) - 8388608);
    d.dy = delta_s * (float)((int)(w.y >> 8) - 8388608);
    d.dz = delta_s * (float)((int)(w.z >> 8) - 8388608);
    d.u = (float)(w.w >> 8) * 0x1p-24f;
    return d;
}

// Periodic wrap of an unwrapped cell index into [0, n); exact for |i| <= 2^23.
__device__ __forceinline__ int wrap_cell(int i, int n, float inv_n)
{
    const int q = (int)floorf((float)i * inv_n);
    int r = i - q * n;
    r = r < 0 ? r + n : r;
    r = r >= n ? r - n : r;
    return r;
}

// Wrap of i in [-n, 2n) into [0, n): exactly one of i, i + n, i - n lies in
// [0, n), and read as unsigned it is the smallest of the three (the others
// are >= n or negative).  For i outside [-n, 2n) all three are >= n, so the
// result is >= n exactly when i was out of that range.
__device__ __forceinline__ int wrap_step(int i, int n)
{
    const uint32_t u = (uint32_t)i, m = (uint32_t)n;
    return (int)min(min(u, u + m), u - m);
}

// ---------------------------------------------------------------------------
// Position representations
// ---------------------------------------------------------------------------
// The system table, the tile tables, the sweep counter and the kernel's own
// arguments are not written while a kernel runs: read through the constant
// address space, a wave-uniform address is a scalar load wherever it stands,
// also behind stores and in divergent code.
#define SOMA_CONST __attribute__((address_space(4)))
using SysPtr = const SOMA_CONST DevSys *;
using TilePtr = const SOMA_CONST Tile *;
using ArgPtr = const SOMA_CONST SweepArgs *;

__device__ __forceinline__ SysPtr sys_at(const DevSys *table, uint32_t k) { return (SysPtr)(uintptr_t)table + k; }
__device__ __forceinline__ Tile tile_at(const Tile *table, int k)
{
    const TilePtr t = (TilePtr)(uintptr_t)table + k;
    return Tile{t->sys, t->chain0, t->slot, t->chain, t->lanes, t->inv_P};
}

// The same pointer as a new value: what is read through it cannot be read
// earlier.  The sweep kernels take the arguments and system scalars of each
// of their phases through such a pointer, so that they do not hold all of
// them in SGPRs from the start (eight waves per SIMD leave a wave 72 SGPRs;
// what does not fit costs a v_writelane and v_readlanes per value: 288 of
// the 1127 vector instructions of the cell + offset stream kernel before).
template <class T>
__device__ __forceinline__ T later(T p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// Element at a byte offset from a wave-uniform base in device memory (one
// 32-bit register of address per lane).
#define SOMA_GLOBAL __attribute__((address_space(1)))
typedef float f2 __attribute__((ext_vector_type(2)));
typedef int i2 __attribute__((ext_vector_type(2)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
template <class T>
__device__ __forceinline__ T ld_off(const void *base, uint32_t off)
{
    return *(const SOMA_GLOBAL T *)((const SOMA_GLOBAL char *)base + off);
}
template <class T>
__device__ __forceinline__ void st_off(void *base, uint32_t off, T v)
{
    *(SOMA_GLOBAL T *)((SOMA_GLOBAL char *)base + off) = v;
}

// Two 32-bit words as one 64-bit value (built as a vector, the first word's
// load is widened to two words and keeps its struct in memory).
template <class T>
__device__ __forceinline__ uint64_t pair_bits(T a, T b)
{
    return (uint64_t)__builtin_bit_cast(uint32_t, a) | (uint64_t)__builtin_bit_cast(uint32_t, b) << 32;
}

struct SysView {            // the per-system scalars a wave needs (SGPR resident)
    int n0, n1, n2;
    float e0, e1, e2;
    float ie0, ie1, ie2;
    bool dyadic;            // every edge a power of two: x * (1/edge) is the exact quotient
    int B1, B2, bs, bm;     // storage order of the cells (see DevSys)
};

struct BeadF32 {
    float x, y, z;
};
struct BeadCell {
    int cx, cy, cz;
    float ox, oy, oz;
};

// Unwrapped cell indexes must stay where the float-reciprocal wrap is exact
// (|i| < 2^24); beyond 2^23 the bead is flagged and counted in cell 0.
constexpr int kCellLimit = 1 << 23;

__device__ __forceinline__ float3 bond(const BeadF32 &a, const BeadF32 &b, const SysView &)
{
    return make_float3(a.x - b.x, a.y - b.y, a.z - b.z);
}
// (the product of a small cell difference and the edge is exact, so the
// fused form rounds exactly like the separate multiply and add)
__device__ __forceinline__ float3 bond(const BeadCell &a, const BeadCell &b, const SysView &v)
{
    return make_float3(fmaf((float)(a.cx - b.cx), v.e0, a.ox - b.ox),
                       fmaf((float)(a.cy - b.cy), v.e1, a.oy - b.oy),
                       fmaf((float)(a.cz - b.cz), v.e2, a.oz - b.oz));
}

__device__ __forceinline__ BeadF32 propose(const BeadF32 &a, const Draw &d, const SysView &)
{
    return BeadF32{a.x + d.dx, a.y + d.dy, a.z + d.dz};
}

// Keep the offset in [0, edge) by whole-cell steps, each one FP32 rounding;
// an offset that rounds up to exactly one edge moves to offset 0 of the next cell.
__device__ __forceinline__ void renorm(int &c, float &o, float e)
{
    while (o < 0.0f) { o = o + e; c -= 1; }
    while (o >= e) { o = o - e; c += 1; }
}

// Lazy renormalisation of a trial offset o + d (|d| < 0.99 edge): the
// offset may lie anywhere in the window [-e, 2e); only an offset that leaves
// it moves one whole cell (one FP32 rounding), which brings it back inside.
// A bead's cell index therefore changes only after a net displacement of
// about one edge, so a sweep rewrites few cell words (renorm, which keeps
// offsets in [0, e), gives the canonical form of a new position).
__device__ __forceinline__ void renorm_window(int &c, float &o, float e)
{
    const bool lo = o < -e;
    const bool hi = o >= 2.0f * e;
    o = lo ? o + e : (hi ? o - e : o);
    c += (int)hi - (int)lo;
}

// NGP index of a bead along one axis: floor((c e + o) / e) = c + floor(o / e)
// exactly, with o in [-e, 2e).
__device__ __forceinline__ int ngp(int c, float o, float e) { return c + (int)(o >= e) - (int)(o < 0.0f); }

__device__ __forceinline__ BeadCell propose(const BeadCell &a, const Draw &d, const SysView &v)
{
    BeadCell n{a.cx, a.cy, a.cz, a.ox + d.dx, a.oy + d.dy, a.oz + d.dz};
    renorm_window(n.cx, n.ox, v.e0);
    renorm_window(n.cy, n.oy, v.e1);
    renorm_window(n.cz, n.oz, v.e2);
    return n;
}

// NGP cell of a bead: wrapped cell coordinates and the unwrapped z index
// (for walls and zones).
struct CellPos {
    int x, y, z, uz;
};

// Unwrapped NGP indexes of M beads: floor of the exact quotient x / e for the
// FP32 cell edge e.  The product with the rounded reciprocal can be one off
// next to a face when e is not a power of two (|x / e| < 2^22, so never more
// than one).  r = x - k e corrects it: one FMA, whose rounding keeps the sign
// and, for r < 2 e (a multiple of the smaller ulp), the comparison with e.
template <int M>
__device__ __forceinline__ void ngp_index(const BeadF32 (&b)[M], const SysView &v, int (&k)[M][3])
{
    float f[M][3];
#pragma unroll
    for (int j = 0; j < M; ++j) {
        f[j][0] = floorf(b[j].x * v.ie0);
        f[j][1] = floorf(b[j].y * v.ie1);
        f[j][2] = floorf(b[j].z * v.ie2);
        for (int d = 0; d < 3; ++d) k[j][d] = (int)f[j][d];
    }
    if (!v.dyadic) {
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const float r0 = fmaf(-f[j][0], v.e0, b[j].x), r1 = fmaf(-f[j][1], v.e1, b[j].y),
                        r2 = fmaf(-f[j][2], v.e2, b[j].z);
            k[j][0] += (int)(r0 >= v.e0) - (int)(r0 < 0.0f);
            k[j][1] += (int)(r1 >= v.e1) - (int)(r1 < 0.0f);
            k[j][2] += (int)(r2 >= v.e2) - (int)(r2 < 0.0f);
        }
    }
}
template <int M>
__device__ __forceinline__ void ngp_index(const BeadCell (&b)[M], const SysView &v, int (&k)[M][3])
{
#pragma unroll
    for (int j = 0; j < M; ++j) {
        k[j][0] = ngp(b[j].cx, b[j].ox, v.e0);
        k[j][1] = ngp(b[j].cy, b[j].oy, v.e1);
        k[j][2] = ngp(b[j].cz, b[j].oz, v.e2);
    }
}

// Cells of M beads, the first M0 of them stored beads, the others trial
// positions.  Beads almost always lie within one image of the box, where
// wrap_step is the wrap; the general form (and the range check) runs only
// for the lanes that need it.  A bead whose unwrapped index leaves the range
// that the general wrap handles (or whose coordinate is not finite: the
// conversion saturates) is counted in cell 0; for a stored bead of a lane
// with `report` that is flagged in *status.
template <int M0, class Bead, int M>
__device__ __forceinline__ void cells_of(const Bead (&b)[M], const SysView &v, SysPtr S, bool report,
                                         uint32_t *status, CellPos (&c)[M])
{
    int k[M][3];
    ngp_index(b, v, k);
    uint32_t m0 = 0, m1 = 0, m2 = 0;
#pragma unroll
    for (int j = 0; j < M; ++j) {
        c[j] = CellPos{wrap_step(k[j][0], v.n0), wrap_step(k[j][1], v.n1), wrap_step(k[j][2], v.n2), k[j][2]};
        m0 = max(m0, (uint32_t)c[j].x);
        m1 = max(m1, (uint32_t)c[j].y);
        m2 = max(m2, (uint32_t)c[j].z);
    }
    if (m0 >= (uint32_t)v.n0 || m1 >= (uint32_t)v.n1 || m2 >= (uint32_t)v.n2) {
        const SysPtr Q = later(S);
        const float i0 = Q->inv_n[0], i1 = Q->inv_n[1], i2 = Q->inv_n[2];
        bool bad = false;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const int lim = j < M0 ? kCellLimit - 1 : kCellLimit;
            bool in = true;
            for (int d = 0; d < 3; ++d) in = in && k[j][d] >= -lim && k[j][d] <= lim;
            if (in) {
                c[j].x = wrap_cell(k[j][0], v.n0, i0);
                c[j].y = wrap_cell(k[j][1], v.n1, i1);
                c[j].z = wrap_cell(k[j][2], v.n2, i2);
            } else {
                c[j] = CellPos{0, 0, 0, 0};
                bad = bad || j < M0;
            }
        }
        if (bad && report) atomicOr(status, ST_CELL_OVERFLOW);
    }
}

// Stored index of a cell (stored_cell; 24-bit multiplies, nx * ny <= 2^24).
// Beads of a chain and the two cells of a move are near each other in all
// directions, so bricks put more of a wave's gathers and updates into one
// 64-byte line than rows of cells do: at two beads per cell and 32-bead
// chains, after the reorder, 0.116 instead of 0.159 lines updated and 0.316
// instead of 0.393 lines gathered per bead (device atomics that leave a wave
// together for one line are one request; without any of them a sweep takes
// 14 to 30 % less).  It costs six vector instructions a cell more.  Sweeps
// with rows of cells -> with bricks: 4.2M beads FP32 50 -> 46 us, 17.2M beads
// FP32 188 -> 164 us, 124.6M beads cell + offset 1.40 -> 1.33 ms, 8192 beads
// (latency) 4.3 -> 4.4 us.
__device__ __forceinline__ int store_index(const CellPos &c, const SysView &v)
{
    const uint32_t y = (uint32_t)c.y, z = (uint32_t)c.z;
    const uint32_t b = __umul24(__umul24((uint32_t)c.x, (uint32_t)v.B1) + (y >> v.bs), (uint32_t)v.B2) + (z >> v.bs);
    return (int)((b << 2 * v.bs) | ((y & v.bm) << v.bs) | (z & v.bm));
}

// Value of the lane before (0 in lane 0) or after (0 in lane 63): a
// whole-wave DPP shift, one VALU move per word, where a shuffle goes through
// the LDS unit and its latency twice per tile.
template <int CTRL, class T>
__device__ __forceinline__ T wave_shift(T x)
{
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
constexpr int kDppShr1 = 0x138, kDppShl1 = 0x130;
template <int CTRL>
__device__ __forceinline__ BeadF32 wave_shift(const BeadF32 &a)
{
    return BeadF32{wave_shift<CTRL>(a.x), wave_shift<CTRL>(a.y), wave_shift<CTRL>(a.z)};
}
template <int CTRL>
__device__ __forceinline__ BeadCell wave_shift(const BeadCell &a)
{
    return BeadCell{wave_shift<CTRL>(a.cx), wave_shift<CTRL>(a.cy), wave_shift<CTRL>(a.cz),
                    wave_shift<CTRL>(a.ox), wave_shift<CTRL>(a.oy), wave_shift<CTRL>(a.oz)};
}

// c ? a : b, component by component and by value (unary plus: a conditional
// of two lvalues would choose between addresses and keep the beads in memory).
__device__ __forceinline__ BeadF32 pick(bool c, BeadF32 a, BeadF32 b)
{
    return BeadF32{c ? +a.x : +b.x, c ? +a.y : +b.y, c ? +a.z : +b.z};
}
__device__ __forceinline__ BeadCell pick(bool c, BeadCell a, BeadCell b)
{
    return BeadCell{c ? +a.cx : +b.cx, c ? +a.cy : +b.cy, c ? +a.cz : +b.cz,
                    c ? +a.ox : +b.ox, c ? +a.oy : +b.oy, c ? +a.oz : +b.oz};
}

// Bond neighbours of a lane's bead pair: the odd bead of the lane before
// (left) and the even bead of the lane after (right).  In block tiles a
// wave's first and last lanes take them from the neighbouring waves through
// LDS; every thread of the block calls these (they hold a barrier).
template <bool BT, class Bead>
__device__ __forceinline__ Bead left_neighbour(const Bead &b1)
{
    Bead l = wave_shift<kDppShr1>(b1);
    if constexpr (BT) {
        __shared__ Bead edge[16];
        const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
        if (lane == 63) edge[w] = b1;
        __syncthreads();
        if (lane == 0 && w > 0) l = edge[w - 1];
    }
    return l;
}
template <bool BT, class Bead>
__device__ __forceinline__ Bead right_neighbour(const Bead &b0)
{
    Bead r = wave_shift<kDppShl1>(b0);
    if constexpr (BT) {
        __shared__ Bead edge[16];
        const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
        if (lane == 0) edge[w] = b0;
        __syncthreads();
        if (lane == 63 && w + 1 < (int)(blockDim.x >> 6)) r = edge[w + 1];
    }
    return r;
}

// Positions: F32 keeps coordinates in P0..P2; CELL keeps offsets in P0..P2
// and cells in C0..C2.  `slot` is even, so pairs are 8-byte aligned.
struct PosArrays {
    float *P0, *P1, *P2;
    int *C0, *C1, *C2;
};
template <class A>
__device__ __forceinline__ PosArrays pos_arrays(const A &a) { return PosArrays{a.P0, a.P1, a.P2, a.C0, a.C1, a.C2}; }
__device__ __forceinline__ PosArrays pos_arrays(ArgPtr a) { return PosArrays{a->P0, a->P1, a->P2, a->C0, a->C1, a->C2}; }

// The pair at byte offset `off` (8 per pair) from slot `first` of each array.
// Consecutive lanes of a tile hold consecutive pairs, so `first` is uniform.
// Position lines stay in the caches between a wave's loads and its stores:
// most stored lines are partial (only changed pairs are written back) and are
// completed in the L2 from the loaded data before they reach memory.
// (Non-temporal loads or stores, which keep lines out of the caches, made the
// sweep slower.)
__device__ __forceinline__ void load_pair(const PosArrays &A, int64_t first, uint32_t off, BeadF32 &a, BeadF32 &b)
{
    const f2 x = ld_off<f2>(A.P0 + first, off), y = ld_off<f2>(A.P1 + first, off),
                 z = ld_off<f2>(A.P2 + first, off);
    a = BeadF32{x.x, y.x, z.x};
    b = BeadF32{x.y, y.y, z.y};
}
__device__ __forceinline__ void load_pair(const PosArrays &A, int64_t first, uint32_t off, BeadCell &a, BeadCell &b)
{
    const i2 cx = ld_off<i2>(A.C0 + first, off), cy = ld_off<i2>(A.C1 + first, off),
               cz = ld_off<i2>(A.C2 + first, off);
    const f2 x = ld_off<f2>(A.P0 + first, off), y = ld_off<f2>(A.P1 + first, off),
                 z = ld_off<f2>(A.P2 + first, off);
    a = BeadCell{cx.x, cy.x, cz.x, x.x, y.x, z.x};
    b = BeadCell{cx.y, cy.y, cz.y, x.y, y.y, z.y};
}
__device__ __forceinline__ void store_pair(const PosArrays &A, int64_t first, uint32_t off, const BeadF32 &a,
                                           const BeadF32 &b)
{
    st_off(A.P0 + first, off, pair_bits(a.x, b.x));
    st_off(A.P1 + first, off, pair_bits(a.y, b.y));
    st_off(A.P2 + first, off, pair_bits(a.z, b.z));
}
__device__ __forceinline__ void store_pair(const PosArrays &A, int64_t first, uint32_t off, const BeadCell &a,
                                           const BeadCell &b)
{
    st_off(A.C0 + first, off, pair_bits(a.cx, b.cx));
    st_off(A.C1 + first, off, pair_bits(a.cy, b.cy));
    st_off(A.C2 + first, off, pair_bits(a.cz, b.cz));
    st_off(A.P0 + first, off, pair_bits(a.ox, b.ox));
    st_off(A.P1 + first, off, pair_bits(a.oy, b.oy));
    st_off(A.P2 + first, off, pair_bits(a.oz, b.oz));
}
// Store what a sweep changed: nothing for a pair whose two moves were
// rejected; in cell mode, each cell word only when a bead of the pair left
// its cell along that axis (a few percent of the beads), so most cell
// sectors are never written back.
__device__ __forceinline__ void store_moved(const PosArrays &A, int64_t first, uint32_t off, const BeadF32 &a,
                                            const BeadF32 &b, const BeadF32 &, const BeadF32 &, bool moved)
{
    if (moved) store_pair(A, first, off, a, b);
}
__device__ __forceinline__ void store_moved(const PosArrays &A, int64_t first, uint32_t off, const BeadCell &a,
                                            const BeadCell &b, const BeadCell &oa, const BeadCell &ob, bool moved)
{
    if (!moved) return;
    if (a.cx != oa.cx || b.cx != ob.cx) st_off(A.C0 + first, off, pair_bits(a.cx, b.cx));
    if (a.cy != oa.cy || b.cy != ob.cy) st_off(A.C1 + first, off, pair_bits(a.cy, b.cy));
    if (a.cz != oa.cz || b.cz != ob.cz) st_off(A.C2 + first, off, pair_bits(a.cz, b.cz));
    st_off(A.P0 + first, off, pair_bits(a.ox, b.ox));
    st_off(A.P1 + first, off, pair_bits(a.oy, b.oy));
    st_off(A.P2 + first, off, pair_bits(a.oz, b.oz));
}

// ---------------------------------------------------------------------------
// Counts and fields
// ---------------------------------------------------------------------------
// U16: one uint32 per cell, A in the low half, B in the high half.
// U32: two uint32 per cell (A, B) interleaved.
template <int CW>
__device__ __forceinline__ uint2 load_counts(const uint32_t *cnt, int64_t cell)
{
    if constexpr (CW == COUNT_U16) {
        const uint32_t w = cnt[cell];
        return make_uint2(w & 0xFFFFu, w >> 16);
    } else {
        return *reinterpret_cast<const uint2 *>(cnt + 2 * cell);
    }
}

// Raw count words of one cell (and, when the fold runs inside the sweep, the
// words of the previous delta), loaded without being combined so that
// several gathers can be in flight before the first use.
struct RawCount {
    uint32_t w0, w1, d0, d1;
};

// (cnt, dprev: first count word of the wave's system; a context has fewer
// than 2^30 count words, so a byte offset fits 32 bits)
template <int CW, bool FI>
__device__ __forceinline__ RawCount load_raw(const uint32_t *cnt, const uint32_t *dprev, int cell)
{
    RawCount r{0u, 0u, 0u, 0u};
    if constexpr (CW == COUNT_U16) {
        r.w0 = ld_off<uint32_t>(cnt, (uint32_t)cell << 2);
        if constexpr (FI) r.d0 = ld_off<uint32_t>(dprev, (uint32_t)cell << 2);
    } else {
        const u2 w = ld_off<u2>(cnt, (uint32_t)cell << 3);
        r.w0 = w.x;
        r.w1 = w.y;
        if constexpr (FI) {
            const u2 d = ld_off<u2>(dprev, (uint32_t)cell << 3);
            r.d0 = d.x;
            r.d1 = d.y;
        }
    }
    return r;
}

// Counts of the cell: base plus delta in modular uint32 arithmetic; for U16
// the packed sum equals nA + 2^16 nB whenever both true counts fit 16 bits.
template <int CW>
__device__ __forceinline__ uint2 counts_of(const RawCount &r)
{
    if constexpr (CW == COUNT_U16) {
        const uint32_t w = r.w0 + r.d0;
        return make_uint2(w & 0xFFFFu, w >> 16);
    } else {
        return make_uint2(r.w0 + r.d0, r.w1 + r.d1);
    }
}

// Per-wave merge of the density changes in LDS before the device atomics.
// Device-scope atomics are executed at the memory side at a fixed rate;
// updates of one chain often hit the same count word (a chain carries a
// count along: one bead leaves a cell that another bead of the same chain
// enters), so merging a wave's updates first removes about a fifth of them.
// About a ninth of a wave's beads change cell in a sweep, so the (word, increment)
// pairs are packed into a list first (two ballots, one 16-byte LDS store per
// bead that moved) and the rest works on full lanes: each entry writes its
// lane into a byte table at its hash, reads the table back, and an entry
// that finds another entry of the same word there adds its increment to it.
// Entries whose slot went to another word are not merged, which costs an
// atomic and no retry, so there is no probe loop and no table to clear.
// (Measured against an open-addressing table with a compare-and-swap per
// update, which runs four loops on lanes that are mostly idle: 8192 beads
// 7.2 -> 5.4 us a sweep, 17.2M beads FP32 230 -> 193 us, 124.6M beads cell +
// offset 1.68 -> 1.55 ms.)  A
// wave makes at most 4 updates per lane with cell words; with face fluxes the
// beads that moved are packed into a list of records first, and every 64 of
// them give at most 3 updates each.
constexpr int kListCells = 4 * kWave;      // 2 words per entry
constexpr int kListFaces = 3 * kWave;      // the face entries of 64 records,
constexpr int kFaceRecs = 2 * kWave;       // and the records (4 words each)
constexpr int kMergeTab = 256;             // bytes of the table (one lane number per slot)
constexpr int list_words(bool faces)
{
    return (faces ? 2 * kListFaces + 4 * kFaceRecs : 2 * kListCells) + kMergeTab / 4;
}

// Multiplicative hash of the low 24 bits of the key.  The product is taken
// with the full-rate 24-bit multiply.
__device__ __forceinline__ uint32_t merge_hash(uint32_t key)
{
    uint32_t p;
    asm("v_mul_u32_u24 %0, 0x9e3779, %1" : "=v"(p) : "v"(key));
    return (p >> 10) & (kMergeTab - 1);
}

// Rank of this lane among the lanes of mask m.
__device__ __forceinline__ uint32_t lane_rank(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Append (k0, v0), (k1, v1) of the lanes with `on` to the wave's list of n
// entries (n even); returns the new length (wave-uniform).
__device__ __forceinline__ uint32_t list_push2(uint32_t *list, uint32_t n, bool on, uint32_t k0, uint32_t v0,
                                               uint32_t k1, uint32_t v1)
{
    const uint64_t m = __builtin_amdgcn_ballot_w64(on);
    if (on) *reinterpret_cast<uint4 *>(list + 2 * n + 4 * lane_rank(m)) = make_uint4(k0, v0, k1, v1);
    return n + 2u * (uint32_t)__popcll(m);
}
__device__ __forceinline__ uint32_t list_push(uint32_t *list, uint32_t n, bool on, uint32_t k, uint32_t v)
{
    const uint64_t m = __builtin_amdgcn_ballot_w64(on);
    if (on) *reinterpret_cast<uint2 *>(list + 2 * (n + lane_rank(m))) = make_uint2(k, v);
    return n + (uint32_t)__popcll(m);
}

// Merge the n entries of the wave's list and add every nonzero sum to its
// word of dst (one device atomic each; without WIDE the byte offsets fit 32
// bits).  LDS operations of one wave execute
// in order; the fences keep the compiler from reordering them.
template <bool WIDE>
__device__ __forceinline__ void list_flush(uint32_t *list, uint8_t *tab, uint32_t n, uint32_t *dst)
{
    const uint32_t lane = threadIdx.x & 63;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (uint32_t b = 0; b < n; b += kWave) {
        const uint32_t i = b + lane;
        if (i < n) {
            const uint2 e = *reinterpret_cast<const uint2 *>(list + 2 * i);
            const uint32_t h = merge_hash(e.x);
            __hip_atomic_store(tab + h, (uint8_t)lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            const uint32_t w = b + __hip_atomic_load(tab + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            const bool dup = w != i && list[2 * w] == e.x;
            if (dup) __hip_atomic_fetch_add(list + 2 * w + 1, e.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            if (!dup) {
                const uint32_t v = list[2 * i + 1];
                uint32_t *word = WIDE ? dst + e.x : reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(dst) + (e.x << 2));
                if (v != 0u) __hip_atomic_fetch_add(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// Word index and packed increment of one bead of type t in a cell.
template <int CW>
__device__ __forceinline__ uint32_t count_word(int cell, int t)
{
    return CW == COUNT_U16 ? (uint32_t)cell : 2u * (uint32_t)cell + (uint32_t)t;
}
template <int CW>
__device__ __forceinline__ uint32_t count_inc(int t)
{
    return CW == COUNT_U16 ? (t ? 0x10000u : 1u) : 1u;
}

// Fold one word: counts' = counts + delta in modular uint32 arithmetic (for
// U16 the packed sum is exact whenever both true counts fit 16 bits); returns
// true if a true count left its range (below zero, or above 65535 for packed
// 16-bit counts).
template <int CW>
__device__ __forceinline__ bool fold_word(uint32_t b, uint32_t d, uint32_t &out)
{
    out = b + d;
    if constexpr (CW == COUNT_U16) {
        const int dA = (int)(int16_t)(d & 0xFFFFu);
        const int dB = (int)(int16_t)((d - (uint32_t)dA) >> 16);
        const int nA = (int)(b & 0xFFFFu) + dA, nB = (int)(b >> 16) + dB;
        return nA < 0 || nA > 0xFFFF || nB < 0 || nB > 0xFFFF;
    } else {
        return (int)d >= 0 ? out < b : out > b;
    }
}

// Adds one bead of type t; returns true if the count overflowed its width.
template <int CW>
__device__ __forceinline__ bool scatter_count(uint32_t *cnt, int64_t cell, int t)
{
    if constexpr (CW == COUNT_U16) {
        const uint32_t old = atomicAdd(cnt + cell, t ? 0x10000u : 1u);
        return ((old >> (t ? 16 : 0)) & 0xFFFFu) == 0xFFFFu;
    } else {
        const uint32_t old = atomicAdd(cnt + 2 * cell + t, 1u);
        return old == 0xFFFFFFFFu;
    }
}

// omega_A = same nA + other nB + c0, omega_B = other nA + same nB + c0
struct FieldCoef {
    float same, other, c0;
};
__device__ __forceinline__ FieldCoef field_coef(SysPtr S) { return FieldCoef{S->c_same, S->c_other, S->c0}; }

// omega_t of a cell from its counts (affine in the counts).  The same
// function produces the fields the sweep uses and the ones soma_fields reports.
__device__ __forceinline__ float omega_of(const FieldCoef &f, uint2 n, int t)
{
    const float ca = t ? f.other : f.same, cb = t ? f.same : f.other;
    return fmaf(ca, (float)n.x, fmaf(cb, (float)n.y, f.c0));
}

// The 32 bead types from bead 32 (i / 32) of a chain of class cls, shifted so
// that bit 0 is bead i's (pat_a and pat_b are consecutive in the table; one
// per-lane load, which the wait for the positions hides, instead of eight
// SGPRs and the selects between them).
__device__ __forceinline__ uint32_t pattern_bits(SysPtr S, int cls, int i)
{
    const uint32_t off = (uint32_t)(cls * 4 + (i >> 5)) << 2;
    return ld_off<uint32_t>((const void *)(uintptr_t)S->pat_a, off) >> (i & 31);
}

// Class of a chain (which pattern it carries): from the class array when
// conversion zones (or the caller) change classes, else chains
// [0, n_chains_a) are class a.
template <bool CPL = true>
__device__ __forceinline__ int chain_cls(SysPtr S, const uint8_t *cc, uint32_t clog)
{
    if constexpr (CPL)
        if (S->cls_array) return (int)cc[S->chain_off + clog];
    return (int)clog < S->n_chains_a ? 0 : 1;
}

// The arguments that lead to the position loads, read together: a wave waits
// once for them, once for its tile (with the sweep counter and the tile's
// acceptance count) and then issues its position loads.  (Read where they
// are used, these are six dependent scalar loads, 1900 to 4000 cycles of a
// wave's 13000 to 23000.)
struct Head {
    const Tile *tiles;
    const uint64_t *ctr;
    const DevSys *systems;
    unsigned long long *acc_tile;
    int n_tiles, waves_per_block, remap;
    uint32_t rel;
    const uint32_t *chain_id;
    PosArrays pos;
    const uint2 *halo;         // stream tiles only
    int64_t halo_cap;
    int one_P, one_G, one_chains;      // the other tiles
    float one_inv_P;
};
__device__ __forceinline__ Head head_of(ArgPtr a, bool cells, bool stream)
{
    Head h{a->wtiles, a->sweep_ctr, a->systems, a->acc_tile, a->n_wtiles, a->waves_per_block, a->remap_blocks, a->rel,
           a->chain_id, pos_arrays(a), a->halo, a->halo_cap, a->one_P, a->one_G, a->one_chains, a->one_inv_P};
    asm volatile("" : "+s"(h.tiles), "+s"(h.ctr), "+s"(h.systems), "+s"(h.acc_tile), "+s"(h.n_tiles),
                      "+s"(h.waves_per_block), "+s"(h.remap), "+s"(h.rel), "+s"(h.chain_id), "+s"(h.pos.P0),
                      "+s"(h.pos.P1), "+s"(h.pos.P2));
    if (cells) asm volatile("" : "+s"(h.pos.C0), "+s"(h.pos.C1), "+s"(h.pos.C2));
    if (stream) asm volatile("" : "+s"(h.halo), "+s"(h.halo_cap));
    else asm volatile("" : "+s"(h.one_P), "+s"(h.one_G), "+s"(h.one_chains), "+s"(h.one_inv_P));
    return h;
}

// Workgroups are dispatched round-robin over the 8 XCDs; the remap gives each
// XCD a contiguous range of tiles, so its L2 sees a compact cell range.
__device__ __forceinline__ int block_index(int remap)
{
    const int bid = (int)blockIdx.x;
    return bid < remap ? (bid & 7) * (remap >> 3) + (bid >> 3) : bid;
}

// Tiling of the sweep.  Wave tiles: a tile is G = floor(64/P) whole chains on
// the lanes of one wave.  Block tiles: a tile is floor(64 W / P) whole chains
// packed over the 64 W lanes of a block, so a chain may span two waves (fewer
// idle lanes when 64 is not a multiple of P); bond neighbours across a wave
// boundary go through LDS.  Stream tiles (uniform moves, no coupling): the
// lanes of a system form one stream in chain order (chain c holds lanes
// [c P, (c + 1) P)), so chains run across wave boundaries and no lane idles
// but in a system's last wave.  Wave w moves the 62 stream lanes
// [62 w, 62 w + 62) on its lanes 1..62; lane 0 holds the stream lane before
// them and lane 63 the one after, which take every step of the sweep but
// store nothing, update no count and count no acceptance.  Lane 1's even
// bead reads lane 0's odd bead (unmoved in the even pass), and lane 62's odd
// bead reads lane 63's even bead after lane 63 has made that bead's even move
// with the same draw, stored state, frozen counts and arithmetic as the wave
// that owns it, so the same decision.  The owners of the two overlap lanes
// rewrite them during the same sweep, so the overlap lanes read them from
// the halo copy taken before the sweep (halo_index): tile w - 1's last and
// tile w + 1's first owned lane.
constexpr int TIL_WAVE = 0, TIL_BLOCK = 1, TIL_STREAM = 2;

template <int TIL>
__device__ __forceinline__ int tile_lane() { return TIL == TIL_BLOCK ? (int)threadIdx.x : (int)(threadIdx.x & 63); }

// Tile t of the launch.  A context of one system needs no table: its tiles
// follow from the arguments, one memory round trip less before the positions
// (740k beads, N = 37: 13.4 -> 12.6 us a sweep with its fold; 8192 beads and
// resident waves: no difference).
template <int TIL>
__device__ __forceinline__ Tile launch_tile(const Head &h, int t)
{
    if (TIL != TIL_STREAM && h.one_P != 0) {
        const int chain0 = t * h.one_G;
        const int n = min(h.one_G, h.one_chains - chain0);
        return Tile{0u, chain0, (int64_t)chain0 * (2 * h.one_P), (int64_t)chain0,
                    tile_word((uint32_t)(n * h.one_P), (uint32_t)h.one_P, true, 0u), h.one_inv_P};
    }
    return tile_at(h.tiles, t);
}

struct TileLane {
    int g, p;       // the lane holds beads 2p and 2p + 1 of chain chain0 + g
    bool valid;     // a bead pair of the system: takes every step
    bool own;       // and belongs to this wave: stores and counts
};

template <int TIL>
__device__ __forceinline__ TileLane lane_of(const Tile &T)
{
    const int lane = tile_lane<TIL>(), P = (int)(T.lanes >> 11 & 127u), n = (int)(T.lanes & 2047u);
    const int q = TIL == TIL_STREAM ? (int)(T.lanes >> 24) + lane : lane;
    TileLane L;
    // q / P: (q + 1/2) / P is at least 1/(2P) from an integer, far more than
    // the FP32 error of the product (q < 1024)
    L.g = (int)(((float)q + 0.5f) * T.inv_P);
    L.p = q - L.g * P;
    if constexpr (TIL == TIL_STREAM) {
        // (single unsigned comparisons; n is at least 2)
        const uint32_t first = 1u - (T.lanes >> 18 & 1u), end = (uint32_t)min(n, kStreamLanes + 1);
        L.valid = (uint32_t)lane - first < (uint32_t)n - first;
        L.own = (uint32_t)lane - 1u < end - 1u;
    } else {
        L.valid = L.own = lane < n;
    }
    return L;
}

// The tile tables (see Tile), one thread per tile.
__global__ __launch_bounds__(256) void k_make_tiles(MakeTilesArgs a)
{
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= a.n_tiles) return;
    int lo = 0, hi = a.n_sys - 1;            // the system with first[lo] <= t < first[lo + 1]
    while (lo < hi) {
        const int mid = lo + (hi - lo + 1) / 2;
        if (a.first[mid] <= t) lo = mid;
        else hi = mid - 1;
    }
    const DevSys &S = a.systems[lo];
    const int64_t w = t - a.first[lo];
    const int P = S.P;
    Tile T;
    T.sys = (uint32_t)lo;
    T.inv_P = S.inv_P;
    if (a.kind == 2) {
        // stream lane 62 w sits on lane 1; lane 0's pair is one before it
        const int64_t l0 = w * kStreamLanes, left = (int64_t)S.n_chains * P - l0;
        const int64_t c = l0 / P;
        T.chain0 = (int32_t)(c - 1);
        T.slot = S.slot_off + 2 * (l0 - 1);
        T.lanes = tile_word((uint32_t)(left + 1 < 64 ? left + 1 : 64), (uint32_t)P, w > 0, (uint32_t)(l0 - c * P + P - 1));
    } else {
        const int G = a.kind == 1 ? a.lanes / P : S.G;
        T.chain0 = (int32_t)(w * G);
        const int n = S.n_chains - T.chain0 < G ? S.n_chains - T.chain0 : G;
        T.slot = S.slot_off + (int64_t)T.chain0 * (2 * P);
        T.lanes = tile_word((uint32_t)(n * P), (uint32_t)P, true, 0u);
    }
    T.chain = S.chain_off + T.chain0;
    a.tiles[t] = T;
}

__device__ __forceinline__ SysView make_view(SysPtr S)
{
    SysView v;
    v.n0 = S->n[0]; v.n1 = S->n[1]; v.n2 = S->n[2];
    v.e0 = S->edge[0]; v.e1 = S->edge[1]; v.e2 = S->edge[2];
    v.ie0 = S->inv_edge[0]; v.ie1 = S->inv_edge[1]; v.ie2 = S->inv_edge[2];
    v.dyadic = S->edge_dyadic != 0;
    v.B1 = S->B1; v.B2 = S->B2; v.bs = S->brick_shift; v.bm = S->brick_mask;
    return v;
}

__device__ __forceinline__ float dot3(float3 a, float3 b) { return fmaf(a.x, b.x, fmaf(a.y, b.y, a.z * b.z)); }
__device__ __forceinline__ float3 add3(float3 a, float3 b) { return make_float3(a.x + b.x, a.y + b.y, a.z + b.z); }

// ---------------------------------------------------------------------------
// The sweep kernel: even pass, odd pass, density update (and, in density
// mode 1, the fold of the previous delta).  One launch per sweep for every
// system.
// ---------------------------------------------------------------------------
// The count words a sweep's field gathers read and the words its changes go
// to, by density mode.  Mode 1: the counts of sweep s are B[s-1] + D[s-1];
// this sweep adds to D[s], writes B[s] and clears D[s+1] (last read by sweep
// s-1).  Mode 2: the face fluxes of sweep s go to flux buffer s mod 2 (three
// W-word arrays).  Mode 3: the counts are B[s mod 2]; the changes go straight
// into its mirror B[(s+1) mod 2], which holds the same counts when the sweep
// starts and is read by no gather of this sweep.
template <int DM>
__device__ __forceinline__ const uint32_t *counts_in(ArgPtr a, uint64_t s)
{
    return DM == 1 ? a->base + ((s + 1) & 1) * a->count_words : (DM == 3 ? a->base + (s & 1) * a->count_words : a->base);
}
// s mod 3 in 32-bit arithmetic (2^32 mod 3 is 1).
__device__ __forceinline__ uint32_t mod3(uint64_t s) { return ((uint32_t)s % 3u + (uint32_t)(s >> 32) % 3u) % 3u; }
template <int DM>
__device__ __forceinline__ const uint32_t *delta_in(ArgPtr a, uint64_t s)
{
    return DM == 1 ? a->delta + mod3(s + 2) * a->count_words : nullptr;
}
template <int DM>
__device__ __forceinline__ uint32_t *changes_out(ArgPtr a, uint64_t s)
{
    return DM == 1   ? a->delta + mod3(s) * a->count_words
           : DM == 2 ? a->flux + (s & 1) * 3 * a->count_words
           : DM == 3 ? a->base + ((s + 1) & 1) * a->count_words
                     : a->delta;
}

// One bead pair in the halo: component k of both beads in one 8-byte word,
// the components of one side contiguous (16-byte accesses).  h: the entry of
// the wave's tile; off: byte offset of the side from there.
__device__ __forceinline__ void halo_put(uint2 *h, uint32_t off, const BeadF32 &a, const BeadF32 &b)
{
    st_off(h, off, u4{__float_as_uint(a.x), __float_as_uint(b.x), __float_as_uint(a.y), __float_as_uint(b.y)});
    st_off(h, off + 16, u2{__float_as_uint(a.z), __float_as_uint(b.z)});
}
__device__ __forceinline__ void halo_put(uint2 *h, uint32_t off, const BeadCell &a, const BeadCell &b)
{
    st_off(h, off, u4{__float_as_uint(a.ox), __float_as_uint(b.ox), __float_as_uint(a.oy), __float_as_uint(b.oy)});
    st_off(h, off + 16, u4{__float_as_uint(a.oz), __float_as_uint(b.oz), (uint32_t)a.cx, (uint32_t)b.cx});
    st_off(h, off + 32, u4{(uint32_t)a.cy, (uint32_t)b.cy, (uint32_t)a.cz, (uint32_t)b.cz});
}
// (read as one 8-byte load per component, like the pairs of the position
// arrays, so both kinds of lanes load into the same registers and the wave
// waits once for all of them)
__device__ __forceinline__ void halo_get(const uint2 *h, uint32_t off, BeadF32 &a, BeadF32 &b)
{
    const f2 x = ld_off<f2>(h, off), y = ld_off<f2>(h, off + 8), z = ld_off<f2>(h, off + 16);
    a = BeadF32{x.x, y.x, z.x};
    b = BeadF32{x.y, y.y, z.y};
}
__device__ __forceinline__ void halo_get(const uint2 *h, uint32_t off, BeadCell &a, BeadCell &b)
{
    const f2 x = ld_off<f2>(h, off), y = ld_off<f2>(h, off + 8), z = ld_off<f2>(h, off + 16);
    const i2 cx = ld_off<i2>(h, off + 24), cy = ld_off<i2>(h, off + 32), cz = ld_off<i2>(h, off + 40);
    a = BeadCell{cx.x, cy.x, cz.x, x.x, y.x, z.x};
    b = BeadCell{cx.y, cy.y, cz.y, x.y, y.y, z.y};
}
constexpr uint32_t kHaloSide = kHaloSlots * sizeof(uint2);     // bytes of one side of an entry

// Load the bead pairs of one tile and the logical chain ids, which key the
// random numbers (with the positions, so the draws do not wait for a second
// memory round trip).  Lanes without a pair of their own read another
// lane's; nothing comes of it.  The overlap lanes of a stream tile (valid
// only next to a tile of the same system: lane 0 when the tile does not
// start its system's stream, lane 63 when the stream goes on) load theirs
// from halo buffer s mod 2.
template <int TIL, class Bead>
__device__ __forceinline__ void tile_load(ArgPtr a, const Head &h, const Tile &T, int tile, uint64_t s, Bead &b0,
                                          Bead &b1, uint32_t &clog)
{
    const TileLane L = lane_of<TIL>(T);
    // (lane 1 of a stream tile is always its own; chain0 + 1 is lane 1's chain)
    const int back = TIL == TIL_STREAM ? 1 : 0;
    clog = ld_off<uint32_t>(h.chain_id + T.chain, (uint32_t)(L.valid ? L.g : back) << 2);
    const uint32_t lane = (uint32_t)tile_lane<TIL>();
    if (TIL == TIL_STREAM && L.valid && !L.own) {
        const uint2 *e = h.halo + halo_index((int)(s & 1), 0, tile, 0, h.halo_cap);
        // tile - 1, side 1 for lane 0; tile + 1, side 0 for lane 63
        halo_get(e - kHaloSlots, lane == 0 ? 0u : 3u * kHaloSide, b0, b1);
    } else {
        load_pair(h.pos, T.slot, (L.own ? lane : (uint32_t)back) * 8u, b0, b1);
    }
}

// Face fluxes of one bead that moved from cell o to cell n (wrapped
// coordinates, at most one step per axis): the move is taken axis by axis,
// x, y, then z, and each step adds the bead to the flux through one face:
// F_a(c) counts the beads that crossed from c to c + e_a, so a step -1 from
// c subtracts one from F_a(c - e_a).  Flux word of face (a, c) for type t:
// a W + word(c, t).
template <int CW>
__device__ __forceinline__ uint32_t emit_faces(uint32_t *list, uint32_t W, CellPos o, const CellPos &n, int t, bool on,
                                               const SysView &v)
{
    const uint32_t inc = count_inc<CW>(t);
    uint32_t len = 0;
    {
        const int k = n.x == o.x ? 0 : (n.x == wrap_step(o.x + 1, v.n0) ? 1 : -1);
        CellPos f = o;
        if (k < 0) f.x = n.x;
        len = list_push(list, len, on && k != 0, count_word<CW>(store_index(f, v), t), k > 0 ? inc : 0u - inc);
        o.x = n.x;
    }
    {
        const int k = n.y == o.y ? 0 : (n.y == wrap_step(o.y + 1, v.n1) ? 1 : -1);
        CellPos f = o;
        if (k < 0) f.y = n.y;
        len = list_push(list, len, on && k != 0, W + count_word<CW>(store_index(f, v), t), k > 0 ? inc : 0u - inc);
        o.y = n.y;
    }
    {
        const int k = n.z == o.z ? 0 : (n.z == wrap_step(o.z + 1, v.n2) ? 1 : -1);
        CellPos f = o;
        if (k < 0) f.z = n.z;
        len = list_push(list, len, on && k != 0, 2u * W + count_word<CW>(store_index(f, v), t), k > 0 ? inc : 0u - inc);
    }
    return len;
}

// Records of the beads that moved (grid coordinates are below 2^15).
__device__ __forceinline__ uint32_t face_push(uint32_t *recs, uint32_t n, bool on, const CellPos &o, const CellPos &f, int t)
{
    const uint64_t m = __builtin_amdgcn_ballot_w64(on);
    if (on)
        *reinterpret_cast<uint4 *>(recs + 4 * (n + lane_rank(m))) =
            make_uint4((uint32_t)o.x | (uint32_t)o.y << 16, (uint32_t)o.z | (uint32_t)t << 16,
                       (uint32_t)f.x | (uint32_t)f.y << 16, (uint32_t)f.z);
    return n + (uint32_t)__popcll(m);
}

// End of a tile: the density change of the beads whose (cell, type)
// changed -- cell words (density modes 0, 1, 3) or face fluxes (mode 2) --
// merged per wave in LDS, then one device atomic per distinct word with a
// nonzero sum; and the acceptance count (into the tile's own counter when
// acc_tile is set: acc_prev + this sweep's count).  Bead j moved from cell o_j
// with type t_j to cell f_j with type u_j (u_j != t_j only for a chain
// converted in a boundary zone, never in mode 2); m_j says that something
// changed.
template <int CW, int DM>
__device__ __forceinline__ void tile_finish(ArgPtr a, SysPtr S, int wave, uint32_t sys, uint64_t s, const SysView &v,
                                            uint32_t *list, uint8_t *tab, bool m0, const CellPos &o0,
                                            const CellPos &f0, int t0, int u0, bool m1, const CellPos &o1,
                                            const CellPos &f1, int t1, int u1, bool acc0, bool acc1,
                                            unsigned long long acc_prev)
{
    const uint32_t lane = threadIdx.x & 63;
    uint32_t *dst = changes_out<DM>(a, s) + (CW == COUNT_U16 ? 1 : 2) * S->cell_off;
    if constexpr (DM == 2) {
        uint32_t *recs = list + 2 * kListFaces;
        const uint32_t n0 = face_push(recs, 0u, m0, o0, f0, t0), n = face_push(recs, n0, m1, o1, f1, t1);
        for (uint32_t b = 0; b < n; b += kWave) {
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            const bool on = b + lane < n;
            const uint4 r = *reinterpret_cast<const uint4 *>(recs + 4 * (on ? b + lane : b));
            const CellPos o{(int)(r.x & 0xFFFFu), (int)(r.x >> 16), (int)(r.y & 0xFFFFu), 0};
            const CellPos f{(int)(r.z & 0xFFFFu), (int)(r.z >> 16), (int)r.w, 0};
            const uint32_t len = emit_faces<CW>(list, (uint32_t)a->count_words, o, f, (int)(r.y >> 16), on, v);
            list_flush<true>(list, tab, len, dst);
        }
    } else {
        uint32_t n = list_push2(list, 0u, m0, count_word<CW>(store_index(o0, v), t0), 0u - count_inc<CW>(t0),
                                count_word<CW>(store_index(f0, v), u0), count_inc<CW>(u0));
        n = list_push2(list, n, m1, count_word<CW>(store_index(o1, v), t1), 0u - count_inc<CW>(t1),
                       count_word<CW>(store_index(f1, v), u1), count_inc<CW>(u1));
        list_flush<false>(list, tab, n, dst);
    }

    const uint64_t nacc = __popcll(__builtin_amdgcn_ballot_w64(acc0)) + __popcll(__builtin_amdgcn_ballot_w64(acc1));
    if (lane == 0 && nacc) {
        if (a->acc_tile)   // this wave owns tile `wave` for the sweep
            a->acc_tile[wave] = acc_prev + nacc;
        else
            atomicAdd(a->accept + ((int64_t)sys * kAcceptSlots + (wave % kAcceptSlots)) * kAcceptStride,
                      (unsigned long long)nacc);
    }
}

// Boundary-zone conversion (Sec. 3.2, "Coupling"), after the moves of a
// sweep: a chain whose binned centre -- the mean of its beads' z-cell
// indexes, compared as the exact integer sum -- lies in the lower zone
// becomes class a, in the upper zone class b.  zf0, zf1: the final z cells of
// this lane's beads.  Returns the chain's new class; the chain's first lane
// stores it and the wave counts the conversions.
__device__ __forceinline__ int zone_convert(ArgPtr a, SysPtr S, uint32_t sys, uint32_t clog, int cls, bool active,
                                            int p, bool has1, int zf0, int zf1)
{
    const int lane = (int)(threadIdx.x & 63), P = S->P;
    int z = active ? zf0 + (has1 ? zf1 : 0) : 0;
    // segmented sum over the chain's P lanes: lane p ends with the sum over
    // [p, P) of its chain, so the chain's first lane holds the total
    for (int o = 1; o < 64; o <<= 1) {
        const int w = __shfl_down(z, o);
        if (p + o < P) z += w;
    }
    const int sum = __shfl(z, lane - p);
    int nc = cls;
    if (S->zone_a && sum < S->zone_a_lim) nc = 0;
    else if (S->zone_b && sum >= S->zone_b_lim) nc = 1;
    const bool conv = active && p == 0 && nc != cls;
    if (conv) a->chain_class[S->chain_off + clog] = (uint8_t)nc;
    const uint64_t to_a = __popcll(__ballot(conv && nc == 0)), to_b = __popcll(__ballot(conv && nc == 1));
    if (lane == 0) {
        if (to_a) atomicAdd(a->conv + 2 * sys, (unsigned long long)to_a);
        if (to_b) atomicAdd(a->conv + 2 * sys + 1, (unsigned long long)to_b);
    }
    return active ? nc : cls;
}

// Trial position outside the walls (z cell outside [wall_lo, wall_hi)).
__device__ __forceinline__ bool outside_walls(SysPtr S, int zc)
{
    return S->walls && (zc < S->wall_lo || zc >= S->wall_hi);
}

// Umbrella part of the field difference of a bead of type t between its
// trial and its old cell: -lambda/N (target_t(new) - target_t(old)).
__device__ __forceinline__ float umb_step(float coef, float2 tn, float2 to, int t)
{
    return coef * (t ? to.y - tn.y : to.x - tn.x);
}

// Field differences between the trial cells nc[j] and the old cells oc[j] of
// M beads of types t[j], where g[j]; all gathers are issued before the first
// use.
template <int CW, int DM, bool CPL, int M>
__device__ __forceinline__ void field_steps(ArgPtr a, SysPtr S, uint64_t s, const int (&nc)[M], const int (&oc)[M],
                                            const int (&t)[M], const bool (&g)[M], float (&dw)[M])
{
    const int64_t cell_off = S->cell_off;
    if (S->frozen) {
        const float2 *om = a->omega + cell_off;
        float2 wn[M], wo[M];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            wn[j] = wo[j] = make_float2(0.0f, 0.0f);
            if (g[j]) { wn[j] = om[nc[j]]; wo[j] = om[oc[j]]; }
        }
#pragma unroll
        for (int j = 0; j < M; ++j) dw[j] = t[j] ? wn[j].y - wo[j].y : wn[j].x - wo[j].x;
        return;
    }
    const uint32_t *cnt = counts_in<DM>(a, s) + (CW == COUNT_U16 ? 1 : 2) * cell_off;
    const uint32_t *dlt = DM == 1 ? delta_in<DM>(a, s) + (CW == COUNT_U16 ? 1 : 2) * cell_off : nullptr;
    const FieldCoef fc = field_coef(S);
    RawCount rn[M], ro[M];
    float2 un[M], uo[M];
    const bool umb = CPL && S->umb != 0;
#pragma unroll
    for (int j = 0; j < M; ++j) {
        rn[j] = ro[j] = RawCount{0u, 0u, 0u, 0u};
        if (g[j]) {
            rn[j] = load_raw<CW, DM == 1>(cnt, dlt, nc[j]);
            ro[j] = load_raw<CW, DM == 1>(cnt, dlt, oc[j]);
        }
        if constexpr (CPL) {
            un[j] = uo[j] = make_float2(0.0f, 0.0f);
            if (umb && g[j]) { un[j] = a->tgt[cell_off + nc[j]]; uo[j] = a->tgt[cell_off + oc[j]]; }
        }
    }
#pragma unroll
    for (int j = 0; j < M; ++j) {
        dw[j] = g[j] ? omega_of(fc, counts_of<CW>(rn[j]), t[j]) - omega_of(fc, counts_of<CW>(ro[j]), t[j]) : 0.0f;
        if constexpr (CPL)
            if (umb) dw[j] += umb_step(S->umb_coef, un[j], uo[j], t[j]);
    }
}

// One tile of the sweep: the even pass, the odd pass and the density change,
// from positions already loaded by tile_load.
//
// What bounds it: with FP32 positions in the 256 MB memory-side cache, vector
// issue and the latency of one wave's chain of loads (8 waves per SIMD are the
// most there are); with cell + offset positions beyond that cache, memory
// (36 to 48 bytes a bead).  Hence: scalars in SGPRs but only while they are
// needed (`later`), 32-bit lane offsets from uniform bases, one range check
// for all four cells, DPP instead of LDS shuffles, and the head of the chain
// read in two scalar round trips (Head, Tile).  Against a form without these
// (64-bit lane addresses, cells one by one, scalars read at the top): 745 ->
// 480 vector instructions a wave for FP32, 967 -> 590 for cell + offset;
// 4.2M beads FP32 59.7 -> 56.1 us a sweep, 124.6M beads cell + offset 1.55
// -> 1.48 ms, smart moves on 4.2M beads 100 -> 90 us.
template <int CW, int DM, bool CPL, int TIL, class Bead>
__device__ __forceinline__ void sweep_tile(ArgPtr a, SysPtr S, const Tile &T, int wave, uint64_t s, uint32_t *list,
                                           uint8_t *tab, const Bead b0, const Bead b1, uint32_t clog,
                                           unsigned long long acc_prev = 0ull)
{
    constexpr bool BT = TIL == TIL_BLOCK;
    const uint32_t sys = T.sys;
    const SysView v = make_view(S);
    const TileLane L = lane_of<TIL>(T);
    const bool valid = L.valid, own = L.own;
    const int N = S->N, p = L.p;
    const int i0 = 2 * p, i1 = 2 * p + 1;
    const bool has1 = valid && i1 < N;

    // the logical chain id keys the random numbers and picks the species, so
    // results do not depend on where a chain sits in memory
    const int cls = chain_cls<CPL>(S, a->chain_class, clog);
    const uint32_t pat = pattern_bits(S, cls, i0);
    const uint32_t k0 = (uint32_t)a->seed, k1 = (uint32_t)(a->seed >> 32);
    const float delta_s = S->delta * 0x1p-23f;
    const Draw d0 = move_draw((uint32_t)i0, clog, (uint32_t)s, S->sys_id, k0, k1, delta_s);
    const Draw d1 = move_draw((uint32_t)i1, clog, (uint32_t)s, S->sys_id, k0, k1, delta_s);

    // Both trial positions are known before either pass (the odd bead's
    // proposal does not depend on the even pass), so the fields of all four
    // cells are gathered together: one memory latency instead of two.
    const Bead n0 = propose(b0, d0, v);
    const Bead n1 = propose(b1, d1, v);
    CellPos c[4];
    {
        const Bead all[4] = {b0, b1, n0, n1};
        cells_of<2>(all, v, S, own, a->status, c);
    }
    const int t[2] = {(int)(pat & 1u), (int)((pat >> 1) & 1u)};
    const int oc[2] = {store_index(c[0], v), store_index(c[1], v)}, nc[2] = {store_index(c[2], v), store_index(c[3], v)};
    const ArgPtr ag = later(a);
    const SysPtr Sg = later(S);
    // walls: a trial position outside the slab is rejected (and needs no field)
    const bool out0 = CPL && outside_walls(Sg, c[2].uz), out1 = CPL && outside_walls(Sg, c[3].uz);
    const bool g[2] = {valid && nc[0] != oc[0] && !out0, has1 && nc[1] != oc[1] && !out1};
    float dw[2];
    field_steps<CW, DM, CPL>(ag, Sg, s, nc, oc, t, g, dw);
    const float kh = Sg->k_half;
    const float3 zero = make_float3(0.0f, 0.0f, 0.0f);

    // even pass: bead 2p, neighbours 2p-1 (previous lane's odd bead) and 2p+1.
    // dE_b = (k/2) sum_j [2 d.(r - r_j) + |d|^2] = (k/2) [2 d.sum_j (r - r_j) + n_j |d|^2]
    bool acc0;
    {
        const Bead left = left_neighbour<BT>(b1);
        const float3 de = bond(n0, b0, v);
        const float3 bl = p > 0 ? bond(b0, left, v) : zero, br = i1 < N ? bond(b0, b1, v) : zero;
        const float nj = (p > 0 ? 1.0f : 0.0f) + (i1 < N ? 1.0f : 0.0f);
        const float dE = fmaf(fmaf(2.0f, dot3(de, add3(bl, br)), nj * dot3(de, de)), kh, dw[0]);
        acc0 = valid && !out0 && (d0.u < __expf(-dE));
    }
    const Bead e0 = pick(acc0, n0, b0);
    // odd pass: bead 2p+1, neighbours 2p (this lane, updated) and 2p+2 (next lane)
    bool acc1;
    {
        const Bead right = right_neighbour<BT>(e0);
        const float3 de = bond(n1, b1, v);
        const float3 br = i1 + 1 < N ? bond(b1, right, v) : zero;
        const float nj = i1 + 1 < N ? 2.0f : 1.0f;
        const float dE = fmaf(fmaf(2.0f, dot3(de, add3(bond(b1, e0, v), br)), nj * dot3(de, de)), kh, dw[1]);
        acc1 = has1 && !out1 && (d1.u < __expf(-dE));
    }
    const Bead e1 = pick(acc1, n1, b1);
    const ArgPtr as = later(a);
    const SysPtr Ss = later(S);
    const uint32_t lane = (uint32_t)tile_lane<TIL>();
    store_moved(pos_arrays(as), T.slot, lane * 8u, e0, e1, b0, b1, own && (acc0 || acc1));
    if constexpr (TIL == TIL_STREAM) {
        // the end lanes' pairs for the overlap lanes of the next sweep
        if (own && (lane == 1 || lane == (uint32_t)kStreamLanes))
            halo_put(as->halo + halo_index((int)((s + 1) & 1), 0, wave, 0, as->halo_cap), lane == 1 ? 0u : kHaloSide, e0,
                     e1);
    }
    // final cells: without coupling a change implies an accepted move, so the
    // trial cells serve (and the selection costs no registers)
    const CellPos f0 = CPL ? (acc0 ? c[2] : c[0]) : c[2], f1 = CPL ? (acc1 ? c[3] : c[1]) : c[3];
    int u0 = t[0], u1 = t[1];
    if (CPL && !BT && Ss->zones) {   // (the host never packs contexts with zones)
        const int ncls = zone_convert(as, Ss, sys, clog, cls, valid, p, has1, f0.uz, f1.uz);
        const uint32_t np = pattern_bits(Ss, ncls, i0);
        u0 = (int)(np & 1u);
        u1 = (int)((np >> 1) & 1u);
    }
    const bool own1 = own && has1;
    tile_finish<CW, DM>(as, Ss, BT ? wave * 16 + (int)(threadIdx.x >> 6) : wave, sys, s, v, list, tab,
                        own && ((acc0 && nc[0] != oc[0]) || (CPL && u0 != t[0])), c[0], f0, t[0], u0,
                        own1 && ((acc1 && nc[1] != oc[1]) || (CPL && u1 != t[1])), c[1], f1, t[1], u1, own && acc0,
                        own1 && acc1, acc_prev);
}

// Fill halo buffer a.buf from the position arrays: one thread per stream
// tile and end lane (side 0: lane 1, side 1: lane 62), for the lanes that
// belong to their system.
template <class Bead>
__global__ __launch_bounds__(256) void k_stream_halo(HaloArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * (int64_t)a.n_ptiles) return;
    const int64_t tile = i >> 1;
    const int side = (int)(i & 1);
    const Tile T = a.ptiles[tile];
    const int lane = side == 0 ? 1 : kStreamLanes;
    if (lane >= (int)(T.lanes & 2047u)) return;
    Bead b0, b1;
    load_pair(pos_arrays(a), T.slot + 2 * lane, 0u, b0, b1);
    halo_put(a.halo + halo_index(a.buf, 0, tile, side, a.halo_cap), 0u, b0, b1);
}

// ---------------------------------------------------------------------------
// Bond-force-biased ("smart") moves (Sec. 2; Rossky, Doll and Friedman 1978)
// ---------------------------------------------------------------------------
// Three standard normals by Box-Muller (FP64) on the Philox block with counter
// (bead, chain, sweep, system): words 0, 1 give the first two, words 2, 3 the
// third; the acceptance variate is word 0 of the block with counter
// (bead + 256, chain, sweep, system) (beads are numbered below 128).
__device__ __forceinline__ void smc_draw(uint32_t bead, uint32_t chain, uint32_t sweep, uint32_t sys,
                                         uint32_t k0, uint32_t k1, double xi[3], float &u)
{
    const uint4 w = philox4x32_10(make_uint4(bead, chain, sweep, sys), k0, k1);
    box_muller3(w.x, w.y, w.z, w.w, xi);
    const uint4 w2 = philox4x32_10(make_uint4(bead + 256u, chain, sweep, sys), k0, k1);
    u = (float)(w2.x >> 8) * 0x1p-24f;
}

// Position in FP64 from the stored representation (exact for FP32; cell
// mode: cell * edge + offset with the FP32 edge).
__device__ __forceinline__ double3 pos64(const BeadF32 &a, const SysView &)
{
    return make_double3((double)a.x, (double)a.y, (double)a.z);
}
__device__ __forceinline__ double3 pos64(const BeadCell &a, const SysView &v)
{
    return make_double3((double)a.cx * (double)v.e0 + (double)a.ox, (double)a.cy * (double)v.e1 + (double)a.oy,
                        (double)a.cz * (double)v.e2 + (double)a.oz);
}

// One smart move of bead b with neighbours nl (if hl) and nr (if hr), which
// hold still.  Returns the trial state and whether the displacement stays
// below 0.99 cell edges; F gets the bond force at b (FP64).
template <class Bead>
__device__ __forceinline__ Bead smc_propose(const Bead &b, const Bead &nl, bool hl, const Bead &nr, bool hr,
                                            SysPtr S, const SysView &v, const double xi[3], double3 &F,
                                            bool &inside)
{
    const double3 r = pos64(b, v);
    double fx = 0.0, fy = 0.0, fz = 0.0;
    if (hl) {
        const double3 q = pos64(nl, v);
        fx += q.x - r.x; fy += q.y - r.y; fz += q.z - r.z;
    }
    if (hr) {
        const double3 q = pos64(nr, v);
        fx += q.x - r.x; fy += q.y - r.y; fz += q.z - r.z;
    }
    F = make_double3(S->k_spring * fx, S->k_spring * fy, S->k_spring * fz);
    Draw d;
    d.dx = (float)(S->smc_A * F.x + S->smc_s2A * xi[0]);
    d.dy = (float)(S->smc_A * F.y + S->smc_s2A * xi[1]);
    d.dz = (float)(S->smc_A * F.z + S->smc_s2A * xi[2]);
    d.u = 0.0f;
    // a displacement of 0.99 cell edges or more is rejected: the condition is
    // symmetric in r and r', so detailed balance holds, and a kept trial move
    // changes each cell index by at most one
    inside = fabsf(d.dx) < S->dmax[0] && fabsf(d.dy) < S->dmax[1] && fabsf(d.dz) < S->dmax[2];
    if (!inside) d.dx = d.dy = d.dz = 0.0f;
    return propose(b, d, v);
}

// log of q(r'->r) / q(r->r') for q(r->r') ~ exp(-|r'-r-A F(r)|^2 / (4A)),
// with de the stored displacement and F(r') = F(r) - k n_nb de (FP32).
__device__ __forceinline__ float smc_log_ratio(SysPtr S, float3 de, double3 F, int n_nb)
{
    const float A = S->smc_Af, kn = S->k_f * (float)n_nb;
    const float fx = (float)F.x, fy = (float)F.y, fz = (float)F.z;
    const float3 f = make_float3(de.x - A * fx, de.y - A * fy, de.z - A * fz);
    const float3 r = make_float3(de.x + A * (fx - kn * de.x), de.y + A * (fy - kn * de.y), de.z + A * (fz - kn * de.z));
    return (dot3(f, f) - dot3(r, r)) * S->smc_inv4A;
}

// One wave tile with smart moves.  The odd bead's proposal depends on the
// even pass (its bond force uses the moved even beads), so the two passes
// gather their fields one after the other.
template <int CW, int DM, bool CPL, int TIL, class Bead>
__device__ __forceinline__ void sweep_tile_smc(ArgPtr a, SysPtr S, const Tile &T, int wave, uint64_t s,
                                               uint32_t *list, uint8_t *tab, const Bead b0, const Bead b1,
                                               uint32_t clog)
{
    constexpr bool BT = TIL == TIL_BLOCK;
    const SysView v = make_view(S);
    const TileLane L = lane_of<TIL>(T);
    const bool active = L.valid;
    const int N = S->N, p = L.p;
    const int i0 = 2 * p, i1 = 2 * p + 1;
    const bool has1 = active && i1 < N;
    const int cls = chain_cls<CPL>(S, a->chain_class, clog);
    const uint32_t pat = pattern_bits(S, cls, i0);
    const int t0 = (int)(pat & 1u), t1 = (int)((pat >> 1) & 1u);
    const uint32_t k0 = (uint32_t)a->seed, k1 = (uint32_t)(a->seed >> 32);
    const float kh = S->k_half;
    CellPos c[2];
    {
        const Bead all[2] = {b0, b1};
        cells_of<2>(all, v, S, active, a->status, c);
    }
    const int old0 = store_index(c[0], v), old1 = store_index(c[1], v);

    // even pass: bead 2p, neighbours 2p-1 (previous lane's odd bead) and 2p+1
    bool acc0;
    Bead e0, e1;   // the pair after its moves
    int nc0;
    CellPos s0;
    {
        double xi[3];
        float u;
        smc_draw((uint32_t)i0, clog, (uint32_t)s, S->sys_id, k0, k1, xi, u);
        const Bead left = left_neighbour<BT>(b1);
        const bool hl = p > 0, hr = i1 < N;
        double3 F;
        bool inside;
        const Bead trial[1] = {smc_propose(b0, left, hl, b1, hr, S, v, xi, F, inside)};
        CellPos tc[1];
        cells_of<0>(trial, v, S, false, a->status, tc);
        s0 = tc[0];
        nc0 = store_index(s0, v);
        if (CPL) inside = inside && !outside_walls(S, s0.uz);
        const int nc[1] = {nc0}, oc[1] = {old0}, t[1] = {t0};
        const bool g[1] = {active && inside && nc0 != old0};
        float dw[1];
        field_steps<CW, DM, CPL>(a, S, s, nc, oc, t, g, dw);
        const float3 de = bond(trial[0], b0, v);
        const float dd = dot3(de, de);
        float dE = 0.0f;
        if (hl) dE += 2.0f * dot3(de, bond(b0, left, v)) + dd;
        if (hr) dE += 2.0f * dot3(de, bond(b0, b1, v)) + dd;
        dE = dE * kh + dw[0] - smc_log_ratio(S, de, F, (hl ? 1 : 0) + (hr ? 1 : 0));
        acc0 = active && inside && (u < __expf(-dE));
        e0 = pick(acc0, trial[0], b0);
    }
    // odd pass: bead 2p+1, neighbours 2p (this lane, moved) and 2p+2 (next lane)
    bool acc1;
    int nc1;
    CellPos s1;
    {
        double xi[3];
        float u;
        smc_draw((uint32_t)i1, clog, (uint32_t)s, S->sys_id, k0, k1, xi, u);
        const Bead right = right_neighbour<BT>(e0);
        const bool hr = i1 + 1 < N;
        double3 F;
        bool inside;
        const Bead trial[1] = {smc_propose(b1, e0, true, right, hr, S, v, xi, F, inside)};
        CellPos tc[1];
        cells_of<0>(trial, v, S, false, a->status, tc);
        s1 = tc[0];
        nc1 = store_index(s1, v);
        if (CPL) inside = inside && !outside_walls(S, s1.uz);
        const int nc[1] = {nc1}, oc[1] = {old1}, t[1] = {t1};
        const bool g[1] = {has1 && inside && nc1 != old1};
        float dw[1];
        field_steps<CW, DM, CPL>(a, S, s, nc, oc, t, g, dw);
        const float3 de = bond(trial[0], b1, v);
        const float dd = dot3(de, de);
        float dE = 2.0f * dot3(de, bond(b1, e0, v)) + dd;
        if (hr) dE += 2.0f * dot3(de, bond(b1, right, v)) + dd;
        dE = dE * kh + dw[0] - smc_log_ratio(S, de, F, 1 + (hr ? 1 : 0));
        acc1 = has1 && inside && (u < __expf(-dE));
        e1 = pick(acc1, trial[0], b1);
    }
    store_moved(pos_arrays(a), T.slot, (uint32_t)tile_lane<TIL>() * 8u, e0, e1, b0, b1,
                active && (acc0 || acc1));
    // final cells: without coupling a change implies an accepted move, so the
    // trial cells serve (and the selection costs no registers)
    const CellPos f0 = CPL ? (acc0 ? s0 : c[0]) : s0, f1 = CPL ? (acc1 ? s1 : c[1]) : s1;
    int u0 = t0, u1 = t1;
    if (CPL && !BT && S->zones) {   // (the host never packs contexts with zones)
        const int ncls = zone_convert(a, S, T.sys, clog, cls, active, p, has1, f0.uz, f1.uz);
        const uint32_t np = pattern_bits(S, ncls, i0);
        u0 = (int)(np & 1u);
        u1 = (int)((np >> 1) & 1u);
    }
    tile_finish<CW, DM>(a, S, BT ? wave * 16 + (int)(threadIdx.x >> 6) : wave, T.sys, s, v, list, tab,
                        active && ((acc0 && nc0 != old0) || u0 != t0), c[0], f0, t0, u0,
                        has1 && ((acc1 && nc1 != old1) || u1 != t1), c[1], f1, t1, u1, acc0, acc1, 0ull);
}

// The sweep kernel: one launch per sweep for every system.  With one tile
// per wave (the default) wave w moves tile w; with a resident grid (fewer
// waves) the waves walk the tiles grid-stride, each prefetching its next
// tile's positions.  One tile's state is live at a
// time, which keeps the register count (and so the occupancy) of the
// one-tile case.  With FI every thread also folds count words of the
// previous sweep: the first word's loads are issued before the move work
// and its stores after it, so they overlap.
template <int R, int CW, bool LOOP, int DM, bool SMC, bool CPL, int TIL>
__device__ __forceinline__ void sweep_body(ArgPtr a)
{
    using Bead = typename std::conditional<R == REPR_F32, BeadF32, BeadCell>::type;
    constexpr bool FI = DM == 1;
    const Head h = head_of(a, R == REPR_CELL, TIL == TIL_STREAM);
    // (wave-uniform; readfirstlane lets the tables be read with scalar loads)
    const int bid = block_index(h.remap);
    const int wave = __builtin_amdgcn_readfirstlane(
        TIL == TIL_BLOCK ? bid : bid * h.waves_per_block + (int)(threadIdx.x >> 6));
    const bool mine = wave < h.n_tiles;
    // the tile, the sweep counter and the tile's acceptance count (see
    // counts_per_tile; acc_tile is null for the other kernels) together
    Tile T = launch_tile<TIL>(h, mine ? wave : 0);
    uint64_t s = *(const SOMA_CONST uint64_t *)(uintptr_t)h.ctr;
    const bool per_tile = !LOOP && TIL != TIL_BLOCK && h.acc_tile != nullptr && mine;
    unsigned long long accp = *(const SOMA_CONST unsigned long long *)(per_tile ? (uintptr_t)(h.acc_tile + wave) : (uintptr_t)h.ctr);
    asm volatile("" : "+s"(T.sys), "+s"(T.chain0), "+s"(T.slot), "+s"(T.chain), "+s"(T.lanes), "+s"(T.inv_P), "+s"(s),
                      "+s"(accp));
    s += h.rel;
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // this wave's list of density changes and its merge table
    HIP_DYNAMIC_SHARED(uint32_t, agg_lds)
    uint32_t *list = agg_lds + (threadIdx.x >> 6) * list_words(DM == 2);
    uint8_t *tab = reinterpret_cast<uint8_t *>(list + list_words(DM == 2) - kMergeTab / 4);
    const int64_t W = FI || DM == 2 ? a->count_words : 0;
    const uint32_t *cin = FI ? counts_in<DM>(a, s) : nullptr, *dprev = FI ? delta_in<DM>(a, s) : nullptr;
    uint32_t fb = 0u, fd = 0u;
    if constexpr (FI) {
        if (gtid < W) {
            fb = cin[gtid];
            fd = dprev[gtid];
        }
    }
    if constexpr (LOOP) {
        // Resident waves walk the tiles grid-stride (wave, wave + n_waves,
        // ...), so the tiles in flight at any time are neighbours in the
        // spatial chain order and their field gathers share the L2.  Software
        // pipeline: the positions of a wave's next tile are loaded before
        // the current tile's field gathers, so their latency overlaps the
        // current tile's work.
        const int n_waves = (int)gridDim.x * h.waves_per_block;
        Bead nb0, nb1;
        uint32_t nclog = 0u;
        Tile NT = T;
        if (mine) tile_load<TIL>(a, h, NT, wave, s, nb0, nb1, nclog);
        for (int t = wave; t < h.n_tiles; t += n_waves) {
            const Bead b0 = nb0, b1 = nb1;
            const uint32_t clog = nclog;
            const Tile C = NT;
            if (t + n_waves < h.n_tiles) {
                NT = launch_tile<TIL>(h, t + n_waves);
                tile_load<TIL>(a, h, NT, t + n_waves, s, nb0, nb1, nclog);
            }
            const SysPtr S = sys_at(h.systems, C.sys);
            if (SMC && S->smc)
                sweep_tile_smc<CW, DM, CPL, TIL>(a, S, C, t, s, list, tab, b0, b1, clog);
            else
                sweep_tile<CW, DM, CPL, TIL>(a, S, C, t, s, list, tab, b0, b1, clog);
        }
    } else {
        // block tiles: the test is uniform over the block, so every thread
        // of a working block reaches the barriers of the tile
        if (mine) {
            Bead b0, b1;
            uint32_t clog;
            tile_load<TIL>(a, h, T, wave, s, b0, b1, clog);
            const SysPtr S = sys_at(h.systems, T.sys);
            if (SMC && S->smc)
                sweep_tile_smc<CW, DM, CPL, TIL>(a, S, T, wave, s, list, tab, b0, b1, clog);
            else
                sweep_tile<CW, DM, CPL, TIL>(a, S, T, wave, s, list, tab, b0, b1, clog, accp);
        }
    }
    if constexpr (FI) {
        uint32_t *bcur = a->base + (s & 1) * W;
        uint32_t *dnext = a->delta + mod3(s + 1) * W;
        const int64_t nthreads = (int64_t)gridDim.x * blockDim.x;
        bool ovf = false;
        if (gtid < W) {
            uint32_t w;
            ovf |= fold_word<CW>(fb, fd, w);
            bcur[gtid] = w;
            dnext[gtid] = 0u;
        }
        for (int64_t i = gtid + nthreads; i < W; i += nthreads) {
            uint32_t w;
            ovf |= fold_word<CW>(cin[i], dprev[i], w);
            bcur[i] = w;
            dnext[i] = 0u;
        }
        if (ovf) atomicOr(a->status, ST_COUNT_OVERFLOW);
    }
    if constexpr (DM == 2) {
        // clear the flux buffer of sweep s + 1 (folded after sweep s - 1);
        // its 3 W words are a multiple of 4 and 16-byte aligned
        uint4 *fn = reinterpret_cast<uint4 *>(a->flux + ((s + 1) & 1) * 3 * W);
        const int64_t n4 = 3 * W / 4, nthreads = (int64_t)gridDim.x * blockDim.x;
        for (int64_t i = gtid; i < n4; i += nthreads) fn[i] = make_uint4(0u, 0u, 0u, 0u);
    }
}

// (the body reads the arguments through the kernel argument segment, see
// `later`; they are the first and only explicit argument)
template <int R, int CW, bool LOOP, int DM, bool SMC, bool CPL, bool BT>
__global__ __launch_bounds__(1024) void k_sweep(SweepArgs)
{
    sweep_body<R, CW, LOOP, DM, SMC, CPL, BT ? TIL_BLOCK : TIL_WAVE>((ArgPtr)__builtin_amdgcn_kernarg_segment_ptr());
}

// The plain one-tile-per-wave sweep (uniform moves, no coupling) fits in 64
// VGPRs: it asks for eight waves per SIMD, the most a SIMD holds (see
// `later` for the SGPRs).
template <int R, int CW, int DM>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_sweep_plain(SweepArgs)
{
    sweep_body<R, CW, false, DM, false, false, TIL_WAVE>((ArgPtr)__builtin_amdgcn_kernarg_segment_ptr());
}

// Stream tiles, with the same register budget.
template <int R, int CW, int DM>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_sweep_stream(SweepArgs)
{
    sweep_body<R, CW, false, DM, false, false, TIL_STREAM>((ArgPtr)__builtin_amdgcn_kernarg_segment_ptr());
}

// i = (x * n1 + y) * n2 + z back into its parts, with the FP64 reciprocals r1,
// r2 and one correction step (exact: i < 2^31), not by integer division.
__device__ __forceinline__ void split_cell(int i, int n1, int n2, double r1, double r2, int &x, int &y, int &z)
{
    int r = (int)((double)i * r2);
    z = i - r * n2;
    if (z < 0) { z += n2; --r; } else if (z >= n2) { z -= n2; ++r; }
    x = (int)((double)r * r1);
    y = r - x * n1;
    if (y < 0) { y += n1; --x; } else if (y >= n1) { y -= n1; ++x; }
}
// Stored index of the cell with linear index c.
__device__ __forceinline__ int64_t stored_of_linear(const DevSys &S, int64_t c)
{
    if (S.brick_shift == 0) return c;
    int x, y, z;
    split_cell((int)c, S.n[1], S.n[2], S.r_n1, S.r_n2, x, y, z);
    return stored_cell(S, x, y, z);
}
// Cell of a stored index (y, z may lie in the padding).
__device__ __forceinline__ void cell_of_stored(const DevSys &S, int64_t c, int &x, int &y, int &z)
{
    const int bs = S.brick_shift;
    split_cell((int)(c >> 2 * bs), S.B1, S.B2, S.r_B1, S.r_B2, x, y, z);
    y = (y << bs) + (int)(c >> bs & S.brick_mask);
    z = (z << bs) + (int)(c & S.brick_mask);
}

__global__ __launch_bounds__(256) void k_store_pairs(const DevSys *sys, int64_t n_cells, const float *in, float2 *out)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < n_cells) out[stored_of_linear(*sys, c)] = make_float2(in[c], in[n_cells + c]);
}

// Density mode 2: counts += divergence of the face fluxes of sweep s, per
// cell c of one system: n(c) += sum_a F_a(c - e_a) - F_a(c) (modular uint32,
// both species at once for packed counts), with the range check of the
// other folds.  (The sweep kernel of sweep s + 1 clears these fluxes.)  One
// block per chunk of kFoldChunk stored cells of one system.
//
// Memory bound (the counts and three flux arrays read, the counts written).
// With bricks a thread takes one row of four cells: the row itself, its
// neighbours in x and y and the counts are 16 bytes in one piece, and only
// the face below the row's first cell is a word of its own; lane by lane
// these are 6 scattered words a cell (2.1M cells: 18 us with the index of each
// neighbour computed from its coordinates, 10.7 us, 4.7 TB/s, so).
template <int CW>
__global__ __launch_bounds__(256) void k_fold_faces(FoldFacesArgs a)
{
    const FoldChunk ch = a.chunks[blockIdx.x];
    const DevSys &S = a.systems[ch.sys];
    const uint64_t s = *a.sweep_ctr + a.rel;
    const int64_t W = a.count_words;
    const int nx = S.n[0], ny = S.n[1], nz = S.n[2], bs = S.brick_shift, m = S.brick_mask;
    const int64_t end = ch.first + kFoldChunk < S.n_store ? ch.first + kFoldChunk : S.n_store;
    constexpr int WPC = CW == COUNT_U16 ? 1 : 2;
    const uint32_t *F = a.flux + (s & 1) * 3 * W + WPC * S.cell_off;
    uint32_t *cnt = a.counts + WPC * S.cell_off;
    // stored distance to the neighbour below, inside a brick, across its
    // edge and around the box
    const int64_t sx = (int64_t)S.B1 * S.B2 << 2 * bs, wx = (nx - 1) * sx;
    const int64_t sy = 1 << bs, by = ((int64_t)S.B2 << 2 * bs) - (m << bs),
                  wy = ((int64_t)((ny - 1) >> bs) * S.B2 << 2 * bs) + (((ny - 1) & m) << bs);
    const int64_t bz = (1 << 2 * bs) - m, wz = ((int64_t)((nz - 1) >> bs) << 2 * bs) + ((nz - 1) & m);
    bool ovf = false;
    if (bs) {
        constexpr int K = 4 * WPC;                     // words of a row
        for (int64_t c = ch.first + 4 * threadIdx.x; c < end; c += 4 * blockDim.x) {
            int ix, iy, iz;
            cell_of_stored(S, c, ix, iy, iz);
            if (iy >= ny) continue;                    // padding
            const int64_t cx = ix == 0 ? c + wx : c - sx;
            const int64_t cy = iy == 0 ? c + wy : (iy & 3 ? c - sy : c - by);
            const int64_t cz = iz == 0 ? c + wz : c - bz;
            uint32_t own[3][K], fx[K], fy[K], n[K], low[WPC];
#pragma unroll
            for (int v = 0; v < WPC; ++v) {
                for (int d = 0; d < 3; ++d)
                    *reinterpret_cast<uint4 *>(own[d] + 4 * v) = *reinterpret_cast<const uint4 *>(F + d * W + WPC * c + 4 * v);
                *reinterpret_cast<uint4 *>(fx + 4 * v) = *reinterpret_cast<const uint4 *>(F + WPC * cx + 4 * v);
                *reinterpret_cast<uint4 *>(fy + 4 * v) = *reinterpret_cast<const uint4 *>(F + W + WPC * cy + 4 * v);
                *reinterpret_cast<uint4 *>(n + 4 * v) = *reinterpret_cast<const uint4 *>(cnt + WPC * c + 4 * v);
                low[v] = F[2 * W + WPC * cz + v];
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t fz = k < WPC ? low[k] : own[2][k - WPC];
                const uint32_t d = (fx[k] - own[0][k]) + (fy[k] - own[1][k]) + (fz - own[2][k]);
                uint32_t out;
                if (iz + k / WPC < nz) {               // (else padding)
                    ovf |= fold_word<CW>(n[k], d, out);
                    n[k] = out;
                }
            }
#pragma unroll
            for (int v = 0; v < WPC; ++v)
                *reinterpret_cast<uint4 *>(cnt + WPC * c + 4 * v) = *reinterpret_cast<const uint4 *>(n + 4 * v);
        }
    } else {
        for (int64_t c = ch.first + threadIdx.x; c < end; c += blockDim.x) {
            int ix, iy, iz;
            cell_of_stored(S, c, ix, iy, iz);
            const int64_t cx = ix == 0 ? c + wx : c - sx, cy = iy == 0 ? c + wy : c - by, cz = iz == 0 ? c + wz : c - bz;
            for (int j = 0; j < WPC; ++j) {
                const int64_t w = WPC * c + j;
                const uint32_t d = (F[WPC * cx + j] - F[w]) + (F[W + WPC * cy + j] - F[W + w]) +
                                   (F[2 * W + WPC * cz + j] - F[2 * W + w]);
                uint32_t out;
                ovf |= fold_word<CW>(cnt[w], d, out);
                cnt[w] = out;
            }
        }
    }
    if (ovf) atomicOr(a.status, ST_COUNT_OVERFLOW);
}

// Fold a density delta into counts and clear it: out = in + delta (out may
// be in), with 16-byte accesses (the arrays are 256-byte aligned), then the
// words past the last full quadruple.
template <int CW>
__global__ __launch_bounds__(256) void k_fold(const uint32_t *in, uint32_t *delta, uint32_t *counts, int64_t n,
                                              uint32_t *status, uint64_t *ctr, uint32_t advance)
{
    // (the last kernel of a batch of sweeps advances the sweep counter, which
    // no kernel of this launch reads)
    if (advance != 0u && blockIdx.x == 0 && threadIdx.x == 0) *ctr += advance;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n4 = n >> 2;
    const uint4 *i4 = reinterpret_cast<const uint4 *>(in);
    uint4 *c4 = reinterpret_cast<uint4 *>(counts);
    uint4 *d4 = reinterpret_cast<uint4 *>(delta);
    bool ovf = false;
    for (int64_t i = tid; i < n4; i += stride) {
        const uint4 b = i4[i], d = d4[i];
        uint4 w;
        ovf |= fold_word<CW>(b.x, d.x, w.x);
        ovf |= fold_word<CW>(b.y, d.y, w.y);
        ovf |= fold_word<CW>(b.z, d.z, w.z);
        ovf |= fold_word<CW>(b.w, d.w, w.w);
        c4[i] = w;
        d4[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    for (int64_t i = 4 * n4 + tid; i < n; i += stride) {
        uint32_t w;
        ovf |= fold_word<CW>(in[i], delta[i], w);
        counts[i] = w;
        delta[i] = 0u;
    }
    if (ovf) atomicOr(status, ST_COUNT_OVERFLOW);
}

// Density mode 3: copy the counts the sweep's atomics produced,
// B[(s+1) mod 2], into B[s mod 2], so both hold them for the next sweep (16-byte
// accesses; the buffers are 256-byte aligned and W is a multiple of 4).
// Packed 16-bit counts: every change of a sweep is a device atomic add of
// +-1 or +-2^16 on the word, and a true count never goes below zero during
// the sweep (a bead leaves only a cell it was counted in at the start), so
// the word is exact unless a count passed 65535: then its carry moves into
// the other half or out of the word, which lowers the sum of all halves, and
// the error stays in the counts.  So each block adds the sum of the halves
// it copied to its running entry of a.part (the same block index copies the
// same words every sweep), and k_mirror_check, once after the last sweep of
// a batch, compares the total with (sweeps) x (beads).  (Plain stores and a
// second kernel instead of a last-block reduction: a device-scope fence per
// block would write back the L2 each time.)
template <int CW>
__global__ __launch_bounds__(256) void k_mirror(MirrorArgs a)
{
    const uint64_t s = *a.sweep_ctr + a.rel;
    const int64_t W = a.count_words;
    const uint4 *src = reinterpret_cast<const uint4 *>(a.base + ((s + 1) & 1) * W);
    uint4 *dst = reinterpret_cast<uint4 *>(a.base + (s & 1) * W);
    const int64_t n4 = W >> 2;
    // four 16-byte loads in flight per thread before the stores
    constexpr int U = kMirrorUnroll;
    const int64_t step = (int64_t)gridDim.x * (256 * U);
    uint64_t sum = 0;
    for (int64_t b = (int64_t)blockIdx.x * (256 * U) + threadIdx.x; b < n4; b += step) {
        uint4 w[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (b + 256 * k < n4) w[k] = src[b + 256 * k];
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (b + 256 * k < n4) {
                dst[b + 256 * k] = w[k];
                if constexpr (CW == COUNT_U16)
                    sum += (uint64_t)((w[k].x & 0xFFFFu) + (w[k].x >> 16) + (w[k].y & 0xFFFFu) + (w[k].y >> 16)) +
                           (uint64_t)((w[k].z & 0xFFFFu) + (w[k].z >> 16) + (w[k].w & 0xFFFFu) + (w[k].w >> 16));
            }
    }
    if constexpr (CW == COUNT_U16) {
        __shared__ unsigned long long part[4];
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0) a.part[blockIdx.x] += part[0] + part[1] + part[2] + part[3];
    }
}

// Running half sums of the copy blocks against (sweeps) x (beads); clears
// them for the next batch (one block; each thread clears what it read).
__global__ __launch_bounds__(1024) void k_mirror_check(unsigned long long *part, int n_part,
                                                       unsigned long long expected, uint32_t *status, uint64_t *ctr,
                                                       uint32_t advance)
{
    __shared__ unsigned long long red[16];
    unsigned long long sum = 0;
    for (int i = threadIdx.x; i < n_part; i += blockDim.x) {
        sum += part[i];
        part[i] = 0ull;
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) t += red[k];
        if (t != expected) atomicOr(status, ST_COUNT_OVERFLOW);
        *ctr += advance;
    }
}

template <int R, int CW>
__global__ __launch_bounds__(256) void k_density(DensityArgs a)
{
    using Bead = typename std::conditional<R == REPR_F32, BeadF32, BeadCell>::type;
    const int wave = __builtin_amdgcn_readfirstlane(
        a.tile_begin + (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    if (wave >= a.tile_end) return;
    const Tile T = tile_at(a.tiles, wave);
    const SysPtr S = sys_at(a.systems, T.sys);
    const SysView v = make_view(S);
    const TileLane L = lane_of<TIL_WAVE>(T);
    if (!L.valid) return;
    const int i0 = 2 * L.p;
    const bool has1 = i0 + 1 < S->N;
    Bead b[2];
    load_pair(pos_arrays(a), T.slot, (uint32_t)tile_lane<TIL_WAVE>() * 8u, b[0], b[1]);
    if (!has1) b[1] = b[0];      // (the padding slot of an odd chain)
    CellPos c[2];
    cells_of<2>(b, v, S, true, a.status, c);
    const int cls = chain_cls(S, a.chain_class, a.chain_id[T.chain + L.g]);
    const uint32_t pat = pattern_bits(S, cls, i0);
    bool ovf = scatter_count<CW>(a.counts, S->cell_off + store_index(c[0], v), (int)(pat & 1u));
    if (has1) ovf |= scatter_count<CW>(a.counts, S->cell_off + store_index(c[1], v), (int)((pat >> 1) & 1u));
    if (ovf) atomicOr(a.status, ST_COUNT_OVERFLOW);
}

// ---------------------------------------------------------------------------
// State transfer (checkpoints): the chains' order and the padding are undone
// and redone here, so the host copies one compact block straight from or to
// the caller's memory.  (The permutation on the host took 40 of the 46 ms of
// a 4.2M-bead cell + offset state; these kernels take tens of microseconds.)
// ---------------------------------------------------------------------------
// The compact index of a lane's pair, or -1 (no pair, or a corrupt chain id).
__device__ __forceinline__ int64_t compact_index(const StateArgs &a, const Tile &T, SysPtr S, const TileLane &L)
{
    if (!L.valid) return -1;
    const uint32_t clog = a.chain_id[T.chain + L.g];
    if (clog >= (uint32_t)S->n_chains) {
        atomicOr(a.status, ST_INTERNAL);
        return -1;
    }
    return (int64_t)clog * S->N + 2 * L.p;
}

template <class V>
__device__ __forceinline__ void put_pair(V *dst, int64_t i, bool two, V a, V b)
{
    dst[i] = a;
    if (two) dst[i + 1] = b;
}
__device__ __forceinline__ void put_state(const StateArgs &a, int64_t B, int64_t i, bool two, const BeadF32 &u, const BeadF32 &w)
{
    put_pair(a.f, i, two, u.x, w.x);
    put_pair(a.f + B, i, two, u.y, w.y);
    put_pair(a.f + 2 * B, i, two, u.z, w.z);
}
__device__ __forceinline__ void put_state(const StateArgs &a, int64_t B, int64_t i, bool two, const BeadCell &u,
                                          const BeadCell &w)
{
    put_pair(a.f, i, two, u.ox, w.ox);
    put_pair(a.f + B, i, two, u.oy, w.oy);
    put_pair(a.f + 2 * B, i, two, u.oz, w.oz);
    put_pair(a.c, i, two, u.cx, w.cx);
    put_pair(a.c + B, i, two, u.cy, w.cy);
    put_pair(a.c + 2 * B, i, two, u.cz, w.cz);
}
// (the padding slot of an odd chain holds a zero bead)
__device__ __forceinline__ void get_state(const StateArgs &a, int64_t B, int64_t i, bool two, BeadF32 &u, BeadF32 &w)
{
    u = BeadF32{a.f[i], a.f[B + i], a.f[2 * B + i]};
    w = BeadF32{0.0f, 0.0f, 0.0f};
    if (two) w = BeadF32{a.f[i + 1], a.f[B + i + 1], a.f[2 * B + i + 1]};
}
__device__ __forceinline__ void get_state(const StateArgs &a, int64_t B, int64_t i, bool two, BeadCell &u, BeadCell &w)
{
    u = BeadCell{a.c[i], a.c[B + i], a.c[2 * B + i], a.f[i], a.f[B + i], a.f[2 * B + i]};
    w = BeadCell{0, 0, 0, 0.0f, 0.0f, 0.0f};
    if (two) w = BeadCell{a.c[i + 1], a.c[B + i + 1], a.c[2 * B + i + 1], a.f[i + 1], a.f[B + i + 1], a.f[2 * B + i + 1]};
}

enum { STATE_OUT, STATE_POS, STATE_CHECK, STATE_IN };

__device__ __forceinline__ double axis64(const BeadF32 &b, int d, SysPtr) { return (double)(d == 0 ? +b.x : d == 1 ? +b.y : +b.z); }
__device__ __forceinline__ double axis64(const BeadCell &b, int d, SysPtr S)
{
    return (double)(d == 0 ? +b.cx : d == 1 ? +b.cy : +b.cz) * (double)S->edge[d] + (double)(d == 0 ? +b.ox : d == 1 ? +b.oy : +b.oz);
}

// What is wrong with a bead set from the host.
__device__ __forceinline__ bool finite3(float x, float y, float z)
{
    const float m = __uint_as_float(0x7F7FFFFFu);   // FLT_MAX; a NaN fails the comparison
    return fabsf(x) <= m && fabsf(y) <= m && fabsf(z) <= m;
}
__device__ __forceinline__ uint32_t state_flaws(const BeadF32 &b, SysPtr S)
{
    if (!finite3(b.x, b.y, b.z)) return ST_BAD_VALUE;
    if (!S->walls) return 0u;
    const BeadF32 one[1] = {b};
    int k[1][3];
    ngp_index(one, make_view(S), k);
    return k[0][2] < S->wall_lo || k[0][2] >= S->wall_hi ? (uint32_t)ST_BAD_WALL : 0u;
}
__device__ __forceinline__ uint32_t state_flaws(const BeadCell &b, SysPtr S)
{
    if (!finite3(b.ox, b.oy, b.oz)) return ST_BAD_VALUE;
    uint32_t f = 0u;
    if (!(b.ox >= -S->edge[0] && b.ox < 2.0f * S->edge[0] && b.oy >= -S->edge[1] && b.oy < 2.0f * S->edge[1] &&
          b.oz >= -S->edge[2] && b.oz < 2.0f * S->edge[2]))
        f |= ST_BAD_OFFSET;
    const int lim = kStateCellLimit;
    if (b.cx <= -lim || b.cx >= lim || b.cy <= -lim || b.cy >= lim || b.cz <= -lim || b.cz >= lim) f |= ST_BAD_CELL;
    if (S->walls && (b.cz < S->wall_lo || b.cz >= S->wall_hi)) f |= ST_BAD_WALL;
    return f;
}

template <int R, int OP>
__global__ __launch_bounds__(256) void k_state(StateArgs a)
{
    using Bead = typename std::conditional<R == REPR_F32, BeadF32, BeadCell>::type;
    const int wave = __builtin_amdgcn_readfirstlane(
        a.tile_begin + (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    if (wave >= a.tile_end) return;
    const Tile T = tile_at(a.tiles, wave);
    const SysPtr S = sys_at(a.systems, T.sys);
    const TileLane L = lane_of<TIL_WAVE>(T);
    const int64_t i = compact_index(a, T, S, L);
    if (i < 0) return;
    const bool two = 2 * L.p + 1 < S->N;
    const int64_t B = (int64_t)S->n_chains * S->N;
    const uint32_t off = (uint32_t)tile_lane<TIL_WAVE>() * 8u;
    Bead u, w;
    if constexpr (OP == STATE_OUT || OP == STATE_POS) {
        load_pair(pos_arrays(a), T.slot, off, u, w);
        if constexpr (OP == STATE_OUT) put_state(a, B, i, two, u, w);
        else put_pair(a.xyz, i, two, axis64(u, a.axis, S), axis64(w, a.axis, S));
    } else {
        get_state(a, B, i, two, u, w);
        if constexpr (OP == STATE_CHECK) {
            const uint32_t f = state_flaws(u, S) | (two ? state_flaws(w, S) : 0u);
            if (f) atomicOr(a.flags, f);
        } else {
            store_pair(pos_arrays(a), T.slot, off, u, w);
        }
    }
}

__device__ __forceinline__ void report_status(const Report &r)
{
    if (r.host && blockIdx.x == 0 && threadIdx.x == 0) *r.host = *r.status;
}
__global__ void k_report(Report r) { report_status(r); }

// The cells of one system in linear order from the stored order.  One thread
// takes four consecutive stored cells (with bricks a row in z: 16 or 32 bytes
// read, 16 written per species; cell by cell the mapping costs more than the
// copy).
struct StoredRow {
    int64_t c;      // first stored cell
    int64_t lin;    // its linear index
    int n;          // cells inside the grid, 0..4
};
__device__ __forceinline__ StoredRow stored_row(const DevSys &S)
{
    StoredRow r;
    r.c = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    r.lin = r.c;
    r.n = r.c < S.n_store ? (int)(S.n_store - r.c < 4 ? S.n_store - r.c : 4) : 0;
    if (S.brick_shift != 0 && r.n != 0) {
        int x, y, z;
        cell_of_stored(S, r.c, x, y, z);
        r.lin = ((int64_t)x * S.n[1] + y) * S.n[2] + z;
        r.n = y < S.n[1] ? min(4, S.n[2] - z) : 0;
    }
    return r;
}
template <int CW>
__device__ __forceinline__ void row_counts(const uint32_t *cnt, const StoredRow &r, uint2 (&n)[4])
{
    // (a row past the end of a linear array still lies in the buffer: cell
    // offsets are multiples of 64)
    if constexpr (CW == COUNT_U16) {
        const uint4 w = *reinterpret_cast<const uint4 *>(cnt + r.c);
        n[0] = make_uint2(w.x & 0xFFFFu, w.x >> 16);
        n[1] = make_uint2(w.y & 0xFFFFu, w.y >> 16);
        n[2] = make_uint2(w.z & 0xFFFFu, w.z >> 16);
        n[3] = make_uint2(w.w & 0xFFFFu, w.w >> 16);
    } else {
        const uint4 u = *reinterpret_cast<const uint4 *>(cnt + 2 * r.c), v = *reinterpret_cast<const uint4 *>(cnt + 2 * r.c + 4);
        n[0] = make_uint2(u.x, u.y);
        n[1] = make_uint2(u.z, u.w);
        n[2] = make_uint2(v.x, v.y);
        n[3] = make_uint2(v.z, v.w);
    }
}
// (out is the caller's: only the element alignment is known)
template <class V>
__device__ __forceinline__ void put_row(V *out, const StoredRow &r, const V (&v)[4])
{
    V *p = out + r.lin;
    if (r.n == 4 && (reinterpret_cast<uintptr_t>(p) & 15u) == 0) {
        u4 w = {__builtin_bit_cast(uint32_t, v[0]), __builtin_bit_cast(uint32_t, v[1]), __builtin_bit_cast(uint32_t, v[2]),
                __builtin_bit_cast(uint32_t, v[3])};
        *reinterpret_cast<u4 *>(p) = w;
    } else {
        for (int k = 0; k < 4; ++k)
            if (k < r.n) p[k] = v[k];
    }
}

// Fields of one system as float [2][M] (A then B), from its counts or its
// frozen array.
template <int CW>
__global__ __launch_bounds__(256) void k_fields(FieldArgs a)
{
    report_status(a.report);
    const DevSys &S = a.systems[a.sys];
    const StoredRow r = stored_row(S);
    if (r.n == 0) return;
    float wa[4] = {0.0f, 0.0f, 0.0f, 0.0f}, wb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (S.frozen) {
        for (int k = 0; k < 4; ++k)
            if (k < r.n) {
                const float2 w = a.omega[S.cell_off + r.c + k];
                wa[k] = w.x;
                wb[k] = w.y;
            }
    } else {
        const FieldCoef fc{S.c_same, S.c_other, S.c0};
        uint2 n[4];
        row_counts<CW>(a.counts + (CW == COUNT_U16 ? 1 : 2) * S.cell_off, r, n);
        for (int k = 0; k < 4; ++k) {
            wa[k] = omega_of(fc, n[k], 0);
            wb[k] = omega_of(fc, n[k], 1);
            if (S.umb && k < r.n) {
                const float2 t = a.tgt[S.cell_off + r.c + k];
                wa[k] -= S.umb_coef * t.x;
                wb[k] -= S.umb_coef * t.y;
            }
        }
    }
    put_row(a.out, r, wa);
    put_row(a.out + a.n_cells, r, wb);
}

// Counts of one system as uint32 [2][M].
template <int CW>
__global__ __launch_bounds__(256) void k_unpack_counts(UnpackArgs a)
{
    report_status(a.report);
    const DevSys &S = *a.sys;
    const StoredRow r = stored_row(S);
    if (r.n == 0) return;
    uint2 n[4];
    row_counts<CW>(a.counts + (CW == COUNT_U16 ? 1 : 2) * a.cell_off, r, n);
    const uint32_t na[4] = {n[0].x, n[1].x, n[2].x, n[3].x}, nb[4] = {n[0].y, n[1].y, n[2].y, n[3].y};
    put_row(a.out, r, na);
    put_row(a.out + a.n_cells, r, nb);
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t *p, int64_t n, uint32_t v)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

__global__ void k_advance(uint64_t *ctr, uint32_t n) { *ctr += n; }

// ---------------------------------------------------------------------------
// Spatial chain reorder: a counting sort of the chains by the block of 4 x 4
// x 4 cells that holds their middle bead (blocks in linear order, context-wide,
// so every system stays inside its own chain range), so that the chains of a
// wave share count lines and the waves in flight work on a compact region.
// Logical chain ids move with the chains, so the sweep's results do not change.
// (A block, not a cell: at two beads per cell a row of cells in z holds one
// chain of 32 beads per 16 cells, so consecutive chains of a sort by cell are
// 16 cells apart, those of a sort by block are in the same block.  The middle
// bead: it is nearest to the others.  Distinct 64-byte count lines that a wave
// of such chains updates: 0.184 per bead by cell of the first bead, 0.159 by
// block of the middle bead; and the histogram is 64 times smaller.)
// ---------------------------------------------------------------------------
template <int R>
__global__ __launch_bounds__(256) void k_reorder_keys(ReorderArgs a)
{
    using Bead = typename std::conditional<R == REPR_F32, BeadF32, BeadCell>::type;
    const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    if (wave >= a.n_tiles) return;
    const Tile T = tile_at(a.tiles, wave);
    const SysPtr S = sys_at(a.systems, T.sys);
    const SysView v = make_view(S);
    const TileLane L = lane_of<TIL_WAVE>(T);
    if (!L.valid || L.p != (int)(T.lanes >> 12 & 63u)) return;      // lane P / 2 of its chain
    Bead b[2];
    load_pair(pos_arrays(a), T.slot, (uint32_t)tile_lane<TIL_WAVE>() * 8u, b[0], b[1]);
    CellPos c[1];
    const Bead mid[1] = {b[0]};
    cells_of<1>(mid, v, S, false, a.status, c);
    const int64_t blk = ((int64_t)(c[0].x / kSortBlock) * S->nb1 + c[0].y / kSortBlock) * S->nb2 + c[0].z / kSortBlock;
    const uint32_t key = (uint32_t)(S->blk_off + blk);
    a.keys[T.chain + L.g] = key;
    atomicAdd(a.hist + key, 1u);
}

// Exclusive scan of hist[0, n) in place: block sums, a scan of the block
// sums by one block, then the block-local scans plus offsets.
constexpr int kScanBlock = 1024, kScanPer = 4, kScanTile = kScanBlock * kScanPer;

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *sh, uint32_t &total)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kScanBlock; off <<= 1) {
        const uint32_t x = t >= off ? sh[t - off] : 0u;
        __syncthreads();
        sh[t] += x;
        __syncthreads();
    }
    total = sh[kScanBlock - 1];
    const uint32_t incl = sh[t];
    __syncthreads();
    return incl - v;
}

__global__ __launch_bounds__(kScanBlock) void k_scan_partials(const uint32_t *hist, int64_t n, uint32_t *bsum)
{
    __shared__ uint32_t sh[kScanBlock];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    uint32_t v = 0;
    for (int k = 0; k < kScanPer; ++k)
        if (base + k < n) v += hist[base + k];
    uint32_t total;
    (void)block_exclusive_scan(v, sh, total);
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanBlock) void k_scan_bsum(uint32_t *bsum, int nb)
{
    __shared__ uint32_t sh[kScanBlock];
    uint32_t carry = 0;
    for (int start = 0; start < nb; start += kScanBlock) {
        const int i = start + (int)threadIdx.x;
        const uint32_t v = i < nb ? bsum[i] : 0u;
        uint32_t total;
        const uint32_t ex = block_exclusive_scan(v, sh, total);
        if (i < nb) bsum[i] = carry + ex;
        carry += total;
    }
}

__global__ __launch_bounds__(kScanBlock) void k_scan_apply(uint32_t *hist, int64_t n, const uint32_t *bsum)
{
    __shared__ uint32_t sh[kScanBlock];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    uint32_t vals[kScanPer];
    uint32_t v = 0;
    for (int k = 0; k < kScanPer; ++k) {
        vals[k] = base + k < n ? hist[base + k] : 0u;
        v += vals[k];
    }
    uint32_t total;
    uint32_t run = bsum[blockIdx.x] + block_exclusive_scan(v, sh, total);
    for (int k = 0; k < kScanPer; ++k)
        if (base + k < n) {
            hist[base + k] = run;
            run += vals[k];
        }
}

// perm[new] = old: each chain takes the next free place of its key.
__global__ __launch_bounds__(256) void k_reorder_scatter(ReorderArgs a)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.total_chains) return;
    const uint32_t pos = atomicAdd(a.hist + a.keys[c], 1u);
    if (pos < (uint64_t)a.total_chains) a.perm[pos] = (uint32_t)c;
    else atomicOr(a.status, ST_INTERNAL);
}

// Move chain perm[new] into place `new` (scratch copy), with its logical id.
template <int R>
__global__ __launch_bounds__(256) void k_reorder_permute(ReorderArgs a)
{
    using Bead = typename std::conditional<R == REPR_F32, BeadF32, BeadCell>::type;
    const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    if (wave >= a.n_tiles) return;
    const Tile T = tile_at(a.tiles, wave);
    const SysPtr S = sys_at(a.systems, T.sys);
    const TileLane L = lane_of<TIL_WAVE>(T);
    if (!L.valid) return;
    const int64_t old = (int64_t)a.perm[T.chain + L.g] - S->chain_off;
    if (old < 0 || old >= S->n_chains) {           // a chain left its system: never expected
        atomicOr(a.status, ST_INTERNAL);
        return;
    }
    Bead b0, b1;
    load_pair(pos_arrays(a), S->slot_off + old * (2 * S->P) + 2 * L.p, 0u, b0, b1);
    store_pair(PosArrays{a.Q0, a.Q1, a.Q2, a.D0, a.D1, a.D2}, T.slot, (uint32_t)tile_lane<TIL_WAVE>() * 8u, b0, b1);
    if (L.p == 0) a.chain_id2[T.chain + L.g] = a.chain_id[S->chain_off + old];
}

// Logical chain ids in system order (identity within each system).
__global__ __launch_bounds__(256) void k_iota_chains(ReorderArgs a)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    if (wave >= a.n_tiles) return;
    const Tile T = tile_at(a.tiles, wave);
    const TileLane L = lane_of<TIL_WAVE>(T);
    if (L.valid && L.p == 0) a.chain_id[T.chain + L.g] = (uint32_t)(T.chain0 + L.g);
}

// ---------------------------------------------------------------------------
// Initial configuration: Gaussian random walks on the GPU (Sec. 2.2 moved
// the generation of bead coordinates to the GPU), on wave tiles: a lane draws
// the bonds of its two beads (FP64, most of the work), one lane per chain adds
// them up in chain order from LDS, and the lanes round and store their pairs.
// (One thread per chain draws N bonds in a row on an N-th of the lanes and
// stores a chain apart: 16.8M beads 1.45 -> 0.49 ms, 524k beads placed 98 ->
// 28 us.)
// ---------------------------------------------------------------------------
// One coordinate as cell and offset (the canonical form of a new position).
__device__ __forceinline__ void quantise(double r, float e, int &c, float &o)
{
    const double cf = floor(r / (double)e);
    c = (int)cf;
    o = (float)(r - cf * (double)e);
    renorm(c, o, e);
}
__device__ __forceinline__ void store_init_pair(const InitArgs &a, int64_t slot, uint32_t off, double3 u, double3 w)
{
    if (a.repr == REPR_F32) {
        store_pair(pos_arrays(a), slot, off, BeadF32{(float)u.x, (float)u.y, (float)u.z},
                   BeadF32{(float)w.x, (float)w.y, (float)w.z});
        return;
    }
    BeadCell b0, b1;
    quantise(u.x, a.edge[0], b0.cx, b0.ox);
    quantise(u.y, a.edge[1], b0.cy, b0.oy);
    quantise(u.z, a.edge[2], b0.cz, b0.oz);
    quantise(w.x, a.edge[0], b1.cx, b1.ox);
    quantise(w.y, a.edge[1], b1.cy, b1.oy);
    quantise(w.z, a.edge[2], b1.cz, b1.oz);
    store_pair(pos_arrays(a), slot, off, b0, b1);
}

// Initial streams: counter word 3 = system id with the top bit set (never a
// move draw); word 2 names the stream and the attempt j (walls only):
// 4j initial walks, 4j + 1 placement targets, 4j + 2 placement walks.
__device__ __forceinline__ uint4 init_block(uint32_t w0, uint32_t chain, uint32_t stream, uint32_t sys_id,
                                            uint64_t seed)
{
    return philox4x32_10(make_uint4(w0, chain, stream, sys_id | 0x80000000u), (uint32_t)seed,
                         (uint32_t)(seed >> 32));
}

__device__ __forceinline__ double top24(uint32_t w) { return (double)(w >> 8) * 0x1p-24; }

// One Gaussian bond, each component N(0, sigma^2), Box-Muller on words (0,1), (2,3).
__device__ __forceinline__ double3 gauss_bond(uint4 w, double sigma)
{
    const double two_pi = 6.283185307179586476925286766559;
    const double u1 = ((double)(w.x >> 8) + 0.5) * 0x1p-24;
    const double u2 = top24(w.y);
    const double u3 = ((double)(w.z >> 8) + 0.5) * 0x1p-24;
    const double u4 = top24(w.w);
    const double r1 = sqrt(-2.0 * log(u1)), r2 = sqrt(-2.0 * log(u3));
    return make_double3(sigma * r1 * cos(two_pi * u2), sigma * r1 * sin(two_pi * u2), sigma * r2 * cos(two_pi * u4));
}

// Walls: the z range a drawn chain must stay in, with a margin of 1/128 cell
// edge so that the stored representation's z cell is inside whatever the
// rounding (|z| < 2^15 edges).
__device__ __forceinline__ void wall_range(const InitArgs &a, double &lo, double &hi)
{
    const double e = (double)a.edge[2];
    lo = (double)a.wall_lo * e + e / 128.0;
    hi = (double)a.wall_hi * e - e / 128.0;
}

// ---------------------------------------------------------------------------
// Placement from target concentration fields (Sec. 3.2, "Coupling"): each
// molecule's centre ends up at most Re/2 (half the ideal end-to-end
// distance) from a target position drawn from the supplied fields.
//   1. Class k (pattern a or b, A fraction f_k) weighs cell c by the integer
//      w_k(c) = floor(2^20 (f_k tA(c) + (1 - f_k) tB(c)) + 1/2) (FP64, exact
//      as the same operations on any IEEE machine); W_k is its exact
//      inclusive prefix sum (uint64).
//   2. A chain of class k takes t = floor(v T_k / 2^64) for the 64-bit word
//      v of its block (0, chain, 4j + 1) and the first cell with W_k > t.
//   3. Target point uniform in that cell; centre of mass uniform in the ball
//      of radius Re/2 around it; conformation a Gaussian walk (blocks
//      (i, chain, 4j + 2)) shifted to that centre.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_place_weights(PlaceArgs a)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.n_cells) return;
    const int N = a.ia.N;
    const float2 t = a.tgt[a.cell_off + stored_of_linear(*a.sys, c)];
    for (int k = 0; k < 2; ++k) {
        const double fa = (double)a.na[k] / (double)N, fb = (double)(N - a.na[k]) / (double)N;
        const double v = fa * (double)t.x + fb * (double)t.y;
        a.W[k * a.n_cells + c] = (unsigned long long)floor(1048576.0 * v + 0.5);
    }
}

// Inclusive scan of 64-bit words in place (block sums, a one-block scan of
// the sums, then block-local scans plus offsets), as for the reorder.
constexpr int kScan64Block = 256, kScan64Per = 8, kScan64Tile = kScan64Block * kScan64Per;

__device__ __forceinline__ unsigned long long block_scan64(unsigned long long v, unsigned long long *sh,
                                                           unsigned long long &total)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kScan64Block; off <<= 1) {
        const unsigned long long x = t >= off ? sh[t - off] : 0ull;
        __syncthreads();
        sh[t] += x;
        __syncthreads();
    }
    total = sh[kScan64Block - 1];
    const unsigned long long incl = sh[t];
    __syncthreads();
    return incl - v;          // exclusive
}

__global__ __launch_bounds__(kScan64Block) void k_scan64_partials(const unsigned long long *x, int64_t n,
                                                                  unsigned long long *bsum)
{
    __shared__ unsigned long long sh[kScan64Block];
    const int64_t base = (int64_t)blockIdx.x * kScan64Tile + (int64_t)threadIdx.x * kScan64Per;
    unsigned long long v = 0;
    for (int k = 0; k < kScan64Per; ++k)
        if (base + k < n) v += x[base + k];
    unsigned long long total;
    (void)block_scan64(v, sh, total);
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScan64Block) void k_scan64_bsum(unsigned long long *bsum, int nb)
{
    __shared__ unsigned long long sh[kScan64Block];
    unsigned long long carry = 0;
    for (int start = 0; start < nb; start += kScan64Block) {
        const int i = start + (int)threadIdx.x;
        const unsigned long long v = i < nb ? bsum[i] : 0ull;
        unsigned long long total;
        const unsigned long long ex = block_scan64(v, sh, total);
        if (i < nb) bsum[i] = carry + ex;
        carry += total;
    }
}

__global__ __launch_bounds__(kScan64Block) void k_scan64_apply(unsigned long long *x, int64_t n,
                                                               const unsigned long long *bsum)
{
    __shared__ unsigned long long sh[kScan64Block];
    const int64_t base = (int64_t)blockIdx.x * kScan64Tile + (int64_t)threadIdx.x * kScan64Per;
    unsigned long long vals[kScan64Per];
    unsigned long long v = 0;
    for (int k = 0; k < kScan64Per; ++k) {
        vals[k] = base + k < n ? x[base + k] : 0ull;
        v += vals[k];
    }
    unsigned long long total;
    unsigned long long run = bsum[blockIdx.x] + block_scan64(v, sh, total);
    for (int k = 0; k < kScan64Per; ++k)
        if (base + k < n) {
            run += vals[k];
            x[base + k] = run;      // inclusive
        }
}

// Target centre of mass of a chain, attempt j (false: its class has no weight).
__device__ __forceinline__ bool place_centre(const PlaceArgs &a, uint32_t chain, int j, double3 &centre)
{
    const InitArgs &ia = a.ia;
    const double two_pi = 6.283185307179586476925286766559;
    const int k = (int)a.chain_class[a.chain_off + chain];
    const unsigned long long *Wk = a.W + k * a.n_cells;
    const unsigned long long T = Wk[a.n_cells - 1];
    if (T == 0) return false;
    const uint4 w = init_block(0u, chain, 4u * (uint32_t)j + 1u, ia.sys_id, ia.seed);
    const uint4 q = init_block(1u, chain, 4u * (uint32_t)j + 1u, ia.sys_id, ia.seed);
    const unsigned long long v = ((unsigned long long)w.x << 32) | w.y;
    const unsigned long long t = __umul64hi(v, T);
    int64_t lo = 0, hi = a.n_cells - 1;     // first cell with Wk > t
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (Wk[mid] > t) hi = mid;
        else lo = mid + 1;
    }
    const int64_t nyz = (int64_t)a.grid[1] * a.grid[2];
    const int64_t ix = lo / nyz, iy = (lo / a.grid[2]) % a.grid[1], iz = lo % a.grid[2];
    const double tx = ((double)ix + top24(w.z)) * a.edge64[0];
    const double ty = ((double)iy + top24(w.w)) * a.edge64[1];
    const double tz = ((double)iz + top24(q.x)) * a.edge64[2];
    const double rad = 0.5 * a.Re * cbrt(top24(q.y));
    const double ct = 2.0 * top24(q.z) - 1.0;
    const double stt = sqrt(fmax(0.0, 1.0 - ct * ct));
    const double ph = two_pi * top24(q.w);
    centre = make_double3(tx + rad * stt * cos(ph), ty + rad * stt * sin(ph), tz + rad * ct);
    return true;
}

// A wave's beads in LDS: bead i of chain g of the tile at g 2P + i.
struct WalkLds {
    double x[2 * kWave], y[2 * kWave], z[2 * kWave];
};
__device__ __forceinline__ void put_bead(WalkLds &l, int i, double3 v)
{
    l.x[i] = v.x;
    l.y[i] = v.y;
    l.z[i] = v.z;
}
__device__ __forceinline__ double3 get_bead(const WalkLds &l, int i) { return make_double3(l.x[i], l.y[i], l.z[i]); }
// Lanes of this lane's chain.
__device__ __forceinline__ uint64_t chain_lanes(int first, int P)
{
    return (P == 64 ? ~0ull : (1ull << P) - 1ull) << first;
}
constexpr int kWalkWaves = 4;

// The walks of one wave tile.  PLACE false: bead 0 uniform in the box (in z
// between the walls when there are walls).  PLACE true: the walk starts at
// the origin and is shifted so that its centre of mass is the chain's target
// centre.  With walls a chain that leaves the slab is drawn again from the
// next attempt's counters (kMaxAttempts at most, else the status bit); the
// last attempt's chain is the one stored.
template <bool PLACE>
__device__ __forceinline__ void walk_tile(const InitArgs &a, const PlaceArgs *pa)
{
    __shared__ WalkLds lds[kWalkWaves];
    WalkLds &l = lds[threadIdx.x >> 6];
    const int wave = __builtin_amdgcn_readfirstlane(
        a.tile_begin + (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    if (wave >= a.tile_end) return;
    const Tile T = tile_at(a.tiles, wave);
    const TileLane L = lane_of<TIL_WAVE>(T);
    const int lane = tile_lane<TIL_WAVE>(), N = a.N, P = (int)(T.lanes >> 11 & 127u), first = lane - L.p;
    const int i0 = 2 * L.p, at = 2 * lane;
    const bool has1 = L.valid && i0 + 1 < N;
    const uint32_t chain = L.valid ? a.chain_id[T.chain + L.g] : 0u;
    double zlo = 0.0, zhi = 0.0;
    if (a.walls) wall_range(a, zlo, zhi);
    double3 u = make_double3(0.0, 0.0, 0.0), w = u;
    bool todo = L.valid, failed = false, drawn = false;
    for (int j = 0; j < kMaxAttempts && __ballot(todo) != 0; ++j) {
        const uint32_t stream = 4u * (uint32_t)j + (PLACE ? 2u : 0u);
        if (todo) {
            double3 b0 = make_double3(0.0, 0.0, 0.0);
            if (i0 > 0) {
                b0 = gauss_bond(init_block((uint32_t)i0, chain, stream, a.sys_id, a.seed), a.sigma);
            } else if (!PLACE) {
                const uint4 r = init_block(0u, chain, stream, a.sys_id, a.seed);
                b0 = make_double3(a.box[0] * top24(r.x), a.box[1] * top24(r.y), a.box[2] * top24(r.z));
                if (a.walls) {
                    const double e = (double)a.edge[2];
                    const double lo = (double)a.wall_lo * e, hi = (double)a.wall_hi * e;
                    b0.z = lo + (hi - lo) * top24(r.z);
                }
            }
            put_bead(l, at, b0);
            if (has1) put_bead(l, at + 1, gauss_bond(init_block((uint32_t)i0 + 1u, chain, stream, a.sys_id, a.seed), a.sigma));
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        // the chain's first lane adds the bonds up in order
        double3 shift = make_double3(0.0, 0.0, 0.0), mean = shift;
        bool reachable = true;
        if (todo && L.p == 0) {
            double3 x = get_bead(l, at), s = make_double3(0.0, 0.0, 0.0);
            for (int i = 1; i < N; ++i) {
                const double3 b = get_bead(l, at + i);
                x = make_double3(x.x + b.x, x.y + b.y, x.z + b.z);
                s = make_double3(s.x + x.x, s.y + x.y, s.z + x.z);
                put_bead(l, at + i, x);
            }
            if constexpr (PLACE) {
                mean = make_double3(s.x / (double)N, s.y / (double)N, s.z / (double)N);
                reachable = place_centre(*pa, chain, j, shift);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if constexpr (PLACE) {
            shift = make_double3(__shfl(shift.x, first), __shfl(shift.y, first), __shfl(shift.z, first));
            mean = make_double3(__shfl(mean.x, first), __shfl(mean.y, first), __shfl(mean.z, first));
            reachable = __shfl((int)reachable, first) != 0;
        }
        bool out = false;
        if (todo && reachable) {
            drawn = true;
            u = get_bead(l, at);
            if (has1) w = get_bead(l, at + 1);
            if constexpr (PLACE) {
                u = make_double3(shift.x + (u.x - mean.x), shift.y + (u.y - mean.y), shift.z + (u.z - mean.z));
                if (has1) w = make_double3(shift.x + (w.x - mean.x), shift.y + (w.y - mean.y), shift.z + (w.z - mean.z));
            }
            out = a.walls && (!(u.z >= zlo && u.z <= zhi) || (has1 && !(w.z >= zlo && w.z <= zhi)));
        }
        const uint64_t bad = __ballot(out || !reachable);
        failed = todo ? (bad & chain_lanes(first, P)) != 0 : failed;
        todo = todo && failed && a.walls && reachable;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    if (__ballot(L.valid && failed) != 0 && lane == 0) atomicOr(a.status, ST_PLACEMENT);
    // (the padding slot of an odd chain holds a zero bead)
    if (drawn) store_init_pair(a, T.slot, (uint32_t)lane * 8u, u, has1 ? w : make_double3(0.0, 0.0, 0.0));
}

__global__ __launch_bounds__(64 * kWalkWaves) void k_init_walks(InitArgs a) { walk_tile<false>(a, nullptr); }

__global__ __launch_bounds__(64 * kWalkWaves) void k_place_chains(PlaceArgs a) { walk_tile<true>(a.ia, &a); }

// ---------------------------------------------------------------------------
// Observables: FP64 per chain, compensated (Neumaier) sums over chains and
// cells (the only FP64 on the GPU besides smart moves and set-up).
//
// Bound by memory: every position and every count read once.  Positions are
// read as the sweep reads them (a wave tile's pairs, 8 bytes a lane and
// array, the next tile's while this one is summed); sums over the lanes of a
// chain are differences of wave prefix sums (DPP, no LDS).  A resident grid
// walks tiles and cells, so few partial sums are left.  Against one thread
// per chain (whose reads are a chain apart in every array), one block sum per
// 256 chains or cells and one block over all of them, the kernels of a call:
// 16.8M beads cell + offset on 256 x 256 x 128 cells 3.23 -> 0.13 ms (3.6
// TB/s), 4.2M beads FP32 on 128^3 cells 195 -> 33 us, 8192 beads 49 -> 10 us.
// ---------------------------------------------------------------------------
struct NSum {
    double s, c;
};
__device__ __forceinline__ void nadd(NSum &a, double v)
{
    const double t = a.s + v;
    a.c += fabs(a.s) >= fabs(v) ? (a.s - t) + v : (v - t) + a.s;
    a.s = t;
}
__device__ __forceinline__ void nmerge(NSum &a, const NSum &b)
{
    nadd(a, b.s);
    a.c += b.c;
}

constexpr int kObsQ = 6;       // Re2, Re2^2, Rg2, Rg2^2, Ebond (chains), Enb (cells)
constexpr int kObsCells = 2048;   // cells per block and step

// A double through a DPP move of its two words (lanes without a source: 0).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp64(double x)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xF, false);
    return __builtin_bit_cast(double, (uint64_t)lo | (uint64_t)hi << 32);
}
// Inclusive prefix sum over the wave: shifts by 1, 2, 4 and 8 within rows of
// 16 lanes, then the last lane of row 0 and 2 to row 1 and 3, and the last
// lane of row 1 to rows 2 and 3.
__device__ __forceinline__ double wave_prefix(double x)
{
    x += dpp64<0x111, 0xF>(x);
    x += dpp64<0x112, 0xF>(x);
    x += dpp64<0x114, 0xF>(x);
    x += dpp64<0x118, 0xF>(x);
    x += dpp64<0x142, 0xA>(x);
    x += dpp64<0x143, 0xC>(x);
    return x;
}

// Position of bead b relative to bead r of the same chain (FP64; the
// difference of the cells is exact).
__device__ __forceinline__ double3 rel64(const BeadF32 &b, const BeadF32 &r, const ObsArgs &)
{
    return make_double3((double)b.x - (double)r.x, (double)b.y - (double)r.y, (double)b.z - (double)r.z);
}
__device__ __forceinline__ double3 rel64(const BeadCell &b, const BeadCell &r, const ObsArgs &a)
{
    return make_double3((double)(b.cx - r.cx) * (double)a.edge[0] + ((double)b.ox - (double)r.ox),
                        (double)(b.cy - r.cy) * (double)a.edge[1] + ((double)b.oy - (double)r.oy),
                        (double)(b.cz - r.cz) * (double)a.edge[2] + ((double)b.oz - (double)r.oz));
}
__device__ __forceinline__ BeadF32 from_lane(const BeadF32 &b, int l)
{
    return BeadF32{__shfl(b.x, l), __shfl(b.y, l), __shfl(b.z, l)};
}
__device__ __forceinline__ BeadCell from_lane(const BeadCell &b, int l)
{
    return BeadCell{__shfl(b.cx, l), __shfl(b.cy, l), __shfl(b.cz, l), __shfl(b.ox, l), __shfl(b.oy, l), __shfl(b.oz, l)};
}

// Deterministic tree reduction of the block's Q Neumaier sums to out[2 Q].
template <int Q>
__device__ __forceinline__ void block_reduce_store(const NSum (&q)[Q], double *out)
{
    __shared__ double sh_s[Q][256], sh_c[Q][256];
    const int t = threadIdx.x;
    for (int k = 0; k < Q; ++k) {
        sh_s[k][t] = q[k].s;
        sh_c[k][t] = q[k].c;
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) {
            for (int k = 0; k < Q; ++k) {
                NSum x{sh_s[k][t], sh_c[k][t]};
                nmerge(x, NSum{sh_s[k][t + w], sh_c[k][t + w]});
                sh_s[k][t] = x.s;
                sh_c[k][t] = x.c;
            }
        }
        __syncthreads();
    }
    if (t < Q) {
        out[2 * t] = sh_s[t][0];
        out[2 * t + 1] = sh_c[t][0];
    }
}

// Chains: the beads of a chain relative to its first bead (q), so that
// Rg^2 = sum |q|^2 / N - |sum q / N|^2 loses at most the factor N + 1 that
// |q|^2 can exceed Rg^2 by.
template <int R>
__device__ __forceinline__ void obs_chains(const ObsArgs &a)
{
    using Bead = typename std::conditional<R == REPR_F32, BeadF32, BeadCell>::type;
    NSum q[kObsQ - 1];
    for (int k = 0; k < kObsQ - 1; ++k) q[k] = NSum{0.0, 0.0};
    const int lane = (int)(threadIdx.x & 63), N = a.N;
    const double inv_N = 1.0 / (double)N;
    const PosArrays A = pos_arrays(a);
    const int n_waves = a.chain_blocks * 4;
    int t = __builtin_amdgcn_readfirstlane(a.tile_begin + (int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    Tile T{};
    Bead n0{}, n1{};
    if (t < a.tile_end) {
        T = tile_at(a.tiles, t);
        load_pair(A, T.slot, lane_of<TIL_WAVE>(T).valid ? (uint32_t)lane * 8u : 0u, n0, n1);
    }
    for (; t < a.tile_end; t += n_waves) {
        const Bead b0 = n0, b1 = n1;
        const TileLane L = lane_of<TIL_WAVE>(T);
        const int P = (int)(T.lanes >> 11 & 127u);
        if (t + n_waves < a.tile_end) {
            T = tile_at(a.tiles, t + n_waves);
            load_pair(A, T.slot, lane_of<TIL_WAVE>(T).valid ? (uint32_t)lane * 8u : 0u, n0, n1);
        }
        const Bead ref = from_lane(b0, lane - L.p);
        const bool has1 = L.valid && 2 * L.p + 1 < N, next = L.valid && 2 * L.p + 2 < N;
        const double3 z = make_double3(0.0, 0.0, 0.0);
        const double3 r0 = L.valid ? rel64(b0, ref, a) : z, r1 = has1 ? rel64(b1, ref, a) : z;
        const double3 rn = make_double3(dpp64<kDppShl1, 0xF>(r0.x), dpp64<kDppShl1, 0xF>(r0.y), dpp64<kDppShl1, 0xF>(r0.z));
        double bond = 0.0;
        if (has1) bond += (r1.x - r0.x) * (r1.x - r0.x) + (r1.y - r0.y) * (r1.y - r0.y) + (r1.z - r0.z) * (r1.z - r0.z);
        if (next) bond += (rn.x - r1.x) * (rn.x - r1.x) + (rn.y - r1.y) * (rn.y - r1.y) + (rn.z - r1.z) * (rn.z - r1.z);
        const double s2 = (r0.x * r0.x + r0.y * r0.y + r0.z * r0.z) + (r1.x * r1.x + r1.y * r1.y + r1.z * r1.z);
        double v[5] = {wave_prefix(r0.x + r1.x), wave_prefix(r0.y + r1.y), wave_prefix(r0.z + r1.z), wave_prefix(s2),
                       wave_prefix(bond)};
        // a chain's last lane takes the sums of its P lanes
        for (int k = 0; k < 5; ++k) {
            const double before = __shfl(v[k], lane - P);
            if (lane >= P) v[k] -= before;
        }
        if (L.valid && L.p == P - 1) {
            const double3 e = has1 ? r1 : r0;
            const double e2e = e.x * e.x + e.y * e.y + e.z * e.z;
            const double mx = v[0] * inv_N, my = v[1] * inv_N, mz = v[2] * inv_N;
            const double g = v[3] * inv_N - (mx * mx + my * my + mz * mz);
            nadd(q[0], e2e);
            nadd(q[1], e2e * e2e);
            nadd(q[2], g);
            nadd(q[3], g * g);
            nadd(q[4], v[4] * a.k_half);
        }
    }
    block_reduce_store<kObsQ - 1>(q, a.partials + (int64_t)blockIdx.x * 2 * (kObsQ - 1));
}

// Cells: f(phiA, phiB); its sum times (B / M) / N is H_nb / kT.
__device__ __forceinline__ double cell_energy(const ObsArgs &a, uint32_t nA, uint32_t nB, int64_t c)
{
    const double pa = (double)nA * a.phi_per_count, pb = (double)nB * a.phi_per_count;
    const double inc = pa + pb - 1.0;
    double f;
    if (a.ham_form == 1)
        f = a.chiN * pa * pb + 0.5 * a.kappaN * inc * inc;
    else
        f = 0.5 * a.kappaN * inc * inc - 0.25 * a.chiN * (pa - pb) * (pa - pb);
    if (a.umb_lambda > 0.0) {
        // umbrella toward the target fields: (lambda/2) sum_t (phi_t - target_t)^2
        const float2 t = a.tgt[a.cell_off + c];
        const double da = pa - (double)t.x, db = pb - (double)t.y;
        f += 0.5 * a.umb_lambda * (da * da + db * db);
    }
    return f;
}

template <int CW>
__device__ __forceinline__ void obs_cells(const ObsArgs &a)
{
    constexpr int WPC = CW == COUNT_U16 ? 1 : 2, V = 4 / WPC;   // cells per 16 bytes
    NSum q[1] = {NSum{0.0, 0.0}};
    const DevSys &S = *a.sys;
    const int ny = S.n[1], nz = S.n[2], bs = S.brick_shift;
    const uint32_t *cnt = a.counts + WPC * a.cell_off;          // (16-byte aligned: cell_off is a multiple of 64)
    const int64_t block = (int64_t)blockIdx.x - a.chain_blocks, stride = (int64_t)a.cell_blocks * 256;
    const int64_t full = a.n_store / V;
    for (int64_t i = block * 256 + threadIdx.x; i < full; i += stride) {
        const uint4 w = reinterpret_cast<const uint4 *>(cnt)[i];
        const int64_t c = V * i;
        int left = V;                 // cells of the 16 bytes inside the grid
        if (bs) {
            int x, y, z;              // (a row of four cells in z of one brick holds the 16 bytes)
            cell_of_stored(S, c, x, y, z);
            left = y < ny ? nz - z : 0;
        }
        if constexpr (CW == COUNT_U16) {
            if (left > 0) nadd(q[0], cell_energy(a, w.x & 0xFFFFu, w.x >> 16, c));
            if (left > 1) nadd(q[0], cell_energy(a, w.y & 0xFFFFu, w.y >> 16, c + 1));
            if (left > 2) nadd(q[0], cell_energy(a, w.z & 0xFFFFu, w.z >> 16, c + 2));
            if (left > 3) nadd(q[0], cell_energy(a, w.w & 0xFFFFu, w.w >> 16, c + 3));
        } else {
            if (left > 0) nadd(q[0], cell_energy(a, w.x, w.y, c));
            if (left > 1) nadd(q[0], cell_energy(a, w.z, w.w, c + 1));
        }
    }
    const int64_t rest = full * V + threadIdx.x;                // (linear order only)
    if (block == 0 && rest < a.n_store) {
        const uint2 n = load_counts<CW>(cnt, rest);
        nadd(q[0], cell_energy(a, n.x, n.y, rest));
    }
    block_reduce_store<1>(q, a.partials + (int64_t)a.chain_blocks * 2 * (kObsQ - 1) + 2 * block);
}

// Blocks [0, chain_blocks) sum chains, the others cells.
template <int R, int CW>
__global__ __launch_bounds__(256) void k_observables(ObsArgs a)
{
    if ((int)blockIdx.x < a.chain_blocks) obs_chains<R>(a);
    else obs_cells<CW>(a);
}

// Wave k < 6 sums the partials of quantity k; wave 6 gathers the counters.
__global__ __launch_bounds__(64 * (kObsQ + 1)) void k_obs_finalize(ObsArgs a, ObsResult *out)
{
    const int k = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    if (k == kObsQ) {
        static_assert(kAcceptSlots == 128, "two slots per lane");
        unsigned long long v = a.accept[(int64_t)lane * kAcceptStride] + a.accept[(int64_t)(lane + 64) * kAcceptStride];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
        if (lane == 0) {
            out->accepted = v;
            out->conv[0] = a.conv[0];
            out->conv[1] = a.conv[1];
            out->status = *a.status;
        }
        return;
    }
    const bool chains = k < kObsQ - 1;
    const double *p = a.partials + (chains ? 2 * k : (int64_t)a.chain_blocks * 2 * (kObsQ - 1));
    const int n = chains ? a.chain_blocks : a.cell_blocks, step = chains ? 2 * (kObsQ - 1) : 2;
    // (four loads in flight; the order of the sums depends on n only)
    NSum acc{0.0, 0.0};
    for (int b = lane; b < n; b += 256) {
        NSum v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t at = (int64_t)(b + 64 * j < n ? b + 64 * j : b) * step;
            v[j] = NSum{p[at], p[at + 1]};
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (b + 64 * j < n) nmerge(acc, v[j]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        const NSum other{__shfl_down(acc.s, o), __shfl_down(acc.c, o)};
        nmerge(acc, other);
    }
    if (lane == 0) out->q[k] = acc.s + acc.c;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
template <int R, int CW, int DM, bool SMC>
static void launch_sweep_d(const SweepArgs &a, int blocks, hipStream_t st)
{
    const dim3 g(blocks), b(64 * a.waves_per_block);
    const size_t lds = sizeof(uint32_t) * list_words(DM == 2) * a.waves_per_block;
    // contexts without walls, zones, umbrella or caller-set classes launch
    // kernels built without that code (fewer registers)
    // block tiles: one tile per block (never with conversion zones, whose
    // chain sums stay within a wave)
    // only the plain and stream kernels count acceptances per tile
    SweepArgs o = a;
    if (!counts_per_tile(a)) o.acc_tile = nullptr;
    const bool stream = !SMC && !o.cpl && o.max_blocks == 0 && o.packed == 2;
    const bool block = o.max_blocks == 0 && o.packed == 1;
    o.wtiles = stream || block ? o.ptiles : o.tiles;
    o.n_wtiles = stream || block ? o.n_ptiles : o.n_tiles;
    o.remap_blocks = o.xcd_remap ? blocks & ~7 : 0;
    o.one_P = o.n_systems == 1 && !stream ? o.sys0_P : 0;
    if (o.one_P) {
        o.one_G = (block ? 64 * o.waves_per_block : kWave) / o.one_P;
        o.one_chains = o.sys0_chains;
        o.one_inv_P = (float)(1.0 / o.one_P);
    }
    if (o.cpl) {
        if (o.max_blocks > 0) hipLaunchKernelGGL((k_sweep<R, CW, true, DM, SMC, true, false>), g, b, lds, st, o);
        else if (o.packed == 1) hipLaunchKernelGGL((k_sweep<R, CW, false, DM, SMC, true, true>), g, b, lds, st, o);
        else hipLaunchKernelGGL((k_sweep<R, CW, false, DM, SMC, true, false>), g, b, lds, st, o);
    } else {
        if (o.max_blocks > 0) hipLaunchKernelGGL((k_sweep<R, CW, true, DM, SMC, false, false>), g, b, lds, st, o);
        else if (o.packed == 1) hipLaunchKernelGGL((k_sweep<R, CW, false, DM, SMC, false, true>), g, b, lds, st, o);
        else if (stream) hipLaunchKernelGGL((k_sweep_stream<R, CW, DM>), g, b, lds, st, o);
        else if (!SMC) hipLaunchKernelGGL((k_sweep_plain<R, CW, DM>), g, b, lds, st, o);
        else hipLaunchKernelGGL((k_sweep<R, CW, false, DM, SMC, false, false>), g, b, lds, st, o);
    }
}

template <int R, int CW, bool SMC>
static hipError_t launch_sweep_s(const SweepArgs &a, int blocks, hipStream_t st)
{
    if (a.density_mode == 1) launch_sweep_d<R, CW, 1, SMC>(a, blocks, st);
    else if (a.density_mode == 2) launch_sweep_d<R, CW, 2, SMC>(a, blocks, st);
    else if (a.density_mode == 3) launch_sweep_d<R, CW, 3, SMC>(a, blocks, st);
    else launch_sweep_d<R, CW, 0, SMC>(a, blocks, st);
    return hipGetLastError();
}

// Contexts with smart moves use the kernels that carry both move kinds (the
// kind is chosen per wave tile); the others keep the smaller uniform-only ones.
template <int R, int CW>
static hipError_t launch_sweep_t(const SweepArgs &a, int blocks, hipStream_t st)
{
    return a.smc ? launch_sweep_s<R, CW, true>(a, blocks, st) : launch_sweep_s<R, CW, false>(a, blocks, st);
}

hipError_t launch_sweep(int repr, int cw, const SweepArgs &a, hipStream_t st)
{
    int blocks = (a.n_tiles + a.waves_per_block - 1) / a.waves_per_block;
    if (a.max_blocks > 0 && blocks > a.max_blocks) blocks = a.max_blocks;
    if (a.packed == 1 && a.max_blocks == 0) blocks = a.n_ptiles;
    // stream tiles only for uniform moves without coupling (the launch below
    // takes wave tiles otherwise)
    if (a.packed == 2 && a.max_blocks == 0 && !a.cpl && !a.smc)
        blocks = (a.n_ptiles + a.waves_per_block - 1) / a.waves_per_block;
    if (blocks <= 0) return hipErrorInvalidConfiguration;   // the tile tables are empty
    if (repr == REPR_F32)
        return cw == COUNT_U16 ? launch_sweep_t<REPR_F32, COUNT_U16>(a, blocks, st)
                               : launch_sweep_t<REPR_F32, COUNT_U32>(a, blocks, st);
    return cw == COUNT_U16 ? launch_sweep_t<REPR_CELL, COUNT_U16>(a, blocks, st)
                           : launch_sweep_t<REPR_CELL, COUNT_U32>(a, blocks, st);
}

hipError_t launch_density(int repr, int cw, const DensityArgs &a, hipStream_t st)
{
    const int n = a.tile_end - a.tile_begin;
    if (n <= 0) return hipSuccess;
    const int blocks = (n + 3) / 4;
    if (repr == REPR_F32) {
        if (cw == COUNT_U16) hipLaunchKernelGGL((k_density<REPR_F32, COUNT_U16>), dim3(blocks), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((k_density<REPR_F32, COUNT_U32>), dim3(blocks), dim3(256), 0, st, a);
    } else {
        if (cw == COUNT_U16) hipLaunchKernelGGL((k_density<REPR_CELL, COUNT_U16>), dim3(blocks), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((k_density<REPR_CELL, COUNT_U32>), dim3(blocks), dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

template <int OP>
static hipError_t launch_state(int repr, const StateArgs &a, hipStream_t st)
{
    const int n = a.tile_end - a.tile_begin;
    if (n <= 0) return hipSuccess;
    const dim3 g((n + 3) / 4), b(256);
    if (repr == REPR_F32) hipLaunchKernelGGL((k_state<REPR_F32, OP>), g, b, 0, st, a);
    else hipLaunchKernelGGL((k_state<REPR_CELL, OP>), g, b, 0, st, a);
    return hipGetLastError();
}
hipError_t launch_export_state(int repr, const StateArgs &a, hipStream_t st) { return launch_state<STATE_OUT>(repr, a, st); }
hipError_t launch_export_positions(int repr, const StateArgs &a, hipStream_t st) { return launch_state<STATE_POS>(repr, a, st); }
hipError_t launch_check_state(int repr, const StateArgs &a, hipStream_t st) { return launch_state<STATE_CHECK>(repr, a, st); }
hipError_t launch_import_state(int repr, const StateArgs &a, hipStream_t st) { return launch_state<STATE_IN>(repr, a, st); }

hipError_t launch_fields(int cw, const FieldArgs &a, hipStream_t st)
{
    const int blocks = (int)((a.n_store + 1023) / 1024);
    if (blocks == 0) return hipSuccess;
    if (cw == COUNT_U16) hipLaunchKernelGGL((k_fields<COUNT_U16>), dim3(blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_fields<COUNT_U32>), dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_unpack_counts(int cw, const UnpackArgs &a, hipStream_t st)
{
    const int blocks = (int)((a.n_store + 1023) / 1024);
    if (blocks == 0) return hipSuccess;
    if (cw == COUNT_U16) hipLaunchKernelGGL((k_unpack_counts<COUNT_U16>), dim3(blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_unpack_counts<COUNT_U32>), dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_store_pairs(const DevSys *sys, int64_t n_cells, const float *in, float2 *out, hipStream_t st)
{
    if (n_cells <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_store_pairs, dim3((unsigned)((n_cells + 255) / 256)), dim3(256), 0, st, sys, n_cells, in, out);
    return hipGetLastError();
}

hipError_t launch_report(const Report &r, hipStream_t st)
{
    hipLaunchKernelGGL(k_report, dim3(1), dim3(1), 0, st, r);
    return hipGetLastError();
}

hipError_t launch_fold_faces(int cw, const FoldFacesArgs &a, int n_chunks, hipStream_t st)
{
    if (n_chunks <= 0) return hipSuccess;
    if (cw == COUNT_U16) hipLaunchKernelGGL((k_fold_faces<COUNT_U16>), dim3(n_chunks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_fold_faces<COUNT_U32>), dim3(n_chunks), dim3(256), 0, st, a);
    return hipGetLastError();
}

static int64_t mirror_blocks(int64_t count_words)
{
    const int64_t blocks = (count_words / 4 + 256 * kMirrorUnroll - 1) / (256 * kMirrorUnroll);
    return blocks > kMirrorBlocks ? kMirrorBlocks : blocks;
}

hipError_t launch_mirror(int cw, const MirrorArgs &a, hipStream_t st)
{
    if (a.count_words <= 0) return hipSuccess;
    const int64_t blocks = mirror_blocks(a.count_words);
    if (cw == COUNT_U16)
        hipLaunchKernelGGL((k_mirror<COUNT_U16>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_mirror<COUNT_U32>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_mirror_check(int cw, const MirrorArgs &a, uint32_t n_sweeps, uint64_t *ctr, hipStream_t st)
{
    if (a.count_words <= 0 || cw != COUNT_U16 || n_sweeps == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mirror_check, dim3(1), dim3(1024), 0, st, a.part, (int)mirror_blocks(a.count_words),
                       a.beads * (unsigned long long)n_sweeps, a.status, ctr, n_sweeps);
    return hipGetLastError();
}

hipError_t launch_stream_halo(int repr, const HaloArgs &a, hipStream_t st)
{
    if (a.n_ptiles <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)((2 * (int64_t)a.n_ptiles + 255) / 256);
    if (repr == REPR_F32)
        hipLaunchKernelGGL((k_stream_halo<BeadF32>), dim3(blocks), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_stream_halo<BeadCell>), dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_acc_fold(const Tile *tiles, int n_tiles, unsigned long long *acc_tile,
                                                  unsigned long long *accept)
{
    // tiles of one system are consecutive: the waves within a system add one sum
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    const bool on = t < n_tiles;
    unsigned long long v = on ? acc_tile[t] : 0ull;
    const uint32_t sys = tiles[on ? t : n_tiles - 1].sys;
    if (on) acc_tile[t] = 0ull;
    const int slot = (t >> 6) % kAcceptSlots;
    if (__all(sys == (uint32_t)__builtin_amdgcn_readfirstlane((int)sys))) {
        for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
        if ((threadIdx.x & 63) != 0) v = 0ull;
    }
    if (v != 0ull) atomicAdd(accept + ((int64_t)sys * kAcceptSlots + slot) * kAcceptStride, v);
}

hipError_t launch_acc_fold(const Tile *tiles, int n_tiles, unsigned long long *acc_tile, unsigned long long *accept,
                           hipStream_t st)
{
    if (n_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_acc_fold, dim3((unsigned)((n_tiles + 255) / 256)), dim3(256), 0, st, tiles, n_tiles, acc_tile,
                       accept);
    return hipGetLastError();
}

hipError_t launch_make_tiles(const MakeTilesArgs &a, hipStream_t st)
{
    if (a.n_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_make_tiles, dim3((unsigned)((a.n_tiles + 255) / 256)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_fold(int cw, const uint32_t *counts_in, uint32_t *delta, uint32_t *counts_out, int64_t n,
                       uint32_t *status, hipStream_t st, uint64_t *ctr, uint32_t advance)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = ((n + 3) / 4 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (cw == COUNT_U16)
        hipLaunchKernelGGL((k_fold<COUNT_U16>), dim3((unsigned)blocks), dim3(256), 0, st, counts_in, delta, counts_out, n, status, ctr, advance);
    else
        hipLaunchKernelGGL((k_fold<COUNT_U32>), dim3((unsigned)blocks), dim3(256), 0, st, counts_in, delta, counts_out, n, status, ctr, advance);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t launch_advance(uint64_t *ctr, uint32_t n, hipStream_t st)
{
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(1), 0, st, ctr, n);
    return hipGetLastError();
}

hipError_t launch_iota_chains(const ReorderArgs &a, hipStream_t st)
{
    const int blocks = (a.n_tiles + 3) / 4;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_iota_chains, dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_reorder(int repr, const ReorderArgs &a, hipStream_t st)
{
    const int tblocks = (a.n_tiles + 3) / 4;
    if (tblocks == 0) return hipSuccess;
    hipError_t e = launch_fill_u32(a.hist, a.total_blocks, 0u, st);
    if (e != hipSuccess) return e;
    if (repr == REPR_F32) hipLaunchKernelGGL((k_reorder_keys<REPR_F32>), dim3(tblocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_reorder_keys<REPR_CELL>), dim3(tblocks), dim3(256), 0, st, a);
    const int nb = (int)((a.total_blocks + kScanTile - 1) / kScanTile);
    hipLaunchKernelGGL(k_scan_partials, dim3(nb), dim3(kScanBlock), 0, st, a.hist, a.total_blocks, a.bsum);
    hipLaunchKernelGGL(k_scan_bsum, dim3(1), dim3(kScanBlock), 0, st, a.bsum, nb);
    hipLaunchKernelGGL(k_scan_apply, dim3(nb), dim3(kScanBlock), 0, st, a.hist, a.total_blocks, a.bsum);
    const int cblocks = (int)((a.total_chains + 255) / 256);
    hipLaunchKernelGGL(k_reorder_scatter, dim3(cblocks), dim3(256), 0, st, a);
    if (repr == REPR_F32) hipLaunchKernelGGL((k_reorder_permute<REPR_F32>), dim3(tblocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_reorder_permute<REPR_CELL>), dim3(tblocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

int64_t reorder_bsum_words(int64_t total_blocks) { return (total_blocks + kScanTile - 1) / kScanTile; }

static dim3 walk_blocks(const InitArgs &a) { return dim3((unsigned)((a.tile_end - a.tile_begin + kWalkWaves - 1) / kWalkWaves)); }

hipError_t launch_init(const InitArgs &a, hipStream_t st)
{
    if (a.tile_end <= a.tile_begin) return hipSuccess;
    hipLaunchKernelGGL(k_init_walks, walk_blocks(a), dim3(64 * kWalkWaves), 0, st, a);
    return hipGetLastError();
}

int64_t place_bsum_words(int64_t n_cells) { return (n_cells + kScan64Tile - 1) / kScan64Tile; }

hipError_t launch_place(const PlaceArgs &a, unsigned long long *bsum, hipStream_t st)
{
    if (a.n_cells <= 0 || a.ia.tile_end <= a.ia.tile_begin) return hipSuccess;
    const int cb = (int)((a.n_cells + 255) / 256);
    hipLaunchKernelGGL(k_place_weights, dim3(cb), dim3(256), 0, st, a);
    const int nb = (int)place_bsum_words(a.n_cells);
    for (int k = 0; k < 2; ++k) {
        unsigned long long *x = a.W + k * a.n_cells;
        hipLaunchKernelGGL(k_scan64_partials, dim3(nb), dim3(kScan64Block), 0, st, x, a.n_cells, bsum);
        hipLaunchKernelGGL(k_scan64_bsum, dim3(1), dim3(kScan64Block), 0, st, bsum, nb);
        hipLaunchKernelGGL(k_scan64_apply, dim3(nb), dim3(kScan64Block), 0, st, x, a.n_cells, bsum);
    }
    hipLaunchKernelGGL(k_place_chains, walk_blocks(a.ia), dim3(64 * kWalkWaves), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_observables(int repr, int cw, const ObsArgs &args, ObsResult *out, hipStream_t st)
{
    ObsArgs a = args;
    const int64_t cb = ((int64_t)a.tile_end - a.tile_begin + 3) / 4, mb = (a.n_store + kObsCells - 1) / kObsCells;
    a.chain_blocks = (int)(cb < kObsBlocks ? cb : kObsBlocks);
    a.cell_blocks = (int)(mb < kObsBlocks ? mb : kObsBlocks);
    const dim3 g(a.chain_blocks + a.cell_blocks), b(256);
    if (repr == REPR_F32) {
        if (cw == COUNT_U16) hipLaunchKernelGGL((k_observables<REPR_F32, COUNT_U16>), g, b, 0, st, a);
        else hipLaunchKernelGGL((k_observables<REPR_F32, COUNT_U32>), g, b, 0, st, a);
    } else {
        if (cw == COUNT_U16) hipLaunchKernelGGL((k_observables<REPR_CELL, COUNT_U16>), g, b, 0, st, a);
        else hipLaunchKernelGGL((k_observables<REPR_CELL, COUNT_U32>), g, b, 0, st, a);
    }
    hipLaunchKernelGGL(k_obs_finalize, dim3(1), dim3(64 * (kObsQ + 1)), 0, st, a, out);
    return hipGetLastError();
}

}  // namespace soma
