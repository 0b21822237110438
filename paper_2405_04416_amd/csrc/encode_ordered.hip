// Hash-grid encode of samples in spatial order (order.hip): forward gather into sample-major rows, and the table gradient
// of the coarser levels.
#include "encode_common.h"
#include "order_common.h"
#include <algorithm>
#include <mutex>
#include <type_traits>

namespace {

using namespace dg_encode;
using namespace dg_order;
using dg::kSplitLevels;

constexpr int kBlock = 256;
constexpr uint32_t kXcds = 8;

// Two lanes per sample (gather_pair), level after level of the same sample.  Consecutive workgroups of an XCD take
// consecutive samples (workgroups are handed out to the XCDs in turn), so the lines that neighbours share meet in one L2.
// The even lane keeps the lower half of the levels, the odd lane the upper half: each writes half of the sample's row.
// Bound by the cache lines fetched past the L2 on the levels too fine for neighbours to share them (T = 2^24, 33.5 M samples:
// levels 13..15 take 7.3 of 10.4 ms at 51 G lines/s, levels 0..9 1.7 ms), by instructions and vector-cache look-ups on the
// others.  Against the gather in ray order, level after level: 33.5 M samples, T = 2^24 21.6 -> 10.4 ms; 19.8 M, T = 2^24
// 12.3 -> 6.8; 13.3 M, T = 2^19 2.38 -> 1.49; scattered rows of 64 bytes instead of planes cost 0.8, 0.47 and 0.3 ms of it.
// LEVELS: 16, or 12 where the finer levels go through encode_planes_kernel; a row is LEVELS x 4 bytes.
template <int LEVELS>
__global__ void __launch_bounds__(kBlock)
encode_fwd_ordered_kernel(dg_grid_desc g, const float2 *__restrict__ table, const float4 *__restrict__ ordered, uint64_t N,
                          bool by_position, uint32_t *__restrict__ feat, uint32_t blocks_per_xcd)
{
    const uint32_t block = (blockIdx.x % kXcds) * blocks_per_xcd + blockIdx.x / kXcds;
    const uint64_t i = (uint64_t)block * (kBlock / 2) + threadIdx.x / 2;
    const uint32_t cx = threadIdx.x & 1u;
    if (i >= N) return;                                   // both lanes of a pair
    const float4 s = ordered[i];
    const float uu[3] = {s.x, s.y, s.z};
    const uint32_t mask = (1u << g.log2_T) - 1u;
    constexpr int kHalfRow = LEVELS / 2;
    uint32_t out[kHalfRow];
#pragma unroll
    for (int l = 0; l < LEVELS; ++l) {
        const float2 v = gather_pair(level_of(g, l), mask, table, uu, cx);
        const uint32_t f = __builtin_bit_cast(uint32_t, __floats2half2_rn(v.x, v.y));
        if (l < kHalfRow) out[l] = f;
        else out[l - kHalfRow] = cx ? f : out[l - kHalfRow];
    }
    uint32_t *half_row = feat + (size_t)(by_position ? (uint32_t)i : __float_as_uint(s.w)) * LEVELS + kHalfRow * cx;
    if constexpr (kHalfRow % 4 == 0) {
#pragma unroll
        for (int k = 0; k < kHalfRow; k += 4) *reinterpret_cast<uint4 *>(half_row + k) = make_uint4(out[k], out[k + 1], out[k + 2], out[k + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < kHalfRow; k += 2) *reinterpret_cast<uint2 *>(half_row + k) = make_uint2(out[k], out[k + 1]);
    }
}

// Levels 12..15 as planes, level after level, so that one level's table at a time lies in the L2s: SORTED from the sorted list, in its
// order, else in ray order.  With T = 2^19 the sixteen levels that the ordered gather walks at once fetch 5 lines per sample past an L2 that
// holds one of them, at the rate of the fabric; the finer ones are most of it, and below some 6 M samples neighbours share few of their
// lines.  T = 2^19, 3.3 M samples: 612 us with all levels in one walk, 186 + 262 this way; 13.3 M: 1471 against 789 + 1023.  Refresh of an
// occupancy grid, 8.4 M sorted candidates: 1190 against 472 + 485.  T = 2^18, 3.3 M: 441 against 178 + 206.
template <bool SORTED>
__global__ void __launch_bounds__(kBlock)
encode_planes_kernel(dg_grid_desc g, const float2 *__restrict__ table, const float *__restrict__ u, uint64_t N, uint32_t *__restrict__ feat, uint32_t n_tiles)
{
    const uint32_t l = kSplitLevels + blockIdx.x / n_tiles;
    const uint64_t s = (uint64_t)(blockIdx.x % n_tiles) * (kBlock / 2) + threadIdx.x / 2;
    const uint32_t cx = threadIdx.x & 1u;
    if (s >= N) return;                                   // both lanes of a pair
    const float *at = u + (SORTED ? 4 : 3) * s;
    const float uu[3] = {at[0], at[1], at[2]};
    const float2 f = gather_pair(level_of(g, l), (1u << g.log2_T) - 1u, table, uu, cx);
    if (cx == 0u) feat[(size_t)l * N + s] = __builtin_bit_cast(uint32_t, __floats2half2_rn(f.x, f.y));
}

// Table gradient of levels [0, n_merged): a workgroup takes a piece of a brick and sums all its contributions in LDS -- the
// brick's vertices at those levels, in 64 bits, one plane per feature -- then adds the sums to the table gradient, one
// global add per vertex the brick touches.
// Levels [0, n_wide) -- the coarse levels, which ray order sums in fp64 -- are summed in fp64, the other levels, which in ray order
// pass through records of 27-bit values, in fixed point.  Over the bricks levels [0, n_fold) are summed in fp64 as well (a vertex of
// the coarsest level gets hundreds of them): into `wide`, which fold_wide_kernel adds to the table.  The others reach the table
// with an fp32 add per brick.  Against 64-bit sums (33.5 M samples, 25200 bricks, 2-norm of levels 0 / 3 / 7): ray order 2.3e-7 / 1.9e-7 /
// 2.5e-7, this 2.6e-8 / 2.5e-8 / 3.9e-8; level 0 in fixed point with fp32 adds 2.6e-7 (13.3 M samples), and nothing was left there of
// gradients below 2^-38 of the largest.
// Clearing and folding `wide` takes some 12 us.
// A value v becomes round(v * 2^k): the add of 1.5 * 2^52 in fp64 leaves it in the low mantissa bits, in two's complement.  k is
// such that the magnitudes of a piece (at most 2^12 samples) sum to less than 2^50; adding the doubles' bit patterns as
// integers adds those low bits, what happens above bit 50 is dropped when the sum is read.  (Integer adds are the fastest LDS
// atomics: random addresses 3.6 T adds/s against 1.95 in fp64.)
// A lane takes two levels and a run of consecutive samples: the eight corner sums of the cell that the run is in stay in registers and
// go to LDS when it leaves the cell, and every eight (six) samples together with those of its neighbours in the same cell: at most 96
// samples of a cell are added up in fp32.  Neighbouring lanes take the same samples at the neighbouring levels, so that what they read of
// a sample's row of the gradient lies side by side and costs the vector cache one or two look-ups, not one per lane.  Two or three of
// the eight wavefronts share the lower half of the levels, whose runs seldom leave a cell, the others the upper half.
// What a level needs is worked out once per workgroup and kept in LDS; the write-out takes 25 vector instructions per 64 sums.
// 13.3 M samples, T = 2^19, levels 0..11: 1.27 ms; 33.5 M, T = 2^24, levels 0..9: 2.33 ms, of which the rows, some 1.6 random lines each,
// take 0.9 at the rate of the fabric.  Full pieces in one cell, terms of either sign: 8.2e-8 from 64-bit sums.  Measured on the way:
// - runs of up to 66 samples and then sums over lanes, up to 512 samples of a cell in fp32: 1.23 and 2.21 ms, but 1.2e-7 from 64-bit sums
//   (pairs of samples and sums over 64 lanes: 8.6e-8); sixteen samples at a time 1.18 and 2.21 ms, 9.3e-8, twelve 1.25 and 2.27 ms, 8.8e-8;
// - eight samples at a time without sums over lanes: 1.40 and 2.79 ms (adds to one address take turns);
// - every wavefront at all levels of an eighth of the samples, two samples per lane at a time: 1.66 and 3.01 ms (the sums over lanes
//   and the adds to LDS come every other sample, and every level is set up eight times for the write-out);
// - a wavefront per pair of levels, every lane at a row of its own: 1.27 and 2.95 ms, of which the loads alone 0.94 and 2.3;
// - and with whole runs: one and two wavefronts at the lower half 1.46 and 3.10 ms, three and four 1.30 and 2.46 ms; 80 registers for six
//   wavefronts per SIMD 2.4 and 4.9 ms (spills).
struct Boxes { uint32_t n_merged, n_wide, n_fold, dim[kMaxMerged][3], first[kMaxMerged + 1]; };

constexpr int kBrickWaves = 8;
static_assert(kMaxMerged <= 12, "at most three pairs of levels to a wavefront");

// First cell of brick i's box along one axis: a hair (kBoxSlack of a cell) below the brick's edge.  A sample of brick i has
// i <= u * n < i + 1 in fp32, so its cell, floor(u * scale) in fp32, differs from what the exact edges give by less than three
// roundings of a position of at most kMaxMergedScale cells -- 1.5e-3 cells --, and a box of floor(scale / n + 2e-2) + 3
// vertices (dg_order_desc_init) has room for every cell the brick's samples can be in.
constexpr float kBoxSlack = 4e-3f;
__device__ __forceinline__ uint32_t box_low(const Bricks &b, uint32_t i, int axis, float scale)
{
    const float edge = (float)i / b.per_unit[axis] * scale - kBoxSlack;
    return edge > 0.0f ? (uint32_t)edge : 0u;
}

// What the sums of a level need, worked out once per workgroup.
struct LevelBox {
    float scale[3];
    uint32_t first;                          // first vertex of the box among the sums
    float last[3];                           // the last cell
    uint32_t last_slot;                      // last slot whose eight corners lie in the box
    float nx, nxy, origin;                   // strides of the box; slot = x + nx y + nxy z - origin (all exact: below 2^24)
    uint32_t wide;
    uint32_t low[3], count;                  // first cell of the box; its vertices
    float per_nx, per_nxy;                   // reciprocals of the strides
    uint32_t unused[2];
};

__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ float uniform(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

__device__ __forceinline__ void add_fixed(unsigned long long *slot, float v, double to_fixed)
{
    __hip_atomic_fetch_add(slot, (unsigned long long)__double_as_longlong(__builtin_fma((double)v, to_fixed, 6755399441055744.0)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void add_wide(unsigned long long *slot, float v)
{
    asm("" : "+v"(v));          // the sixteen conversions stay on this side of the branch: ahead of it they hold 32 registers
    __hip_atomic_fetch_add(reinterpret_cast<double *>(slot), (double)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// the eight corner sums of the cell whose corner 0 is vertex d of the box
__device__ __forceinline__ void add_to_box(unsigned long long *d, bool wide, double to_fixed, uint32_t nx, uint32_t nxy, uint32_t plane, const float (&vx)[8],
                                           const float (&vy)[8])
{
    unsigned long long *const row[4] = {d, d + nx, d + nxy, d + nx + nxy};
    // one branch around all sixteen adds (a choice per add puts a branch between any two of them)
    if (wide) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            add_wide(row[c >> 1] + (c & 1), vx[c]);
            add_wide(row[c >> 1] + (c & 1) + plane, vy[c]);
        }
    } else {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            add_fixed(row[c >> 1] + (c & 1), vx[c], to_fixed);
            add_fixed(row[c >> 1] + (c & 1) + plane, vy[c], to_fixed);
        }
    }
}

// Adds the sums that lanes hold; lanes STRIDE apart are at the same levels.  A segmented sum along those lanes
// within each row of 16 (a run of lanes in the same cell starts where `head` is set), then its last lane adds.
template <int STRIDE, int STEP>
__device__ __forceinline__ void row_step(float (&vx)[8], float (&vy)[8], int &f)
{
    if constexpr (STRIDE * STEP < 16) seg_step<0x110 + STRIDE * STEP, 0xF>(vx, vy, f);
}

template <int STRIDE>
__device__ __forceinline__ void finish_runs(unsigned long long *sums, const LevelBox (&box)[2], const uint32_t (&slot)[2], float (&vx)[2][8], float (&vy)[2][8],
                                            bool live, int lane, double to_fixed, uint32_t plane)
{
    static_assert(STRIDE <= 3, "steps of 1, 2, 4 and 8 runs cover a row");
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        const uint32_t mine = live ? slot[which] : ~0u;               // lanes without samples are runs of their own
        const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0x110 + STRIDE, 0xF, 0xF, true);
        const int head = (lane & 15) < STRIDE || before != mine ? 1 : 0;
        const int next = __builtin_amdgcn_update_dpp(1, head, 0x100 + STRIDE, 0xF, 0xF, false);        // of the lane STRIDE above; 1 past the row's end
        int f = head;
        row_step<STRIDE, 1>(vx[which], vy[which], f);
        row_step<STRIDE, 2>(vx[which], vy[which], f);
        row_step<STRIDE, 4>(vx[which], vy[which], f);
        row_step<STRIDE, 8>(vx[which], vy[which], f);
        if (live && next) {
            const LevelBox &v = box[which];
            add_to_box(sums + v.first + slot[which], v.wide, to_fixed, (uint32_t)v.nx, (uint32_t)v.nxy, plane, vx[which], vy[which]);
        }
    }
}

__global__ void __launch_bounds__(kBrickWaves * 64, 4)       // two workgroups per compute unit: four wavefronts per SIMD, 128 registers
brick_bwd_kernel(dg_grid_desc g, Bricks b, Boxes boxes, const uint2 *__restrict__ pieces, const float4 *__restrict__ ordered,
                 const float4 *__restrict__ dfeat, const uint32_t *__restrict__ largest, float *__restrict__ dtable, double *__restrict__ wide_table)
{
    extern __shared__ __attribute__((aligned(16))) unsigned long long sums[];
    __shared__ LevelBox levels[kMaxMerged];
    if (blockIdx.x >= pieces[0].x) return;
    const uint2 piece = pieces[1 + blockIdx.x];
    const uint32_t begin = piece.y, n = pieces[2 + blockIdx.x].y - begin;
    const uint32_t n_vertices = boxes.first[boxes.n_merged];
    const uint32_t brick[3] = {piece.x % b.n[0], piece.x / b.n[0] % b.n[1], piece.x / (b.n[0] * b.n[1])};
    if (threadIdx.x < boxes.n_merged) {
        const uint32_t l = threadIdx.x, nx = boxes.dim[l][0], nxy = nx * boxes.dim[l][1];
        LevelBox v;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v.scale[a] = g.scale[l][a];
            v.last[a] = (float)(g.res[l][a] - 1u);
            v.low[a] = box_low(b, brick[a], a, v.scale[a]);
        }
        v.first = boxes.first[l];
        v.count = boxes.first[l + 1] - v.first;
        v.last_slot = v.count - 2u - nx - nxy;
        v.nx = (float)nx;
        v.nxy = (float)nxy;
        v.origin = (float)(v.low[0] + nx * v.low[1] + nxy * v.low[2]);
        v.wide = l < boxes.n_wide;
        v.per_nx = 1.0f / v.nx;
        v.per_nxy = 1.0f / v.nxy;
        levels[l] = v;
    }
    uint4 *const clear = reinterpret_cast<uint4 *>(sums);
    for (uint32_t i = threadIdx.x; i < n_vertices; i += blockDim.x) clear[i] = make_uint4(0u, 0u, 0u, 0u);
    const uint32_t mask = (1u << g.log2_T) - 1u;
    const int lane = threadIdx.x % dg::kWave;
    const uint32_t pairs = boxes.n_merged / 2;
    const uint32_t top = *largest >> 23;                             // biased exponent (0: no smaller k needed)
    if (top == 255u) {      // not finite: no scale fits, the gradient is marked instead
        for (uint32_t l = threadIdx.x; l < boxes.n_merged; l += blockDim.x) {
            const LevelGeom lv = level_of(g, l);
            const uint32_t e = vertex_entry(lv, mask, box_low(b, brick[0], 0, lv.scale[0]), box_low(b, brick[1], 1, lv.scale[1]), box_low(b, brick[2], 2, lv.scale[2]));
            dtable[2 * ((size_t)lv.offset + e)] = __uint_as_float(0x7fc00000u);
        }
        return;
    }
    static_assert(kPiece <= 1u << 12, "2^12 samples of the largest magnitude sum to less than 2^50 units");
    const int k_scale = 50 - 12 - 1 - ((int)(top ? top : 1u) - 127);
    const double to_fixed = __longlong_as_double((long long)(1023 + k_scale) << 52), from_fixed = __longlong_as_double((long long)(1023 - k_scale) << 52);
    __syncthreads();
    {
        const char *const list = reinterpret_cast<const char *>(ordered + begin);
        const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / dg::kWave));
        const uint32_t lower = pairs / 2, lower_waves = lower == 0u ? 0u : lower < pairs - lower ? 2u : 3u;
        const bool is_lower = wave < lower_waves;
        const uint32_t here = is_lower ? lower : pairs - lower, per_wave = dg::kWave / here;            // pairs of levels, runs per wavefront
        const uint32_t runs = (is_lower ? lower_waves : kBrickWaves - lower_waves) * per_wave;
        const uint32_t in_wave = lane / here, q = (is_lower ? 0u : lower) + lane % here;
        const uint32_t run = (n + runs - 1u) / runs;                                                    // samples per lane
        // lanes that are left over start past the end
        const uint32_t i0 = in_wave < per_wave ? ((is_lower ? wave : wave - lower_waves) * per_wave + in_wave) * run : n;
        const LevelBox box[2] = {levels[2 * q], levels[2 * q + 1]};
        float vx[2][8], vy[2][8];
        uint32_t slot[2] = {0u, 0u};                                  // of the cells whose sums vx, vy are
        // a sample's coordinates are asked for two samples ahead, its row of the gradient one ahead
        const uint32_t last = (n - 1u) * (uint32_t)sizeof(float4);
        uint32_t at = i0 * (uint32_t)sizeof(float4);
        auto sample = [&](uint32_t offset) { return *reinterpret_cast<const float4 *>(list + min(offset, last)); };
        float4 s = sample(at), s_next = sample(at + (uint32_t)sizeof(float4));
        float4 row = dfeat[(size_t)__float_as_uint(s.w) * pairs + q];
        // samples that a lane adds up in fp32 before the sums over lanes, which take four steps with runs next to one another, else three: on
        // average 7.5 roundings per sample either way
        const uint32_t in_fp32 = here == 1u ? 6u : 8u;
#pragma unroll 1
        for (uint32_t k0 = 0; k0 < run; k0 += in_fp32) {
            const bool live = at <= last;                                 // the lane has samples among these
#pragma unroll
            for (int which = 0; which < 2; ++which)
#pragma unroll
                for (int c = 0; c < 8; ++c) { vx[which][c] = 0.0f; vy[which][c] = 0.0f; }
            const uint32_t k1 = min(k0 + in_fp32, run);
#pragma unroll 1
            for (uint32_t k = k0; k < k1; ++k, at += (uint32_t)sizeof(float4)) {
                const float uu[3] = {unit(s.x), unit(s.y), unit(s.z)}, gx[2] = {row.x, row.z}, gy[2] = {row.y, row.w};
                s = s_next;
                row = dfeat[(size_t)__float_as_uint(s.w) * pairs + q];
                s_next = sample(at + 2u * (uint32_t)sizeof(float4));
                if (at > last) continue;                                  // past the end of the piece
#pragma unroll
                for (int which = 0; which < 2; ++which) {
                    const LevelBox &v = box[which];
                    float cell[3], w1[3], w0[3];
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        locate_unit(uu[a], v.scale[a], v.last[a], cell[a], w1[a]);
                        w0[a] = 1.0f - w1[a];
                    }
                    // whole numbers below 2^24: exact in fp32
                    const uint32_t now = min((uint32_t)__builtin_fmaf(cell[2], v.nxy, __builtin_fmaf(cell[1], v.nx, cell[0] - v.origin)), v.last_slot);
                    if (k > k0 && now != slot[which]) {
                        add_to_box(sums + v.first + slot[which], v.wide, to_fixed, (uint32_t)v.nx, (uint32_t)v.nxy, n_vertices, vx[which], vy[which]);
#pragma unroll
                        for (int c = 0; c < 8; ++c) { vx[which][c] = 0.0f; vy[which][c] = 0.0f; }
                    }
                    slot[which] = now;
                    const float px[2] = {gx[which] * w0[0], gx[which] * w1[0]}, py[2] = {gy[which] * w0[0], gy[which] * w1[0]};
                    const float yz[4] = {w0[1] * w0[2], w1[1] * w0[2], w0[1] * w1[2], w1[1] * w1[2]};
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        vx[which][c] = __builtin_fmaf(px[c & 1], yz[c >> 1], vx[which][c]);
                        vy[which][c] = __builtin_fmaf(py[c & 1], yz[c >> 1], vy[which][c]);
                    }
                }
            }
            // what the lanes then hold, first summed over the lanes of a row of 16 that are in the same cell: on the coarser levels
            // these are most of them, and adds to one address take turns
            if (here == 1u) finish_runs<1>(sums, box, slot, vx, vy, live, lane, to_fixed, n_vertices);
            else if (here == 2u) finish_runs<2>(sums, box, slot, vx, vy, live, lane, to_fixed, n_vertices);
            else finish_runs<3>(sums, box, slot, vx, vy, live, lane, to_fixed, n_vertices);
        }
    }
    __syncthreads();
    for (uint32_t l = 0; l < boxes.n_merged; ++l) {
        const LevelGeom lv = level_of(g, l);
        const LevelBox &v = levels[l];
        const uint32_t low[3] = {uniform(v.low[0]), uniform(v.low[1]), uniform(v.low[2])}, first = uniform(v.first), count = uniform(v.count);
        const float fnx = uniform(v.nx), fnxy = uniform(v.nxy), per_nx = uniform(v.per_nx), per_nxy = uniform(v.per_nxy);
        const uint32_t origin = lv.dense ? vertex_entry(lv, mask, low[0], low[1], low[2]) : 0u, ny1 = lv.res[1] + 1u, nx1 = lv.res[0] + 1u;
        // neighbouring lanes add the two features of neighbouring vertices: whole cache lines per instruction
        auto write_out = [&](auto dense, auto add) {
            const uint32_t f = threadIdx.x & 1u;                     // blockDim.x is even
            const unsigned long long *from = sums + f * n_vertices + first;
            for (uint32_t v = threadIdx.x >> 1; v < count; v += blockDim.x >> 1) {
                // quotients of v + 1/2: a whole number below 2^13 is half a unit from the next multiple, far more than the products' rounding
                const float fv = (float)v, fz = floorf(__builtin_fmaf(fv, per_nxy, 0.5f * per_nxy)), in_z = __builtin_fmaf(-fz, fnxy, fv);
                const float fy = floorf(__builtin_fmaf(in_z, per_nx, 0.5f * per_nx));
                const uint32_t x = (uint32_t)__builtin_fmaf(-fy, fnx, in_z), y = (uint32_t)fy, z = (uint32_t)fz;
                const uint32_t e = dense ? origin + x + nx1 * (y + ny1 * z) : ((low[0] + x) ^ (low[1] + y) * kPrimeY ^ (low[2] + z) * kPrimeZ) & mask;
                add(from[v], 2u * e + f);                            // below 2^25
            }
        };
        auto write_level = [&](auto add) {
            if (lv.dense) write_out(std::true_type{}, add);
            else write_out(std::false_type{}, add);
        };
        if (l < boxes.n_fold) {
            double *dst = wide_table + 2 * (size_t)lv.offset;
            const bool wide = l < boxes.n_wide;
            write_level([&](unsigned long long held, uint32_t at) {
                const double sum = wide ? __longlong_as_double((long long)held) : from_low_bits(held) * from_fixed;
                if (sum != 0.0) unsafeAtomicAdd(dst + at, sum);
            });
        } else {
            float *dst = dtable + 2 * (size_t)lv.offset;
            write_level([&](unsigned long long held, uint32_t at) {
                const float sum = (float)(from_low_bits(held) * from_fixed);
                if (sum != 0.0f) unsafeAtomicAdd(dst + at, sum);
            });
        }
    }
}

// ---- forward, brick by brick
constexpr int kFwdThreads = 1024;
constexpr uint32_t kFwdChunk = 16;

// what a gather from the brick's box of a level needs
struct FwdBox {
    float scale[3], origin;                  // slot = x + nx y + nxy z - origin (all exact: below 2^24)
    float last[3], nx;
    float nxy;
    uint32_t first, last_slot, nx_bytes;     // first: of the level's sums, in bytes; last_slot: whose eight corners lie in the box
    uint32_t nxy_bytes, unused[3];
};
// and what filling it does: its place in the grid and in the table
struct FwdFill {
    float nx, nxy, per_nx, per_nxy;
    uint32_t low[3], dense;
    uint32_t res[3], offset;                 // offset: of the level's entries in the table
};

// Rows of the first kSplitLevels levels, the finer ones of which come as planes (encode_planes_kernel).  What bounds the walk above is the vector cache,
// a look-up per clock and compute unit, whatever the walk finds there.  Here a workgroup takes a piece of a brick and first copies the
// brick's vertices at the merged levels to LDS -- 5000 of them, where its samples make 30 000 look-ups --; a sample's two lanes then take half of these
// levels each, eight corners from LDS.  Levels between the merged and the split ones are gathered as above, asked for before the others' arithmetic.
// 3.3 M samples, T = 2^19, ten levels of twelve merged 213 -> 134 us; 8.4 M 473 -> 280.  Rows of all sixteen levels this way are no faster: the finer levels
// bound them, and the LDS of the boxes leaves room for fewer wavefronts to wait for their lines (13.3 M, T = 2^19 1486 / 1512 us; 33.5 M,
// T = 2^24 10.3 / 10.4 ms; 1.55 M with eight merged levels 177 / 348 us).  Boxes filled level by level, without loads under way together: 147 us
// instead of 138; equal numbers of pieces to every XCD in one stretch: 16.4 ms instead of 10.7, as one gets the crowded side of the box.
template <int MERGED>
__global__ void __launch_bounds__(kFwdThreads)
encode_fwd_bricks_kernel(dg_grid_desc g, Bricks b, Boxes boxes, const uint2 *__restrict__ pieces, const float2 *__restrict__ table,
                         const float4 *__restrict__ ordered, bool by_position, uint32_t *__restrict__ feat)
{
    constexpr int LEVELS = kSplitLevels;
    extern __shared__ __attribute__((aligned(16))) float2 box[];
    __shared__ __attribute__((aligned(16))) FwdBox levels[MERGED];
    __shared__ __attribute__((aligned(16))) FwdFill fills[MERGED];
    // an XCD takes kFwdChunk consecutive pieces, the next one the next: neighbours meet in one L2, and no XCD gets the empty side of the box
    const uint32_t in_xcd = blockIdx.x / kXcds, index = (in_xcd / kFwdChunk * kXcds + blockIdx.x % kXcds) * kFwdChunk + in_xcd % kFwdChunk;
    if (index >= pieces[0].x) return;
    const uint2 piece = pieces[1 + index];
    const uint32_t begin = piece.y, n = pieces[2 + index].y - begin;
    const uint32_t mask = (1u << g.log2_T) - 1u;
    if (threadIdx.x < MERGED) {
        const uint32_t l = threadIdx.x, nx = boxes.dim[l][0], nxy = nx * boxes.dim[l][1], count = boxes.first[l + 1] - boxes.first[l];
        const uint32_t brick[3] = {piece.x % b.n[0], piece.x / b.n[0] % b.n[1], piece.x / (b.n[0] * b.n[1])};
        FwdBox v{};
        FwdFill w;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v.scale[a] = g.scale[l][a];
            v.last[a] = (float)(g.res[l][a] - 1u);
            w.low[a] = box_low(b, brick[a], a, v.scale[a]);
            w.res[a] = g.res[l][a];
        }
        v.origin = (float)(w.low[0] + nx * w.low[1] + nxy * w.low[2]);
        v.nx = w.nx = (float)nx;
        v.nxy = w.nxy = (float)nxy;
        v.first = boxes.first[l] * (uint32_t)sizeof(float2);
        v.last_slot = count - 2u - nx - nxy;
        v.nx_bytes = nx * (uint32_t)sizeof(float2);
        v.nxy_bytes = nxy * (uint32_t)sizeof(float2);
        w.per_nx = 1.0f / w.nx;
        w.per_nxy = 1.0f / w.nxy;
        w.dense = g.dense[l];
        w.offset = g.offset[l];
        levels[l] = v;
        fills[l] = w;
    }
    __syncthreads();
    // The boxes of all levels in one go: a thread's vertices are asked for before the first of them is waited for
    {
        constexpr int kPer = (int)((kMaxBoxVertices + kFwdThreads - 1) / kFwdThreads);
        const uint32_t n_vertices = boxes.first[MERGED];
        float2 entry[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const uint32_t at = min(k * kFwdThreads + threadIdx.x, n_vertices - 1u);
            uint32_t l = 0, first = 0;
#pragma unroll
            for (int m = 1; m < MERGED; ++m)
                if (at >= boxes.first[m]) { l = m; first = boxes.first[m]; }
            const FwdFill w = fills[l];
            // quotients as in brick_bwd_kernel; vertices beyond the grid, which no cell has, repeat the last one
            const float fv = (float)(at - first), fz = floorf(__builtin_fmaf(fv, w.per_nxy, 0.5f * w.per_nxy)), in_z = __builtin_fmaf(-fz, w.nxy, fv);
            const float fy = floorf(__builtin_fmaf(in_z, w.per_nx, 0.5f * w.per_nx));
            const uint32_t x = min(w.low[0] + (uint32_t)__builtin_fmaf(-fy, w.nx, in_z), w.res[0]), y = min(w.low[1] + (uint32_t)fy, w.res[1]),
                           z = min(w.low[2] + (uint32_t)fz, w.res[2]);
            // indices of at most 24 bits
            const uint32_t e = w.dense ? x + __umul24(w.res[0] + 1u, y + __umul24(w.res[1] + 1u, z)) : (x ^ hash_y(y) ^ hash_z(z)) & mask;
            entry[k] = table[(size_t)w.offset + e];
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (k * kFwdThreads + threadIdx.x < n_vertices) box[k * kFwdThreads + threadIdx.x] = entry[k];
    }
    __syncthreads();
    const uint32_t odd = threadIdx.x & 1u;
    for (uint32_t i = threadIdx.x / 2; i < n; i += kFwdThreads / 2) {
        const float4 s = ordered[begin + i];
        const float uu[3] = {unit(s.x), unit(s.y), unit(s.z)};
        // the finer levels' corners are asked for first, and waited for last
        PairCorners finer[LEVELS > MERGED ? LEVELS - MERGED : 1];
#pragma unroll
        for (int l = MERGED; l < LEVELS; ++l) finer[l - MERGED] = ask_pair(level_of(g, l), mask, table, uu, odd);
        __builtin_amdgcn_sched_barrier(0);
        uint32_t mine[MERGED / 2];                           // levels 0 .. MERGED / 2 - 1 on the even lane, the others on the odd one
        // read where it is used: held in registers for all levels it would leave no room for the wavefronts
        uint32_t from = odd * (MERGED / 2);
        asm volatile("" : "+v"(from));
        const FwdBox *const here = levels + from;
#pragma unroll
        for (int l = 0; l < MERGED / 2; ++l) {
            const FwdBox q = here[l];
            float cell[3], w1[3], w0[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                locate_unit(uu[a], q.scale[a], q.last[a], cell[a], w1[a]);
                w0[a] = 1.0f - w1[a];
            }
            // whole numbers below 2^24: exact in fp32
            const uint32_t slot = min((uint32_t)__builtin_fmaf(cell[2], q.nxy, __builtin_fmaf(cell[1], q.nx, cell[0] - q.origin)), q.last_slot);
            const char *const at = reinterpret_cast<const char *>(box) + q.first + slot * (uint32_t)sizeof(float2);
            float2 v[8];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float2 *row = reinterpret_cast<const float2 *>(at + ((r & 1) ? q.nx_bytes : 0u) + ((r & 2) ? q.nxy_bytes : 0u));
                v[2 * r] = row[0];
                v[2 * r + 1] = row[1];
            }
            const float yz[4] = {w0[1] * w0[2], w1[1] * w0[2], w0[1] * w1[2], w1[1] * w1[2]};
            float f0 = 0.0f, f1 = 0.0f;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float w = (c & 1 ? w1[0] : w0[0]) * yz[c >> 1];
                f0 = __builtin_fmaf(w, v[c].x, f0);
                f1 = __builtin_fmaf(w, v[c].y, f1);
            }
            mine[l] = __builtin_bit_cast(uint32_t, __floats2half2_rn(f0, f1));
            asm volatile("" : "+v"(mine[l]));                // done here: put off to where the rows are written, all levels' corners would wait for it
        }
        // half of the sample's row per lane
        constexpr int kHalfRow = LEVELS / 2;
        uint32_t out[kHalfRow];
#pragma unroll
        for (int l = 0; l < LEVELS; ++l) {
            uint32_t f;
            if (l < MERGED / 2) f = mine[l];
            else if (l < MERGED) f = l < kHalfRow ? from_pair(mine[l - MERGED / 2]) : mine[l - MERGED / 2];
            else {
                const float2 v = finish_pair(finer[l - MERGED], odd);
                f = __builtin_bit_cast(uint32_t, __floats2half2_rn(v.x, v.y));
            }
            if (l < kHalfRow) out[l] = f;
            else out[l - kHalfRow] = odd ? f : out[l - kHalfRow];
        }
        uint32_t *half_row = feat + (size_t)(by_position ? begin + i : __float_as_uint(s.w)) * LEVELS + kHalfRow * odd;
        static_assert(kHalfRow % 2 == 0, "halves of rows are written in steps of 8 bytes");
#pragma unroll
        for (int k = 0; k < kHalfRow; k += 2) *reinterpret_cast<uint2 *>(half_row + k) = make_uint2(out[k], out[k + 1]);
    }
}

__global__ void __launch_bounds__(kBlock)
fold_wide_kernel(const double *__restrict__ wide_table, uint32_t n, float *__restrict__ dtable)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const float v = (float)wide_table[i];
    if (v != 0.0f) unsafeAtomicAdd(dtable + i, v);
}

Boxes boxes_of(const dg_order_desc *order)
{
    Boxes boxes{};
    boxes.n_merged = order->n_merged;
    for (uint32_t l = 0; l < order->n_merged; ++l) {
        for (int a = 0; a < 3; ++a) boxes.dim[l][a] = order->box[l][a];
        boxes.first[l + 1] = order->box_first[l + 1];
    }
    return boxes;
}

// Merged levels whose bricks are summed in fp64: tables of at most 2^18 entries, which get many adds per entry -- the coarse levels
// because many bricks share a cell, hashed ones because many vertices share an entry (some 100 with 2^18 entries and 16 000 bricks,
// where fp32 adds are as far from 64-bit sums as ray order, 1.5e-7 in 2-norm; some 55 with 2^19, 1.1e-7 against 1.3e-7).  Up to 29 MB
// to clear and fold.
constexpr uint32_t kFoldEntries = 1u << 18;
uint32_t fold_levels(const dg_grid_desc *d, const dg_order_desc *order)
{
    uint32_t l = 0;
    while (l < order->n_merged && d->offset[l + 1] - d->offset[l] <= kFoldEntries) ++l;
    return l;
}

// bytes of their sums
size_t wide_bytes(const dg_grid_desc *d, const dg_order_desc *order) { return (2 * (size_t)d->offset[fold_levels(d, order)] * sizeof(double) + 255) / 256 * 256; }

}  // namespace

namespace dg {

// the merged levels of the ordered backward pass (N samples; dfeat rows of 2 * n_merged floats; wide: wide_bytes of scratch)
int brick_bwd(const char *who, const dg_grid_desc *d, const dg_order_desc *order, const uint32_t *pieces, const void *ordered, const float *dfeat,
              const uint32_t *largest, uint64_t N, float *dtable, double *wide, hipStream_t st)
{
    static std::once_flag lds_once;
    static hipError_t lds_status = hipSuccess;
    std::call_once(lds_once, [] {
        lds_status = hipFuncSetAttribute(reinterpret_cast<const void *>(&brick_bwd_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)(kMaxBoxVertices * 2 * sizeof(double)));
    });
    if (lds_status != hipSuccess) return fail(DG_ERR_HIP, "%s: cannot reserve LDS: %s", who, hipGetErrorString(lds_status));
    Boxes boxes = boxes_of(order);
    boxes.n_wide = std::min(coarse_levels(d), order->n_merged);
    boxes.n_fold = fold_levels(d, order);
    const size_t lds = (size_t)boxes.first[boxes.n_merged] * 2 * sizeof(double);
    const uint32_t n_wide_sums = 2 * d->offset[boxes.n_fold];
    if (int rc = dg_clear(wide, n_wide_sums * sizeof(double), st)) return rc;
    brick_bwd_kernel<<<(uint32_t)piece_bound(order->total, N), kBrickWaves * 64, lds, st>>>(
        *d, bricks_of(order), boxes, (const uint2 *)pieces, (const float4 *)ordered, (const float4 *)dfeat, largest, dtable, wide);
    if (n_wide_sums) fold_wide_kernel<<<(n_wide_sums + kBlock - 1) / kBlock, kBlock, 0, st>>>(wide, n_wide_sums, dtable);
    return launch_status(who);
}

}  // namespace dg

extern "C" int dg_hashgrid_encode_fwd_ordered(const dg_grid_desc *desc, const float *table, const void *ordered, uint64_t N,
                                              uint32_t by_position, void *feat, void *stream)
{
    const char *who = "dg_hashgrid_encode_fwd_ordered";
    if (int rc = dg::check_grid_desc(desc, who)) return rc;
    DG_REQUIRE(desc->n_levels == 16, DG_ERR_UNSUPPORTED, "%s: needs 16 levels", who);
    if (N == 0) return DG_OK;
    DG_REQUIRE(table && ordered && feat, DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(dg::aligned(table, 8) && dg::aligned(ordered, 16) && dg::aligned(feat, 16), DG_ERR_ARG, "%s: misaligned pointer", who);
    const uint64_t blocks = (2 * N + kBlock - 1) / kBlock, per_xcd = (blocks + kXcds - 1) / kXcds;
    DG_REQUIRE(per_xcd * kXcds <= 0x7fffffffull, DG_ERR_UNSUPPORTED, "%s: N too large for one launch", who);
    encode_fwd_ordered_kernel<16><<<(uint32_t)(per_xcd * kXcds), kBlock, 0, (hipStream_t)stream>>>(
        *desc, (const float2 *)table, (const float4 *)ordered, N, by_position != 0, (uint32_t *)feat, (uint32_t)per_xcd);
    return dg::launch_status(who);
}

namespace {
void launch_planes(const dg_grid_desc &d, const float *table, const void *ordered, const float *u, uint64_t N, uint32_t by_position, void *feat, hipStream_t st)
{
    const uint32_t blocks = (uint32_t)((2 * N + kBlock - 1) / kBlock), grid = (16 - kSplitLevels) * blocks;
    if (by_position) encode_planes_kernel<true><<<grid, kBlock, 0, st>>>(d, (const float2 *)table, (const float *)ordered, N, (uint32_t *)feat, blocks);
    else encode_planes_kernel<false><<<grid, kBlock, 0, st>>>(d, (const float2 *)table, u, N, (uint32_t *)feat, blocks);
}
}  // namespace

extern "C" int dg_hashgrid_encode_fwd_split(const dg_grid_desc *desc, const float *table, const void *ordered, const float *u, uint64_t N,
                                            uint32_t by_position, void *feat, void *stream)
{
    const char *who = "dg_hashgrid_encode_fwd_split";
    if (int rc = dg::check_grid_desc(desc, who)) return rc;
    DG_REQUIRE(desc->n_levels == 16, DG_ERR_UNSUPPORTED, "%s: needs 16 levels", who);
    if (N == 0) return DG_OK;
    DG_REQUIRE(table && ordered && feat && (u || by_position), DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(dg::aligned(table, 8) && dg::aligned(ordered, 16) && dg::aligned(feat, 16), DG_ERR_ARG, "%s: misaligned pointer", who);
    const uint64_t blocks = (2 * N + kBlock - 1) / kBlock, per_xcd = (blocks + kXcds - 1) / kXcds;
    DG_REQUIRE(per_xcd * kXcds <= 0x7fffffffull && (16 - kSplitLevels) * blocks <= 0x7fffffffull, DG_ERR_UNSUPPORTED, "%s: N too large for one launch", who);
    hipStream_t st = (hipStream_t)stream;
    encode_fwd_ordered_kernel<kSplitLevels><<<(uint32_t)(per_xcd * kXcds), kBlock, 0, st>>>(*desc, (const float2 *)table, (const float4 *)ordered, N, by_position != 0,
                                                                                           (uint32_t *)feat, (uint32_t)per_xcd);
    launch_planes(*desc, table, ordered, u, N, by_position, feat, st);
    return dg::launch_status(who);
}

namespace {

int ordered_ok(const char *who, const dg_grid_desc *desc, const dg_order_desc *order)
{
    if (int rc = dg::check_grid_desc(desc, who)) return rc;
    if (int rc = order_ok(order, who)) return rc;
    DG_REQUIRE(desc->n_levels == 16 && order->n_merged <= kMaxMerged && order->n_merged % 2 == 0 && order->n_merged > 0, DG_ERR_UNSUPPORTED,
               "%s: needs 16 levels and at least two merged ones", who);
    return order_fits(order, desc, who);
}

int bwd_ordered(const char *who, const dg_grid_desc *desc, const dg_order_desc *order, const void *ordered, const uint32_t *pieces, const float *u,
                const float *dfeat, const uint32_t *largest, uint64_t N, float *dtable, void *ws, size_t ws_bytes, bool counted, void *stream)
{
    if (int rc = ordered_ok(who, desc, order)) return rc;
    if (N == 0) return DG_OK;
    DG_REQUIRE(ordered && pieces && u && dfeat && largest && dtable && ws, DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(dg::aligned(ordered, 16) && dg::aligned(pieces, 8) && dg::aligned(dfeat, 16) && dg::aligned(dtable, 8) && dg::aligned(ws, 256), DG_ERR_ARG,
               "%s: misaligned pointer", who);
    const size_t wide = wide_bytes(desc, order);
    DG_REQUIRE(ws_bytes >= wide, DG_ERR_WORKSPACE, "%s: workspace %zu bytes cannot hold the %zu of the coarser levels", who, ws_bytes, wide);
    // the rows of the merged levels take the place of those levels' planes: plane l of the others lies where it always does
    if (int rc = dg::brick_bwd(who, desc, order, pieces, ordered, dfeat, largest, N, dtable, (double *)ws, (hipStream_t)stream)) return rc;
    return dg::encode_bwd_binned(who, desc, order->n_merged, u, dfeat, N, dtable, (char *)ws + wide, ws_bytes - wide, counted, (hipStream_t)stream);
}

}  // namespace

extern "C" size_t dg_hashgrid_encode_bwd_ordered_workspace_bytes(const dg_grid_desc *desc, const dg_order_desc *order, uint64_t N)
{
    if (ordered_ok("dg_hashgrid_encode_bwd_ordered_workspace_bytes", desc, order)) return 0;
    return wide_bytes(desc, order) + dg::encode_bwd_binned_workspace_bytes(desc, order->n_merged, N);
}

extern "C" int dg_hashgrid_encode_bwd_ordered_count(const dg_grid_desc *desc, const dg_order_desc *order, const float *u, uint64_t N, void *ws,
                                                    size_t ws_bytes, void *stream)
{
    const char *who = "dg_hashgrid_encode_bwd_ordered_count";
    if (int rc = ordered_ok(who, desc, order)) return rc;
    if (N == 0) return DG_OK;
    DG_REQUIRE(u && ws, DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(dg::aligned(ws, 256), DG_ERR_ARG, "%s: workspace must be 256-byte aligned", who);
    const size_t wide = wide_bytes(desc, order);
    DG_REQUIRE(ws_bytes >= wide, DG_ERR_WORKSPACE, "%s: workspace %zu bytes cannot hold the %zu of the coarser levels", who, ws_bytes, wide);
    return dg::encode_bwd_binned_count(who, desc, order->n_merged, u, N, (char *)ws + wide, ws_bytes - wide, (hipStream_t)stream);
}

extern "C" int dg_hashgrid_encode_bwd_ordered(const dg_grid_desc *desc, const dg_order_desc *order, const void *ordered, const uint32_t *pieces,
                                              const float *u, const float *dfeat, const uint32_t *largest, uint64_t N, float *dtable, void *ws,
                                              size_t ws_bytes, uint32_t counted, void *stream)
{
    return bwd_ordered("dg_hashgrid_encode_bwd_ordered", desc, order, ordered, pieces, u, dfeat, largest, N, dtable, ws, ws_bytes, counted != 0, stream);
}

// With eight merged levels the corners of four more are under way, 96 registers a lane, which leave room for one workgroup per compute unit: enough while the L2s
// hold those levels' tables.  Rows walked / from bricks, with the planes, in us: T = 2^17, 1.2 M samples 154 / 147, T = 2^18 152 / 149, T = 2^19 179 / 181,
// T = 2^20, 0.8 M 186 / 200, T = 2^21 (2048 cells) 233 / 241, T = 2^21 and 2^22 (8192 cells), 4.0 M and 2.5 M 1316 / 1417 and 1048 / 1116.
constexpr uint32_t kBricks8Log2T = 18;

extern "C" int dg_hashgrid_encode_fwd_bricks(const dg_grid_desc *desc, const dg_order_desc *order, const float *table, const void *ordered,
                                             const uint32_t *pieces, const float *u, uint64_t N, uint32_t by_position, void *feat, void *stream)
{
    const char *who = "dg_hashgrid_encode_fwd_bricks";
    if (int rc = ordered_ok(who, desc, order)) return rc;
    if (N == 0) return DG_OK;
    DG_REQUIRE(table && ordered && pieces && feat && (u || by_position), DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(dg::aligned(table, 8) && dg::aligned(ordered, 16) && dg::aligned(pieces, 8) && dg::aligned(feat, 16), DG_ERR_ARG, "%s: misaligned pointer", who);
    DG_REQUIRE((16 - kSplitLevels) * ((2 * N + kBlock - 1) / kBlock) <= 0x7fffffffull, DG_ERR_UNSUPPORTED, "%s: N too large for one launch", who);
    hipStream_t st = (hipStream_t)stream;
    const Boxes boxes = boxes_of(order);
    auto launch = [&](auto kernel) {
        const uint64_t stretch = kXcds * kFwdChunk, grid = (piece_bound(order->total, N) + stretch - 1) / stretch * stretch;
        kernel<<<(uint32_t)grid, kFwdThreads, boxes.first[boxes.n_merged] * sizeof(float2), st>>>(
            *desc, bricks_of(order), boxes, (const uint2 *)pieces, (const float2 *)table, (const float4 *)ordered, by_position != 0, (uint32_t *)feat);
    };
    if (order->n_merged == 12) launch(encode_fwd_bricks_kernel<12>);
    else if (order->n_merged == 10) launch(encode_fwd_bricks_kernel<10>);
    else if (order->n_merged == 8 && desc->log2_T <= kBricks8Log2T) launch(encode_fwd_bricks_kernel<8>);
    else return dg_hashgrid_encode_fwd_split(desc, table, ordered, u, N, by_position, feat, stream);
    launch_planes(*desc, table, ordered, u, N, by_position, feat, st);
    return dg::launch_status(who);
}
