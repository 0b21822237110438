// Device helpers shared by the hash-grid encode kernels: level geometry, cell lookup, corner entries
// and trilinear weights (Sec. 3.2, Sec. 4.1; hash of Instant-NGP Eq. 4).  Internal, not part of the ABI.
#pragma once
#include "dg_internal.h"

namespace dg_encode {

constexpr uint32_t kPrimeY = 2654435761u, kPrimeZ = 805459861u;   // Instant-NGP Eq. 4 (x prime is 1)

// Products with the hash's primes, as far as an index of at most 24 bits needs them: one full-rate instruction where a 32-bit product takes
// four times as long
__device__ __forceinline__ uint32_t hash_y(uint32_t y) { return __umul24(y, kPrimeY & 0xffffffu); }
__device__ __forceinline__ uint32_t hash_z(uint32_t z) { return __umul24(z, kPrimeZ & 0xffffffu); }

struct LevelGeom {
    uint32_t res[3];
    uint32_t dense;
    uint32_t offset;
    float scale[3];
};

__device__ __forceinline__ LevelGeom level_of(const dg_grid_desc &g, uint32_t l)
{
    LevelGeom v;
    v.res[0] = g.res[l][0]; v.res[1] = g.res[l][1]; v.res[2] = g.res[l][2];
    v.dense = g.dense[l];
    v.offset = g.offset[l];
    v.scale[0] = g.scale[l][0]; v.scale[1] = g.scale[l][1]; v.scale[2] = g.scale[l][2];
    return v;
}

// cell and fractional position along one axis: one fp32 multiply, no contraction
__device__ __forceinline__ void locate_axis(float c, float scale, uint32_t last, uint32_t &cell, float &frac)
{
#pragma clang fp contract(off)
    const float pos = c * scale;
    uint32_t i = (uint32_t)floorf(pos);
    i = i > last ? last : i;
    cell = i;
    frac = pos - (float)i;
}

__device__ __forceinline__ float clamp_unit(float c)
{
    c = c >= 0.0f ? c : 0.0f;     // NaN lands on 0 as well
    return c > 1.0f ? 1.0f : c;
}

// clamp_unit, and locate_axis with the cell left in floating point, in one instruction per clamp: the middle of three values, which takes NaN for
// the smallest
__device__ __forceinline__ float unit(float c) { return __builtin_amdgcn_fmed3f(c, 0.0f, 1.0f); }
__device__ __forceinline__ void locate_unit(float c, float scale, float last, float &cell, float &frac)
{
#pragma clang fp contract(off)
    const float pos = c * scale;
    cell = __builtin_amdgcn_fmed3f(floorf(pos), 0.0f, last);
    frac = pos - cell;
}

// cell and fractional position of a sample at one level
__device__ __forceinline__ void locate(const LevelGeom &lv, const float u[3], uint32_t cell[3], float frac[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) locate_axis(clamp_unit(u[a]), lv.scale[a], lv.res[a] - 1u, cell[a], frac[a]);
}

// entry indices (relative to the level) of the 8 corners, corner c = cx + 2cy + 4cz
__device__ __forceinline__ void corner_entries(const LevelGeom &lv, uint32_t mask, const uint32_t cell[3], uint32_t e[8])
{
    if (lv.dense) {
        const uint32_t nx = lv.res[0] + 1u, nxy = nx * (lv.res[1] + 1u);
        const uint32_t base = cell[0] + nx * cell[1] + nxy * cell[2];
#pragma unroll
        for (int c = 0; c < 8; ++c) e[c] = base + (c & 1) + ((c >> 1) & 1) * nx + ((c >> 2) & 1) * nxy;
    } else {
        const uint32_t hy0 = cell[1] * kPrimeY, hy1 = hy0 + kPrimeY;
        const uint32_t hz0 = cell[2] * kPrimeZ, hz1 = hz0 + kPrimeZ;
#pragma unroll
        for (int c = 0; c < 8; ++c)
            e[c] = ((cell[0] + (c & 1)) ^ ((c & 2) ? hy1 : hy0) ^ ((c & 4) ? hz1 : hz0)) & mask;
    }
}

// entry of one vertex (relative to the level)
__device__ __forceinline__ uint32_t vertex_entry(const LevelGeom &lv, uint32_t mask, uint32_t x, uint32_t y, uint32_t z)
{
    return lv.dense ? x + (lv.res[0] + 1u) * (y + (lv.res[1] + 1u) * z) : (x ^ y * kPrimeY ^ z * kPrimeZ) & mask;
}

__device__ __forceinline__ void corner_weights(const float frac[3], float w[8])
{
    const float wx[2] = {1.0f - frac[0], frac[0]}, wy[2] = {1.0f - frac[1], frac[1]}, wz[2] = {1.0f - frac[2], frac[2]};
#pragma unroll
    for (int c = 0; c < 8; ++c) w[c] = wx[c & 1] * wy[(c >> 1) & 1] * wz[(c >> 2) & 1];
}


// the whole number, less than 2^50 in magnitude, that the low 51 bits of a sum of doubles' bit patterns hold in two's complement
__device__ __forceinline__ double from_low_bits(unsigned long long held)
{
    // shifted up by 2^50 the number is the low mantissa bits of a double from 2^52 on; the upper bits of `held` go
    const uint32_t high = (((uint32_t)(held >> 32) + (1u << 18)) & ((1u << 19) - 1u)) | 0x43300000u;
    return __longlong_as_double((long long)((unsigned long long)high << 32 | (uint32_t)held)) - 0x1.4p52;
}

// value of the other lane of a pair (quad_perm 1, 0, 3, 2)
__device__ __forceinline__ uint32_t from_pair(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true); }

// Features of one sample at one level by two lanes: cx = 0 takes the four corners with x of the cell, its neighbour cx = 1 those with x + 1
// -- the two entries of an x-pair nearly always share a cache line, which then costs one look-up -- and a DPP move adds the halves.
struct PairCorners {
    float2 v[4];
    float frac[3];
};

// asks for the lane's four corners; uu within [0, 1]
__device__ __forceinline__ PairCorners ask_pair(const LevelGeom &lv, uint32_t mask, const float2 *__restrict__ table, const float (&uu)[3], uint32_t cx)
{
    PairCorners q;
    float at[3];
    uint32_t cell[3], e[4];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        locate_unit(uu[a], lv.scale[a], (float)(lv.res[a] - 1u), at[a], q.frac[a]);
        cell[a] = (uint32_t)at[a];
    }
    if (lv.dense) {
        const uint32_t nx = lv.res[0] + 1u, nxy = nx * (lv.res[1] + 1u);
        const uint32_t base = cell[0] + cx + nx * cell[1] + nxy * cell[2];
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] = base + (k & 1) * nx + (k >> 1) * nxy;
    } else {
        const uint32_t hy0 = hash_y(cell[1]), hy1 = hy0 + kPrimeY;
        const uint32_t hz0 = hash_z(cell[2]), hz1 = hz0 + kPrimeZ;
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] = ((cell[0] + cx) ^ ((k & 1) ? hy1 : hy0) ^ ((k & 2) ? hz1 : hz0)) & mask;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) q.v[k] = table[(size_t)lv.offset + e[k]];
    return q;
}

// both lanes get the sum
__device__ __forceinline__ float2 finish_pair(const PairCorners &q, uint32_t cx)
{
    const float wx = cx ? q.frac[0] : 1.0f - q.frac[0];
    const float wy[2] = {1.0f - q.frac[1], q.frac[1]}, wz[2] = {1.0f - q.frac[2], q.frac[2]};
    float f0 = 0.0f, f1 = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float w = wx * wy[k & 1] * wz[k >> 1];
        f0 = fmaf(w, q.v[k].x, f0);
        f1 = fmaf(w, q.v[k].y, f1);
    }
    f0 += __uint_as_float(from_pair(__float_as_uint(f0)));
    f1 += __uint_as_float(from_pair(__float_as_uint(f1)));
    return make_float2(f0, f1);
}

__device__ __forceinline__ float2 gather_pair(const LevelGeom &lv, uint32_t mask, const float2 *__restrict__ table, const float (&uu)[3], uint32_t cx)
{
    const float at[3] = {unit(uu[0]), unit(uu[1]), unit(uu[2])};
    return finish_pair(ask_pair(lv, mask, table, at, cx), cx);
}

// value of the lane below (lane - 1) in the wavefront; lane 0 gets its own.  A DPP move: no LDS traffic, no wait.
__device__ __forceinline__ uint32_t from_lane_below(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
}

// ---- segmented sum over the wavefront with DPP moves (no LDS traffic, no waits) ----------------------
// Lanes form runs (a run starts where `head` is set; lane 0 always starts one).  After the call the last
// lane of every run holds the sum of that run's 16 values.  One step combines each lane with a lane
// further down: (v, f) <- (f ? v : v + v_src, f | f_src), f meaning "a run start lies in the span summed so
// far".  Steps: row_shr 1, 2, 4, 8 inside rows of 16 lanes, then row_bcast:15 into rows 1 and 3 and
// row_bcast:31 into rows 2 and 3 -- the classic wavefront scan, made segment-aware.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void seg_step(float (&vx)[8], float (&vy)[8], int &f)
{
    const int fs = __builtin_amdgcn_update_dpp(0, f, CTRL, ROW_MASK, 0xF, true);
    const float take = f ? 0.0f : 1.0f;      // v + 1 * t is exact, so one multiply-add (which can carry the DPP move) does the step
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float tx = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(vx[c]), CTRL, ROW_MASK, 0xF, true));
        const float ty = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(vy[c]), CTRL, ROW_MASK, 0xF, true));
        vx[c] = __builtin_fmaf(tx, take, vx[c]);
        vy[c] = __builtin_fmaf(ty, take, vy[c]);
    }
    f |= fs;
}

__device__ __forceinline__ void segmented_sum(float (&vx)[8], float (&vy)[8], bool head, unsigned long long heads)
{
    int f = head ? 1 : 0;
    // wavefront-uniform: steps that no run needs are skipped.  Bit i of the k-th mask: the lanes up to i continue a run for
    // at least 1, 2, 4, 8 lanes, i.e. some run is longer than that.
    const unsigned long long r1 = ~heads, r2 = r1 & r1 << 1, r4 = r2 & r2 << 2, r8 = r4 & r4 << 4;
    if (r1) seg_step<0x111, 0xF>(vx, vy, f);
    if (r2) seg_step<0x112, 0xF>(vx, vy, f);
    if (r4) seg_step<0x114, 0xF>(vx, vy, f);
    if (r8) seg_step<0x118, 0xF>(vx, vy, f);
    if (!((heads >> 16) & 1ull) || !((heads >> 48) & 1ull)) seg_step<0x142, 0xA>(vx, vy, f);
    if (!((heads >> 32) & 1ull)) seg_step<0x143, 0xC>(vx, vy, f);
}

}  // namespace dg_encode
