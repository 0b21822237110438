// Count and fill sweep of the table-gradient pass: how many records every workgroup has for every bin, then the records, bin by bin.
//
// Memory takes whole lines written one after the other at some 54 G/s and 128 aligned bytes better than 64, so records are collected in LDS: every
// bin has a ring of queue lines, 64 or 128 KB for all bins of a level.  A record takes the next place in its bin's ring with an LDS add; after a barrier
// the bins that hold a whole unit (UNIT lines) write their units out, four lanes a line, and move on.  The count sweep has sized the
// workgroup's slice of every bin for exactly its records; a slice ends in zero records, which add nothing.  A record that finds its ring full
// waits for the write-out where the ring is a single line (2048 bins: one record in twenty), else, or where there are too many of
// them, it goes to the queue directly, where the place that it took says.
//
// Samples in the order of their rays: 16-byte records of pairs of corners along x, runs of lanes that share a cell in one (struct Merged).  Bound by
// the arithmetic (some 490 vector instructions per wavefront and level), below 0.1 M samples by the steps' latency.  Whole training steps with appends sorted through LDS tiles (up to 64
// bins) or one queue granule per bin (above) / rings as first built: eight sub-models, T = 2^19 and 2^22, 0.4 M samples each 6.20 / 6.11 ms; T = 2^23, 0.32 M 1.08 / 0.91;
// T = 2^24, 0.37 M 1.75 / 1.27, 27 k 1.12 / 0.55.
//
// Samples in spatial order, the levels above those that are summed brick by brick: their cells are so small that few neighbours along a ray share one
// (T = 2^19, 13.3 M samples, levels 12..15: 4 % of the lanes; T = 2^24, levels 10..15: 1 %), so nothing is merged, and what a pair of corners along x gets
// is one gradient times the weights 1 - fx and fx.  A record is 12 bytes (struct Compact): where the sums of corner 0 lie in its bin's table (14 bits),
// how corner 1's entry differs (4 bits), the two gradient values times their y and z weights (27-bit floats, as in the other queues) and fx in units of
// 2^-23 (24 bits: exact but for the first cell along x, see values).  Five records and a spare word make a queue line of 64 bytes.
// Bound by the writes: T = 2^19, 13.3 M samples, 4 levels 0.75 ms, 57 G lines/s (records of 16 bytes sorted in LDS: 0.88); four sub-models, T = 2^22,
// 13 M samples, 6 levels 1.31 ms (granules of four 16-byte records: 2.14);
// T = 2^24, 33.5 M samples, 6 levels 4.43 ms (6.10).  Measured on the way, T = 2^19: a ring per wavefront, without barriers, nine wavefronts per
// compute unit 1.18 ms; four workgroups of 512 threads per compute unit 0.80, with appends of single lines 0.95; T = 2^22: appends of single
// lines, 64 KB of rings, two workgroups 1.54 ms, 32 KB, four workgroups 1.95; T = 2^24: records that find their ring full to the queue at once
// 5.20 ms (a third of the writes is then less than a line), two rounds instead of four the same, all bins looked at instead of listed 7.47.
#include "encode_binned_common.h"

namespace dg_encode_binned {

// ------------------------------------------------------------------ records of pairs whose runs are merged
// One record serves a pair of corners along x: (entry of corner 0 within the bin, entry of corner 1
// within the bin, 4 values).  The two entries of a pair are neighbours in a dense level and differ only
// in their low index bits in a hashed one, so they share a bin -- except where the pair straddles a bin
// boundary (one pair in 8192 of a dense level).  Then the record carries corner 0 alone and corner 1 is
// added to the table directly with global atomics; both sweeps see exactly four records per emitting
// sample and level.

// A queue record is 16 bytes: the entry of corner 0 within the bin (13 bits), how corner 1's entry differs from it (4
// bits: the two differ in their k low bits, all of them -- x and x + 1 do, and both index forms keep that: a sum of
// x with multiples of the resolution, or an exclusive-or of x with hashes of y and z) and the pair's four values as
// 27-bit floats (sign, 8 exponent bits, 18 mantissa bits: fp32 rounded to nearest at bit 5, relative error at most
// 2^-19 per value, the same for both signs).  Four of them make a queue line of 64 bytes.  (With 20-byte records of fp32 values, probes
// of the store side alone measured 3.0 ms for 9.1 GB appended as it comes and 1.8 ms in whole lines.)
// k such that eb == ea ^ (2^k - 1), or 15 when the two do not differ that way (ea, eb < 2^13)
__device__ __forceinline__ uint32_t pair_code(uint32_t ea, uint32_t eb)
{
    const uint32_t x = ea ^ eb, k = 32u - (uint32_t)__clz((int)x);       // __clz(0) == 32
    return x == (1u << k) - 1u ? k : 15u;
}

// (entry of corner 0 < 2^13, pair_code < 15, four values) <-> record.  A value keeps its top 27 bits, rounded to nearest
// (half a unit is added to the magnitude before the cut: ties go away from zero, the same way for both signs).
// x: entry, code and the low 15 bits of value 3; y, z, w: values 0..2 in the low 27 bits, more bits of value 3 above.
__device__ __forceinline__ uint4 pack_record(uint32_t ea, uint32_t code, float v0, float v1, float v2, float v3)
{
    const uint32_t q0 = (__float_as_uint(v0) + 16u) >> 5, q1 = (__float_as_uint(v1) + 16u) >> 5, q2 = (__float_as_uint(v2) + 16u) >> 5,
                   q3 = (__float_as_uint(v3) + 16u) >> 5;
    return make_uint4(ea | code << 13 | q3 << 17, q0 | (q3 >> 15) << 27, q1 | (q3 >> 20) << 27, q2 | (q3 >> 25) << 27);
}

// Which records a sample emits at a level (both sweeps take the same decision from the same data).  A
// wavefront holds 64 consecutive samples of a ray; lanes that share a cell form a run whose 16 values are
// summed into the run's last lane, which alone emits records.  Skipped where no two lanes share a cell.
struct Emission {
    uint32_t e[8];
    float frac[3];
    unsigned long long heads;
    bool head, merge, emit;
};

__device__ __forceinline__ Emission classify(const LevelGeom &lv, uint32_t mask, const float (&uu)[3], bool live, int lane)
{
    Emission o;
    uint32_t cell[3];
    locate(lv, uu, cell, o.frac);
    corner_entries(lv, mask, cell, o.e);
    o.head = lane == 0 || !live;
#pragma unroll
    for (int a = 0; a < 3; ++a) o.head |= from_lane_below(cell[a]) != cell[a];
    o.heads = __ballot(o.head);
    o.merge = __popcll(o.heads) < dg::kWave;      // any run at all: the merge steps cost less than the records they save
    const bool tail = lane == dg::kWave - 1 || ((o.heads >> ((lane + 1) & 63)) & 1ull);
    o.emit = live && (!o.merge || tail);
    return o;
}

// values of the 8 corners of one sample at one level, runs merged where the emission says so; `largest` follows the
// largest magnitude (as the bit pattern of |v|, which orders like the value) of anything a lane emits
__device__ __forceinline__ void corner_values(const Emission &em, float2 gfe, float (&vx)[8], float (&vy)[8], uint32_t &largest)
{
    float w[8];
    corner_weights(em.frac, w);
#pragma unroll
    for (int c = 0; c < 8; ++c) { vx[c] = w[c] * gfe.x; vy[c] = w[c] * gfe.y; }
    if (em.merge) segmented_sum(vx, vy, em.head, em.heads);
    if (em.emit) {
        float m = 0.0f;
#pragma unroll
        for (int c = 0; c < 8; ++c) m = fmaxf(m, fmaxf(fabsf(vx[c]), fabsf(vy[c])));
        largest = max(largest, __float_as_uint(m));
    }
    // fmaxf passes over NaN: a NaN gradient is reported as such (its bit pattern orders above infinity's), by whichever
    // lane holds it, whether or not that lane emits
    if (gfe.x != gfe.x || gfe.y != gfe.y) largest = max(largest, 0x7fc00000u);
}

// the record of pair p; a pair that straddles a bin boundary (or, against every expectation, differs in some other way
// than a record can say) keeps corner 0 only and its corner 1 goes to the table directly
__device__ __forceinline__ uint4 make_record(const Emission &em, int p, const float (&vx)[8], const float (&vy)[8], uint32_t level_offset,
                                             float *__restrict__ dtable)
{
    const uint32_t ea = em.e[2 * p], eb = em.e[2 * p + 1];
    uint32_t code = pair_code(ea & (kChunk - 1u), eb & (kChunk - 1u));
    const bool together = (ea >> kChunkLog2) == (eb >> kChunkLog2) && code != 15u;
    if (!together) {
        code = 0u;
        float *dst = dtable + 2 * ((size_t)level_offset + eb);
        if (vx[2 * p + 1] != 0.0f) unsafeAtomicAdd(dst, vx[2 * p + 1]);
        if (vy[2 * p + 1] != 0.0f) unsafeAtomicAdd(dst + 1, vy[2 * p + 1]);
    }
    return pack_record(ea & (kChunk - 1u), code, vx[2 * p], vy[2 * p], together ? vx[2 * p + 1] : 0.0f, together ? vy[2 * p + 1] : 0.0f);
}

// What a sample gives at a level, for the sweeps.  Merged: 16-byte records, runs of lanes that share a cell in one
struct Merged {
    static constexpr uint32_t kLine = kPairLine;
    typedef uint4 Record;
    Emission em;
    float vx[8], vy[8];

    static __device__ __forceinline__ uint32_t line_of(uint32_t p) { return p / kLine; }
    __device__ __forceinline__ bool locate_sample(const LevelGeom &lv, uint32_t mask, const float (&uu)[3], bool live, int lane)
    {
        em = classify(lv, mask, uu, live, lane);
        return em.emit;
    }
    __device__ __forceinline__ uint32_t entry(int p) const { return em.e[2 * p]; }
    __device__ __forceinline__ void values(const LevelGeom &, uint32_t, float2 gfe, bool, float *, uint32_t &largest) { corner_values(em, gfe, vx, vy, largest); }
    // once per pair: it may add to the table
    __device__ __forceinline__ Record record(int p, const LevelGeom &lv, float *__restrict__ dtable) const { return make_record(em, p, vx, vy, lv.offset, dtable); }
};

// ------------------------------------------------------------------ compact records
// p / 5, p < 2^14
__device__ __forceinline__ uint32_t fifth(uint32_t p) { return __umul24(p, 13108u) >> 16; }

struct CompactRecord { uint32_t w[3]; };

// Where the sums of an entry of a bin lie in LDS (8 bytes each): those of the first feature here, those of the second kChunk / 2 further on,
// which an LDS address can say in its offset.
__device__ __forceinline__ uint32_t slot_of(uint32_t e) { return (e & (kChunk / 2 - 1u)) | (e & kChunk / 2) << 1; }

// top 27 bits of a float, rounded to nearest (ties away from zero), below the low five bits of `above`
__device__ __forceinline__ uint32_t pack_value(float v, uint32_t above) { return __builtin_amdgcn_alignbit(above, __float_as_uint(v) + 16u, 5u); }

// corner 0 of each pair of corners along x, as entries of the level
__device__ __forceinline__ void pair_entries(const LevelGeom &lv, uint32_t mask, uint32_t x, uint32_t y, uint32_t z, uint32_t (&e)[4])
{
    if (lv.dense) {
        const uint32_t nx = lv.res[0] + 1u, nxy = nx * (lv.res[1] + 1u), base = x + nx * y + nxy * z;
#pragma unroll
        for (int p = 0; p < 4; ++p) e[p] = base + (p & 1) * nx + (p >> 1) * nxy;
    } else {
        const uint32_t hy0 = hash_y(y), hy1 = hy0 + kPrimeY, hz0 = hash_z(z), hz1 = hz0 + kPrimeZ;
#pragma unroll
        for (int p = 0; p < 4; ++p) e[p] = (x ^ ((p & 1) ? hy1 : hy0) ^ ((p & 2) ? hz1 : hz0)) & mask;
    }
}

struct Compact {
    static constexpr uint32_t kLine = kCompactLine;
    typedef CompactRecord Record;
    uint32_t e[4], x, codes, fx;                                      // codes: pair_code of each pair, at bits 14 + 4 p
    float frac[3], vx[4], vy[4];

    static __device__ __forceinline__ uint32_t line_of(uint32_t p) { return fifth(p); }
    __device__ __forceinline__ bool locate_sample(const LevelGeom &lv, uint32_t mask, const float (&uu)[3], bool live, int)
    {
        float cell[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) locate_unit(unit(uu[a]), lv.scale[a], (float)(lv.res[a] - 1u), cell[a], frac[a]);
        x = (uint32_t)cell[0];
        pair_entries(lv, mask, x, (uint32_t)cell[1], (uint32_t)cell[2], e);
        return live;
    }
    __device__ __forceinline__ uint32_t entry(int p) const { return e[p]; }
    // A pair's entries may lie in different bins or halves of one (one in thousands), or the x fraction may not fit the record: corner 1 then
    // goes to the table directly, and the record's second entry is corner 0 again, whose value the record's two shares add up to
    __device__ __forceinline__ void apart(int p, uint32_t other, const LevelGeom &lv, float *__restrict__ dtable)
    {
        float *dst = dtable + 2 * ((size_t)lv.offset + other);
        if (vx[p] * frac[0] != 0.0f) unsafeAtomicAdd(dst, vx[p] * frac[0]);
        if (vy[p] * frac[0] != 0.0f) unsafeAtomicAdd(dst + 1, vy[p] * frac[0]);
        vx[p] *= 1.0f - frac[0];
        vy[p] *= 1.0f - frac[0];
    }
    __device__ __forceinline__ void values(const LevelGeom &lv, uint32_t mask, float2 gfe, bool live, float *__restrict__ dtable, uint32_t &largest)
    {
        const float wy[2] = {1.0f - frac[1], frac[1]}, wz[2] = {1.0f - frac[2], frac[2]};
        float most = 0.0f;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const float w = wy[p & 1] * wz[p >> 1];
            vx[p] = w * gfe.x;
            vy[p] = w * gfe.y;
            most = fmaxf(most, fmaxf(fabsf(vx[p]), fabsf(vy[p])));
        }
        largest = max(largest, __float_as_uint(most));
        if (gfe.x != gfe.x || gfe.y != gfe.y) largest = 0x7fc00000u;                  // fmaxf passes over NaN
        // In a level's first cell along x fractions have more bits than units of 2^-23 can say.  Rounded to these a share is off by 2^-21 of itself at most while
        // the fraction lies in [1/8, 7/8], a quarter of what its 27-bit value may be off; nearer to a face of the cell it could lose all of its bits, and the
        // pair goes apart: one sample in hundreds.  Ordered pass without and with this, T = 2^19, 13.3 M samples 2600 / 2599 us, 3.3 M 780 / 788 (798 if
        // pairs went apart all over the cell); half a million with a sixth of all in the first cell 282 / 366.
        const float units = frac[0] * 0x1p23f;
        fx = (uint32_t)(units + 0.5f);
        const bool finer = units != (float)fx && fabsf(units - 0x1p22f) > 0x1.8p21f;
        codes = 0u;
        if (lv.dense) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const uint32_t differ = e[p] ^ (e[p] + 1u);
                if (differ < kChunk / 2 && !finer) codes |= (uint32_t)__popc(differ) << (14 + 4 * p);
                else if (live) apart(p, e[p] + 1u, lv, dtable);
            }
        } else {
            const uint32_t differ = (x ^ (x + 1u)) & mask;
            if (differ < kChunk / 2 && !finer) codes = (uint32_t)__popc(differ) * 0x4444000u;
            else if (live) {
#pragma unroll
                for (int p = 0; p < 4; ++p) apart(p, e[p] ^ differ, lv, dtable);
            }
        }
    }
    __device__ __forceinline__ Record record(int p, const LevelGeom &, float *) const
    {
        Record rec;
        rec.w[0] = slot_of(e[p]) | (codes >> (4 * p) & 15u << 14) | fx << 18;
        rec.w[1] = pack_value(vx[p], fx >> 14);
        rec.w[2] = pack_value(vy[p], fx >> 19);
        return rec;
    }
};

// ------------------------------------------------------------------ sweeps
// Both sweeps: a workgroup takes tiles of kFillTile samples, me, me + width, ..., of the nb at u
template <class K>
__global__ void __launch_bounds__(kFillTile)
count_kernel(dg_grid_desc g, Plan plan, Sweep sw, const float *__restrict__ u, uint32_t nb, uint32_t *__restrict__ rows)
{
    extern __shared__ uint32_t smem[];
    uint32_t *row = smem;                                // [n_keys]
    const uint32_t me = blockIdx.x % sw.width, first_level = plan.first_level + blockIdx.x / sw.width, tid = threadIdx.x;
    const int lane = tid % dg::kWave;
    const uint32_t mask = (1u << g.log2_T) - 1u;
    for (uint32_t i = tid; i < plan.n_keys; i += kFillTile) row[i] = 0u;
    __syncthreads();
    const uint32_t n_tiles = (nb + kFillTile - 1u) / kFillTile;
    for (uint32_t tile = me; tile < n_tiles; tile += sw.width) {
        const uint32_t rel = tile * kFillTile + tid;
        const bool live = rel < nb;
        const size_t n = live ? rel : nb - 1u;
        const float uu[3] = {u[3 * n], u[3 * n + 1], u[3 * n + 2]};
        for (uint32_t l = first_level; l < g.n_levels; l += sw.groups) {
            K k;
            if (!k.locate_sample(level_of(g, l), mask, uu, live, lane)) continue;
            uint32_t *c = row + plan.key_base[l];
#pragma unroll
            for (int p = 0; p < 4; ++p) atomicAdd(&c[k.entry(p) >> kChunkLog2], 1u);
        }
    }
    __syncthreads();
    uint32_t *row_global = rows + (size_t)me * plan.n_keys;
    for (uint32_t l = first_level; l < g.n_levels; l += sw.groups)
        for (uint32_t i = plan.key_base[l] + tid; i < plan.key_base[l + 1]; i += kFillTile) row_global[i] = row[i];
}

// a step's inputs
struct StepAhead {
    float u[3];
    float2 g;
};

// UNIT: lines of an append.  A step's records go in ROUNDS rounds, each followed by its own write-out: the fewer records a bin gets per round, the
// less often its ring overflows.  LIST: bins that have a unit are listed, otherwise all are looked at.  WAIT: where a ring is a single line, records
// beyond it wait for the write-out.
// Merged records, of which a step has fewer, take one round.  The pass on samples in ray order, four rounds (two with 1024 bins) and lists at all levels / one and lists where
// there are more than 128 bins, in us: T = 2^24, oblique rays, 25.6 M samples 17 291 / 13 530, 5.1 M 4080 / 3246, views from above 16.1 M 8980 / 7970, 0.5 M 877 / 827;
// T = 2^23, 0.64 M 1141 / 724, 6.4 M 4190 / 3600.
template <class K, int PER_UNIT, int UNIT, int ROUNDS, bool LIST, bool WAIT>
__global__ void __launch_bounds__(kFillTile, PER_UNIT == 1 ? 4 : 8)          // wavefronts per SIMD
fill_kernel(dg_grid_desc g, Plan plan, Sweep sw, const float *__restrict__ u, const float2 *__restrict__ dfeat, uint64_t N, uint32_t nb,
                    const uint32_t *__restrict__ rows, const uint32_t *__restrict__ binbase, uint32_t *__restrict__ queue,
                    float *__restrict__ dtable, uint32_t *__restrict__ largest_out)
{
    constexpr int kLinesLog2 = ring_lines_log2(PER_UNIT), kLines = 1 << kLinesLog2;
    constexpr int kPer = 4 / ROUNDS;                                  // pairs of corners per round
    constexpr uint32_t kLine = K::kLine, kWords = kLine == kPairLine ? 4u : 3u;      // records of a line, words of a record
    constexpr uint32_t kUnit = UNIT * kLine, kLanes = 4 * UNIT, kGroups = kFillTile / kLanes;
    constexpr uint32_t kDirect = 0x80u;                               // in `kept`: what was beyond the ring went to the queue
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    const uint32_t cap = plan.max_bins;
    uint32_t *ring = smem;                                            // [kLines][16]
    uint32_t *books = ring + 16 * kLines;                      // [cap] records in the bin's ring | its first line << 16
    uint32_t *line0 = books + cap;                                    // [cap] queue line of the ring's first
    uint32_t *n_list = line0 + cap;                                   // [2] entries of the two lists (+ 2 unused words)
    uint16_t *list = reinterpret_cast<uint16_t *>(n_list + 4);        // [2][cap] bins that got a whole unit in a round
    uint8_t *kept = reinterpret_cast<uint8_t *>(list + (LIST ? 2 * cap : 0));      // [cap] records of the first line that are in the queue already
    const uint32_t tid = threadIdx.x;
    const int lane = tid % dg::kWave;
    const uint32_t mask = (1u << g.log2_T) - 1u;
    const uint32_t me = blockIdx.x % sw.width, first_level = plan.first_level + blockIdx.x / sw.width;
    const uint32_t *row = rows + (size_t)me * plan.n_keys;
    uint32_t parity = 0;
    uint32_t largest = 0;                                             // bits of the largest magnitude; infinity or more where a gradient is not a number
    const uint32_t n_tiles = (nb + kFillTile - 1u) / kFillTile;
    StepAhead ahead = {{0.0f, 0.0f, 0.0f}, make_float2(0.0f, 0.0f)};
    // the tile's addresses are the same for all lanes, a lane's offset in it fits 32 bits
    auto load = [&](uint32_t tile, uint32_t l) {
        const uint32_t n = min(tid, nb - 1u - tile * kFillTile);
        const float *at = reinterpret_cast<const float *>(reinterpret_cast<const char *>(u + (size_t)tile * (3 * kFillTile)) + n * 12u);
        ahead.u[0] = at[0]; ahead.u[1] = at[1]; ahead.u[2] = at[2];
        ahead.g = *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(dfeat + (size_t)l * N + (size_t)tile * kFillTile) + n * 8u);
    };
    const bool has_work = me < n_tiles && first_level < g.n_levels;
    if (has_work) load(me, first_level);
    for (uint32_t i = tid; i < kLines; i += kFillTile) ring[16 * i + 15] = 0u;      // the spare words
    if (tid < 2) n_list[tid] = 0u;
    if (blockIdx.x == 0 && tid == 0) largest_out[1] = 0u;             // pieces taken by the accumulate kernel
    for (uint32_t l = first_level; l < g.n_levels; l += sw.groups) {
        const uint32_t n_bins = plan.n_bins[l], key0 = plan.key_base[l];
        const LevelGeom lv = level_of(g, l);
        // all of LDS is shared out among the level's bins, in powers of two
        const uint32_t bins_log2 = n_bins > 1u ? 32u - __clz((int)(n_bins - 1u)) : 0u;
        const uint32_t lines_log2 = kLinesLog2 - bins_log2, line_mask = (1u << lines_log2) - 1u, room = kLine << lines_log2;
        __syncthreads();                                              // the last level's books are closed
        for (uint32_t i = tid; i < n_bins; i += kFillTile) {
            books[i] = 0u;
            line0[i] = (row[key0 + i] + binbase[key0 + i]) / kLine;
            kept[i] = 0;
        }
        __syncthreads();
        // a bin's units are written out by groups of lanes that sit in one wavefront, several where there are more groups than bins
        const bool wait = WAIT && lines_log2 == 0u;
        constexpr uint32_t kGroupsLog2 = 31 - __builtin_clz(kGroups), kPerWaveLog2 = 31 - __builtin_clz(dg::kWave / kLanes);
        // A level of few bins is not listed: a bin that gets hundreds of lines a round would have one group of lanes to write them.  (Compact records come from
        // finer levels, where all bins are listed.)
        constexpr bool kChoose = LIST && kLine == kPairLine;
        const uint32_t subs_log2 = LIST && !kChoose ? 0u : min(kPerWaveLog2, bins_log2 < kGroupsLog2 ? kGroupsLog2 - bins_log2 : 0u);
        const bool listed = LIST && (!kChoose || subs_log2 == 0u);
        const uint32_t group = tid / kLanes, sub = group & ((1u << subs_log2) - 1u), subs = 1u << subs_log2;
        const uint32_t first_group = group >> subs_log2, group_step = kGroups >> subs_log2;
        for (uint32_t tile = me; tile < n_tiles; tile += sw.width) {
            const bool live = tile * kFillTile + tid < nb;
            const float uu[3] = {ahead.u[0], ahead.u[1], ahead.u[2]};
            const float2 gfe = live ? ahead.g : make_float2(0.0f, 0.0f);
            // the next step's inputs are asked for before this step's stores (loads and stores of a wavefront retire in order)
            const bool same_level = tile + sw.width < n_tiles;
            if (same_level || l + sw.groups < g.n_levels) load(same_level ? tile + sw.width : me, same_level ? l : l + sw.groups);
            K k0;
            const bool emit = k0.locate_sample(lv, mask, uu, live, lane);
            k0.values(lv, mask, gfe, live, dtable, largest);
#pragma unroll
            for (int round = 0; round < ROUNDS; ++round, parity ^= 1u) {
                uint32_t at[kPer], bin[kPer];                         // place of each record in its bin's ring
                typename K::Record rec[kPer];
                uint32_t beyond[kPer];                                // queue line of the ring's first, of records that found their ring full
                auto to_queue = [&](uint32_t line, uint32_t place, const typename K::Record &rec) {
                    const uint32_t q = K::line_of(place);
                    *reinterpret_cast<typename K::Record *>(queue + ((size_t)(line + q) * 16 + kWords * (place - kLine * q))) = rec;
                };
#pragma unroll
                for (int k = 0; k < kPer; ++k) bin[k] = k0.entry(kPer * round + k) >> kChunkLog2;
                if (emit) {
#pragma unroll
                    for (int k = 0; k < kPer; ++k) at[k] = atomicAdd(&books[bin[k]], 1u);
#pragma unroll
                    for (int k = 0; k < kPer; ++k) {
                        const int p = kPer * round + k;
                        const uint32_t head = at[k] >> 16;
                        at[k] &= 0xffffu;
                        const uint32_t q = K::line_of(at[k]), in_line = kWords * (at[k] - kLine * q);
                        rec[k] = k0.record(p, lv, dtable);
                        if (at[k] < room) *reinterpret_cast<typename K::Record *>(ring + ((((bin[k] << lines_log2) + ((head + q) & line_mask)) << 4) + in_line)) = rec[k];
                        else if (wait) beyond[k] = line0[bin[k]];
                        else to_queue(line0[bin[k]], at[k], rec[k]);
                    }
                }
                if (listed) {
                    // bins that get their first whole unit go into the list: one LDS add per wavefront and pair of corners
#pragma unroll
                    for (int k = 0; k < kPer; ++k) {
                        const bool full = emit && at[k] == kUnit - 1u;
                        const unsigned long long votes = __ballot(full);
                        if (votes == 0ull) continue;                  // wavefront-uniform
                        const int leader = __ffsll((long long)votes) - 1;
                        uint32_t first = 0u;
                        if (lane == leader) first = atomicAdd(&n_list[parity], (uint32_t)__popcll(votes));
                        first = lane_value(first, (uint32_t)leader);
                        if (full) list[parity * cap + first + __popcll(votes & ((1ull << lane) - 1ull))] = (uint16_t)bin[k];
                    }
                }
                __syncthreads();                                      // records placed, list complete
                const uint32_t n = listed ? n_list[parity] : n_bins, c = tid % kLanes;
                for (uint32_t i = first_group; i < n; i += group_step) {
                    const uint32_t bin = listed ? list[parity * cap + i] : i;
                    const uint32_t book = books[bin], total = book & 0xffffu, head = book >> 16;
                    const uint32_t units = K::line_of(min(total, room)) / UNIT;
                    if (!units) continue;
                    const uint32_t first = line0[bin], skip = kept[bin] & (kDirect - 1u);
                    const uint4 *from = reinterpret_cast<const uint4 *>(ring) + ((size_t)bin << lines_log2) * 4;
                    uint4 *to = reinterpret_cast<uint4 *>(queue);
                    for (uint32_t k = sub; k < units; k += subs) {
                        const uint32_t line = UNIT * k + c / 4;
                        if (k == 0 && skip != 0u) {                   // the unit's first records are in the queue already
                            for (uint32_t s = skip + c; s < kUnit; s += kLanes) {
                                const uint32_t q = K::line_of(s), in_line = kWords * (s - kLine * q);
                                *reinterpret_cast<typename K::Record *>(queue + ((size_t)(first + q) * 16 + in_line)) =
                                    *reinterpret_cast<const typename K::Record *>(ring + ((((bin << lines_log2) + ((head + q) & line_mask)) << 4) + in_line));
                            }
                            continue;
                        }
                        to[(size_t)(first + line) * 4 + c % 4] = from[((head + line) & line_mask) * 4 + c % 4];
                    }
                    if (sub == 0 && c == 0) {                         // the other groups of the bin, in this wavefront, have read the books
                        // What is beyond the ring goes to the queue -- or waits, if it fits the emptied ring
                        const bool beyond_ring = total > room, waits = beyond_ring && wait && total < room + kUnit;
                        const uint32_t gone = beyond_ring && !waits ? K::line_of(total) / UNIT : units, left = total - kUnit * gone;
                        line0[bin] = first + UNIT * gone;
                        books[bin] = left | ((head + UNIT * gone) & line_mask) << 16;
                        kept[bin] = beyond_ring && !waits ? (uint8_t)(left | kDirect) : 0;
                    }
                }
                if (LIST && tid == 0) n_list[parity ^ 1u] = 0u;       // the other list: last read before the barrier above
                __syncthreads();                                      // lines read, bins moved on
                if constexpr (WAIT) {
#pragma unroll
                    for (int k = 0; k < kPer; ++k) {
                        if (!wait || !emit || at[k] < room) continue;
                        if (kept[bin[k]] & kDirect) to_queue(beyond[k], at[k], rec[k]);
                        else *reinterpret_cast<typename K::Record *>(ring + 16u * bin[k] + kWords * (at[k] - room)) = rec[k];
                    }
                }
            }
        }
        // end of the level: open units go out, filled up with zero records
        if constexpr (WAIT) __syncthreads();                          // those that waited are in
        for (uint32_t bin = tid / kLanes; bin < n_bins; bin += kGroups) {
            const uint32_t left = books[bin] & 0xffffu, head = books[bin] >> 16, first = line0[bin];
            for (uint32_t s = (kept[bin] & (kDirect - 1u)) + tid % kLanes; left && s < kUnit; s += kLanes) {
                const uint32_t q = K::line_of(s), in_line = kWords * (s - kLine * q);
                const uint32_t *from = ring + ((((bin << lines_log2) + ((head + q) & line_mask)) << 4) + in_line);
                uint32_t *to = queue + ((size_t)(first + q) * 16 + in_line);
#pragma unroll
                for (uint32_t k = 0; k < kWords; ++k) to[k] = s < left ? from[k] : 0u;
            }
        }
    }
    publish_largest(largest, n_list, largest_out);
}

namespace {

// calls f with the plan's fill kernel
template <class F>
auto with_kernel(const Plan &p, F f)
{
    if (p.compact) {
        if (p.max_bins <= 512u) return f(fill_kernel<Compact, 1, 2, 1, false, false>);
        if (p.max_bins <= 1024u) return f(fill_kernel<Compact, 1, 1, 2, true, false>);
        return f(fill_kernel<Compact, 1, 1, 4, true, true>);
    }
    if (p.per_unit == 2u) return f(fill_kernel<Merged, 2, 2, 1, false, false>);
    if (p.max_bins <= 1024u) return f(fill_kernel<Merged, 1, 1, 1, true, false>);
    return f(fill_kernel<Merged, 1, 1, 1, true, true>);
}

// rings, the books of the bins (13 bytes each) and the lists' lengths
size_t fill_lds(const Plan &p) { return (64u << ring_lines_log2((int)p.per_unit)) + (p.max_bins * 13 + 16 + 15) / 16 * 16; }

}  // namespace

int reserve_fill()
{
    hipError_t rc = hipSuccess;
    auto most = [&](auto kernel, size_t lds) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) rc = e;
    };
    most(count_kernel<Merged>, kMaxKeys * 4);
    most(count_kernel<Compact>, kMaxKeys * 4);
    for (const uint32_t compact : {0u, 1u})
        for (const uint32_t bins : {512u, 1024u, 2048u}) {
            Plan p{};
            p.max_bins = bins;
            p.compact = compact;
            p.per_unit = per_unit(p);
            with_kernel(p, [&](auto kernel) { most(kernel, fill_lds(p)); });
        }
    return (int)rc;
}

void count_records(const dg_grid_desc *d, const Plan &p, const Sweep &sw, const float *u, uint64_t n0, uint64_t nb, uint32_t *rows, hipStream_t st)
{
    auto launch = [&](auto kernel) { kernel<<<sw.width * sw.groups, kFillTile, p.n_keys * 4, st>>>(*d, p, sw, u + 3 * n0, (uint32_t)nb, rows); };
    if (p.compact) launch(count_kernel<Compact>);
    else launch(count_kernel<Merged>);
}

void fill_queues(const dg_grid_desc *d, const Plan &p, const Sweep &sw, const float *u, const float *dfeat, uint64_t N, uint64_t n0, uint64_t nb,
                 const uint32_t *rows, uint32_t *binbase, void *queue, float *dtable, hipStream_t st)
{
    with_kernel(p, [&](auto kernel) {
        kernel<<<sw.width * sw.groups, kFillTile, fill_lds(p), st>>>(*d, p, sw, u + 3 * n0, (const float2 *)dfeat + n0, N, (uint32_t)nb, rows,
                                                                                        binbase, (uint32_t *)queue, dtable, binbase + p.n_keys + 1);
    });
}

}  // namespace dg_encode_binned
