// Occupancy grid and occupancy-guided sampling (Sec. 3.2: per-voxel densities let marching skip empty space;
// Sec. 4.1: the grid is deformable like the hash grid; Sec. 5.1: its hyper-parameters; refresh rule of
// Instant-NGP App. E.2: decay, candidate cells, maximum, threshold).
//
// Marching: sixteen lanes per segment (64 where there are few), one stratum per lane and pass.  The lanes of a pass lie next to
// each other on the ray, so their bit lookups fall into a few cache lines of a bit field that stays in L2
// (512 x 512 x 64 cells are 2 MiB).  Segments are placed by an exclusive scan over their sample counts, so the layout is
// deterministic: count, scan, write.
//
// Cells, bits and sample counts are decided in fp32 with one rounding per operation (built with
// -ffp-contract=off).
#include "dg_internal.h"
#include "sample_common.h"
#include <cmath>
#include <cstring>
#include <type_traits>

#pragma clang fp contract(off)

namespace {

using dg_sample::BoxArgs;
using dg_sample::jitter_base;
using dg_sample::kGolden;
using dg_sample::mix_out;
using dg_sample::mix64;
using dg_sample::unit_float;

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / dg::kWave;
constexpr int kScanItems = 8;                          // values per thread
constexpr int kScanTile = kBlock * kScanItems;         // values per workgroup of the scan
constexpr int kSumsBlock = 1024;

struct OccArgs { uint32_t res[3]; uint32_t n_cells; float scale[3]; };

__device__ __forceinline__ uint32_t cell_of(const OccArgs &g, const float (&u)[3])
{
    uint32_t c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float v = u[a];
        v = v >= 0.0f ? v : 0.0f;          // NaN lands on 0 as well
        v = v > 1.0f ? 1.0f : v;
        const float pos = v * g.scale[a];
        uint32_t i = (uint32_t)floorf(pos);
        const uint32_t last = g.res[a] - 1u;
        c[a] = i > last ? last : i;
    }
    return c[0] + g.res[0] * (c[1] + g.res[1] * c[2]);
}

__device__ __forceinline__ bool bit_of(const uint32_t *__restrict__ bits, uint32_t c) { return (bits[c >> 5] >> (c & 31u)) & 1u; }

// ---------------------------------------------------------------- refresh
__device__ __forceinline__ uint64_t candidate_counter(uint32_t iteration, uint32_t i, uint32_t attempt, uint32_t q)
{
    return ((uint64_t)iteration << 36) | ((uint64_t)i << 8) | ((uint64_t)attempt << 2) | q;
}

__global__ void __launch_bounds__(kBlock)
candidates_kernel(OccArgs g, const uint32_t *__restrict__ bits, uint32_t i0, uint32_t M, uint32_t n_uniform, int warmup,
                  uint64_t seed, uint32_t iteration, uint32_t tries, uint32_t *__restrict__ cell, float *__restrict__ u)
{
    const uint32_t j = blockIdx.x * kBlock + threadIdx.x;       // position in this call's output
    if (j >= M) return;
    const uint32_t i = i0 + j;                                   // index of the candidate within the refresh
    uint32_t c = i, attempt = 0;
    if (!warmup) {
        const uint32_t allowed = i < n_uniform ? 1u : tries;
        for (attempt = 0; attempt < allowed; ++attempt) {
            const uint64_t z = mix64(seed, candidate_counter(iteration, i, attempt, 0));
            c = (uint32_t)(((z >> 32) * (uint64_t)g.n_cells) >> 32);
            if (i < n_uniform || bit_of(bits, c)) break;
        }
        if (attempt == allowed) attempt = allowed - 1u;     // no occupied cell met: the last draw stands
    }
    cell[j] = c;
    const uint32_t idx[3] = {c % g.res[0], (c / g.res[0]) % g.res[1], c / (g.res[0] * g.res[1])};
#pragma unroll
    for (uint32_t a = 0; a < 3; ++a) {
        const float xi = unit_float(mix64(seed, candidate_counter(iteration, i, attempt, a + 1u)));
        u[3 * (size_t)j + a] = ((float)idx[a] + xi) / g.scale[a];
    }
}

__global__ void __launch_bounds__(kBlock)
decay_kernel(float *__restrict__ density, uint32_t n_cells, float factor)
{
    const uint32_t c = blockIdx.x * kBlock + threadIdx.x;
    if (c < n_cells) density[c] = density[c] * factor;
}

// densities are >= 0, so their bit patterns order like unsigned integers and the maximum is one integer atomic
__global__ void __launch_bounds__(kBlock)
update_kernel(float *__restrict__ density, uint32_t n_cells, const uint32_t *__restrict__ cell, const float *__restrict__ sigma,
              uint32_t M)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= M) return;
    const uint32_t c = cell[i];
    const float s = sigma[i];
    if (c < n_cells && s > 0.0f) atomicMax(reinterpret_cast<unsigned int *>(density) + c, __float_as_uint(s));
}

constexpr int kBitsRounds = 16;                        // cells per thread and turn of the bit-field pass
constexpr uint32_t kBitsGrid = 512;

// Thresholds kBlock * kBitsRounds consecutive cells per workgroup and turn, all loads of a turn under way before the first
// value is used.  Set bits are counted per workgroup, and there are at most kBitsGrid of them: same-address atomics take turns
// at some 12 ns each (16.8 M cells: one per 4096 cells 51 us, this 26 us = 2.6 TB/s).
__global__ void __launch_bounds__(kBlock)
bits_kernel(const float *__restrict__ density, uint32_t n_cells, float threshold, uint32_t *__restrict__ bits,
            uint32_t *__restrict__ n_set)
{
    __shared__ uint32_t wave_count[kWavesPerBlock];
    const uint32_t n_words = (n_cells + 31u) >> 5;
    uint32_t mine = 0;
    for (uint64_t base = (uint64_t)blockIdx.x * (kBitsRounds * kBlock); base < n_cells; base += (uint64_t)gridDim.x * (kBitsRounds * kBlock)) {
        float v[kBitsRounds];
#pragma unroll
        for (int round = 0; round < kBitsRounds; ++round) {
            const uint32_t c = (uint32_t)base + round * kBlock + threadIdx.x;       // n_cells <= 2^31: no wrap
            v[round] = density[c < n_cells ? c : n_cells - 1u];
        }
#pragma unroll
        for (int round = 0; round < kBitsRounds; ++round) {
            const uint32_t c = (uint32_t)base + round * kBlock + threadIdx.x;
            const bool on = c < n_cells && v[round] > threshold;
            const unsigned long long mask = __ballot(on);
            if (threadIdx.x % dg::kWave == 0 && c < n_cells) {
                const uint32_t w = c >> 5;
                bits[w] = (uint32_t)mask;
                if (w + 1u < n_words) bits[w + 1u] = (uint32_t)(mask >> 32);
                mine += (uint32_t)__popcll(mask);
            }
        }
    }
    if (!n_set) return;
    if (threadIdx.x % dg::kWave == 0) wave_count[threadIdx.x / dg::kWave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int w = 0; w < kWavesPerBlock; ++w) total += wave_count[w];
        if (total) atomicAdd(n_set, total);
    }
}

// ---------------------------------------------------------------- marching
struct MarchOut { float *u, *delta, *t; uint32_t *sample_ray; };

// Segments are short (some eighty strata where the box is flat): sixteen lanes take one, four to a wavefront, so that few lanes run past its end.
// The counting pass is bound by its look-ups, a cache line of the bit field per stratum, and by the arithmetic, two 64-bit products for the jitter and
// the cell; what it finds out about the first kMaskStrata strata stays in the workspace as bits, and the writing pass works on the kept ones
// alone.  208 k segments, 1.55 M of 16 M strata kept: 57 + 23 us (a wavefront per segment, both passes over all strata: 76 + 79).
// Where there are few, little more than the 8192 wavefronts that the chip holds, each gets one: what counts is then the chain along a segment.  The whole march with sixteen / 64 lanes, in us: flat box, tenth of the cells
// set 4000 segments 24 / 23, 10 000 26.5 / 25.9, 20 000 31 / 34, 260 000 141 / 217; cube, some 400 strata a segment, a layer set 1000 segments 36 / 22, 4000 38 / 28, 10 000 49 / 41,
// 20 000 64 / 61, 60 000 130 / 135; cube, all cells set 1000 44 / 25, 4000 53 / 35.
constexpr uint32_t kFewSegments = 10240, kFewLanes = dg::kWave, kManyLanes = 16;
constexpr uint32_t kMaskWords = 8, kMaskStrata = 32 * kMaskWords;

struct MarchIn {
    const float *o, *d, *seg_t;
    const uint32_t *seg_ray, *seg_slot;
    uint32_t n_seg, k_max;
    BoxArgs box;
    float dt;
    uint32_t max_steps;
    uint64_t seed;
};

// one segment, cut into n strata of equal width
struct Strata {
    uint32_t ray, n;
    uint64_t jitter;
    float t_in, width, o[3], d[3];

    __device__ __forceinline__ Strata(const MarchIn &in, uint32_t j)
    {
        ray = in.seg_ray[j];
        const uint32_t slot = in.seg_slot[j];
        jitter = jitter_base(in.seed, ray, slot);
        const size_t at = (size_t)ray * in.k_max + slot;
        t_in = in.seg_t[2 * at];
        const float len = in.seg_t[2 * at + 1] - t_in;
        const float wanted = ceilf(len / in.dt);               // strata no wider than the marching step
        n = wanted >= (float)in.max_steps ? in.max_steps : (wanted >= 1.0f ? (uint32_t)wanted : 1u);
        width = len / (float)n;
#pragma unroll
        for (int a = 0; a < 3; ++a) { o[a] = in.o[3 * (size_t)ray + a]; d[a] = in.d[3 * (size_t)ray + a]; }
    }
    // distance and unit coordinates of the sample in stratum s; z: jitter + golden * s
    __device__ __forceinline__ float sample(const MarchIn &in, uint32_t s, uint64_t z, float (&u)[3]) const
    {
        const float t = t_in + ((float)s + unit_float(mix_out(z))) * width;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float x = __builtin_fmaf(t, d[a], o[a]);
            u[a] = (x - in.box.lo[a]) * in.box.inv_ext[a];
        }
        return t;
    }
};

// `on` of the lane's segment, as its low bits
template <uint32_t LANES>
__device__ __forceinline__ uint64_t segment_ballot(bool on, uint32_t lane)
{
    const uint64_t wave = __ballot(on);
    return LANES == dg::kWave ? wave : (wave >> (lane & ~(LANES - 1u))) & ((1ull << (LANES % dg::kWave)) - 1ull);
}

template <uint32_t LANES>
__global__ void __launch_bounds__(kBlock)
march_count_kernel(MarchIn in, OccArgs occ, const uint32_t *__restrict__ bits, uint32_t *__restrict__ first, uint32_t *__restrict__ masks)
{
    const uint32_t j = blockIdx.x * (kBlock / LANES) + threadIdx.x / LANES, lane = threadIdx.x % dg::kWave, in_seg = threadIdx.x % LANES;
    if (blockIdx.x == 0 && threadIdx.x == 0) first[in.n_seg] = 0;            // the scan turns it into the total
    if (j >= in.n_seg) return;                                              // all lanes of a segment
    const Strata strata(in, j);
    uint32_t kept = 0;
    uint64_t z = strata.jitter + kGolden * in_seg, word = 0u;
    for (uint32_t base = 0; base < strata.n; base += LANES, z += kGolden * LANES) {
        float u[3];
        const uint32_t s = base + in_seg;
        strata.sample(in, s, z, u);
        const uint64_t mask = segment_ballot<LANES>(s < strata.n && bit_of(bits, cell_of(occ, u)), lane);      // empty space is skipped
        kept += (uint32_t)__popcll(mask);
        word |= mask << (base % 64u);
        if ((base + LANES) % 64u == 0u || base + LANES >= strata.n) {
            if (in_seg == 0 && base < kMaskStrata) {                        // words: the workspace may be aligned for no more
                uint32_t *at = masks + (size_t)kMaskWords * j + base / 64u * 2u;
                at[0] = (uint32_t)word;
                at[1] = (uint32_t)(word >> 32);
            }
            word = 0u;
        }
    }
    if (in_seg == 0) first[j] = kept;
}

// place of the set bit of x that has `rank` set bits below it
__device__ __forceinline__ uint32_t select_bit(uint32_t x, uint32_t rank)
{
    uint32_t at = 0;
#pragma unroll
    for (uint32_t half = 16; half > 0; half >>= 1) {
        const uint32_t below = (uint32_t)__popc(x & ((1u << half) - 1u));
        const bool above = rank >= below;
        rank -= above ? below : 0u;
        at += above ? half : 0u;
        x = above ? x >> half : x;
    }
    return at;
}

template <uint32_t LANES>
__global__ void __launch_bounds__(kBlock)
march_write_kernel(MarchIn in, OccArgs occ, const uint32_t *__restrict__ bits, uint32_t capacity, const uint32_t *__restrict__ first,
                   const uint32_t *__restrict__ masks, MarchOut out, uint32_t *__restrict__ status)
{
    const uint32_t j = blockIdx.x * (kBlock / LANES) + threadIdx.x / LANES, lane = threadIdx.x % dg::kWave, in_seg = threadIdx.x % LANES;
    if (j >= in.n_seg) return;                                              // all lanes of a segment
    const uint32_t begin = first[j], total = first[j + 1] - begin;
    if (total == 0u) return;
    const Strata strata(in, j);
    bool dropped = false;
    auto write = [&](uint32_t at, uint32_t s) {
        const uint32_t pos = begin + at;
        if (pos < capacity) {
            float u[3];
            out.t[pos] = strata.sample(in, s, strata.jitter + kGolden * s, u);
            out.u[3 * (size_t)pos] = u[0]; out.u[3 * (size_t)pos + 1] = u[1]; out.u[3 * (size_t)pos + 2] = u[2];
            out.delta[pos] = strata.width;
            out.sample_ray[pos] = strata.ray;
        } else {
            dropped = true;
        }
    };
    uint32_t word[kMaskWords], below[kMaskWords + 1];                       // kept samples in the words before
    below[0] = 0u;
#pragma unroll
    for (uint32_t w = 0; w < kMaskWords; ++w) {
        word[w] = 32u * w < strata.n ? masks[(size_t)kMaskWords * j + w] : 0u;
        below[w + 1] = below[w] + (uint32_t)__popc(word[w]);
    }
    for (uint32_t i = in_seg; i < below[kMaskWords]; i += LANES) {
        uint32_t mine = word[0], rank = i, base = 0;
#pragma unroll
        for (uint32_t w = 1; w < kMaskWords; ++w)
            if (i >= below[w]) { mine = word[w]; rank = i - below[w]; base = 32u * w; }
        write(i, base + select_bit(mine, rank));
    }
    // strata that the bits do not reach are looked at again
    uint32_t kept = below[kMaskWords];
    for (uint32_t base = kMaskStrata; base < strata.n; base += LANES) {
        float u[3];
        const uint32_t s = base + in_seg;
        strata.sample(in, s, strata.jitter + kGolden * s, u);
        const bool keep = s < strata.n && bit_of(bits, cell_of(occ, u));
        const uint64_t mask = segment_ballot<LANES>(keep, lane);
        if (keep) write(kept + (uint32_t)__popcll(mask & ((1ull << in_seg) - 1ull)), s);
        kept += (uint32_t)__popcll(mask);
    }
    if (dropped) atomicOr(status, 2u);
}

// ---------------------------------------------------------------- exclusive scan of uint32 values, in place
__device__ __forceinline__ uint32_t wave_inclusive(uint32_t v, uint32_t lane)
{
#pragma unroll
    for (int off = 1; off < dg::kWave; off <<= 1) {
        const uint32_t up = __shfl_up(v, off, dg::kWave);
        if (lane >= (uint32_t)off) v += up;
    }
    return v;
}

// exclusive prefix of x over the workgroup (WAVES wavefronts); total receives the sum of all
template <int WAVES>
__device__ __forceinline__ uint32_t block_exclusive(uint32_t x, uint32_t *wave_sums, uint32_t &total)
{
    const uint32_t lane = threadIdx.x % dg::kWave, wave = threadIdx.x / dg::kWave;
    const uint32_t incl = wave_inclusive(x, lane);
    if (lane == dg::kWave - 1) wave_sums[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const uint32_t v = wave_sums[w];
        before += (uint32_t)w < wave ? v : 0u;
        all += v;
    }
    __syncthreads();                                      // wave_sums may be reused by the caller's next round
    total = all;
    return before + incl - x;
}

__global__ void __launch_bounds__(kBlock)
scan_tile_sums_kernel(const uint32_t *__restrict__ v, uint32_t n, uint32_t *__restrict__ sums)
{
    __shared__ uint32_t wave_sums[kWavesPerBlock];
    const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) mine += base + i < n ? v[base + i] : 0u;
    uint32_t total;
    block_exclusive<kWavesPerBlock>(mine, wave_sums, total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kSumsBlock)
scan_sums_kernel(uint32_t *__restrict__ sums, uint32_t n_tiles)
{
    __shared__ uint32_t wave_sums[kSumsBlock / dg::kWave];
    uint32_t carry = 0;
    for (uint32_t base = 0; base < n_tiles; base += kSumsBlock) {         // the bound is uniform over the workgroup
        const uint32_t i = base + threadIdx.x;
        const uint32_t x = i < n_tiles ? sums[i] : 0u;
        uint32_t total;
        const uint32_t excl = block_exclusive<kSumsBlock / dg::kWave>(x, wave_sums, total);
        if (i < n_tiles) sums[i] = carry + excl;
        carry += total;
    }
}

__global__ void __launch_bounds__(kBlock)
scan_apply_kernel(uint32_t *__restrict__ v, uint32_t n, const uint32_t *__restrict__ sums)
{
    __shared__ uint32_t wave_sums[kWavesPerBlock];
    const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
    uint32_t x[kScanItems], mine = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) { x[i] = base + i < n ? v[base + i] : 0u; mine += x[i]; }
    uint32_t total;
    uint32_t run = sums[blockIdx.x] + block_exclusive<kWavesPerBlock>(mine, wave_sums, total);
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        if (base + i < n) v[base + i] = run;
        run += x[i];
    }
}

uint32_t scan_tiles(uint32_t n) { return (uint32_t)(((uint64_t)n + kScanTile - 1) / kScanTile); }

OccArgs occ_args(const dg_occ_desc *desc)
{
    OccArgs g;
    for (int a = 0; a < 3; ++a) { g.res[a] = desc->res[a]; g.scale[a] = desc->scale[a]; }
    g.n_cells = desc->n_cells;
    return g;
}

int occ_desc_ok(const dg_occ_desc *desc, const char *who)
{
    DG_REQUIRE(desc, DG_ERR_ARG, "%s: null descriptor", who);
    DG_REQUIRE(desc->res[0] && desc->res[1] && desc->res[2] &&
                   (uint64_t)desc->res[0] * desc->res[1] * desc->res[2] == desc->n_cells,
               DG_ERR_ARG, "%s: descriptor not initialised by dg_occ_desc_init", who);
    return DG_OK;
}

}  // namespace

extern "C" int dg_occ_desc_init(dg_occ_desc *desc, uint32_t N, const double extent[3])
{
    DG_REQUIRE(desc && extent, DG_ERR_ARG, "dg_occ_desc_init: null pointer");
    DG_REQUIRE(N >= 1, DG_ERR_ARG, "dg_occ_desc_init: resolution must be at least 1");
    DG_REQUIRE(extent[0] > 0 && extent[1] > 0 && extent[2] > 0, DG_ERR_ARG, "dg_occ_desc_init: box extents must be positive");
    std::memset(desc, 0, sizeof *desc);
    const double longest = std::fmax(extent[0], std::fmax(extent[1], extent[2]));
    uint64_t cells = 1;
    for (int a = 0; a < 3; ++a) {
        const double along = extent[a] / longest * (double)N;       // the hash grid's rule at one resolution (Sec. 4.1)
        const uint32_t r = (uint32_t)std::ceil(along);
        desc->res[a] = r ? r : 1u;
        desc->scale[a] = (float)along;
        cells *= desc->res[a];
        DG_REQUIRE(cells <= 0x80000000ull, DG_ERR_UNSUPPORTED, "dg_occ_desc_init: more than 2^31 cells");
    }
    desc->n_cells = (uint32_t)cells;
    return DG_OK;
}

extern "C" void dg_occ_schedule(uint64_t iteration, int *update_now, int *warmup, float *decay, float *threshold)
{
    if (update_now) *update_now = iteration % 16 == 0;
    if (warmup) *warmup = iteration < 4096;
    if (decay) *decay = 0.99f;
    if (threshold) *threshold = iteration < 10000 ? 0.6f : 60.0f;
}

extern "C" int dg_occ_candidates(const dg_occ_desc *desc, const uint32_t *bits, uint32_t i0, uint32_t M, uint32_t n_uniform,
                                 int warmup, uint64_t seed, uint32_t iteration, uint32_t tries, uint32_t *cell, float *u,
                                 void *stream)
{
    if (int rc = occ_desc_ok(desc, "dg_occ_candidates")) return rc;
    DG_REQUIRE((uint64_t)i0 + M <= (1u << 28) && iteration < (1u << 28), DG_ERR_UNSUPPORTED,
               "dg_occ_candidates: candidate indices and iteration must be below 2^28");
    DG_REQUIRE(tries >= 1 && tries <= 64, DG_ERR_ARG, "dg_occ_candidates: tries=%u outside 1..64", tries);
    DG_REQUIRE(!warmup || (uint64_t)i0 + M <= desc->n_cells, DG_ERR_ARG, "dg_occ_candidates: the warm-up rule visits cell i, i0 + M exceeds n_cells");
    if (M == 0) return DG_OK;
    DG_REQUIRE(cell && u && (warmup || n_uniform >= i0 + M || bits), DG_ERR_ARG, "dg_occ_candidates: null pointer");
    candidates_kernel<<<(M + kBlock - 1) / kBlock, kBlock, 0, (hipStream_t)stream>>>(occ_args(desc), bits, i0, M, n_uniform, warmup,
                                                                                    seed, iteration, tries, cell, u);
    return dg::launch_status("dg_occ_candidates");
}

extern "C" int dg_occ_decay(float *density, uint32_t n_cells, float factor, void *stream)
{
    if (n_cells == 0) return DG_OK;
    DG_REQUIRE(density, DG_ERR_ARG, "dg_occ_decay: null pointer");
    const uint32_t n_blocks = (uint32_t)(((uint64_t)n_cells + kBlock - 1) / kBlock);
    decay_kernel<<<n_blocks, kBlock, 0, (hipStream_t)stream>>>(density, n_cells, factor);
    return dg::launch_status("dg_occ_decay");
}

extern "C" int dg_occ_update(float *density, uint32_t n_cells, const uint32_t *cell, const float *sigma, uint32_t M, void *stream)
{
    if (M == 0) return DG_OK;
    DG_REQUIRE(density && cell && sigma, DG_ERR_ARG, "dg_occ_update: null pointer");
    const uint32_t n_blocks = (uint32_t)(((uint64_t)M + kBlock - 1) / kBlock);
    update_kernel<<<n_blocks, kBlock, 0, (hipStream_t)stream>>>(density, n_cells, cell, sigma, M);
    return dg::launch_status("dg_occ_update");
}

extern "C" int dg_occ_bits(const float *density, uint32_t n_cells, float threshold, uint32_t *bits, uint32_t *n_set, void *stream)
{
    if (n_cells == 0) return DG_OK;
    DG_REQUIRE(density && bits, DG_ERR_ARG, "dg_occ_bits: null pointer");
    const uint64_t per_block = (uint64_t)kBlock * kBitsRounds;
    const uint64_t blocks = ((uint64_t)n_cells + per_block - 1) / per_block;
    bits_kernel<<<(uint32_t)(blocks < kBitsGrid ? blocks : kBitsGrid), kBlock, 0, (hipStream_t)stream>>>(density, n_cells, threshold, bits, n_set);
    return dg::launch_status("dg_occ_bits");
}

namespace {
size_t march_sums_bytes(uint32_t n_seg)
{
    const size_t bytes = (size_t)scan_tiles(n_seg + 1u) * sizeof(uint32_t);      // n_seg < 2^32 - 1 is checked at the call
    return (bytes + 255u) / 256u * 256u;
}
}  // namespace

extern "C" size_t dg_march_workspace_bytes(uint32_t n_seg)
{
    return march_sums_bytes(n_seg) + (size_t)n_seg * kMaskWords * sizeof(uint32_t);
}

extern "C" int dg_march_segments(const float *o, const float *d, const float *seg_t, const uint32_t *seg_ray,
                                 const uint32_t *seg_slot, uint32_t n_seg, uint32_t k_max, const float *box,
                                 const dg_occ_desc *occ, const uint32_t *bits, float dt, uint32_t max_steps, uint64_t seed,
                                 uint32_t capacity, uint32_t *first, float *u, float *delta, float *t, uint32_t *sample_ray,
                                 uint32_t *status, void *ws, size_t ws_bytes, void *stream)
{
    if (int rc = occ_desc_ok(occ, "dg_march_segments")) return rc;
    DG_REQUIRE(box && k_max >= 1 && dt > 0.0f && max_steps >= 1 && max_steps <= 65535, DG_ERR_ARG,
               "dg_march_segments: bad box, k_max, dt or max_steps (1..65535)");
    DG_REQUIRE(n_seg < 0xffffffffu, DG_ERR_UNSUPPORTED, "dg_march_segments: too many segments");
    DG_REQUIRE(first && status && ws, DG_ERR_ARG, "dg_march_segments: null pointer");
    DG_REQUIRE(ws_bytes >= dg_march_workspace_bytes(n_seg), DG_ERR_WORKSPACE, "dg_march_segments: workspace of %zu bytes, %zu needed",
               ws_bytes, dg_march_workspace_bytes(n_seg));
    DG_REQUIRE(n_seg == 0 || (o && d && seg_t && seg_ray && seg_slot && bits), DG_ERR_ARG, "dg_march_segments: null pointer");
    DG_REQUIRE(capacity == 0 || (u && delta && t && sample_ray), DG_ERR_ARG, "dg_march_segments: null output");
    BoxArgs b;
    for (int a = 0; a < 3; ++a) {
        DG_REQUIRE(box[3 + a] > box[a], DG_ERR_ARG, "dg_march_segments: empty box");
        b.lo[a] = box[a];
        b.inv_ext[a] = 1.0f / (box[3 + a] - box[a]);
    }
    hipStream_t st = (hipStream_t)stream;
    const OccArgs g = occ_args(occ);
    const MarchOut out = {u, delta, t, sample_ray};
    const MarchIn in = {o, d, seg_t, seg_ray, seg_slot, n_seg, k_max, b, dt, max_steps, seed};
    uint32_t *sums = (uint32_t *)ws;
    uint32_t *masks = sums + march_sums_bytes(n_seg) / sizeof(uint32_t);
    const uint32_t n_vals = n_seg + 1u, n_tiles = scan_tiles(n_vals);
    auto march = [&](auto lanes) {
        constexpr uint32_t kLanes = decltype(lanes)::value;
        const uint32_t blocks = (uint32_t)(((uint64_t)n_seg * kLanes + kBlock - 1) / kBlock);
        march_count_kernel<kLanes><<<blocks ? blocks : 1u, kBlock, 0, st>>>(in, g, bits, first, masks);
        scan_tile_sums_kernel<<<n_tiles, kBlock, 0, st>>>(first, n_vals, sums);
        scan_sums_kernel<<<1, kSumsBlock, 0, st>>>(sums, n_tiles);
        scan_apply_kernel<<<n_tiles, kBlock, 0, st>>>(first, n_vals, sums);
        if (n_seg) march_write_kernel<kLanes><<<blocks, kBlock, 0, st>>>(in, g, bits, capacity, first, masks, out, status);
    };
    if (n_seg <= kFewSegments) march(std::integral_constant<uint32_t, kFewLanes>{});
    else march(std::integral_constant<uint32_t, kManyLanes>{});
    return dg::launch_status("dg_march_segments");
}
