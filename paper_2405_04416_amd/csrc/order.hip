// Samples in spatial order: a two-step counting sort that puts the samples of a sub-model next to the samples they
// share table lines with.
//
// Rays are drawn at random over all images, so samples in ray order meet the tables of the fine levels at random: every
// corner row costs a cache line of its own, and runs of equal cells end with the ray.  In spatial order the lines that
// neighbours share are fetched once, and the coarser levels' gradients can be summed on chip before they go anywhere.
//
//   1. bricks: the box is cut into equal bricks.  Aimed at are 700 to 1200 samples each; the number along every axis is then
//      rounded down and the total is at most 2^15, so that a brick holds some 700 to 2400 samples on average (2^19 samples: a few
//      hundred bricks; the limit rules from some 39 M samples on).  Count, scan, scatter with one persistent tiling; the
//      counters of all bricks live in LDS, so there are no global atomics.
//      A sample becomes 16 bytes: its coordinates and the index it came from (or a number of the caller's).
//   2. inside a brick: pencils along x (the table's contiguous direction), sorted in LDS.
// The order is a matter of speed alone: any order gives the same results.
// Bound by the scatter's lone 16-byte writes (33.5 M samples: 0.53 of 1.05 ms) and the LDS sort.
#include "order_common.h"
#include <cmath>
#include <cstring>
#include <mutex>

namespace {

using namespace dg_order;

constexpr int kSweepBlock = 1024, kSweepGrid = 256;      // one workgroup per compute unit: its counters fill LDS
constexpr int kScanKeys = 32, kScanGroups = 32;

__device__ __forceinline__ float unit(float u)
{
    u = u >= 0.0f ? u : 0.0f;          // NaN lands on 0 as well
    return u > 1.0f ? 1.0f : u;
}

__device__ __forceinline__ uint32_t brick_axis(float u, float n, uint32_t last)
{
    const uint32_t i = (uint32_t)(unit(u) * n);
    return i > last ? last : i;
}

__device__ __forceinline__ uint32_t brick_of(const Bricks &b, float x, float y, float z)
{
    return brick_axis(x, b.per_unit[0], b.n[0] - 1u) + b.n[0] * (brick_axis(y, b.per_unit[1], b.n[1] - 1u) + b.n[1] * brick_axis(z, b.per_unit[2], b.n[2] - 1u));
}

// every workgroup counts the samples of each brick in its tiles -> rows[workgroup][brick]
__global__ void __launch_bounds__(kSweepBlock)
brick_count_kernel(Bricks b, const float *__restrict__ u, uint64_t N, uint32_t *__restrict__ rows)
{
    extern __shared__ uint32_t counts[];
    for (uint32_t i = threadIdx.x; i < b.total; i += kSweepBlock) counts[i] = 0u;
    __syncthreads();
    for (uint64_t n = (uint64_t)blockIdx.x * kSweepBlock + threadIdx.x; n < N; n += (uint64_t)gridDim.x * kSweepBlock)
        atomicAdd(&counts[brick_of(b, u[3 * n], u[3 * n + 1], u[3 * n + 2])], 1u);
    __syncthreads();
    uint32_t *row = rows + (size_t)blockIdx.x * b.total;
    for (uint32_t i = threadIdx.x; i < b.total; i += kSweepBlock) row[i] = counts[i];
}

// rows -> exclusive prefix over the workgroups, per brick; totals per brick
__global__ void __launch_bounds__(kScanKeys * kScanGroups)
brick_scan_rows_kernel(uint32_t *__restrict__ rows, uint32_t n_rows, uint32_t n_keys, uint32_t *__restrict__ totals)
{
    __shared__ uint32_t part[kScanGroups][kScanKeys];
    const uint32_t col = threadIdx.x % kScanKeys, group = threadIdx.x / kScanKeys;
    const uint32_t k = blockIdx.x * kScanKeys + col;
    const uint32_t per = (n_rows + kScanGroups - 1) / kScanGroups;
    const uint32_t lo = min(group * per, n_rows), hi = min(lo + per, n_rows);
    uint32_t sum = 0;
    if (k < n_keys)
        for (uint32_t r = lo; r < hi; ++r) sum += rows[(size_t)r * n_keys + k];
    part[group][col] = sum;
    __syncthreads();
    if (k >= n_keys) return;
    uint32_t run = 0;
    for (uint32_t g = 0; g < group; ++g) run += part[g][col];
    for (uint32_t r = lo; r < hi; ++r) {
        const uint32_t t = rows[(size_t)r * n_keys + k];
        rows[(size_t)r * n_keys + k] = run;
        run += t;
    }
    if (group == kScanGroups - 1) totals[k] = run;
}

// exclusive prefix over the bricks, and the list of pieces: a brick's samples in pieces of at most kPiece (one workgroup; at
// most kMaxBricks bricks).  pieces[0] = (number of pieces, 0 for the caller's use), then (brick, first sample) of each, then (0, N).
__global__ void __launch_bounds__(1024)
brick_scan_totals_kernel(const uint32_t *__restrict__ totals, uint32_t n_keys, uint32_t *__restrict__ first, uint2 *__restrict__ pieces)
{
    __shared__ uint32_t wave_sum[16], wave_pieces[16];
    const uint32_t per = (n_keys + 1023u) / 1024u, lo = min(threadIdx.x * per, n_keys), hi = min(lo + per, n_keys);
    const uint32_t lane = threadIdx.x % dg::kWave, wave = threadIdx.x / dg::kWave;
    uint32_t sum = 0, sum_p = 0;
    for (uint32_t i = lo; i < hi; ++i) { sum += totals[i]; sum_p += (totals[i] + kPiece - 1u) / kPiece; }
    uint32_t incl = sum, incl_p = sum_p;
#pragma unroll
    for (int off = 1; off < dg::kWave; off <<= 1) {
        const uint32_t up = __shfl_up(incl, off, dg::kWave), up_p = __shfl_up(incl_p, off, dg::kWave);
        if ((int)lane >= off) { incl += up; incl_p += up_p; }
    }
    if (lane == dg::kWave - 1) { wave_sum[wave] = incl; wave_pieces[wave] = incl_p; }
    __syncthreads();
    uint32_t run = incl - sum, run_p = incl_p - sum_p;
    for (uint32_t w = 0; w < wave; ++w) { run += wave_sum[w]; run_p += wave_pieces[w]; }
    for (uint32_t i = lo; i < hi; ++i) {
        first[i] = run;
        for (uint32_t at = 0; at < totals[i]; at += kPiece) pieces[1 + run_p++] = make_uint2(i, run + at);
        run += totals[i];
    }
    if (threadIdx.x == 1023) {
        pieces[0] = make_uint2(run_p, 0u);
        pieces[1 + run_p] = make_uint2(0u, run);
    }
}

// same tiling as the count: a sample takes its place with an LDS add on its brick's counter
__global__ void __launch_bounds__(kSweepBlock)
brick_scatter_kernel(Bricks b, const float *__restrict__ u, const uint32_t *__restrict__ ids, uint64_t N, const uint32_t *__restrict__ rows,
                     const uint32_t *__restrict__ first, float4 *__restrict__ ordered)
{
    extern __shared__ uint32_t next[];
    const uint32_t *row = rows + (size_t)blockIdx.x * b.total;
    for (uint32_t i = threadIdx.x; i < b.total; i += kSweepBlock) next[i] = row[i] + first[i];
    __syncthreads();
    for (uint64_t n = (uint64_t)blockIdx.x * kSweepBlock + threadIdx.x; n < N; n += (uint64_t)gridDim.x * kSweepBlock) {
        const float x = u[3 * n], y = u[3 * n + 1], z = u[3 * n + 2];
        const uint32_t at = atomicAdd(&next[brick_of(b, x, y, z)], 1u);
        ordered[at] = make_float4(x, y, z, __uint_as_float(ids ? ids[n] : (uint32_t)n));
    }
}

// Inside a brick: 16 x 8 x 8 cells, x fastest.  A piece is sorted in LDS, up to kSortRun samples at a time (a brick that holds many more
// samples than the average is only sorted run by run).  Bound by the chain from the loads over the counts to the stores, so the runs are as short
// as the bricks of most batches and four workgroups fit a compute unit: 13.3 M samples 82 us, 19.8 M 152
// (4096 samples, two workgroups: 137 and 410).
constexpr int kSortBlock = 512, kCells = 1024, kSortRun = 2048, kPerThread = kSortRun / kSortBlock;
__global__ void __launch_bounds__(kSortBlock)
brick_sort_kernel(Bricks b, const uint2 *__restrict__ pieces, float4 *__restrict__ ordered)
{
    __shared__ float4 stage[kSortRun];
    __shared__ uint32_t count[kCells];
    __shared__ uint32_t wave_sum[kSortBlock / dg::kWave];
    if (blockIdx.x >= pieces[0].x) return;
    const uint32_t lane = threadIdx.x % dg::kWave, wave = threadIdx.x / dg::kWave;
    const uint32_t end = pieces[2 + blockIdx.x].y;
    for (uint32_t base = pieces[1 + blockIdx.x].y; base < end; base += kSortRun) {
        const uint32_t n = min(end - base, (uint32_t)kSortRun);
        float4 s[kPerThread];
        uint32_t place[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const uint32_t i = k * kSortBlock + threadIdx.x;
            if (i < n) s[k] = ordered[base + i];
        }
        for (uint32_t i = threadIdx.x; i < kCells; i += kSortBlock) count[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const uint32_t i = k * kSortBlock + threadIdx.x;
            if (i >= n) continue;
            // sixteenths and eighths of the brick (the brick's own number drops out of the low bits)
            const uint32_t cx = (uint32_t)(unit(s[k].x) * b.per_unit[0] * 16.0f) & 15u, cy = (uint32_t)(unit(s[k].y) * b.per_unit[1] * 8.0f) & 7u,
                           cz = (uint32_t)(unit(s[k].z) * b.per_unit[2] * 8.0f) & 7u;
            const uint32_t yz = (cy & 1u) | (cz & 1u) << 1 | (cy & 2u) << 1 | (cz & 2u) << 2 | (cy & 4u) << 2 | (cz & 4u) << 3;
            const uint32_t cell = yz << 4 | cx;
            place[k] = cell << 16 | atomicAdd(&count[cell], 1u);
        }
        __syncthreads();
        // exclusive scan of the cell counts, two per thread
        const uint32_t c0 = count[2 * threadIdx.x], c1 = count[2 * threadIdx.x + 1];
        uint32_t incl = c0 + c1;
#pragma unroll
        for (int off = 1; off < dg::kWave; off <<= 1) {
            const uint32_t up = __shfl_up(incl, off, dg::kWave);
            if ((int)lane >= off) incl += up;
        }
        if (lane == dg::kWave - 1) wave_sum[wave] = incl;
        __syncthreads();
        uint32_t run = incl - c0 - c1;
        for (uint32_t w = 0; w < wave; ++w) run += wave_sum[w];
        count[2 * threadIdx.x] = run;
        count[2 * threadIdx.x + 1] = run + c0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const uint32_t i = k * kSortBlock + threadIdx.x;
            if (i < n) stage[count[place[k] >> 16] + (place[k] & 0xffffu)] = s[k];
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < n; i += kSortBlock) ordered[base + i] = stage[i];
        __syncthreads();                                                  // counts and sums of the next run
    }
}

}  // namespace

namespace {

inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Vertices of a brick at one level, along one axis.  A brick of width w voxels meets at most floor(w) + 2 voxels, floor(w) + 3
// vertices (2e-2: room for the slack and the fp32 rounding of the edges).
uint32_t box_vertices(const dg_grid_desc *desc, uint32_t l, int a, uint32_t n_bricks)
{
    const uint32_t box = (uint32_t)std::floor((double)desc->scale[l][a] / n_bricks + 2e-2) + 3u;
    return box < desc->res[l][a] + 1u ? box : desc->res[l][a] + 1u;
}

double finest_scale(const dg_grid_desc *desc, uint32_t l) { return std::fmax(desc->scale[l][0], std::fmax(desc->scale[l][1], desc->scale[l][2])); }

// bricks of about per_brick samples, and the levels that such a brick has in LDS together
void cut_bricks(dg_order_desc *order, const dg_grid_desc *desc, uint64_t N, uint32_t per_brick)
{
    std::memset(order, 0, sizeof *order);
    // the box's proportions, from the finest level's voxels along each axis
    const float *ext = desc->scale[desc->n_levels - 1];
    const double want = std::fmin((double)kMaxBricks, std::fmax(1.0, (double)N / per_brick));
    const double per_side = std::cbrt(want / ((double)ext[0] * ext[1] * ext[2]));
    uint64_t total = 1;
    for (int a = 0; a < 3; ++a) {
        double n = std::floor(ext[a] * per_side);
        n = std::fmin(std::fmax(n, 1.0), 1024.0);
        order->n_bricks[a] = (uint32_t)n;
        total *= order->n_bricks[a];
    }
    while (total > kMaxBricks) {          // a flat box rounds up to one brick along its short axes: fewer along the longest
        int a = 0;
        for (int k = 1; k < 3; ++k) if (order->n_bricks[k] > order->n_bricks[a]) a = k;
        order->n_bricks[a] = (order->n_bricks[a] + 1) / 2;
        total = (uint64_t)order->n_bricks[0] * order->n_bricks[1] * order->n_bricks[2];
    }
    order->total = (uint32_t)total;
    for (int a = 0; a < 3; ++a) order->per_unit[a] = (float)order->n_bricks[a];
    // levels summed brick by brick in the backward pass: as many as have their brick's vertices in LDS together
    uint32_t at = 0, l = 0;
    for (; l < kMaxMerged; ++l) {
        uint64_t vertices = 1;
        uint32_t box[3];
        for (int a = 0; a < 3; ++a) {
            box[a] = box_vertices(desc, l, a, order->n_bricks[a]);
            vertices *= box[a];
        }
        if (at + vertices > kMaxBoxVertices || finest_scale(desc, l) > kMaxMergedScale) break;
        for (int a = 0; a < 3; ++a) order->box[l][a] = box[a];
        order->box_first[l] = at;
        at += (uint32_t)vertices;
        order->box_first[l + 1] = at;
    }
    order->n_merged = l & ~1u;
}

}  // namespace

namespace dg_order {
int order_ok(const dg_order_desc *o, const char *who)
{
    DG_REQUIRE(o, DG_ERR_ARG, "%s: null order descriptor", who);
    DG_REQUIRE(o->n_bricks[0] && o->n_bricks[1] && o->n_bricks[2] && o->total <= kMaxBricks &&
                   (uint64_t)o->n_bricks[0] * o->n_bricks[1] * o->n_bricks[2] == o->total,
               DG_ERR_ARG, "%s: descriptor not initialised by dg_order_desc_init", who);
    return DG_OK;
}

// the boxes are those of this grid: with another grid's the brick sums would land outside the levels
int order_fits(const dg_order_desc *o, const dg_grid_desc *d, const char *who)
{
    bool fits = o->n_merged <= kMaxMerged && o->n_merged <= d->n_levels && o->box_first[0] == 0;
    for (int a = 0; a < 3; ++a) fits = fits && o->per_unit[a] == (float)o->n_bricks[a];
    for (uint32_t l = 0; fits && l < o->n_merged; ++l) {
        uint64_t vertices = 1;
        for (int a = 0; a < 3; ++a) {
            fits = fits && o->box[l][a] == box_vertices(d, l, a, o->n_bricks[a]);
            vertices *= o->box[l][a];
        }
        fits = fits && o->box_first[l] + vertices == o->box_first[l + 1] && o->box_first[l + 1] <= kMaxBoxVertices && finest_scale(d, l) <= kMaxMergedScale;
    }
    DG_REQUIRE(fits, DG_ERR_ARG, "%s: the order descriptor was made for another grid", who);
    return DG_OK;
}
}  // namespace dg_order

extern "C" int dg_order_desc_init(dg_order_desc *order, const dg_grid_desc *desc, uint64_t N)
{
    const char *who = "dg_order_desc_init";
    DG_REQUIRE(order && desc, DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(desc->n_levels == 16 && desc->n_features == 2, DG_ERR_UNSUPPORTED, "%s: needs L = 16, F = 2", who);
    std::memset(order, 0, sizeof *order);
    // Bricks of about 1200 samples, or smaller ones, down to 700, where more levels then fit LDS (two more levels summed per
    // brick save 2 / 16 of the table-gradient pass: 13.3 M samples, T = 2^19, 9680 bricks and 10 levels 3.85 ms, 16 854 bricks and
    // 12 levels 3.54 ms; with bricks of 500 and 350 samples 3.70 and 3.66 ms).
    for (uint32_t per_brick = kPerBrickMax; per_brick >= kPerBrickMin; per_brick -= 100) {
        dg_order_desc trial;
        cut_bricks(&trial, desc, N, per_brick);
        if (trial.n_merged > order->n_merged || order->total == 0) *order = trial;
    }
    return DG_OK;
}

extern "C" size_t dg_order_workspace_bytes(const dg_order_desc *order)
{
    if (order_ok(order, "dg_order_workspace_bytes")) return 0;
    return align256((size_t)kSweepGrid * order->total * sizeof(uint32_t)) + align256((size_t)order->total * sizeof(uint32_t)) +
           align256(((size_t)order->total + 1) * sizeof(uint32_t));
}

extern "C" size_t dg_order_pieces_words(const dg_order_desc *order, uint64_t N)
{
    if (order_ok(order, "dg_order_pieces_words")) return 0;
    return 2 * (2 + piece_bound(order->total, N));
}

extern "C" int dg_order_samples(const dg_order_desc *order, const float *u, const uint32_t *ids, uint64_t N, void *ordered, uint32_t *pieces,
                                void *ws, size_t ws_bytes, void *stream)
{
    const char *who = "dg_order_samples";
    if (int rc = order_ok(order, who)) return rc;
    DG_REQUIRE(pieces && ws, DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(N == 0 || (u && ordered), DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(N < 0xffffffffull, DG_ERR_UNSUPPORTED, "%s: too many samples", who);
    DG_REQUIRE(dg::aligned(ordered, 16) && dg::aligned(pieces, 8) && dg::aligned(ws, 256), DG_ERR_ARG, "%s: misaligned pointer", who);
    DG_REQUIRE(ws_bytes >= dg_order_workspace_bytes(order), DG_ERR_WORKSPACE, "%s: workspace %zu < %zu bytes", who, ws_bytes,
               dg_order_workspace_bytes(order));
    static std::once_flag lds_once;
    static hipError_t lds_status = hipSuccess;
    std::call_once(lds_once, [] {
        const int bytes = (int)(kMaxBricks * sizeof(uint32_t));
        const hipError_t e[2] = {
            hipFuncSetAttribute(reinterpret_cast<const void *>(&brick_count_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes),
            hipFuncSetAttribute(reinterpret_cast<const void *>(&brick_scatter_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes)};
        for (const hipError_t x : e)
            if (x != hipSuccess) lds_status = x;
    });
    if (lds_status != hipSuccess) return dg::fail(DG_ERR_HIP, "%s: cannot reserve LDS: %s", who, hipGetErrorString(lds_status));
    const Bricks b = bricks_of(order);
    hipStream_t st = (hipStream_t)stream;
    uint32_t *rows = static_cast<uint32_t *>(ws);
    uint32_t *totals = rows + align256((size_t)kSweepGrid * b.total * sizeof(uint32_t)) / sizeof(uint32_t);
    uint32_t *first = totals + align256((size_t)b.total * sizeof(uint32_t)) / sizeof(uint32_t);
    const size_t lds = (size_t)b.total * sizeof(uint32_t);
    brick_count_kernel<<<kSweepGrid, kSweepBlock, lds, st>>>(b, u, N, rows);
    brick_scan_rows_kernel<<<(b.total + kScanKeys - 1) / kScanKeys, kScanKeys * kScanGroups, 0, st>>>(rows, kSweepGrid, b.total, totals);
    brick_scan_totals_kernel<<<1, 1024, 0, st>>>(totals, b.total, first, (uint2 *)pieces);
    brick_scatter_kernel<<<kSweepGrid, kSweepBlock, lds, st>>>(b, u, ids, N, rows, first, (float4 *)ordered);
    brick_sort_kernel<<<(uint32_t)piece_bound(b.total, N), kSortBlock, 0, st>>>(b, (const uint2 *)pieces, (float4 *)ordered);
    return dg::launch_status(who);
}
