// Hash-grid encode backward without global atomics in the inner loop (Sec. 3.2: the transpose of the
// encode).
//
// Global fp32 atomics on MI355X retire at a fixed rate per distinct cache line an instruction touches
// (about 21 G lines/s measured, whatever the scope or table size), far below what the 8 x N x L
// scattered adds of this pass need.  LDS atomics do not have that limit.  So the table gradient is
// built by binning:
//   * levels whose tables fit LDS together (the coarse prefix) are accumulated directly: persistent
//     workgroups sweep the samples, merge runs of lanes that share a cell, add into an LDS copy of
//     those tables and flush it once;
//   * every other level is cut into bins of 8192 entries (128 KB of 64-bit sums in LDS).  A counting sweep
//     and a filling sweep over the samples (same persistent tiling, so each workgroup owns a private,
//     pre-computed slice of every bin's queue: no global atomics, no overflow) write one 16-byte record
//     (two entries within the bin, 4 values) per pair of corners along x, or one of 12 bytes, collected in LDS so that each
//     bin receives whole lines (encode_bwd_fill.hip).  Then workgroups balanced by record count stream the queue,
//     accumulate in LDS (as scaled 64-bit integers: integer adds are the fastest LDS atomics) and add the
//     finished bin into dtable with coalesced atomics.
//     Many bins of few records are taken by workgroups that stay (sparse_bins).
// Where there are few bins altogether, all of them are accumulated directly, without queues (direct_bins).
#include "encode_binned_common.h"
#include <algorithm>
#include <mutex>

namespace dg_encode_binned {

// ------------------------------------------------------------------ accumulate in LDS directly
// Groups of `width` workgroups, each for a table region that fits LDS: the coarse prefix, if there is one, and then every bin of the
// other levels where direct_bins takes this way.  A group's workgroups sweep all samples at their region's levels and add what falls
// into it.
__global__ void __launch_bounds__(kCoarseBlock)
coarse_kernel(dg_grid_desc g, Plan plan, uint32_t from_level, uint32_t width, const float *__restrict__ u, const float2 *__restrict__ dfeat,
              uint64_t N, float *__restrict__ dtable)
{
    // 2 sums per entry of the region, one plane per feature (an add instruction then spreads over all LDS banks); fp64 LDS atomics
    // run ~7x faster than fp32 ones
    extern __shared__ double tab[];
    const uint32_t group = blockIdx.x / width, me = blockIdx.x % width, prefix = plan.first_level > from_level ? 1u : 0u;
    uint32_t first = from_level, end = plan.first_level, base = g.offset[first], n_entries = g.offset[end] - base;      // levels, entries
    if (group >= prefix) {
        const uint32_t key = group - prefix;
        first = plan.first_level;
        while (first + 1 < g.n_levels && key >= plan.key_base[first + 1]) ++first;
        end = first + 1;
        base = g.offset[first] + (key - plan.key_base[first]) * kChunk;
        n_entries = min(kChunk, g.offset[end] - base);
    }
    const uint32_t n_floats = 2u * n_entries;
    for (uint32_t i = threadIdx.x; i < n_floats; i += kCoarseBlock) tab[i] = 0.0;
    __syncthreads();
    const int lane = threadIdx.x % dg::kWave;
    const uint32_t mask = (1u << g.log2_T) - 1u;
    const uint64_t n_tiles = (N + kCoarseBlock - 1) / kCoarseBlock;
    for (uint64_t tile = me; tile < n_tiles; tile += width) {
        const uint64_t n = tile * kCoarseBlock + threadIdx.x;
        const bool live = n < N;
        const uint64_t nn = live ? n : N - 1;
        const float uu[3] = {u[3 * nn], u[3 * nn + 1], u[3 * nn + 2]};
        for (uint32_t l = first; l < end; ++l) {
            const LevelGeom lv = level_of(g, l);
            uint32_t cell[3], e[8];
            float frac[3], w[8];
            locate(lv, uu, cell, frac);
            corner_entries(lv, mask, cell, e);
            corner_weights(frac, w);
            float2 gfe = dfeat[(size_t)l * N + nn];
            if (!live) gfe = make_float2(0.0f, 0.0f);
            bool head = lane == 0;
#pragma unroll
            for (int a = 0; a < 3; ++a) head |= from_lane_below(cell[a]) != cell[a];
            const unsigned long long heads = __ballot(head);
            float vx[8], vy[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) { vx[c] = w[c] * gfe.x; vy[c] = w[c] * gfe.y; }
            if (__popcll(heads) < dg::kWave) segmented_sum(vx, vy, head, heads);     // merge each run into its last lane
            const bool tail = lane == dg::kWave - 1 || ((heads >> ((lane + 1) & 63)) & 1ull);
            if (tail) {
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const uint32_t slot = lv.offset + e[c] - base;
                    if (slot >= n_entries) continue;                 // another bin's
                    if (vx[c] != 0.0f) __hip_atomic_fetch_add(&tab[slot], (double)vx[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (vy[c] != 0.0f) __hip_atomic_fetch_add(&tab[n_entries + slot], (double)vy[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_floats; i += kCoarseBlock) {
        const float v = (float)tab[(i & 1u) * n_entries + (i >> 1)];
        if (v != 0.0f) unsafeAtomicAdd(dtable + 2 * (size_t)base + i, v);
    }
}

// ------------------------------------------------------------------ queues
// The records are those of encode_bwd_fill.hip.
template <typename R>
__device__ __forceinline__ void unpack_record(const R &r, uint32_t &ea, uint32_t &eb, float &v0, float &v1, float &v2, float &v3)
{
    ea = r.x & (kChunk - 1u);
    eb = ea ^ ((1u << (r.x >> 13 & 15u)) - 1u);
    v0 = __uint_as_float(r.y << 5);
    v1 = __uint_as_float(r.z << 5);
    v2 = __uint_as_float(r.w << 5);
    v3 = __uint_as_float((r.x >> 17 | (r.y >> 27) << 15 | (r.z >> 27) << 20 | (r.w >> 27) << 25) << 5);
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// rows[b][k] (per-workgroup counts, each rounded up to a multiple of `round`) -> exclusive prefix over workgroups;
// totals[k].  A workgroup serves 32 keys; 32 groups of threads each take a contiguous stretch of the rows, whose counts stay
// in registers between the two passes (all loads under way at once: 3 times as fast as a loop over the rows).
constexpr int kScanKeys = 32, kScanGroups = 32;
template <int PER>      // rows per group
__global__ void __launch_bounds__(kScanKeys * kScanGroups)
scan_rows_kernel(uint32_t *__restrict__ rows, uint32_t n_rows, uint32_t n_keys, uint32_t round, uint32_t *__restrict__ totals)
{
    __shared__ uint32_t part[kScanGroups][kScanKeys];
    const uint32_t col = threadIdx.x % kScanKeys, group = threadIdx.x / kScanKeys;
    const uint32_t k = blockIdx.x * kScanKeys + col, lo = group * PER;
    uint32_t count[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) count[i] = k < n_keys && lo + i < n_rows ? rows[(size_t)(lo + i) * n_keys + k] : 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) { count[i] = (count[i] + round - 1u) / round * round; sum += count[i]; }     // a slice is padded to whole granules
    part[group][col] = sum;
    __syncthreads();
    if (k >= n_keys) return;
    uint32_t run = 0;
    for (uint32_t g = 0; g < group; ++g) run += part[g][col];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (lo + i < n_rows) rows[(size_t)(lo + i) * n_keys + k] = run;
        run += count[i];
    }
    if (group == kScanGroups - 1) totals[k] = run;
}

// binbase = exclusive scan of totals, and the list of pieces the accumulate workgroups take: pieces[0].x of them, each (key,
// first record, end) -- a bin is cut into acc_pieces of its record count, in equal shares, so that work is balanced whatever
// the bins hold, and a workgroup finds its share with one load.  (One workgroup; n_keys is at most a few tens of thousands.)
__global__ void __launch_bounds__(1024)
scan_totals_kernel(const uint32_t *__restrict__ totals, uint32_t n_keys, uint32_t piece_log2, uint32_t round, uint32_t *__restrict__ binbase, uint4 *__restrict__ pieces)
{
    __shared__ uint32_t wave_sum[16], wave_pieces[16];
    const uint32_t per = (n_keys + 1023) / 1024, lo = min(threadIdx.x * per, n_keys), hi = min(lo + per, n_keys);
    const uint32_t lane = threadIdx.x % dg::kWave, wave = threadIdx.x / dg::kWave;
    uint32_t s = 0, sp = 0;
    for (uint32_t i = lo; i < hi; ++i) { s += totals[i]; sp += acc_pieces(totals[i], piece_log2); }
    const uint32_t incl = wave_inclusive_scan(s), incl_p = wave_inclusive_scan(sp);
    if (lane == dg::kWave - 1) { wave_sum[wave] = incl; wave_pieces[wave] = incl_p; }
    __syncthreads();
    uint32_t run = incl - s, run_p = incl_p - sp;
    for (uint32_t w = 0; w < wave; ++w) { run += wave_sum[w]; run_p += wave_pieces[w]; }
    for (uint32_t i = lo; i < hi; ++i) {
        const uint32_t total = totals[i], n = acc_pieces(total, piece_log2), share = n ? ((total + n - 1u) / n + round - 1u) / round * round : 0u;
        binbase[i] = run;
        for (uint32_t q = 0; q < n; ++q) pieces[1 + run_p++] = make_uint4(i, run + (uint32_t)min((uint64_t)q * share, (uint64_t)total), run + (uint32_t)min((q + 1ull) * share, (uint64_t)total), 0u);
        run += total;
    }
    if (threadIdx.x == 1023) {
        binbase[n_keys] = run;
        binbase[n_keys + 1] = 0u;        // the fill sweep leaves the largest record magnitude of the batch here
        pieces[0] = make_uint4(run_p, 0u, 0u, 0u);
    }
}

// ------------------------------------------------------------------ accumulate one (bin, split)
// The sums are kept as 64-bit integers in LDS: integer adds there run at almost twice the rate of fp64 adds
// (2.7 against 1.5 T adds/s measured).  A value v becomes round(v * 2^k) with k chosen from the largest record
// magnitude of the batch so that the sum of a workgroup's records (fewer than 2^kAccMaxLog2) stays below 2^50; the
// conversion is the add of 1.5 * 2^52 in fp64, after which the low mantissa bits hold the integer in two's complement.
// The quantum is 2^-31 of the largest magnitude or finer, hundreds of times below the fp32 rounding of the value itself,
// and integer sums do not depend on the order of the additions.
// A sum of doubles' bit patterns adds their low bits; what happens above bit 50 is dropped when the sum is read.
__device__ __forceinline__ void add_fixed(unsigned long long *slot, float v, double scale)
{
    __hip_atomic_fetch_add(slot, (unsigned long long)__double_as_longlong(__builtin_fma((double)v, scale, 6755399441055744.0 /* 1.5 * 2^52 */)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The two kinds of records in the queues.  A thread takes kDepth records at a time, kAccBlock apart, 64 bytes.
struct PairRecords {
    static constexpr int kDepth = 4;
    typedef u32x4 Record;
    static __device__ __forceinline__ uint32_t offset(uint32_t i) { return i * 16u; }                  // of record i, in bytes
    static __device__ __forceinline__ uint32_t slot(uint32_t entry, uint32_t feature) { return feature * kChunk + entry; }      // of the sum
    // records that fill a slice up are zero: they would all add to one sum in turn
    static __device__ __forceinline__ bool empty(const Record &rec) { return (rec.x >> 17 | rec.y | rec.z | rec.w) == 0u; }
    static __device__ __forceinline__ void add(unsigned long long *tab, const Record &rec, double scale)
    {
        uint32_t ea, eb;
        float v0, v1, v2, v3;
        unpack_record(rec, ea, eb, v0, v1, v2, v3);
        add_fixed(&tab[ea], v0, scale);
        add_fixed(&tab[kChunk + ea], v1, scale);
        add_fixed(&tab[eb], v2, scale);
        add_fixed(&tab[kChunk + eb], v3, scale);
    }
};
// slot of the entry's sums (slot_of, 14 bits), pair_code (4 bits), gradient times y and z weights (27-bit floats), x fraction in units of 2^-23
struct CompactRecords {
    static constexpr int kDepth = kCompactLine;
    typedef uint32_t Record __attribute__((ext_vector_type(3), aligned(4)));
    static __device__ __forceinline__ uint32_t offset(uint32_t i) { return i / kCompactLine * 64u + i % kCompactLine * 12u; }
    static __device__ __forceinline__ uint32_t slot(uint32_t entry, uint32_t feature)
    {
        return (entry & (kChunk / 2 - 1u)) | (entry & kChunk / 2) << 1 | feature * (kChunk / 2);
    }
    static __device__ __forceinline__ bool empty(const Record &rec) { return ((rec.y | rec.z) & 0x7ffffffu) == 0u; }
    static __device__ __forceinline__ void add(unsigned long long *tab, const Record &rec, double scale)
    {
        const uint32_t a = (rec.x & 0x3fffu) << 3, b = a ^ ((1u << (rec.x >> 14 & 15u)) - 1u) << 3;
        const uint32_t fx = __builtin_amdgcn_alignbit(__builtin_amdgcn_alignbit(rec.z >> 27, rec.y, 27u), rec.x, 18u);
        const double at1 = (double)fx, at0 = 8388608.0 - at1, unit = scale * 0x1p-23;
        const double gx = (double)__uint_as_float(rec.y << 5) * unit, gy = (double)__uint_as_float(rec.z << 5) * unit;
        char *const sums = reinterpret_cast<char *>(tab);
        add_scaled(sums + a, gx, at0);
        add_scaled(sums + a + kChunk / 2 * 8, gy, at0);
        add_scaled(sums + b, gx, at1);
        add_scaled(sums + b + kChunk / 2 * 8, gy, at1);
    }
    // adds round(v * w)
    static __device__ __forceinline__ void add_scaled(char *sum, double v, double w)
    {
        __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(sum), (unsigned long long)__double_as_longlong(__builtin_fma(v, w, 6755399441055744.0 /* 1.5 * 2^52 */)),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

// A thread's records of a piece: several in flight so that the queue streams at memory speed.  The loads are unconditional (clamped to the
// piece's last record) so that they issue back to back, and non-temporal: what is read once streams faster past the caches (measured).
template <class R>
struct PieceReader {
    static constexpr uint32_t kStride = R::kDepth * kAccBlock;           // records per turn of the workgroup
    static constexpr uint32_t kStrideBytes = 64u * kAccBlock;
    uint32_t offset[R::kDepth];
    __device__ __forceinline__ PieceReader()
    {
#pragma unroll
        for (int j = 0; j < R::kDepth; ++j) offset[j] = R::offset(j * kAccBlock + threadIdx.x);
    }
    // the records of turn `turn` of a piece whose last record lies at `last`
    __device__ __forceinline__ void load(typename R::Record (&rec)[R::kDepth], const char *piece, uint32_t turn, uint32_t last) const
    {
#pragma unroll
        for (int j = 0; j < R::kDepth; ++j)
            rec[j] = __builtin_nontemporal_load(reinterpret_cast<const typename R::Record *>(piece + min(turn * kStrideBytes + offset[j], last)));
    }
    // adds them, n records in the piece
    __device__ __forceinline__ void add(unsigned long long *tab, const typename R::Record (&rec)[R::kDepth], uint32_t turn, uint32_t n, double scale) const
    {
#pragma unroll
        for (int j = 0; j < R::kDepth; ++j)
            if (turn * kStride + j * kAccBlock + threadIdx.x < n && !R::empty(rec[j])) R::add(tab, rec[j], scale);
    }
};
static_assert(PairRecords::kDepth * 16 == 64 && CompactRecords::kDepth == kCompactLine, "a thread takes 64 bytes of the queue per turn");

template <class R>
__device__ __forceinline__ const char *piece_records(const char *queue, uint32_t first)
{
    return queue + (R::kDepth == kCompactLine ? (size_t)(first / kCompactLine) * 64 : (size_t)first * 16);
}

template <class R>
__global__ void __launch_bounds__(kAccBlock)
accumulate_kernel(dg_grid_desc g, Plan plan, const uint32_t *__restrict__ binbase, const uint4 *__restrict__ pieces,
                  const char *__restrict__ queue, float *__restrict__ dtable)
{
    // [2][kChunk] sums, one plane per feature: an add instruction then spreads over all LDS banks instead of every other pair
    extern __shared__ unsigned long long acc_tab[];
    unsigned long long *tab = acc_tab;
    const uint4 piece = pieces[1 + blockIdx.x];                           // the list has room for every workgroup of the grid
    if (blockIdx.x >= pieces[0].x) return;
    const uint32_t key = piece.x, n = piece.z - piece.y;                  // fewer than 2^kAccMaxLog2 records
    // 2^k with k = 50 - kAccMaxLog2 - 1 - (exponent of the largest magnitude): 2^kAccMaxLog2 values of that size sum to < 2^50
    const uint32_t top = binbase[plan.n_keys + 1] >> 23;                 // biased exponent (0 for zero / denormal: no smaller k needed)
    const int k = 50 - kAccMaxLog2 - 1 - ((int)(top ? top : 1u) - 127);
    const double scale = __longlong_as_double((long long)(1023 + k) << 52);
    const double inv_scale = __longlong_as_double((long long)(1023 - k) << 52);
    if (top == 255u) {
        // an infinite or NaN contribution somewhere in the batch: the scale above means nothing and integer sums cannot
        // carry it.  The gradient is marked instead: every bin that has records gets NaN in its first entry, as sums
        // with fp32 atomics would end up non-finite too.
        if (threadIdx.x == 0 && n) {
            uint32_t lv = plan.first_level;
            while (lv + 1 < g.n_levels && key >= plan.key_base[lv + 1]) ++lv;
            dtable[2 * ((size_t)g.offset[lv] + (size_t)(key - plan.key_base[lv]) * kChunk)] = __uint_as_float(0x7fc00000u);
        }
        return;
    }
    for (uint32_t i = threadIdx.x; i < 2 * kChunk; i += kAccBlock) tab[i] = 0ull;
    __syncthreads();
    if (n) {
        const PieceReader<R> reader;
        const char *records = piece_records<R>(queue, piece.y);
        const uint32_t last = R::offset(n - 1u);
        typename R::Record rec[R::kDepth];
        reader.load(rec, records, 0u, last);
        for (uint32_t turn = 0; turn * PieceReader<R>::kStride < n; ++turn) {
            typename R::Record now[R::kDepth];
#pragma unroll
            for (int j = 0; j < R::kDepth; ++j) now[j] = rec[j];
            reader.load(rec, records, turn + 1u, last);
            reader.add(tab, now, turn, n, scale);
        }
    }
    __syncthreads();
    uint32_t l = plan.first_level;
    while (l + 1 < g.n_levels && key >= plan.key_base[l + 1]) ++l;
    const uint32_t bin = key - plan.key_base[l];
    const uint32_t level_len = g.offset[l + 1] - g.offset[l];
    const uint32_t first = bin * kChunk, n_valid = min(kChunk, level_len - first);
    float *dst = dtable + 2 * ((size_t)g.offset[l] + first);
    for (uint32_t i = threadIdx.x; i < 2 * n_valid; i += kAccBlock) {
        const float sum = (float)(from_low_bits(tab[R::slot(i >> 1, i & 1u)]) * inv_scale);
        if (sum != 0.0f) unsafeAtomicAdd(dst + i, sum);
    }
}

// The same for bins of few records, which are bound not by the queue but by the chain of a bin -- its piece, the first records from
// memory, the adds, the table's way in and out -- in a compute unit that one table fills.  One workgroup per compute unit stays
// and takes piece after piece from a common counter: the next piece's first records are on their way while the table goes out,
// which also clears it.
// Where it serves: sparse_bins.  Eight sub-models, four of them with 4074 bins of 5.7 k records: 243 -> 219 us each.  (Bins that come in one piece
// stored instead, with what the gradient held added: 183 us, but then an add of another stream to the same gradient is lost.)
template <class R>
__global__ void __launch_bounds__(kAccBlock)
accumulate_sparse_kernel(dg_grid_desc g, Plan plan, const uint32_t *__restrict__ binbase, const uint4 *__restrict__ pieces,
                  const char *__restrict__ queue, float *__restrict__ dtable, uint32_t *__restrict__ taken)
{
    // [2][kChunk] sums, one plane per feature: an add instruction then spreads over all LDS banks instead of every other pair
    extern __shared__ __attribute__((aligned(16))) unsigned long long acc_tab[];
    __shared__ uint32_t next_piece;
    constexpr int kPerThread = 2 * (int)kChunk / kAccBlock;              // sums of the table
    unsigned long long *tab = acc_tab;
    const uint32_t n_pieces = pieces[0].x;
    uint32_t index = blockIdx.x;                                         // the list has room for every workgroup of the grid
    // 2^k with k = 50 - kAccMaxLog2 - 1 - (exponent of the largest magnitude): 2^kAccMaxLog2 values of that size sum to < 2^50
    const uint32_t top = binbase[plan.n_keys + 1] >> 23;                 // biased exponent (0 for zero / denormal: no smaller k needed)
    const int k = 50 - kAccMaxLog2 - 1 - ((int)(top ? top : 1u) - 127);
    const double scale = __longlong_as_double((long long)(1023 + k) << 52);
    const double inv_scale = __longlong_as_double((long long)(1023 - k) << 52);
    if (top == 255u) {
        // an infinite or NaN contribution somewhere in the batch: the scale above means nothing and integer sums cannot
        // carry it.  The gradient is marked instead: every bin that has records gets NaN in its first entry, as sums
        // with fp32 atomics would end up non-finite too.
        for (uint32_t i = blockIdx.x * kAccBlock + threadIdx.x; i < n_pieces; i += gridDim.x * kAccBlock) {
            const uint32_t key = pieces[1 + i].x;
            uint32_t lv = plan.first_level;
            while (lv + 1 < g.n_levels && key >= plan.key_base[lv + 1]) ++lv;
            dtable[2 * ((size_t)g.offset[lv] + (size_t)(key - plan.key_base[lv]) * kChunk)] = __uint_as_float(0x7fc00000u);
        }
        return;
    }
    if (index >= n_pieces) return;
    const PieceReader<R> reader;
    uint4 piece = pieces[1 + index];                                     // key, first record, end: fewer than 2^kAccMaxLog2 records, at least one
    typename R::Record rec[R::kDepth];
    reader.load(rec, piece_records<R>(queue, piece.y), 0u, R::offset(piece.z - piece.y - 1u));
    uint4 *const clear = reinterpret_cast<uint4 *>(tab);
    for (uint32_t i = threadIdx.x; i < kChunk; i += kAccBlock) clear[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    for (;;) {
        const uint32_t key = piece.x, n = piece.z - piece.y, last = R::offset(n - 1u);
        const char *const records = piece_records<R>(queue, piece.y);
        if (threadIdx.x == 0) next_piece = gridDim.x + atomicAdd(taken, 1u);
        uint32_t l = plan.first_level;
        while (l + 1 < g.n_levels && key >= plan.key_base[l + 1]) ++l;
        const uint32_t first = (key - plan.key_base[l]) * kChunk, n_values = 2 * min(kChunk, g.offset[l + 1] - g.offset[l] - first);
        float *dst = dtable + 2 * ((size_t)g.offset[l] + first);
        for (uint32_t turn = 0;; ++turn) {
            typename R::Record now[R::kDepth];
#pragma unroll
            for (int j = 0; j < R::kDepth; ++j) now[j] = rec[j];
            const bool more = (turn + 1u) * PieceReader<R>::kStride < n;
            if (more) reader.load(rec, records, turn + 1u, last);
            reader.add(tab, now, turn, n, scale);
            if (!more) break;
        }
        __syncthreads();
        index = next_piece;
        const bool another = index < n_pieces;
        if (another) {
            piece = pieces[1 + index];
            reader.load(rec, piece_records<R>(queue, piece.y), 0u, R::offset(piece.z - piece.y - 1u));
        }
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            const uint32_t i = j * kAccBlock + threadIdx.x;
            if (i >= n_values) continue;
            unsigned long long *from = tab + R::slot(i >> 1, i & 1u);
            const unsigned long long bits = *from;
            *from = 0ull;
            const float sum = (float)(from_low_bits(bits) * inv_scale);
            if (sum != 0.0f) unsafeAtomicAdd(dst + i, sum);
        }
        if (!another) break;
        __syncthreads();
    }
}

// from_level > 0: the caller sums the levels below it (brick_bwd); what is left of the coarse prefix is taken here
Plan make_plan(const dg_grid_desc *d, uint32_t from_level)
{
    Plan p{};
    uint32_t l = std::max(from_level, dg::coarse_levels(d));
    p.first_level = l;
    uint32_t key = 0;
    for (; l < d->n_levels; ++l) {
        p.key_base[l] = key;
        p.n_bins[l] = (d->offset[l + 1] - d->offset[l] + kChunk - 1) / kChunk;
        key += p.n_bins[l];
        if (p.n_bins[l] > p.max_bins) p.max_bins = p.n_bins[l];
    }
    p.compact = from_level > 0u;
    uint32_t bins = 1;
    while (bins < p.max_bins) bins *= 2;
    p.max_bins = bins;
    p.per_unit = per_unit(p);
    p.key_base[d->n_levels] = key;
    p.n_keys = key;
    return p;
}

inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }

struct Layout {
    size_t rows, totals, binbase, pieces, queue, total;
    uint64_t batch;      // samples per batch
    uint64_t records;    // queue capacity: the records of a batch plus the padding of the slices
};

// width and groups of the sweeps over nb samples at n_levels levels: the split with the fewest (tile, level) steps per
// workgroup, one group unless another saves a thirtieth.  A level costs half a step beyond its tiles (rings opened and written out).  (80 k samples
// at 12 levels, 79 tiles for 512 workgroups: 6 groups of 85 would do with 3 such steps, 12 of 42 with 2.5: the fill takes 41.3 and 39.0 us.)
Sweep choose_sweep(const Plan &p, uint32_t n_levels, uint64_t nb)
{
    const uint64_t n_tiles = (nb + kFillTile - 1) / kFillTile;
    const uint32_t grid = fill_grid(p), levels = n_levels - p.first_level;
    Sweep best = {grid, 1};
    double least = 0.0;
    for (uint32_t k = 1; k <= levels; ++k) {
        const uint32_t width = grid / k;
        const double steps = ((double)((n_tiles + width - 1) / width) + 0.5) * ((levels + k - 1) / k);
        if (k == 1 || steps < least * (29.0 / 30.0)) { best = {width, k}; least = steps; }
    }
    best.width = (uint32_t)std::min<uint64_t>(best.width, n_tiles);          // the others would have no tile, but counters to clear and rows to scan
    return best;
}
// Zero records that fill up the slices of nb samples, at most: a workgroup without a tile has no records and no slice.  (A level of 512 bins is
// 512 workgroups' appends of 128 bytes, 29 MB of padding a level where all have tiles, 57 KB where one tile is all a workspace has room for.)
uint64_t slice_padding(const Plan &p, uint64_t nb)
{
    return std::min<uint64_t>(fill_grid(p), (nb + kFillTile - 1) / kFillTile) * p.n_keys * (slice_round(p) - 1u);
}

uint32_t piece_log2(uint64_t records)
{
    uint32_t k = kPieceLog2Min;
    while (k < (uint32_t)kPieceLog2Max && records >> (k + 1) >= 512) ++k;
    return k;
}

// accumulate workgroups that `records` records need at most
uint32_t acc_grid(const Plan &p, uint64_t records) { return (uint32_t)(records >> piece_log2(records)) + p.n_keys; }

// All bins summed in LDS directly, in the sweep that serves the coarse prefix (coarse_kernel): one launch instead of six and no queue,
// but every bin's workgroups go through all samples: 8 us + 12.6 ps per sample and bin against some 45 us + 34 ps per sample and level
// through the queues, which the line below follows.  In us, direct / queues: 6 bins in 3 levels 33 k samples 18 / 52, 1.6 M 129 / 186,
// 4 M 326 / 567; 17 bins in 3 levels 0.3 M 70 / 120, 3 M 618 / 425; 30 bins in 15 levels 30 k 23 / 76, 3 M 1086 / 1796; 58 bins in 13
// levels 30 k 31 / 73, 0.3 M 219 / 247, 3 M 2203 / 1625.  At most as many bins as workgroups are resident at once.
bool direct_bins(const Plan &p, uint32_t n_levels, uint64_t N)
{
    const uint64_t free = 5ull * (n_levels - p.first_level) / 2;
    return p.n_keys < (uint32_t)kCoarseGrid && (p.n_keys <= free || N * (p.n_keys - free) < 5000000ull);
}

// Many bins: accumulate_sparse_kernel.  Its time against accumulate_kernel's in us, with `bins` bins and `records` records per bin at most.  Compact records:
// 12 288 bins, 65 500 records 2212 / 2275; 12 288, 38 700 1426 / 1466; four calls of 3072, 25 400 1068 / 1122; few bins: 256 bins, 832 000 records 519 / 522; 390,
// 203 000 281 / 239; 512, 97 000 171 / 166.  Records of 16 bytes: 4074, 5700 211 / 243; 15 923, 1300 955 / 1014; 611, 4800 49 / 47; the whole pass, for more records
// than entries: 3731, 8500 438 / 427; 3731, 17 000 645 / 669; 3731, 113 000 3720 / 3733; 4566, 23 000 1124 / 1157; 8662, 48 000 4148 / 4174; 15 923, 53 000 9037 / 9126.
bool sparse_bins(const Plan &p) { return p.n_keys >= 2048u; }

// records that nb samples make at most, with the padding of the slices
uint64_t batch_records(const Plan &p, uint32_t n_levels, uint64_t nb) { return nb * 4ull * (n_levels - p.first_level) + slice_padding(p, nb); }

// workspace layout for a batch of `batch` samples
Layout make_layout(const dg_grid_desc *d, const Plan &p, uint64_t batch)
{
    Layout L{};
    const uint64_t records = (batch_records(p, d->n_levels, batch) + 79ull) / 80ull * 80ull;
    size_t off = 0;
    L.rows = off; off = align256(off + (size_t)fill_grid(p) * p.n_keys * 4);
    L.totals = off; off = align256(off + (size_t)p.n_keys * 4);
    L.binbase = off; off = align256(off + (size_t)(p.n_keys + 3) * 4);      // + the largest record magnitude, the pieces taken
    // a smaller batch may have smaller pieces: never more than 1024 beyond one per bin while they are not at their largest
    L.pieces = off; off = align256(off + (size_t)(1 + std::max(acc_grid(p, records), 1024u + p.n_keys)) * 16);
    L.queue = off; off = align256(off + records / line_records(p) * 64);
    L.total = off;
    L.batch = batch;
    L.records = records;
    return L;
}

uint64_t max_batch(const dg_grid_desc *d, const Plan &p)
{
    const uint64_t per_sample = 4ull * (d->n_levels - p.first_level);
    if (per_sample == 0) return ~0ull;
    return ((0xffffffffull - slice_padding(p, ~0ull / 2) - 80ull) / per_sample) / kTile * kTile;           // record offsets stay below 2^32
}

}  // namespace dg_encode_binned

namespace dg {

uint32_t coarse_levels(const dg_grid_desc *d)
{
    uint32_t l = 0;
    while (l < d->n_levels && d->offset[l + 1] <= dg_encode_binned::kChunk) ++l;
    return l;
}

size_t encode_bwd_binned_workspace_bytes(const dg_grid_desc *d, uint32_t from_level, uint64_t N)
{
    using namespace dg_encode_binned;
    const Plan p = make_plan(d, from_level);
    if (p.n_keys == 0) return 256;
    uint64_t batch = (N + kTile - 1) / kTile * kTile;
    const uint64_t cap = max_batch(d, p);
    if (batch > cap) batch = cap;
    if (batch == 0) batch = kTile;
    return make_layout(d, p, batch).total;
}

namespace {

using namespace dg_encode_binned;

// what a call works with: the plan of the grid, the batch the workspace holds and the workspace's parts
struct Prepared {
    Plan p;
    Layout L;
    uint32_t *rows, *totals, *binbase;
    uint4 *pieces;
    char *queue;
};

int prepare(const char *who, const dg_grid_desc *d, uint32_t from_level, uint64_t N, void *ws, size_t ws_bytes, Prepared &q)
{
    q.p = make_plan(d, from_level);
    // kernels that use more LDS than a launch gets by default: asked for once per process, whichever thread comes first
    static std::once_flag lds_once;
    static hipError_t lds_status = hipSuccess;
    std::call_once(lds_once, [] {
        const int acc_lds = 2 * kChunk * (int)sizeof(double);
        const hipError_t e[] = {
            (hipError_t)reserve_fill(),
            hipFuncSetAttribute(reinterpret_cast<const void *>(&accumulate_kernel<PairRecords>), hipFuncAttributeMaxDynamicSharedMemorySize, acc_lds),
            hipFuncSetAttribute(reinterpret_cast<const void *>(&accumulate_kernel<CompactRecords>), hipFuncAttributeMaxDynamicSharedMemorySize, acc_lds),
            hipFuncSetAttribute(reinterpret_cast<const void *>(&accumulate_sparse_kernel<PairRecords>), hipFuncAttributeMaxDynamicSharedMemorySize, acc_lds),
            hipFuncSetAttribute(reinterpret_cast<const void *>(&accumulate_sparse_kernel<CompactRecords>), hipFuncAttributeMaxDynamicSharedMemorySize, acc_lds),
            hipFuncSetAttribute(reinterpret_cast<const void *>(&coarse_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, acc_lds)};
        for (const hipError_t x : e)
            if (x != hipSuccess) lds_status = x;
    });
    if (lds_status != hipSuccess) return dg::fail(DG_ERR_HIP, "%s: cannot reserve LDS: %s", who, hipGetErrorString(lds_status));
    if (q.p.n_keys == 0) return DG_OK;
    if (q.p.n_keys > kMaxKeys) return dg::fail(DG_ERR_UNSUPPORTED, "%s: %u table regions exceed %u", who, q.p.n_keys, kMaxKeys);
    // largest batch the workspace holds
    uint64_t batch = (N + kTile - 1) / kTile * kTile;
    const uint64_t cap = max_batch(d, q.p);
    if (batch > cap) batch = cap;
    while (batch > kTile && make_layout(d, q.p, batch).total > ws_bytes) batch = (batch / 2 + kTile - 1) / kTile * kTile;
    q.L = make_layout(d, q.p, batch);
    if (q.L.total > ws_bytes)
        return dg::fail(DG_ERR_WORKSPACE, "%s: workspace %zu bytes cannot hold one tile (%zu needed)", who, ws_bytes, q.L.total);
    char *base = static_cast<char *>(ws);
    q.rows = reinterpret_cast<uint32_t *>(base + q.L.rows);
    q.totals = reinterpret_cast<uint32_t *>(base + q.L.totals);
    q.binbase = reinterpret_cast<uint32_t *>(base + q.L.binbase);
    q.pieces = reinterpret_cast<uint4 *>(base + q.L.pieces);
    q.queue = base + q.L.queue;
    return DG_OK;
}

// count sweep and scans of samples [n0, n0 + nb): every workgroup's slice of every bin's queue, the bins' queue ranges,
// the accumulate workgroups per bin; also clears the slot of the batch's largest magnitude
void launch_count(const Prepared &q, const dg_grid_desc *d, const float *u, uint64_t n0, uint64_t nb, hipStream_t st)
{
    const Plan &p = q.p;
    const Sweep sw = choose_sweep(p, d->n_levels, nb);
    count_records(d, p, sw, u, n0, nb, q.rows, st);
    const uint32_t scan_grid = (p.n_keys + kScanKeys - 1) / kScanKeys;
    auto scan = [&](auto kernel) { kernel<<<scan_grid, kScanKeys * kScanGroups, 0, st>>>(q.rows, sw.width, p.n_keys, slice_round(p), q.totals); };
    if (sw.width <= 8u * kScanGroups) scan(scan_rows_kernel<8>);
    else scan(scan_rows_kernel<16>);
    scan_totals_kernel<<<1, 1024, 0, st>>>(q.totals, p.n_keys, piece_log2(batch_records(p, d->n_levels, nb)), slice_round(p), q.binbase, q.pieces);
}

}  // namespace

int encode_bwd_binned_count(const char *who, const dg_grid_desc *d, uint32_t from_level, const float *u, uint64_t N, void *ws, size_t ws_bytes, hipStream_t st)
{
    Prepared q;
    if (int rc = prepare(who, d, from_level, N, ws, ws_bytes, q)) return rc;
    if (q.p.n_keys == 0) return DG_OK;
    if (q.L.batch < N)
        return fail(DG_ERR_WORKSPACE, "%s: counting ahead needs a workspace that holds all %llu samples in one batch (it holds %llu)", who,
                    (unsigned long long)N, (unsigned long long)q.L.batch);
    if (direct_bins(q.p, d->n_levels, N)) return DG_OK;                  // no queues to size
    launch_count(q, d, u, 0, N, st);
    return launch_status(who);
}

int encode_bwd_binned(const char *who, const dg_grid_desc *d, uint32_t from_level, const float *u, const float *dfeat, uint64_t N,
                      float *dtable, void *ws, size_t ws_bytes, bool counted, hipStream_t st)
{
    Prepared q;
    if (int rc = prepare(who, d, from_level, N, ws, ws_bytes, q)) return rc;
    const Plan &p = q.p;
    if (counted && p.n_keys && q.L.batch < N)
        return fail(DG_ERR_WORKSPACE, "%s: the workspace holds %llu of %llu samples: no counts from dg_hashgrid_encode_bwd_count can be in it",
                    who, (unsigned long long)q.L.batch, (unsigned long long)N);
    const bool direct = direct_bins(p, d->n_levels, N);
    const uint32_t groups = (p.first_level > from_level ? 1u : 0u) + (direct ? p.n_keys : 0u);
    if (groups) {
        const uint64_t tiles = (N + kCoarseBlock - 1) / kCoarseBlock;
        const uint32_t width = std::max(1u, (uint32_t)std::min<uint64_t>(tiles, kCoarseGrid / groups));
        const uint32_t entries = direct && p.n_keys ? kChunk : d->offset[p.first_level] - d->offset[from_level];
        coarse_kernel<<<groups * width, kCoarseBlock, 2 * entries * sizeof(double), st>>>(*d, p, from_level, width, u, (const float2 *)dfeat, N, dtable);
    }
    if (p.n_keys == 0 || direct) return launch_status(who);
    const uint64_t batch = q.L.batch;
    for (uint64_t n0 = 0; n0 < N; n0 += batch) {
        const uint64_t nb = N - n0 < batch ? N - n0 : batch;
        if (!counted) launch_count(q, d, u, n0, nb, st);
        const Sweep sw = choose_sweep(p, d->n_levels, nb);
        fill_queues(d, p, sw, u, dfeat, N, n0, nb, q.rows, q.binbase, q.queue, dtable, st);
        const uint64_t records = batch_records(p, d->n_levels, nb);
        const uint32_t grid = acc_grid(p, records);
        constexpr size_t table = 2 * kChunk * sizeof(double);
        auto accumulate = [&](auto kind) {
            typedef decltype(kind) R;
            if (sparse_bins(p))
                accumulate_sparse_kernel<R><<<std::min(grid, (uint32_t)kAccGrid), kAccBlock, table, st>>>(*d, p, q.binbase, q.pieces, q.queue, dtable,
                                                                                                         q.binbase + p.n_keys + 2);
            else accumulate_kernel<R><<<grid, kAccBlock, table, st>>>(*d, p, q.binbase, q.pieces, q.queue, dtable);
        };
        if (p.compact) accumulate(CompactRecords{});
        else accumulate(PairRecords{});
    }
    return launch_status(who);
}

}  // namespace dg
