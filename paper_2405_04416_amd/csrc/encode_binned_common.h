// What the table-gradient passes that go through bins share: bins, plans of a sweep, the sweeps' look-ahead.  Internal, not part of the ABI.
#pragma once
#include "encode_common.h"

namespace dg_encode_binned {

using namespace dg_encode;

constexpr int kChunkLog2 = 13;
constexpr uint32_t kChunk = 1u << kChunkLog2;      // entries per bin
constexpr int kMaxBins = 2048;                     // per level: 2^24 entries / 8192
constexpr int kTile = 512;                         // samples per tile == threads per binning workgroup
constexpr int kKeeper = 64;                        // narrow fill sweep: one more wavefront, which keeps the books of the 64 bins
constexpr int kPairs = kTile * 4;                  // records staged per (tile, level): one per pair of corners along x
constexpr uint32_t kMaxKeys = DG_MAX_LEVELS * kMaxBins;   // (level, bin) pairs at most: the count sweep keeps one counter each in LDS (128 KB)
constexpr int kBinGrid = 768;                      // persistent binning workgroups (three per compute unit)
constexpr int kAccBlock = 1024, kAccGrid = 256;    // threads of an accumulate workgroup (one per compute unit: its table fills LDS), compute units
// An accumulate workgroup sums at least 2^piece_log2 records of a bin (or all it has) and fewer than twice as many: a bin is
// cut into floor(records / 2^piece_log2) equal pieces, so a bin with less than two pieces' worth stays whole (a second
// workgroup would clear and write out a table of its own for little).  2^17 records where there are plenty; where the bins
// are few and the records too, pieces shrink until some 512 workgroups have one (c1's grid, 33 k samples in three bins of 131 k
// records: 46 -> 17 us).
constexpr int kPieceLog2Min = 13, kPieceLog2Max = 17;
constexpr int kAccMaxLog2 = kPieceLog2Max + 1;
__host__ __device__ __forceinline__ uint32_t acc_pieces(uint32_t total, uint32_t piece_log2) { return total == 0u ? 0u : (total >> piece_log2 ? total >> piece_log2 : 1u); }
constexpr int kCoarseBlock = 1024;                 // coarse prefix: threads per workgroup, persistent workgroups (one per compute unit)
constexpr int kCoarseGrid = 256;

// How a sweep's workgroups share the work: `groups` groups of `width` workgroups; workgroup w of group k takes the tiles w,
// w + width, ... at the levels first_level + k, + groups, ...  One group where there are tiles enough for every workgroup
// (neighbouring appends then meet in L2, level after level); with few tiles several groups go through fewer levels each.
struct Sweep { uint32_t width, groups; };

struct Plan {
    uint32_t first_level;                  // levels below are accumulated directly in LDS
    uint32_t n_keys;                       // (level, bin) pairs of the binned levels
    uint32_t key_base[DG_MAX_LEVELS + 1];  // first key of each level
    uint32_t n_bins[DG_MAX_LEVELS];
    uint32_t max_bins;                     // of a level: rounded up to a multiple of 64, or a power of two where records are compact
    uint32_t compact;                      // 0, or records of an append where records are compact (encode_bwd_compact.hip)
};

// Queues of compact records: lines of 64 bytes, five records and a spare word.
constexpr uint32_t kLineRecords = 5;
constexpr int kCompactTile = 1024;                 // samples that a workgroup takes per step == its threads
constexpr int kCompactGrid = 256;                  // persistent workgroups, one per compute unit: their rings fill LDS
constexpr uint32_t kRingLinesLog2 = 11, kRingLines = 1u << kRingLinesLog2;
constexpr uint64_t kCompactBatch = 1ull << 28;     // samples: their coordinates' offsets stay below 2^32 bytes
inline size_t compact_lds(uint32_t max_bins) { return 64 * kRingLines + (max_bins * 13 + 16 + 15) / 16 * 16; }

void set_compact(Plan &p);                 // p.max_bins: of a level
int reserve_compact();                     // sets the kernels' LDS limits; returns a hipError_t
// the sweeps over samples [n0, n0 + nb)
void count_compact(const dg_grid_desc *d, const Plan &p, const Sweep &sw, const float *u, uint64_t n0, uint64_t nb, uint32_t *rows, hipStream_t st);
void fill_compact(const dg_grid_desc *d, const Plan &p, const Sweep &sw, const float *u, const float *dfeat, uint64_t N, uint64_t n0, uint64_t nb,
                  const uint32_t *rows, uint32_t *binbase, void *queue, float *dtable, hipStream_t st);

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void scan_step(uint32_t &v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, true);
}

// inclusive prefix sum over the wavefront (DPP moves: rows of 16 lanes, then across rows)
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v)
{
    scan_step<0x111, 0xF>(v);
    scan_step<0x112, 0xF>(v);
    scan_step<0x114, 0xF>(v);
    scan_step<0x118, 0xF>(v);
    scan_step<0x142, 0xA>(v);
    scan_step<0x143, 0xC>(v);
    return v;
}

// inclusive running maximum over the wavefront, same moves (a lane that receives nothing takes 0)
__device__ __forceinline__ uint32_t wave_inclusive_max(uint32_t v)
{
#define DG_MAX_STEP(CTRL, ROW_MASK) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, true))
    DG_MAX_STEP(0x111, 0xF); DG_MAX_STEP(0x112, 0xF); DG_MAX_STEP(0x114, 0xF); DG_MAX_STEP(0x118, 0xF);
    DG_MAX_STEP(0x142, 0xA); DG_MAX_STEP(0x143, 0xC);
#undef DG_MAX_STEP
    return v;
}

__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane); }

struct StepAhead {
    float u[3];
    float2 g;
};

__device__ __forceinline__ void load_ahead(StepAhead &a, const float *__restrict__ u, const float2 *__restrict__ dfeat, uint64_t N,
                                           uint64_t n0, uint64_t nb, uint64_t tile, uint32_t l, uint32_t tid)
{
    const uint64_t rel = tile * kTile + tid, n = n0 + (rel < nb ? rel : nb - 1);
    a.u[0] = u[3 * n]; a.u[1] = u[3 * n + 1]; a.u[2] = u[3 * n + 2];
    a.g = dfeat[(size_t)l * N + n];
}

// largest over the workgroup -> *dst (one atomic per workgroup); `word` is an LDS word nobody else uses any more
__device__ __forceinline__ void publish_largest(uint32_t largest, uint32_t *word, uint32_t *__restrict__ dst)
{
    __syncthreads();
    if (threadIdx.x == 0) *word = 0u;
    __syncthreads();
#pragma unroll
    for (int off = dg::kWave / 2; off > 0; off >>= 1) largest = max(largest, (uint32_t)__shfl_xor((int)largest, off, dg::kWave));
    if (threadIdx.x % dg::kWave == 0 && largest) atomicMax(word, largest);
    __syncthreads();
    if (threadIdx.x == 0 && *word) atomicMax(dst, *word);
}

}  // namespace dg_encode_binned
