// What the parts of the table-gradient pass that goes through bins share: bins, plans of a sweep, queue lines.  Internal, not part of the ABI.
#pragma once
#include "encode_common.h"

namespace dg_encode_binned {

using namespace dg_encode;

constexpr int kChunkLog2 = 13;
constexpr uint32_t kChunk = 1u << kChunkLog2;      // entries per bin
constexpr int kMaxBins = 2048;                     // per level: 2^24 entries / 8192
constexpr int kTile = 512;                         // batches are multiples of this many samples
constexpr uint32_t kMaxKeys = DG_MAX_LEVELS * kMaxBins;   // (level, bin) pairs at most: the count sweep keeps one counter each in LDS (128 KB)
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
    uint32_t max_bins;                     // of a level, rounded up to a power of two
    uint32_t compact;                      // compact records
    uint32_t per_unit;                     // workgroups of a sweep per compute unit: 1 or 2
};

// Queues are lines of 64 bytes: four records, or five compact ones and a spare word.  The sweeps that fill them (encode_bwd_fill.hip):
constexpr uint32_t kPairLine = 4, kCompactLine = 5;
constexpr int kFillTile = 1024;                    // samples that a workgroup takes per step == its threads
constexpr int kUnits = 256;                        // compute units, one or two persistent workgroups each, whose rings of lines fill LDS
__host__ __device__ constexpr int ring_lines_log2(int per_unit) { return per_unit == 1 ? 11 : 10; }
inline uint32_t line_records(const Plan &p) { return p.compact ? kCompactLine : kPairLine; }
inline uint32_t append_lines(uint32_t max_bins) { return max_bins <= 512u ? 2u : 1u; }      // lines of an append: two where rings have at least four
inline uint32_t slice_round(const Plan &p) { return line_records(p) * append_lines(p.max_bins); }       // a workgroup's slice of a bin is padded to this many records
// Workgroups per compute unit.  A second one hides barriers and latency, but its rings are half as long and appends of two lines need two of them.
// Merged records, whose arithmetic takes longer than the writes, fill pass in us with one / two: 8 sub-models, T = 2^19 and 2^22, 0.4 M samples each
// 1402 / 1218, 80 k samples, T = 2^19 41.9 / 39.0 (four of 512 threads 49.7).  Compact ones are bound by the writes: T = 2^19, 13.3 M samples 751 / 808.
inline uint32_t per_unit(const Plan &p) { return p.compact || p.max_bins > 512u ? 1u : 2u; }
inline uint32_t fill_grid(const Plan &p) { return kUnits * p.per_unit; }

int reserve_fill();                        // sets the kernels' LDS limits; returns a hipError_t
// the sweeps over samples [n0, n0 + nb)
void count_records(const dg_grid_desc *d, const Plan &p, const Sweep &sw, const float *u, uint64_t n0, uint64_t nb, uint32_t *rows, hipStream_t st);
void fill_queues(const dg_grid_desc *d, const Plan &p, const Sweep &sw, const float *u, const float *dfeat, uint64_t N, uint64_t n0, uint64_t nb,
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

__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane); }

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
