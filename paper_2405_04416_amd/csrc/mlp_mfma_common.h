// Matrix-core building blocks of the field MLPs: operand images, the product, transposes, weight-gradient
// shares.  Internal, not part of the ABI.
//
// Operand and result layouts (lane = 32 h + c, element j / register r):
//   A[row c][k = 8 h + j]     B[k = 8 h + j][col c]     D[row 8 (r / 4) + 4 h + r % 4][col c]
// "Images" are weight tiles pre-arranged in LDS so that one 16-byte read per lane yields an operand.
#pragma once
#include "dg_internal.h"

namespace dg_mlp_mfma {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / 64;

// feature held by slot j of lane half h in k-step ks
__device__ __forceinline__ int feat_tiled(int ks, int h, int j) { return 32 * (ks >> 1) + 8 * (2 * (ks & 1) + (j >> 2)) + 4 * h + (j & 3); }
__device__ __forceinline__ int feat_natural(int ks, int h, int j) { return 16 * ks + 8 * h + j; }

// kind: 0 tiled, 1 natural, 2 colour-net input (k-step 0 tiled geometry, k-step 1 natural direction)
__device__ __forceinline__ int feat_of(int kind, int ks, int h, int j)
{
    if (kind == 0) return feat_tiled(ks, h, j);
    if (kind == 1) return feat_natural(ks, h, j);
    return ks == 0 ? feat_tiled(0, h, j) : feat_natural(1, h, j);
}

// A-operand image of a weight matrix W[n_out][n_in] (row-major): rows = outputs (transpose == false)
// or rows = inputs (transpose == true, for the data gradient).  A thread makes whole operands of 8 halves, whose loads are under way
// together: the images are built once per workgroup, and with few tiles per workgroup the kernels wait for little else.
template <int N_IN, int ROWS_REAL, int K_REAL, int N_MT, int N_KS, int KIND, bool TRANSPOSE>
__device__ __forceinline__ void build_image(__half *img, const __half *__restrict__ W)
{
#pragma unroll
    for (int i = 0; i < (N_MT * N_KS * 64 + kBlock - 1) / kBlock; ++i) {
        const int slot = i * kBlock + threadIdx.x;
        if (N_MT * N_KS * 64 % kBlock != 0 && slot >= N_MT * N_KS * 64) break;
        const int lane = slot & 63, chunk = slot >> 6, ks = chunk % N_KS, mt = chunk / N_KS;
        const int row = 32 * mt + (lane & 31);
        const _Float16 *w = reinterpret_cast<const _Float16 *>(W);
        h8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = feat_of(KIND, ks, lane >> 5, j);
            const bool real = (ROWS_REAL >= 32 * N_MT || row < ROWS_REAL) && (K_REAL >= 16 * N_KS || k < K_REAL);
            v[j] = real ? (TRANSPOSE ? w[k * N_IN + row] : w[row * N_IN + k]) : (_Float16)0.0f;
        }
        reinterpret_cast<h8 *>(img)[slot] = v;
    }
}

__device__ __forceinline__ h8 image(const __half *lds, int chunk, int lane)
{
    return reinterpret_cast<const h8 *>(lds)[chunk * 64 + lane];
}

// Returns its argument, in a way the compiler cannot see through: LDS reads indexed with the result are
// issued where they are used, not hoisted out of the tile loop and held in registers for its whole length.
__device__ __forceinline__ int opaque(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

__device__ __forceinline__ f16v mma(h8 a, h8 b, f16v c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }

__device__ __forceinline__ f16v zero16()
{
    f16v z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.0f;
    return z;
}

__device__ __forceinline__ float fast_sigmoid(float x)
{
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}
// the same with the library's exponential and a rounded division
__device__ __forceinline__ float full_sigmoid(float x) { return 1.0f / (1.0f + expf(-x)); }
__device__ __forceinline__ float clip15(float x) { return fminf(fmaxf(x, -15.0f), 15.0f); }

// max(x, 0) on four pairs of halves, one instruction per pair.  Not in inline assembly: the compiler keeps two wait states between a vector
// instruction and a matrix instruction that reads its result, and does not see one that stands there.
__device__ __forceinline__ h8 relu_pairs(h8 x) { return __builtin_elementwise_max(x, (h8)(_Float16)0.0f); }

// registers 8p .. 8p+7 of a result tile, activated, rounded to fp16 and packed: k-step (m, p) of the next operand
template <int ACT>   // 0 identity, 1 ReLU, 2 sigmoid, 3 sigmoid at full fp32 precision
__device__ __forceinline__ h8 pack_half(const f16v &c, int p)
{
    h8 out;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float v = c[8 * p + j];
        if (ACT == 2) v = fast_sigmoid(v);
        if (ACT == 3) v = full_sigmoid(v);
        out[j] = (_Float16)v;
    }
    // ReLU after the rounding gives the same values as before it (rounding is monotone and keeps 0) and works on pairs
    if (ACT == 1) out = relu_pairs(out);
    // the packed halves are what later uses read: without this the compiler rounds every value a second time, unpacked
    if (ACT >= 2) asm("" : "+v"(out));
    return out;
}

// Transposes of 32-feature tiles through LDS, for the weight gradients, which need the samples on the k axis.  A wavefront writes a tile
// as rows of a sample's features (a lane holds eight of them per k-step, in two stretches of four) and reads columns: the
// transposing read gives a lane four samples of one feature.  What the lane then holds in slot j of sample k-step p is sample
// feat_tiled(p, h, j) of feature lane & 31.  LDS operations of a wavefront stay in order, so a tile's place can be used again at once.
// Rows are 72 bytes apart: writes of 32 samples fall on different banks.
// (Products with 0/1 selection matrices on the matrix cores do the same, 19 of then 73 in the colour kernel, with a result tile to round
// and pack for each: 0.65 M samples, colour and density kernel 65 + 32 us against 64 + 30; 5.1 M with 48 appearance inputs 548 + 228 against
// 530 + 222.  The colour kernel's chain of dependent products and LDS round trips at two wavefronts per SIMD bounds both forms: as
// straight-line code without the branches around its loads and its output layer it is slower, 1050 against 1018 us at 13.3 M samples.)
constexpr int kTileRow = 36, kTileHalves = 32 * kTileRow, kScratchHalves = 2 * kTileHalves;       // two tiles per wavefront

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
enum TileKind { kTiled, kNatural };

// What a lane reads of a tile, other lanes wrote.  The hardware keeps a wavefront's LDS operations in order, but the compiler sees
// only that a lane's own addresses differ: this keeps it from moving LDS accesses of one side to the other.  Emits no instruction.
__device__ __forceinline__ void tile_exchange()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// k-step ks of a packed tensor (its features 16 ks .. 16 ks + 15) into a tile
template <TileKind KIND>
__device__ __forceinline__ void put_step(_Float16 *tile, int lane, int ks, h8 x)
{
    _Float16 *row = tile + (lane & 31) * kTileRow + 16 * ks + (KIND == kTiled ? 4 : 8) * (lane >> 5);
    *reinterpret_cast<h4 *>(row) = __builtin_shufflevector(x, x, 0, 1, 2, 3);
    *reinterpret_cast<h4 *>(row + (KIND == kTiled ? 8 : 4)) = __builtin_shufflevector(x, x, 4, 5, 6, 7);
}

// the two sample k-steps of the transposed tile, whose place can be written again at once
__device__ __forceinline__ void get_transposed(const _Float16 *tile, int lane, h8 out[2])
{
    typedef __fp16 g4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) g4 *lds_g4;
    const int i = lane & 15;
    const _Float16 *at = tile + (4 * (lane >> 5) + (i >> 2)) * kTileRow + (lane & 16) + 4 * (i & 3);
    tile_exchange();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const h4 lo = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_g4)(at + 16 * p * kTileRow)));
        const h4 hi = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_g4)(at + (16 * p + 8) * kTileRow)));
        out[p] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
    tile_exchange();
}

template <TileKind KIND0 = kTiled, TileKind KIND1 = KIND0>
__device__ __forceinline__ void transpose_tile(_Float16 *tile, int lane, h8 x0, h8 x1, h8 out[2])
{
    put_step<KIND0>(tile, lane, 0, x0);
    put_step<KIND1>(tile, lane, 1, x1);
    get_transposed(tile, lane, out);
}
// features 16..31 of the result are whatever the tile held: rows or columns of a weight gradient that nobody reads
template <TileKind KIND = kTiled>
__device__ __forceinline__ void transpose_half_tile(_Float16 *tile, int lane, h8 x0, h8 out[2])
{
    put_step<KIND>(tile, lane, 0, x0);
    get_transposed(tile, lane, out);
}

// delta = fp16(g * act'(a)) for one k-step; a is the packed (rounded) activation
template <int ACT>   // 1 ReLU, 2 sigmoid
__device__ __forceinline__ h8 delta_from(const f16v &g, int p, h8 a)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    h8 out;
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        f2 v;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float av = (float)a[j + k];
            // a (1 - a) as one multiply-add on the halves: 1 - a is exact in fp32 for all but the smallest a, so this rounds the
            // same value once
            v[k] = g[8 * p + j + k] * (ACT == 2 ? __builtin_fmaf(-av, av, av) : (av > 0.0f ? 1.0f : 0.0f));
        }
        const h2 r = __builtin_convertvector(v, h2);
        out[j] = r[0];
        out[j + 1] = r[1];
    }
    return out;
}

// one tile of a wavefront's weight gradient into the workgroup's share in LDS; every word belongs to one lane
__device__ __forceinline__ void add_share(float *share, bool first, int n_in, int rows_real, int cols_real, int ot, int it, int lane, const f16v &acc)
{
    const int h = lane >> 5, i = 32 * it + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int o = 32 * ot + 8 * (r >> 2) + 4 * h + (r & 3);
        if (o < rows_real && i < cols_real) share[o * n_in + i] = first ? acc[r] : share[o * n_in + i] + acc[r];
    }
}

// The wavefronts of a workgroup add their weight gradients up in LDS before the workgroup writes its share: a quarter of the
// shares to write and to fold (fold_shares_kernel 37 -> 8 us).  The gradient comes in four groups of tiles; in turn t
// wavefront w adds group (w + t) % 4, so that all four work at once and every word still gets its addends in a fixed order.
// The space is that of the weight images, which nobody needs any more.
template <int N_WORDS, class Add>
__device__ __forceinline__ void write_share(float *share, float *__restrict__ dst, Add add)
{
    static_assert(kWavesPerBlock == 4, "four wavefronts, four groups");
    const uint32_t w = threadIdx.x >> 6;
    for (uint32_t t = 0; t < 4; ++t) {
        __syncthreads();
        add(share, (w + t) & 3u, t == 0);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < N_WORDS; i += kBlock) dst[i] = share[i];
}

// dW[e] += (sum of the workgroups' shares of element e) / loss_scale, in a fixed order, e < n_total.  Elements below n_first
// come from first_shares [n_a][n_first], the rest from rest_shares [n_b][n_total - n_first]; n_first is n_total or a multiple
// of kFoldElems.  A workgroup serves 64 consecutive elements; 16 groups of threads each sum every 16th share, then the 16
// partial sums are added in a fixed order.
constexpr int kFoldElems = 64, kFoldGroups = 16;
static __global__ void __launch_bounds__(kFoldElems * kFoldGroups)
fold_shares_kernel(const float *__restrict__ first_shares, uint32_t n_a, uint32_t n_first, const float *__restrict__ rest_shares, uint32_t n_b,
                   uint32_t n_total, float inv_scale, float *__restrict__ dW)
{
    __shared__ float part[kFoldGroups][kFoldElems];
    const uint32_t col = threadIdx.x % kFoldElems, group = threadIdx.x / kFoldElems;
    const uint32_t e = blockIdx.x * kFoldElems + col;
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (e < n_total) {
        const bool in_first = e < n_first;
        const float *src = in_first ? first_shares + e : rest_shares + (e - n_first);
        const uint32_t stride = in_first ? n_first : n_total - n_first, n = in_first ? n_a : n_b;
        uint32_t b = group;
        for (; b + 3 * kFoldGroups < n; b += 4 * kFoldGroups) {
#pragma unroll
            for (int k = 0; k < 4; ++k) s[k] += src[(size_t)(b + k * kFoldGroups) * stride];
        }
        for (; b < n; b += kFoldGroups) s[0] += src[(size_t)b * stride];
    }
    part[group][col] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    if (group == 0 && e < n_total) {
        float sum = 0.0f;
#pragma unroll
        for (int k = 0; k < kFoldGroups; ++k) sum += part[k][col];
        dW[e] += sum * inv_scale;
    }
}

// Tiles of 32 samples that a wavefront takes, w, w + n_waves, ..., and where the tile lies in the rows of S samples each.  All of it is
// the same for the whole wavefront and lives in scalar registers: rows are followed instead of divided out, and addresses are a
// scalar base plus a lane's constant offset.
struct TileWalk {
    uint64_t tile, n_tiles, n_waves, n_samples, row, rem, row_step, rem_step;       // row, rem: row of the tile's first sample, and its place in that row
    uint32_t S;

    __device__ __forceinline__ TileWalk(uint64_t N, uint32_t S_) : n_samples(N), S(S_)
    {
        n_tiles = (N + 31) / 32;
        n_waves = (uint64_t)gridDim.x * kWavesPerBlock;
        tile = (uint64_t)blockIdx.x * kWavesPerBlock + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        row = tile * 32 / S;
        rem = tile * 32 - row * S;
        row_step = n_waves * 32 / S;
        rem_step = n_waves * 32 - row_step * S;
    }
    __device__ __forceinline__ bool more() const { return tile < n_tiles; }
    __device__ __forceinline__ void next()
    {
        tile += n_waves;
        row += row_step;
        rem += rem_step;
        if (rem >= S) { rem -= S; ++row; }
    }
    // samples of the tile
    __device__ __forceinline__ uint32_t count() const { return n_samples - tile * 32 < 32 ? (uint32_t)(n_samples - tile * 32) : 32u; }
    // row of sample s of the tile (s < 32), counted from `row`: rows of 32 or more samples change at most once; shorter ones:
    // integers below 63 divided through a float reciprocal, which the slack of 1e-3 makes exact
    __device__ __forceinline__ uint32_t local_row(uint32_t s) const
    {
        if (S >= 32) return s >= S - rem ? 1u : 0u;
        return (uint32_t)((float)((uint32_t)rem + s) * (1.0f / (float)S) + 1e-3f);
    }
};

inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace dg_mlp_mfma
