// Field MLPs on the matrix cores (v_mfma_f32_32x32x16_f16) for the 32 -> 64 -> 16 density net and
// the (16 + 16) -> 64 -> 64 -> 3 colour net (Sec. 3.2; activations and output clip of Sec. 5.1).
//
// One wavefront owns a tile of 32 samples and keeps every activation of the tile in registers.
// Layers are evaluated transposed, out^T = W . in^T: the weight matrix is the A operand (rows = output
// features), the activations are the B operand (columns = samples).  The result tile then has the
// sample on the lane and the features on the registers, which is again a B operand for the next
// layer once the registers are rounded to fp16 and packed -- the feature order this produces is
// baked into the weight images, so layers chain with no data movement.
//
// Operand layouts, images, transposes: mlp_mfma_common.h.
//
// What the kernels spend on a tile (13.3 M samples): forward 394 vector instructions of which 135 are transcendental and take two issue
// slots; the vector units are busy 0.84 of the time, the matrix cores 0.30.  Colour backward: busy 0.60 and 0.33, with little overlap
// at two wavefronts per SIMD, so it goes by the number of instructions: a compile-time choice of the activation (branches around each
// of its uses cut the schedule into pieces), a (1 - a) as one multiply-add on halves, rows followed on the scalar unit instead of
// divided out and images built from loads under way together took it from 1206 to 1050 us (0.65 M samples: 79 -> 65; 0.15 M: 35 -> 26),
// transposes through LDS instead of products with selection matrices to 1020; the forward went from 482 to 470 (40 -> 33; 17 -> 16).
//
// Backward recomputes the forward, then walks the chain back.  Weight gradients contract over the
// samples, so they need each (delta, activation) pair with the samples on the k axis: tiles are transposed through LDS.  Every
// wavefront accumulates its share of dW in registers over all its tiles; the workgroup adds its wavefronts' shares up, writes the
// sum to the workspace once, and a second kernel folds the workgroups' in a fixed order.
//
// Appearance features (Sec. 4.4.3: a fixed per-image vector of 16 or 48 values as extra colour-net inputs) widen the
// first colour layer to 48 or 80 inputs.  Forward: NA / 16 more k-steps from a second row table.  Backward: the
// features are constant along a row of samples, so the gradient of their weight columns is
// sum_rows (sum of delta over the row's samples) x (row's features): the per-row delta sums come from one more
// matrix-core product of the transposed delta tile with a 0/1 sample-to-row matrix and are added into a [rows, 64]
// buffer; a small kernel contracts that buffer with the feature rows.  No accumulator registers are added.
#include "mlp_mfma_common.h"
#include <type_traits>

namespace dg_mlp_mfma {

using dg::FeatureLayout;
using dg::kPlanes;
using dg::kRows;
using dg::kSplit;
using dg::kSplitLevels;

constexpr int NF = 32, HD = 64, NG = 16, ND = 16, HC = 64, CI = NG + ND;
constexpr int oWd1 = 0, oWd2 = oWd1 + HD * NF, oWc1 = oWd2 + NG * HD, oWc2 = oWc1 + HC * CI, oWc3 = oWc2 + HC * HC;
constexpr int kTotal = oWc3 + 3 * HC;

// image chunks (1 KB each: 64 lanes x 8 halves)
constexpr int cD1 = 0, cD2 = 4, cC1 = 8, cC2 = 12, cC3 = 20, kFwdChunks = 24;
constexpr int cC3T = 24, cC2T = 26, cC1T = 34, kAllChunks = 38;

__device__ void build_forward_images(__half *lds, const __half *w)
{
    build_image<NF, HD, NF, 2, 2, 1, false>(lds + cD1 * 512, w + oWd1);
    build_image<HD, NG, HD, 1, 4, 0, false>(lds + cD2 * 512, w + oWd2);
    build_image<CI, HC, CI, 2, 2, 2, false>(lds + cC1 * 512, w + oWc1);
    build_image<HC, HC, HC, 2, 4, 0, false>(lds + cC2 * 512, w + oWc2);
    build_image<HC, 3, HC, 1, 4, 0, false>(lds + cC3 * 512, w + oWc3);
}

__device__ void build_backward_images(__half *lds, const __half *w)
{
    build_image<HC, HC, 3, 2, 1, 0, true>(lds + cC3T * 512, w + oWc3);
    build_image<HC, HC, HC, 2, 4, 0, true>(lds + cC2T * 512, w + oWc2);
    build_image<CI, NG, HC, 1, 4, 0, true>(lds + cC1T * 512, w + oWc1);     // direction inputs get no gradient
}

struct Tile {
    h8 x0[2], h1[4], xc[2], xa[3], c1[4], c2[4];      // xa: appearance inputs (unused without them)
    float geo0, sigma, raw[3], rgb[3];     // meaningful on lanes with h == 0
};

// NA: appearance inputs (0, 16 or 48); their weight images start at chunk c_app.  SIG: the colour net's hidden layers are sigmoids
// (else ReLU); a compile-time choice, because a branch around every activation keeps the scheduler from filling the matrix
// instructions' latency with it.
template <int NA, bool SIG>
__device__ __forceinline__ void forward_tile(const __half *lds, int lane, Tile &t, int c_app = 0)
{
    f16v acc[2];
    // density layer 1: 32 -> 64, ReLU
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        acc[mt] = zero16();
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) acc[mt] = mma(image(lds, cD1 + mt * 2 + ks, lane), t.x0[ks], acc[mt]);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) t.h1[ks] = pack_half<1>(acc[ks >> 1], ks & 1);
    // density layer 2: 64 -> 16, raw
    f16v geo = zero16();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) geo = mma(image(lds, cD2 + ks, lane), t.h1[ks], geo);
    t.geo0 = geo[0];
    t.sigma = __expf(clip15(geo[0]));
    t.xc[0] = pack_half<0>(geo, 0);
    // colour layer 1: (16 + 16) -> 64
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        acc[mt] = zero16();
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) acc[mt] = mma(image(lds, cC1 + mt * 2 + ks, lane), t.xc[ks], acc[mt]);
#pragma unroll
        for (int ks = 0; ks < NA / 16; ++ks) acc[mt] = mma(image(lds, c_app + mt * (NA / 16) + ks, lane), t.xa[ks], acc[mt]);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) t.c1[ks] = pack_half<SIG ? 2 : 1>(acc[ks >> 1], ks & 1);
    // colour layer 2: 64 -> 64
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        acc[mt] = zero16();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) acc[mt] = mma(image(lds, cC2 + mt * 4 + ks, lane), t.c1[ks], acc[mt]);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) t.c2[ks] = pack_half<SIG ? 2 : 1>(acc[ks >> 1], ks & 1);
    // colour layer 3: 64 -> 3, raw
    f16v out = zero16();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) out = mma(image(lds, cC3 + ks, lane), t.c2[ks], out);
#pragma unroll
    for (int c = 0; c < 3; ++c) { t.raw[c] = out[c]; t.rgb[c] = fast_sigmoid(clip15(out[c])); }
}

// the density net's first output, before its activation (lanes with h == 0); same arithmetic as in forward_tile
__device__ __forceinline__ float density_net(const __half *lds, int lane, const h8 (&x0)[2])
{
    f16v acc[2], geo = zero16();
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        acc[mt] = zero16();
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) acc[mt] = mma(image(lds, cD1 + mt * 2 + ks, lane), x0[ks], acc[mt]);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) geo = mma(image(lds, cD2 + ks, lane), pack_half<1>(acc[ks >> 1], ks & 1), geo);
    return geo[0];
}

// Features arrive as level-major planes [16][n_samples] of half2 -- slot j of k-step ks on lane half h is feature
// 16 ks + 8 h + j, i.e. component j % 2 of level 8 ks + 4 h + j / 2 -- as rows of 32 halves, or as rows of 24 halves and the planes of levels 12..15.
// base: first sample of a tile or segment, the same for the whole wavefront; s: the lane's sample from there.
template <FeatureLayout LAYOUT>
__device__ __forceinline__ void load_features(const __half *feat, uint64_t n_samples, uint64_t base, uint32_t s, int h, h8 x0[2])
{
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    const uint32_t *words = reinterpret_cast<const uint32_t *>(feat);
    if (LAYOUT == kRows) {
        const h8 *row = reinterpret_cast<const h8 *>(feat) + 4 * base;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) x0[ks] = row[4 * s + 2 * ks + h];
    } else if (LAYOUT == kPlanes) {
        const uint32_t *planes = words + (size_t)(4 * h) * n_samples + s;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            u4 bits;
#pragma unroll
            for (int q = 0; q < 4; ++q) bits[q] = planes[(size_t)(8 * ks + q) * n_samples + base];
            x0[ks] = __builtin_bit_cast(h8, bits);
        }
    } else {
        static_assert(kSplitLevels == 12, "a row is three operands, the fourth comes from planes");
        const h8 *row = reinterpret_cast<const h8 *>(feat) + 3 * base;
        x0[0] = row[3 * s + h];
        if (h == 0) {
            x0[1] = row[3 * s + 2];
        } else {
            const uint32_t *planes = words + base;
            u4 bits;
#pragma unroll
            for (int q = 0; q < 4; ++q) bits[q] = (planes + (size_t)(12 + q) * n_samples)[s];
            x0[1] = __builtin_bit_cast(h8, bits);
        }
    }
}

// row: of the sample at base, r: the lane's row from there
template <int NA, FeatureLayout LAYOUT>
__device__ __forceinline__ void load_inputs(const __half *feat, const __half *dir_enc, const __half *app, uint64_t n_samples, uint64_t base, uint32_t s,
                                            uint64_t row, uint32_t r, int h, Tile &t)
{
    load_features<LAYOUT>(feat, n_samples, base, s, h, t.x0);
    t.xc[1] = reinterpret_cast<const h8 *>(dir_enc + row * ND)[2 * r + h];
#pragma unroll
    for (int ks = 0; ks < NA / 16; ++ks) t.xa[ks] = reinterpret_cast<const h8 *>(app + row * NA)[NA / 8 * r + 2 * ks + h];
}

// Inputs of the walk's tile.  Lanes past the last sample read it again: no branch, and what they compute is not stored and gets no
// gradient.  (Asked for a tile ahead: no gain at five wavefronts per SIMD forward, spills at two backward.)
template <int NA, FeatureLayout LAYOUT>
__device__ __forceinline__ void load_tile(const __half *feat, const __half *dir_enc, const __half *app, const TileWalk &walk, int lane, Tile &t)
{
    const uint32_t s = min((uint32_t)lane & 31u, walk.count() - 1u);
    load_inputs<NA, LAYOUT>(feat, dir_enc, app, walk.n_samples, walk.tile * 32, s, walk.row, walk.local_row(s), lane >> 5, t);
}

template <int NA, FeatureLayout LAYOUT, bool SIG>
__global__ void __launch_bounds__(kBlock, 4)
fwd_kernel(const __half *__restrict__ weights, const __half *__restrict__ feat, const __half *__restrict__ dir_enc,
           const __half *__restrict__ app, uint32_t S, uint64_t n_samples, float *__restrict__ sigma, float *__restrict__ rgb)
{
    __shared__ __attribute__((aligned(16))) __half lds[(kFwdChunks + 2 * (NA / 16)) * 512];
    build_forward_images(lds, weights);
    if constexpr (NA > 0) build_image<NA, HC, NA, 2, NA / 16, 1, false>(lds + kFwdChunks * 512, weights + kTotal);
    __syncthreads();
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const uint32_t s = lane & 31;
    for (TileWalk walk(n_samples, S); walk.more(); walk.next()) {
        const uint64_t base = walk.tile * 32;
        const bool valid = s < walk.count();
        Tile t;
        load_tile<NA, LAYOUT>(feat, dir_enc, app, walk, lane, t);
        forward_tile<NA, SIG>(lds, opaque(lane), t, kFwdChunks);
        if (valid && h == 0) {
            (sigma + base)[s] = t.sigma;
            float *c = rgb + 3 * base;
            c[3 * s] = t.rgb[0]; c[3 * s + 1] = t.rgb[1]; c[3 * s + 2] = t.rgb[2];
        }
    }
}

// ---------------------------------------------------------------------------------------- densities of grid cells
// Refresh of the occupancy grid: the density net alone, its output straight into the grid.  Densities are > 0 -- the clip before the
// exponential turns a NaN of the network into -15 --, so their bit patterns order like unsigned integers and the maximum is one
// integer atomic.
// Bound by the rows it reads and the atomics' cache lines.  8.4 M candidates, 16.8 M cells: whole networks and a separate maximum
// 304 + 323 us, this kernel on candidates in spatial order 215 us (neighbours' cells then share lines).
template <FeatureLayout LAYOUT>
__global__ void __launch_bounds__(kBlock, 8)
density_max_kernel(const __half *__restrict__ weights, const __half *__restrict__ feat, const uint32_t *__restrict__ cell, uint32_t cell_stride,
                   uint64_t n_samples, float *__restrict__ density, uint32_t n_cells)
{
    __shared__ __attribute__((aligned(16))) __half lds[cC1 * 512];
    build_image<NF, HD, NF, 2, 2, 1, false>(lds + cD1 * 512, weights + oWd1);
    build_image<HD, NG, HD, 1, 4, 0, false>(lds + cD2 * 512, weights + oWd2);
    __syncthreads();
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const uint64_t n_tiles = (n_samples + 31) / 32;
    const uint64_t wave = (uint64_t)blockIdx.x * kWavesPerBlock + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t n_waves = (uint64_t)gridDim.x * kWavesPerBlock;
    for (uint64_t tile = wave; tile < n_tiles; tile += n_waves) {
        const uint64_t n = tile * 32 + (lane & 31), nn = n < n_samples ? n : n_samples - 1;
        h8 x0[2];
        load_features<LAYOUT>(feat, n_samples, tile * 32, (uint32_t)(nn - tile * 32), h, x0);
        const uint32_t c = cell[nn * cell_stride];
        const float sigma = __expf(clip15(density_net(lds, opaque(lane), x0)));
        if (h == 0 && n < n_samples && c < n_cells) atomicMax(reinterpret_cast<unsigned int *>(density) + c, __float_as_uint(sigma));
    }
}

// ---------------------------------------------------------------------------------------- evaluation rendering, fused
// Forward-only rendering (Sec. 4.4.2: every sub-model renders its segments, the partial colour, depth and transmittance
// are merged afterwards): the field networks and the local volume rendering (Eq. 3) of one segment in one wavefront.
// A segment of S <= 64 samples is two tiles of the forward above (samples 0..31 and 32..S-1); their densities and
// colours end up on lanes 0..31, the second tile's are moved to lanes 32..63, and the front-to-back product over the
// 64 lanes is a prefix scan -- sigma and rgb never leave the registers.  The arithmetic of the scan is that of the
// separate compositing kernels (alpha from expm1, transmittance as a running product of exp(-sigma delta)).
__device__ __forceinline__ float wave_inclusive_product(float v, int lane)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float up = __shfl_up(v, off, 64);
        if (lane >= off) v *= up;
    }
    return v;
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int NA, FeatureLayout LAYOUT, bool SIG>
__global__ void __launch_bounds__(kBlock, 4)
render_fwd_kernel(const __half *__restrict__ weights, const __half *__restrict__ feat, const __half *__restrict__ dir_enc,
                  const __half *__restrict__ app, uint32_t S, uint32_t n_seg, const float *__restrict__ delta,
                  const float *__restrict__ t_samples, const uint32_t *__restrict__ seg_ray, const uint32_t *__restrict__ seg_slot,
                  uint32_t k_max, float *__restrict__ Ck, float *__restrict__ Tk, float *__restrict__ Dk)
{
    __shared__ __attribute__((aligned(16))) __half lds[(kFwdChunks + 2 * (NA / 16)) * 512];
    build_forward_images(lds, weights);
    if constexpr (NA > 0) build_image<NA, HC, NA, 2, NA / 16, 1, false>(lds + kFwdChunks * 512, weights + kTotal);
    __syncthreads();
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const uint64_t n_samples = (uint64_t)n_seg * S;
    const uint32_t wave = blockIdx.x * kWavesPerBlock + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), n_waves = gridDim.x * kWavesPerBlock;
    for (uint32_t seg = wave; seg < n_seg; seg += n_waves) {
        const uint64_t first = (uint64_t)seg * S;
        float sig[2], col[2][3];
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            const uint32_t s = 32u * part + (lane & 31);
            const bool valid = s < S;
            Tile t;
            load_inputs<NA, LAYOUT>(feat, dir_enc, app, n_samples, first, valid ? s : 0u, seg, 0u, h, t);
            forward_tile<NA, SIG>(lds, opaque(lane), t, kFwdChunks);
            sig[part] = t.sigma;
            col[part][0] = t.rgb[0]; col[part][1] = t.rgb[1]; col[part][2] = t.rgb[2];
        }
        // sample `lane` of the segment: first tile on lanes 0..31 as it stands, second tile fetched from lanes 0..31
        // (every lane takes part in the exchange; the choice comes afterwards: a lane must not read from lanes that a
        // branch has switched off)
        const float s_up = __shfl(sig[1], lane & 31, 64), a_up = __shfl(col[1][0], lane & 31, 64);
        const float b_up = __shfl(col[1][1], lane & 31, 64), c_up = __shfl(col[1][2], lane & 31, 64);
        const float sigma_s = h ? s_up : sig[0], r0 = h ? a_up : col[0][0], r1 = h ? b_up : col[0][1], r2 = h ? c_up : col[0][2];
        const bool live = (uint32_t)lane < S;
        const uint64_t n = first + (live ? lane : 0);
        const float x = live ? sigma_s * delta[n] : 0.0f;
        const float incl = wave_inclusive_product(expf(-x), lane);
        float before = __shfl_up(incl, 1, 64);
        if (lane == 0) before = 1.0f;
        const float wgt = live ? before * -expm1f(-x) : 0.0f;
        const float c0 = wave_sum(wgt * r0), c1 = wave_sum(wgt * r1), c2 = wave_sum(wgt * r2);
        const float depth = t_samples ? wave_sum(live ? wgt * t_samples[n] : 0.0f) : 0.0f;
        const float trans = __shfl(incl, 63, 64);
        if (lane == 0) {
            const size_t dst = (size_t)seg_ray[seg] * k_max + seg_slot[seg];
            Ck[3 * dst] = c0; Ck[3 * dst + 1] = c1; Ck[3 * dst + 2] = c2;
            Tk[dst] = trans;
            if (Dk) Dk[dst] = depth;
        }
    }
}

// ---------------------------------------------------------------------------------------- backward

// The backward pass runs as two kernels so that neither has to hold all twelve dW tiles (192
// accumulator registers) next to the activations:
//   colour_bwd : recomputes the whole forward, back-propagates the colour net, accumulates dWc1..3
//                (8 tiles = 128 registers; the weight images are re-read from LDS tile by tile so that
//                the rest fits the 256 registers of two wavefronts per SIMD, which keeps every MFMA
//                result in ordinary registers) and leaves delta_geo (gradient of the 16 density outputs, sigma term included,
//                already scaled and rounded to fp16, in operand order) in the workspace;
//   density_bwd: recomputes the density hidden layer, back-propagates it from delta_geo, accumulates
//                dWd1..2 and writes the feature gradient planes.
template <int NA, FeatureLayout LAYOUT, bool SIG>
__global__ void __launch_bounds__(kBlock, 2)
colour_bwd_kernel(const __half *__restrict__ weights, const __half *__restrict__ feat, const __half *__restrict__ dir_enc,
                  const __half *__restrict__ app, uint32_t S, uint64_t n_samples,
                  const float *__restrict__ dsigma, const float *__restrict__ drgb, float loss_scale, h8 *__restrict__ dgeo,
                  float *__restrict__ shares, float *__restrict__ row_delta)
{
    __shared__ __attribute__((aligned(16))) __half lds[(kAllChunks + 2 * (NA / 16)) * 512];
    __shared__ float acc3[kWavesPerBlock * 2 * 3 * 32];
    __shared__ __attribute__((aligned(16))) _Float16 scratch[kWavesPerBlock * kScratchHalves];
    build_forward_images(lds, weights);
    build_backward_images(lds, weights);
    if constexpr (NA > 0) build_image<NA, HC, NA, 2, NA / 16, 1, false>(lds + kAllChunks * 512, weights + kTotal);
    __syncthreads();
    const int lane_fixed = threadIdx.x & 63, h = lane_fixed >> 5;
    const h8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};

    f16v gWc2[2][2], gWc1[2];               // [output tile][input tile]
#pragma unroll
    for (int a = 0; a < 2; ++a) { gWc1[a] = zero16(); gWc2[a][0] = zero16(); gWc2[a][1] = zero16(); }
    // The output layer has 3 rows: its gradient tiles are 3 real rows of 32, too little to deserve 32 accumulator
    // registers next to the others.  Each wavefront keeps those 3 x 64 sums in LDS words of its own (one owner lane
    // per word, plain read-add-write, so the order of the additions is fixed).
    float *gWc3 = acc3 + (threadIdx.x >> 6) * (2 * 3 * 32);      // [input tile][row][column]
    _Float16 *const tile0 = scratch + (threadIdx.x >> 6) * kScratchHalves, *const tile1 = tile0 + kTileHalves;
    if (h == 0) {
#pragma unroll
        for (int k = 0; k < 6; ++k) gWc3[k * 32 + (lane_fixed & 31)] = 0.0f;
    }

    const uint32_t s = lane_fixed & 31;
    for (TileWalk walk(n_samples, S); walk.more(); walk.next()) {
        const uint64_t base = walk.tile * 32;
        const bool valid = s < walk.count();
        const int lane = opaque(lane_fixed);
        Tile t;
        load_tile<NA, LAYOUT>(feat, dir_enc, app, walk, lane_fixed, t);
        float ds = 0.0f, dc[3] = {0.0f, 0.0f, 0.0f};
        if (valid && h == 0) {                 // issued before the forward so the latency hides behind it
            const float *c = drgb + 3 * base;
            ds = (dsigma + base)[s];
            dc[0] = c[3 * s]; dc[1] = c[3 * s + 1]; dc[2] = c[3 * s + 2];
        }
        forward_tile<NA, SIG>(lds, lane, t, kAllChunks);

        // ---- output layer of the colour net
        h8 d3 = zero8;
        if (valid && h == 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const bool pass = t.raw[c] >= -15.0f && t.raw[c] <= 15.0f;
                d3[c] = (_Float16)(pass ? loss_scale * dc[c] * t.rgb[c] * (1.0f - t.rgb[c]) : 0.0f);
            }
        }
        h8 td[2][2], ta[2][2];      // transposed delta / activation: [feature tile][sample k-step]
        transpose_half_tile(tile0, lane, d3, td[0]);
        transpose_tile(tile1, lane, t.c2[0], t.c2[1], ta[0]);
        transpose_tile(tile0, lane, t.c2[2], t.c2[3], ta[1]);
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            f16v part = mma(td[0][0], ta[it][0], zero16());
            part = mma(td[0][1], ta[it][1], part);
            if (h == 0) {                  // rows 0..2 of the tile are registers 0..2 of the lower half's lanes
#pragma unroll
                for (int o = 0; o < 3; ++o) gWc3[(it * 3 + o) * 32 + (lane_fixed & 31)] += part[o];
            }
        }
        f16v g[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) g[mt] = mma(image(lds, cC3T + mt, lane), d3, zero16());

        // ---- second hidden layer of the colour net
        h8 dl[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) dl[ks] = delta_from<SIG ? 2 : 1>(g[ks >> 1], ks & 1, t.c2[ks]);
        transpose_tile(tile0, lane, t.c1[0], t.c1[1], ta[0]);
        transpose_tile(tile1, lane, t.c1[2], t.c1[3], ta[1]);
        transpose_tile(tile0, lane, dl[0], dl[1], td[0]);
        transpose_tile(tile1, lane, dl[2], dl[3], td[1]);
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
            for (int it = 0; it < 2; ++it)
#pragma unroll
                for (int p = 0; p < 2; ++p) gWc2[ot][it] = mma(td[ot][p], ta[it][p], gWc2[ot][it]);
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            g[mt] = zero16();
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) g[mt] = mma(image(lds, cC2T + mt * 4 + ks, lane), dl[ks], g[mt]);
        }

        // ---- first hidden layer of the colour net
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) dl[ks] = delta_from<SIG ? 2 : 1>(g[ks >> 1], ks & 1, t.c1[ks]);
        transpose_tile<kTiled, kNatural>(tile0, lane, t.xc[0], t.xc[1], ta[0]);
        transpose_tile(tile1, lane, dl[0], dl[1], td[0]);
        transpose_tile(tile0, lane, dl[2], dl[3], td[1]);
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
            for (int p = 0; p < 2; ++p) gWc1[ot] = mma(td[ot][p], ta[0][p], gWc1[ot]);
        if (NA > 0) {
            // per-row sums of delta for the appearance columns: delta^T (features x samples) times the 0/1 matrix
            // "sample s lies in the tile's local row c"; column c of the result is the sum over that row's samples
            const uint32_t c = s, n_local = walk.local_row(walk.count() - 1u) + 1u;   // rows with samples in this tile
            h8 in_row[2];
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int j = 0; j < 8; ++j)      // slot j of k-step p holds sample feat_tiled(p, h, j) of the tile, as in td
                    in_row[p][j] = (_Float16)(walk.local_row((uint32_t)feat_tiled(p, h, j)) == c ? 1.0f : 0.0f);
#pragma unroll
            for (int ot = 0; ot < 2; ++ot) {
                f16v sums = mma(td[ot][0], in_row[0], zero16());
                sums = mma(td[ot][1], in_row[1], sums);
                if (c < n_local) {
                    float *dst = row_delta + (walk.row + c) * HC + 32 * ot + 4 * h;
#pragma unroll
                    for (int r = 0; r < 16; ++r) unsafeAtomicAdd(dst + 8 * (r >> 2) + (r & 3), sums[r]);
                }
            }
        }
        f16v gx = zero16();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) gx = mma(image(lds, cC1T + ks, lane), dl[ks], gx);

        // ---- density net output: geometry features feed the colour net, output 0 also feeds exp()
        if (valid && h == 0) {
            const bool pass0 = t.geo0 >= -15.0f && t.geo0 <= 15.0f;
            gx[0] += pass0 ? loss_scale * ds * t.sigma : 0.0f;
        }
        if (valid) (dgeo + 2 * base)[2 * s + h] = pack_half<0>(gx, 0);
    }

    static_assert((kTotal - oWc1) * 4 <= kAllChunks * 1024, "the share fits the space of the images");
    write_share<kTotal - oWc1>(reinterpret_cast<float *>(lds), shares + (size_t)blockIdx.x * (kTotal - oWc1), [&](float *share, uint32_t group, bool first) {
        const int lane = lane_fixed;
        share -= oWc1;                                          // colour shares hold elements [oWc1, kTotal)
        if (group < 2) {
#pragma unroll
            for (uint32_t ot = 0; ot < 2; ++ot)
                if (group == ot) {
                    add_share(share + oWc2, first, HC, HC, HC, ot, 0, lane, gWc2[ot][0]);
                    add_share(share + oWc2, first, HC, HC, HC, ot, 1, lane, gWc2[ot][1]);
                }
        } else if (group == 2) {
#pragma unroll
            for (int ot = 0; ot < 2; ++ot) add_share(share + oWc1, first, CI, HC, CI, ot, 0, lane, gWc1[ot]);
        } else if (h == 0) {
#pragma unroll
            for (int it = 0; it < 2; ++it)
#pragma unroll
                for (int o = 0; o < 3; ++o) {
                    float *at = share + oWc3 + o * HC + 32 * it + (lane & 31);
                    const float v = gWc3[(it * 3 + o) * 32 + (lane & 31)];
                    *at = first ? v : *at + v;
                }
        }
    });
}

// Other than with planes, the gradient of levels [0, n_merged) goes into rows of 2 n_merged floats, that of the others into planes behind them
template <FeatureLayout LAYOUT>
__global__ void __launch_bounds__(kBlock, 2)
density_bwd_kernel(const __half *__restrict__ weights, const __half *__restrict__ feat, uint64_t n_samples,
                   const h8 *__restrict__ dgeo, float loss_scale, uint32_t n_merged, float *__restrict__ dfeat, uint32_t *__restrict__ largest,
                   float *__restrict__ shares)
{
    // images: density layer 1 forward (4 chunks), Wd2^T (2), Wd1^T (4); the share of the weight gradient takes their place
    constexpr bool kGradRows = LAYOUT != kPlanes;
    constexpr int kD1 = 0, kD2T = 4, kD1T = 6, kChunks = 12;
    __shared__ __attribute__((aligned(16))) __half lds[kChunks * 512];
    __shared__ __attribute__((aligned(16))) _Float16 scratch[kWavesPerBlock * kScratchHalves];
    build_image<NF, HD, NF, 2, 2, 1, false>(lds + kD1 * 512, weights + oWd1);
    build_image<HD, HD, NG, 2, 1, 0, true>(lds + kD2T * 512, weights + oWd2);
    build_image<NF, NF, HD, 1, 4, 0, true>(lds + kD1T * 512, weights + oWd1);
    __syncthreads();
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const uint64_t n_tiles = (n_samples + 31) / 32;
    const uint64_t wave = (uint64_t)blockIdx.x * kWavesPerBlock + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t n_waves = (uint64_t)gridDim.x * kWavesPerBlock;
    const float inv_scale = 1.0f / loss_scale;
    _Float16 *const tile0 = scratch + (threadIdx.x >> 6) * kScratchHalves, *const tile1 = tile0 + kTileHalves;
    const h8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};

    float most = 0.0f;                                          // largest magnitude of the feature gradient, before the division by the loss scale
    f16v gWd2[2], gWd1[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) { gWd2[a] = zero16(); gWd1[a] = zero16(); }

    h8 x_next[2], dg_next;
    auto load = [&](uint64_t tile) {            // lanes past the last sample read it again; their gradient is set to zero below
        const uint64_t base = tile * 32, left = n_samples - base;
        const uint32_t s = min((uint32_t)lane & 31u, left < 32 ? (uint32_t)left - 1u : 31u);
        load_features<LAYOUT>(feat, n_samples, base, s, h, x_next);
        dg_next = (dgeo + 2 * base)[2 * s + h];
    };
    if (wave < n_tiles) load(wave);
    for (uint64_t tile = wave; tile < n_tiles; tile += n_waves) {
        const uint64_t n = tile * 32 + (lane & 31);
        const bool valid = n < n_samples;
        Tile t;
        t.x0[0] = x_next[0]; t.x0[1] = x_next[1];
        const h8 dg = valid ? dg_next : zero8;
        if (tile + n_waves < n_tiles) load(tile + n_waves);         // a tile ahead
        f16v acc[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            acc[mt] = zero16();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) acc[mt] = mma(image(lds, kD1 + mt * 2 + ks, lane), t.x0[ks], acc[mt]);
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) t.h1[ks] = pack_half<1>(acc[ks >> 1], ks & 1);

        h8 td[2][2], ta[2][2];
        transpose_half_tile(tile0, lane, dg, td[0]);
        transpose_tile(tile1, lane, t.h1[0], t.h1[1], ta[0]);
        transpose_tile(tile0, lane, t.h1[2], t.h1[3], ta[1]);
#pragma unroll
        for (int it = 0; it < 2; ++it)
#pragma unroll
            for (int p = 0; p < 2; ++p) gWd2[it] = mma(td[0][p], ta[it][p], gWd2[it]);
        f16v g[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) g[mt] = mma(image(lds, kD2T + mt, lane), dg, zero16());

        h8 dl[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) dl[ks] = delta_from<1>(g[ks >> 1], ks & 1, t.h1[ks]);
        transpose_tile<kNatural>(tile1, lane, t.x0[0], t.x0[1], ta[0]);
        transpose_tile(tile0, lane, dl[0], dl[1], td[0]);
        transpose_tile(tile1, lane, dl[2], dl[3], td[1]);
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
            for (int p = 0; p < 2; ++p) gWd1[ot] = mma(td[ot][p], ta[0][p], gWd1[ot]);
        f16v gf = zero16();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) gf = mma(image(lds, kD1T + ks, lane), dl[ks], gf);
        if (kGradRows && valid) {
            bool nan = false;                                   // fmaxf passes over NaN
#pragma unroll
            for (int k = 0; k < 16; ++k) { most = fmaxf(most, fabsf(gf[k])); nan |= gf[k] != gf[k]; }
            if (nan) most = INFINITY;
        }
        if (valid) {
            // registers 4q .. 4q+3 hold features 8q + 4h .. + 3: levels 4q + 2h and 4q + 2h + 1 of the planes [16][n_samples][2]
            float2 *planes = reinterpret_cast<float2 *>(dfeat);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (kGradRows && 4u * q + 2u * h < n_merged) {          // n_merged is even: a lane's two levels go the same way
                    reinterpret_cast<float4 *>(dfeat)[n * (n_merged / 2) + 2 * q + h] =
                        make_float4(gf[4 * q] * inv_scale, gf[4 * q + 1] * inv_scale, gf[4 * q + 2] * inv_scale, gf[4 * q + 3] * inv_scale);
                    continue;
                }
                planes[(size_t)(4 * q + 2 * h) * n_samples + n] = make_float2(gf[4 * q] * inv_scale, gf[4 * q + 1] * inv_scale);
                planes[(size_t)(4 * q + 2 * h + 1) * n_samples + n] = make_float2(gf[4 * q + 2] * inv_scale, gf[4 * q + 3] * inv_scale);
            }
        }
    }

    if (kGradRows) {
        // one atomic per workgroup at most: same-address atomics take turns (one per wavefront cost 15 us)
        __shared__ uint32_t most_word;
        if (threadIdx.x == 0) most_word = 0u;
        __syncthreads();
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) most = fmaxf(most, __shfl_xor(most, off, 64));
        if (lane == 0) atomicMax(&most_word, __float_as_uint(most * inv_scale));      // bit patterns of values >= 0 order like the values
        __syncthreads();
        if (threadIdx.x == 0 && most_word > __hip_atomic_load(largest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(largest, most_word);
    }
    static_assert(oWc1 * 4 <= kChunks * 1024, "the share fits the space of the images");
    write_share<oWc1>(reinterpret_cast<float *>(lds), shares + (size_t)blockIdx.x * oWc1, [&](float *share, uint32_t group, bool first) {
#pragma unroll
        for (uint32_t t = 0; t < 2; ++t) {
            if (group == t) add_share(share + oWd1, first, NF, HD, NF, t, 0, lane, gWd1[t]);
            if (group == 2 + t) add_share(share + oWd2, first, HD, NG, HD, 0, t, lane, gWd2[t]);
        }
    });
}

// dW[kTotal + o * NA + a] += inv_scale * sum_rows row_delta[row][o] * app[row][a].  A workgroup of four row groups
// walks rows with a grid stride, eight rows in flight per thread (independent loads); thread (o, quarter q) of a row
// group keeps NA / 4 sums; the groups' sums meet in LDS and the workgroup issues one atomic per weight (atomics on the
// same few thousand addresses serialise, so there are few workgroups).
constexpr int kWgradGroups = 4, kWgradBlock = kWgradGroups * 256, kWgradGrid = 256;
template <int NA>
__global__ void __launch_bounds__(kWgradBlock)
appearance_wgrad_kernel(const float *__restrict__ row_delta, const __half *__restrict__ app, uint64_t n_rows, float inv_scale,
                        float *__restrict__ dW)
{
    constexpr int kPer = NA / 4, kBatch = 8;
    __shared__ float part[kWgradGroups - 1][HC * NA];
    const int o = threadIdx.x & 63, q = (threadIdx.x >> 6) & 3, group = threadIdx.x >> 8;
    float acc[kPer];
#pragma unroll
    for (int a = 0; a < kPer; ++a) acc[a] = 0.0f;
    for (uint64_t first = ((uint64_t)blockIdx.x * kWgradGroups + group) * kBatch; first < n_rows;
         first += (uint64_t)gridDim.x * kWgradGroups * kBatch) {
        float d[kBatch];
        uint2 x[kBatch][kPer / 4];                          // kPer halves = kPer / 4 words of 8 bytes
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const uint64_t row = first + b < n_rows ? first + b : n_rows - 1;
            d[b] = first + b < n_rows ? row_delta[row * HC + o] : 0.0f;
            const uint2 *src = reinterpret_cast<const uint2 *>(app + row * NA + q * kPer);
#pragma unroll
            for (int w = 0; w < kPer / 4; ++w) x[b][w] = src[w];
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
#pragma unroll
            for (int w = 0; w < kPer / 4; ++w) {
                const __half2 lo = __builtin_bit_cast(__half2, x[b][w].x), hi = __builtin_bit_cast(__half2, x[b][w].y);
                acc[4 * w] = __builtin_fmaf(d[b], __low2float(lo), acc[4 * w]);
                acc[4 * w + 1] = __builtin_fmaf(d[b], __high2float(lo), acc[4 * w + 1]);
                acc[4 * w + 2] = __builtin_fmaf(d[b], __low2float(hi), acc[4 * w + 2]);
                acc[4 * w + 3] = __builtin_fmaf(d[b], __high2float(hi), acc[4 * w + 3]);
            }
    }
    if (group > 0) {
#pragma unroll
        for (int a = 0; a < kPer; ++a) part[group - 1][o * NA + q * kPer + a] = acc[a];
    }
    __syncthreads();
    if (group == 0) {
#pragma unroll
        for (int a = 0; a < kPer; ++a) {
            float v = acc[a];
#pragma unroll
            for (int g = 0; g < kWgradGroups - 1; ++g) v += part[g][o * NA + q * kPer + a];
            unsafeAtomicAdd(dW + kTotal + o * NA + q * kPer + a, v * inv_scale);
        }
    }
}

__global__ void __launch_bounds__(kBlock)
zero_kernel(float *__restrict__ p, uint64_t n)
{
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock) p[i] = 0.0f;
}

// Forward: five workgroups per compute unit, all resident at once.  0.65 M samples: 33 us against 36 with 2048 workgroups, each of which
// builds the weight images; 13.3 M samples: the same within 1 %.
constexpr uint32_t kGridForward = 1280;
constexpr uint32_t kGridColour = 512;      // persistent workgroups: two per compute unit of MI355X
constexpr uint32_t kGridDensity = 512;     // the lighter kernel fits two workgroups per compute unit

}  // namespace dg_mlp_mfma

namespace dg {

size_t mlp_mfma_workspace_bytes(uint64_t N, uint32_t n_app, uint32_t S)
{
    using namespace dg_mlp_mfma;
    const uint64_t n_rows = n_app ? (N + S - 1) / S : 0;
    return align256((size_t)kGridDensity * oWc1 * sizeof(float)) +
           align256((size_t)kGridColour * (kTotal - oWc1) * sizeof(float)) + align256((size_t)N * 32) +
           align256((size_t)n_rows * HC * sizeof(float));
}

size_t mlp_mfma_weight_count(uint32_t n_app) { return (size_t)dg_mlp_mfma::kTotal + (size_t)dg_mlp_mfma::HC * n_app; }

// calls launch(appearance inputs, layout of the features, sigmoid) with all three as compile-time constants
template <class F>
static void for_shape(uint32_t n_app, FeatureLayout layout, uint32_t act_c, F launch)
{
    auto with_act = [&](auto na, auto in_rows) {
        if (act_c) launch(na, in_rows, std::true_type{});
        else launch(na, in_rows, std::false_type{});
    };
    auto with_rows = [&](auto na) {
        if (layout == kPlanes) with_act(na, std::integral_constant<FeatureLayout, kPlanes>{});
        else if (layout == kRows) with_act(na, std::integral_constant<FeatureLayout, kRows>{});
        else with_act(na, std::integral_constant<FeatureLayout, kSplit>{});
    };
    if (n_app == 0) with_rows(std::integral_constant<int, 0>{});
    else if (n_app == 16) with_rows(std::integral_constant<int, 16>{});
    else with_rows(std::integral_constant<int, 48>{});
}

void mlp_mfma_fwd(const void *weights, const void *feat, FeatureLayout layout, const void *dir_enc, const void *app, uint32_t n_app, uint32_t S,
                  uint64_t N, uint32_t act_c, float *sigma, float *rgb, hipStream_t st)
{
    using namespace dg_mlp_mfma;
    const uint64_t tiles = (N + 31) / 32, blocks_needed = (tiles + kWavesPerBlock - 1) / kWavesPerBlock;
    const uint32_t grid = (uint32_t)(blocks_needed < kGridForward ? blocks_needed : kGridForward);
    for_shape(n_app, layout, act_c, [&](auto na, auto in_rows, auto sig) {
        fwd_kernel<decltype(na)::value, decltype(in_rows)::value, decltype(sig)::value><<<grid, kBlock, 0, st>>>(
            (const __half *)weights, (const __half *)feat, (const __half *)dir_enc, (const __half *)app, S, N, sigma, rgb);
    });
}

void mlp_mfma_density_max(const void *weights, const void *feat, FeatureLayout layout, const uint32_t *cell, uint32_t cell_stride, uint64_t N, float *density,
                          uint32_t n_cells, hipStream_t st)
{
    using namespace dg_mlp_mfma;
    const uint64_t tiles = (N + 31) / 32, blocks_needed = (tiles + kWavesPerBlock - 1) / kWavesPerBlock;
    const uint32_t grid = (uint32_t)(blocks_needed < 2048 ? blocks_needed : 2048);
    const __half *w = (const __half *)weights, *f = (const __half *)feat;
    if (layout == kPlanes) density_max_kernel<kPlanes><<<grid, kBlock, 0, st>>>(w, f, cell, cell_stride, N, density, n_cells);
    else if (layout == kRows) density_max_kernel<kRows><<<grid, kBlock, 0, st>>>(w, f, cell, cell_stride, N, density, n_cells);
    else density_max_kernel<kSplit><<<grid, kBlock, 0, st>>>(w, f, cell, cell_stride, N, density, n_cells);
}

int mlp_mfma_render(const char *who, const void *weights, const void *feat, FeatureLayout layout, const void *dir_enc, const void *app, uint32_t n_app, uint32_t S,
                    uint32_t n_seg, uint32_t act_c, const float *delta, const float *t, const uint32_t *seg_ray,
                    const uint32_t *seg_slot, uint32_t k_max, float *Ck, float *Tk, float *Dk, hipStream_t st)
{
    using namespace dg_mlp_mfma;
    DG_REQUIRE(layout != kSplit, DG_ERR_UNSUPPORTED, "%s: views take planes or rows, not split features", who);
    const uint32_t blocks_needed = (n_seg + kWavesPerBlock - 1) / kWavesPerBlock;
    const uint32_t grid = blocks_needed < 2048 ? blocks_needed : 2048;
    for_shape(n_app, layout, act_c, [&](auto na, auto in_rows, auto sig) {
        if constexpr (decltype(in_rows)::value != kSplit)              // refused above
            render_fwd_kernel<decltype(na)::value, decltype(in_rows)::value, decltype(sig)::value><<<grid, kBlock, 0, st>>>(
                (const __half *)weights, (const __half *)feat, (const __half *)dir_enc, (const __half *)app, S, n_seg, delta, t, seg_ray,
                seg_slot, k_max, Ck, Tk, Dk);
    });
    return launch_status(who);
}

void mlp_mfma_bwd(const void *weights, const void *feat, FeatureLayout layout, uint32_t n_merged, const void *dir_enc, const void *app, uint32_t n_app,
                  uint32_t S, uint64_t N, uint32_t act_c, const float *dsigma, const float *drgb, float loss_scale, float *dfeat, uint32_t *largest,
                  float *dW, void *ws, hipStream_t st)
{
    using namespace dg_mlp_mfma;
    const uint64_t tiles = (N + 31) / 32, blocks_needed = (tiles + kWavesPerBlock - 1) / kWavesPerBlock;
    const uint32_t grid_c = (uint32_t)(blocks_needed < kGridColour ? blocks_needed : kGridColour);
    const uint32_t grid_d = (uint32_t)(blocks_needed < kGridDensity ? blocks_needed : kGridDensity);
    char *base = static_cast<char *>(ws);
    float *density_shares = reinterpret_cast<float *>(base);
    float *colour_shares = reinterpret_cast<float *>(base + align256((size_t)kGridDensity * oWc1 * sizeof(float)));
    h8 *dgeo = reinterpret_cast<h8 *>(reinterpret_cast<char *>(colour_shares) +
                                      align256((size_t)kGridColour * (kTotal - oWc1) * sizeof(float)));
    float *row_delta = reinterpret_cast<float *>(reinterpret_cast<char *>(dgeo) + align256((size_t)N * 32));
    const uint64_t n_rows = n_app ? (N + S - 1) / S : 0;
    const __half *w = (const __half *)weights, *f = (const __half *)feat, *dr = (const __half *)dir_enc, *ap = (const __half *)app;
    if (n_app) {
        const uint64_t n = n_rows * HC, want = (n + kBlock - 1) / kBlock;
        zero_kernel<<<(uint32_t)(want < 4096 ? want : 4096), kBlock, 0, st>>>(row_delta, n);
    }
    for_shape(n_app, layout, act_c, [&](auto na, auto in_rows, auto sig) {
        colour_bwd_kernel<decltype(na)::value, decltype(in_rows)::value, decltype(sig)::value><<<grid_c, kBlock, 0, st>>>(w, f, dr, ap, S, N, dsigma, drgb, loss_scale, dgeo,
                                                                                                   colour_shares, row_delta);
    });
    if (layout == kPlanes) density_bwd_kernel<kPlanes><<<grid_d, kBlock, 0, st>>>(w, f, N, dgeo, loss_scale, 0, dfeat, nullptr, density_shares);
    else if (layout == kRows) density_bwd_kernel<kRows><<<grid_d, kBlock, 0, st>>>(w, f, N, dgeo, loss_scale, n_merged, dfeat, largest, density_shares);
    else density_bwd_kernel<kSplit><<<grid_d, kBlock, 0, st>>>(w, f, N, dgeo, loss_scale, n_merged, dfeat, largest, density_shares);
    static_assert(oWc1 % kFoldElems == 0, "a fold workgroup must not span both share regions");
    fold_shares_kernel<<<(kTotal + kFoldElems - 1) / kFoldElems, kFoldElems * kFoldGroups, 0, st>>>(density_shares, grid_d, oWc1, colour_shares, grid_c,
                                                                                                   kTotal, 1.0f / loss_scale, dW);
    if (n_app) {
        const uint64_t batches = (n_rows + 8 * kWgradGroups - 1) / (8 * kWgradGroups);
        const uint32_t grid_a = (uint32_t)(batches < kWgradGrid ? batches : kWgradGrid);
        if (n_app == 16) appearance_wgrad_kernel<16><<<grid_a, kWgradBlock, 0, st>>>(row_delta, ap, n_rows, 1.0f / loss_scale, dW);
        else appearance_wgrad_kernel<48><<<grid_a, kWgradBlock, 0, st>>>(row_delta, ap, n_rows, 1.0f / loss_scale, dW);
    }
}

}  // namespace dg
