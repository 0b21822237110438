// The small field networks, 8 -> 32 -> 16 and (16 + 4) -> 32 -> 3, on the matrix cores: one wavefront owns a tile of 32 samples,
// as in mlp_mfma.hip, but every layer is a single 32-row tile, so the whole backward pass fits one kernel: four weight-gradient
// tiles of 16 registers.
// These calls are small (a batch of 1024 rays has 1024 tiles): what bounds them is the chain of dependent layers and the
// launch, not a rate.  33 k samples: forward 33 -> 5 us, backward with its fold 131 -> 15 us against one sample per lane with
// scalar multiply-adds.
#include "mlp_mfma_common.h"

namespace dg_mlp_small {

using namespace dg_mlp_mfma;

constexpr int sNF = 8, sHD = 32, sNG = 16, sND = 4, sHC = 32, sCI = sNG + sND;
constexpr int pWd1 = 0, pWd2 = pWd1 + sHD * sNF, pWc1 = pWd2 + sNG * sHD, pWc3 = pWc1 + sHC * sCI, sTotal = pWc3 + 3 * sHC;

// image chunks: forward, then the transposed weights of the backward pass
constexpr int iD1 = 0, iD2 = 1, iC1 = 3, iC3 = 5, kFwdImages = 7;
constexpr int iC3T = 7, iC1T = 8, iD2T = 10, iD1T = 11, kAllImages = 13;

__device__ void build_small_forward(__half *lds, const __half *w)
{
    build_image<sNF, sHD, sNF, 1, 1, 1, false>(lds + iD1 * 512, w + pWd1);
    build_image<sHD, sNG, sHD, 1, 2, 0, false>(lds + iD2 * 512, w + pWd2);
    build_image<sCI, sHC, sCI, 1, 2, 2, false>(lds + iC1 * 512, w + pWc1);
    build_image<sHC, 3, sHC, 1, 2, 0, false>(lds + iC3 * 512, w + pWc3);
}

__device__ void build_small_backward(__half *lds, const __half *w)
{
    build_image<sHC, sHC, 3, 1, 1, 0, true>(lds + iC3T * 512, w + pWc3);
    build_image<sCI, sNG, sHC, 1, 2, 0, true>(lds + iC1T * 512, w + pWc1);        // direction inputs get no gradient
    build_image<sHD, sHD, sNG, 1, 1, 0, true>(lds + iD2T * 512, w + pWd2);
    build_image<sNF, sNF, sHD, 1, 2, 0, true>(lds + iD1T * 512, w + pWd1);
}

struct SmallTile {
    h8 x0, h1[2], xc[2], c1[2];
    float geo0, sigma, raw[3], rgb[3];     // meaningful on lanes with h == 0
};

// features: level-major planes [4][n_samples][2], in slots 0..7 of the lower half; direction row: 4 values
__device__ __forceinline__ void load_small(const __half *feat, const __half *dir_enc, uint32_t S, uint64_t n_samples, uint64_t n, bool valid, int h, SmallTile &t)
{
    const h8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    t.x0 = zero;
    t.xc[1] = zero;
    if (valid && h == 0) {
        const _Float16 *f = reinterpret_cast<const _Float16 *>(feat), *d = reinterpret_cast<const _Float16 *>(dir_enc) + (n / S) * sND;
#pragma unroll
        for (int j = 0; j < 8; ++j) t.x0[j] = f[((size_t)(j >> 1) * n_samples + n) * 2 + (j & 1)];
#pragma unroll
        for (int j = 0; j < sND; ++j) t.xc[1][j] = d[j];
    }
}

__device__ __forceinline__ void small_forward(const __half *lds, int lane, uint32_t act_c, SmallTile &t)
{
    f16v acc = mma(image(lds, iD1, lane), t.x0, zero16());
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) t.h1[ks] = pack_half<1>(acc, ks);
    f16v geo = mma(image(lds, iD2, lane), t.h1[0], zero16());
    geo = mma(image(lds, iD2 + 1, lane), t.h1[1], geo);
    t.geo0 = geo[0];
    t.sigma = expf(clip15(geo[0]));
    t.xc[0] = pack_half<0>(geo, 0);
    acc = mma(image(lds, iC1, lane), t.xc[0], zero16());
    acc = mma(image(lds, iC1 + 1, lane), t.xc[1], acc);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) t.c1[ks] = act_c ? pack_half<3>(acc, ks) : pack_half<1>(acc, ks);
    f16v out = mma(image(lds, iC3, lane), t.c1[0], zero16());
    out = mma(image(lds, iC3 + 1, lane), t.c1[1], out);
#pragma unroll
    for (int c = 0; c < 3; ++c) { t.raw[c] = out[c]; t.rgb[c] = full_sigmoid(clip15(out[c])); }
}

__global__ void __launch_bounds__(kBlock)
small_fwd_kernel(const __half *__restrict__ weights, const __half *__restrict__ feat, const __half *__restrict__ dir_enc, uint32_t S, uint64_t n_samples,
                 uint32_t act_c, float *__restrict__ sigma, float *__restrict__ rgb)
{
    __shared__ __attribute__((aligned(16))) __half lds[kFwdImages * 512];
    build_small_forward(lds, weights);
    __syncthreads();
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const uint64_t n_tiles = (n_samples + 31) / 32, n_waves = (uint64_t)gridDim.x * kWavesPerBlock;
    for (uint64_t tile = (uint64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6); tile < n_tiles; tile += n_waves) {
        const uint64_t n = tile * 32 + (lane & 31);
        const bool valid = n < n_samples;
        SmallTile t;
        load_small(feat, dir_enc, S, n_samples, n, valid, h, t);
        small_forward(lds, lane, act_c, t);
        if (valid && h == 0) {
            sigma[n] = t.sigma;
            rgb[3 * n] = t.rgb[0]; rgb[3 * n + 1] = t.rgb[1]; rgb[3 * n + 2] = t.rgb[2];
        }
    }
}

__global__ void __launch_bounds__(kBlock)
small_bwd_kernel(const __half *__restrict__ weights, const __half *__restrict__ feat, const __half *__restrict__ dir_enc, uint32_t S, uint64_t n_samples,
                 uint32_t act_c, const float *__restrict__ dsigma, const float *__restrict__ drgb, float loss_scale, float *__restrict__ dfeat,
                 float *__restrict__ shares)
{
    __shared__ __attribute__((aligned(16))) __half lds[kAllImages * 512];
    __shared__ __attribute__((aligned(16))) _Float16 scratch[kWavesPerBlock * kScratchHalves];
    build_small_forward(lds, weights);
    build_small_backward(lds, weights);
    __syncthreads();
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const uint64_t n_tiles = (n_samples + 31) / 32, n_waves = (uint64_t)gridDim.x * kWavesPerBlock;
    const float inv_scale = 1.0f / loss_scale;
    _Float16 *const tile0 = scratch + (threadIdx.x >> 6) * kScratchHalves, *const tile1 = tile0 + kTileHalves;
    f16v gWd1 = zero16(), gWd2 = zero16(), gWc1 = zero16(), gWc3 = zero16();
    for (uint64_t tile = (uint64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6); tile < n_tiles; tile += n_waves) {
        const uint64_t n = tile * 32 + (lane & 31);
        const bool valid = n < n_samples;
        SmallTile t;
        load_small(feat, dir_enc, S, n_samples, n, valid, h, t);
        float ds = 0.0f, dc[3] = {0.0f, 0.0f, 0.0f};
        if (valid && h == 0) {
            ds = dsigma[n];
            dc[0] = drgb[3 * n]; dc[1] = drgb[3 * n + 1]; dc[2] = drgb[3 * n + 2];
        }
        small_forward(lds, lane, act_c, t);
        // output layer of the colour net
        h8 d3 = {0, 0, 0, 0, 0, 0, 0, 0};
        if (valid && h == 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const bool pass = t.raw[c] >= -15.0f && t.raw[c] <= 15.0f;
                d3[c] = (_Float16)(pass ? loss_scale * dc[c] * t.rgb[c] * (1.0f - t.rgb[c]) : 0.0f);
            }
        }
        h8 td[2], ta[2];                        // transposed delta / activation: samples on the k axis
        transpose_half_tile(tile0, lane, d3, td);
        transpose_tile(tile1, lane, t.c1[0], t.c1[1], ta);
        gWc3 = mma(td[0], ta[0], gWc3);
        gWc3 = mma(td[1], ta[1], gWc3);
        f16v g = mma(image(lds, iC3T, lane), d3, zero16());
        // hidden layer of the colour net
        h8 dl[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) dl[ks] = act_c ? delta_from<2>(g, ks, t.c1[ks]) : delta_from<1>(g, ks, t.c1[ks]);
        transpose_tile(tile0, lane, dl[0], dl[1], td);
        transpose_tile<kTiled, kNatural>(tile1, lane, t.xc[0], t.xc[1], ta);
        gWc1 = mma(td[0], ta[0], gWc1);
        gWc1 = mma(td[1], ta[1], gWc1);
        f16v gx = mma(image(lds, iC1T, lane), dl[0], zero16());
        gx = mma(image(lds, iC1T + 1, lane), dl[1], gx);
        // density net output: geometry features feed the colour net, output 0 also feeds exp()
        if (valid && h == 0) {
            const bool pass0 = t.geo0 >= -15.0f && t.geo0 <= 15.0f;
            gx[0] += pass0 ? loss_scale * ds * t.sigma : 0.0f;
        }
        const h8 dgeo = pack_half<0>(gx, 0);
        transpose_half_tile(tile0, lane, dgeo, td);
        transpose_tile(tile1, lane, t.h1[0], t.h1[1], ta);
        gWd2 = mma(td[0], ta[0], gWd2);
        gWd2 = mma(td[1], ta[1], gWd2);
        g = mma(image(lds, iD2T, lane), dgeo, zero16());
        // hidden layer of the density net
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) dl[ks] = delta_from<1>(g, ks, t.h1[ks]);
        transpose_tile(tile0, lane, dl[0], dl[1], td);
        transpose_half_tile<kNatural>(tile1, lane, t.x0, ta);
        gWd1 = mma(td[0], ta[0], gWd1);
        gWd1 = mma(td[1], ta[1], gWd1);
        f16v gf = mma(image(lds, iD1T, lane), dl[0], zero16());
        gf = mma(image(lds, iD1T + 1, lane), dl[1], gf);
        if (valid) {            // registers 0..3 hold features 4h .. 4h + 3: levels 2h and 2h + 1
#pragma unroll
            for (int r = 0; r < 4; ++r) dfeat[((size_t)(2 * h + (r >> 1)) * n_samples + n) * 2 + (r & 1)] = gf[r] * inv_scale;
        }
    }
    static_assert(sTotal * 4 <= kAllImages * 1024, "the share fits the space of the images");
    write_share<sTotal>(reinterpret_cast<float *>(lds), shares + (size_t)blockIdx.x * sTotal, [&](float *share, uint32_t group, bool first) {
        if (group == 0) add_share(share + pWd1, first, sNF, sHD, sNF, 0, 0, lane, gWd1);
        if (group == 1) add_share(share + pWd2, first, sHD, sNG, sHD, 0, 0, lane, gWd2);
        if (group == 2) add_share(share + pWc1, first, sCI, sHC, sCI, 0, 0, lane, gWc1);
        if (group == 3) add_share(share + pWc3, first, sHC, 3, sHC, 0, 0, lane, gWc3);
    });
}

constexpr uint32_t kGridFwd = 2048, kGridBwd = 512;

uint32_t grid_of(uint64_t N, uint32_t most)
{
    const uint64_t tiles = (N + 31) / 32, blocks = (tiles + kWavesPerBlock - 1) / kWavesPerBlock;
    return (uint32_t)(blocks < most ? blocks : most);
}

}  // namespace dg_mlp_small

namespace dg {

size_t mlp_small_workspace_bytes() { return (size_t)dg_mlp_small::kGridBwd * dg_mlp_small::sTotal * sizeof(float); }

void mlp_small_fwd(const void *weights, const void *feat, const void *dir_enc, uint32_t S, uint64_t N, uint32_t act_c, float *sigma, float *rgb, hipStream_t st)
{
    using namespace dg_mlp_small;
    small_fwd_kernel<<<grid_of(N, kGridFwd), kBlock, 0, st>>>((const __half *)weights, (const __half *)feat, (const __half *)dir_enc, S, N, act_c, sigma, rgb);
}

void mlp_small_bwd(const void *weights, const void *feat, const void *dir_enc, uint32_t S, uint64_t N, uint32_t act_c, const float *dsigma,
                   const float *drgb, float loss_scale, float *dfeat, float *dW, void *ws, hipStream_t st)
{
    using namespace dg_mlp_small;
    float *shares = static_cast<float *>(ws);
    const uint32_t grid = grid_of(N, kGridBwd);
    small_bwd_kernel<<<grid, kBlock, 0, st>>>((const __half *)weights, (const __half *)feat, (const __half *)dir_enc, S, N, act_c, dsigma, drgb, loss_scale,
                                              dfeat, shares);
    fold_shares_kernel<<<(sTotal + kFoldElems - 1) / kFoldElems, kFoldElems * kFoldGroups, 0, st>>>(shares, grid, sTotal, shares, 0, sTotal, 1.0f / loss_scale, dW);
}

}  // namespace dg
