// Field MLPs (Sec. 3.2; activations and output clip of Sec. 5.1): argument checks and the choice of the network's kernels --
// mlp_mfma.hip for 32-64-16 / (32 + n_app)-64-64-3, mlp_small.hip for 8-32-16 / 20-32-3.
#include "dg_internal.h"

namespace {

int which_net(const dg_mlp_desc *m, const char *who)
{
    DG_REQUIRE(m, DG_ERR_ARG, "%s: null descriptor", who);
    DG_REQUIRE(m->act_c <= 1, DG_ERR_ARG, "%s: act_c must be 0 or 1", who);
    if (m->n_feat == 32 && m->n_hidden_d == 64 && m->n_geo == 16 && m->n_dir == 16 && m->n_hidden_c == 64 && m->n_layers_c == 2 &&
        (m->n_app == 0 || m->n_app == 16 || m->n_app == 48))
        return 1;
    if (m->n_feat == 8 && m->n_hidden_d == 32 && m->n_geo == 16 && m->n_dir == 4 && m->n_hidden_c == 32 && m->n_layers_c == 1 &&
        m->n_app == 0)
        return 2;
    return dg::fail(DG_ERR_UNSUPPORTED, "%s: unsupported MLP shape (%u,%u,%u,%u,%u,%u) with %u appearance inputs", who, m->n_feat,
                    m->n_hidden_d, m->n_geo, m->n_dir, m->n_hidden_c, m->n_layers_c, m->n_app);
}

}  // namespace

namespace {

// layout: of the features; only the matrix-core networks take other than planes
int mlp_fwd(const char *who, const dg_mlp_desc *desc, const void *weights, const void *feat, dg::FeatureLayout layout, const void *dir_enc, const void *app, uint32_t S,
            uint64_t N, float *sigma, float *rgb, void *stream)
{
    const int net = which_net(desc, who);
    if (net < 0) return net;
    DG_REQUIRE(layout == dg::kPlanes || net == 1, DG_ERR_UNSUPPORTED, "%s: only the 32-64-16 / 64-64-3 networks take feature rows", who);
    DG_REQUIRE(S >= 1, DG_ERR_ARG, "%s: S must be >= 1", who);
    if (N == 0) return DG_OK;
    DG_REQUIRE(weights && feat && dir_enc && sigma && rgb, DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(desc->n_app == 0 || (app && dg::aligned(app, 16)), DG_ERR_ARG, "%s: appearance rows missing or not 16-byte aligned", who);
    hipStream_t st = (hipStream_t)stream;
    if (net == 1) {
        DG_REQUIRE(dg::aligned(feat, layout != dg::kPlanes ? 16 : 4) && dg::aligned(dir_enc, 16), DG_ERR_ARG, "%s: feat must be %d-byte, dir_enc 16-byte aligned", who,
                   layout != dg::kPlanes ? 16 : 4);
        dg::mlp_mfma_fwd(weights, feat, layout, dir_enc, app, desc->n_app, S, N, desc->act_c, sigma, rgb, st);
    } else
        dg::mlp_small_fwd(weights, feat, dir_enc, S, N, desc->act_c, sigma, rgb, st);
    return dg::launch_status(who);
}

int mlp_composite_fwd(const char *who, const dg_mlp_desc *desc, const void *weights, const void *feat, dg::FeatureLayout layout, const void *dir_enc, const void *app,
                      uint32_t S, uint32_t n_seg, const float *delta, const float *t, const uint32_t *seg_ray, const uint32_t *seg_slot,
                      uint32_t k_max, float *Ck, float *Tk, float *Dk, void *stream)
{
    const int net = which_net(desc, who);
    if (net < 0) return net;
    DG_REQUIRE(net == 1, DG_ERR_UNSUPPORTED, "%s: only the 32-64-16 / 64-64-3 networks have a fused kernel", who);
    DG_REQUIRE(S >= 1 && S <= 64, DG_ERR_UNSUPPORTED, "%s: S=%u outside 1..64 (one wavefront renders a segment)", who, S);
    DG_REQUIRE(k_max >= 1, DG_ERR_ARG, "%s: k_max must be >= 1", who);
    if (n_seg == 0) return DG_OK;
    DG_REQUIRE(weights && feat && dir_enc && delta && seg_ray && seg_slot && Ck && Tk, DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE((t == nullptr) == (Dk == nullptr), DG_ERR_ARG, "%s: t and Dk go together", who);
    DG_REQUIRE(desc->n_app == 0 || (app && dg::aligned(app, 16)), DG_ERR_ARG, "%s: appearance rows missing or not 16-byte aligned", who);
    DG_REQUIRE(dg::aligned(feat, layout != dg::kPlanes ? 16 : 4) && dg::aligned(dir_enc, 16), DG_ERR_ARG, "%s: feat must be %d-byte, dir_enc 16-byte aligned", who,
               layout != dg::kPlanes ? 16 : 4);
    return dg::mlp_mfma_render(who, weights, feat, layout, dir_enc, app, desc->n_app, S, n_seg, desc->act_c, delta, t, seg_ray, seg_slot, k_max, Ck, Tk, Dk,
                               (hipStream_t)stream);
}

int mlp_bwd(const char *who, const dg_mlp_desc *desc, const void *weights, const void *feat, dg::FeatureLayout layout, uint32_t n_merged, const void *dir_enc,
            const void *app, uint32_t S, uint64_t N, const float *dsigma, const float *drgb, float loss_scale, float *dfeat, uint32_t *largest,
            float *dW, void *ws, size_t ws_bytes, void *stream)
{
    const int net = which_net(desc, who);
    if (net < 0) return net;
    DG_REQUIRE(layout == dg::kPlanes || net == 1, DG_ERR_UNSUPPORTED, "%s: only the 32-64-16 / 64-64-3 networks take feature rows", who);
    DG_REQUIRE(n_merged % 2 == 0 && n_merged <= desc->n_feat / 2, DG_ERR_ARG, "%s: n_merged=%u must be even and at most the number of levels", who, n_merged);
    DG_REQUIRE(S >= 1 && loss_scale > 0.0f, DG_ERR_ARG, "%s: S >= 1 and loss_scale > 0 required", who);
    if (N == 0) return DG_OK;
    DG_REQUIRE(weights && feat && dir_enc && dsigma && drgb && dfeat && dW && (layout == dg::kPlanes || largest), DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(desc->n_app == 0 || (app && dg::aligned(app, 16)), DG_ERR_ARG, "%s: appearance rows missing or not 16-byte aligned", who);
    DG_REQUIRE(ws && ws_bytes >= dg_mlp_bwd_app_workspace_bytes(desc, N, S), DG_ERR_WORKSPACE, "%s: workspace %zu < %zu bytes", who, ws_bytes,
               dg_mlp_bwd_app_workspace_bytes(desc, N, S));
    DG_REQUIRE(dg::aligned(ws, 256), DG_ERR_ARG, "%s: workspace must be 256-byte aligned", who);
    hipStream_t st = (hipStream_t)stream;
    if (net == 1) {
        DG_REQUIRE(dg::aligned(feat, layout != dg::kPlanes ? 16 : 4) && dg::aligned(dir_enc, 16) && dg::aligned(dfeat, layout != dg::kPlanes ? 16 : 8), DG_ERR_ARG,
                   "%s: feat must be %d-byte, dfeat %d-byte, dir_enc 16-byte aligned", who, layout != dg::kPlanes ? 16 : 4, layout != dg::kPlanes ? 16 : 8);
        dg::mlp_mfma_bwd(weights, feat, layout, n_merged, dir_enc, app, desc->n_app, S, N, desc->act_c, dsigma, drgb, loss_scale, dfeat, largest, dW, ws, st);
        return dg::launch_status(who);
    }
    dg::mlp_small_bwd(weights, feat, dir_enc, S, N, desc->act_c, dsigma, drgb, loss_scale, dfeat, dW, ws, st);
    return dg::launch_status(who);
}

}  // namespace

extern "C" int dg_mlp_fwd(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                          uint32_t S, uint64_t N, float *sigma, float *rgb, void *stream)
{
    DG_REQUIRE(!desc || desc->n_app == 0, DG_ERR_ARG, "dg_mlp_fwd: a network with appearance inputs needs dg_mlp_fwd_app");
    return dg_mlp_fwd_app(desc, weights, feat, dir_enc, nullptr, S, N, sigma, rgb, stream);
}

extern "C" int dg_mlp_fwd_app(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                              const void *app, uint32_t S, uint64_t N, float *sigma, float *rgb, void *stream)
{
    return mlp_fwd("dg_mlp_fwd", desc, weights, feat, dg::kPlanes, dir_enc, app, S, N, sigma, rgb, stream);
}

extern "C" int dg_mlp_fwd_rows(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                               const void *app, uint32_t S, uint64_t N, float *sigma, float *rgb, void *stream)
{
    return mlp_fwd("dg_mlp_fwd_rows", desc, weights, feat, dg::kRows, dir_enc, app, S, N, sigma, rgb, stream);
}

extern "C" int dg_mlp_composite_fwd(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                                    const void *app, uint32_t S, uint32_t n_seg, const float *delta, const float *t,
                                    const uint32_t *seg_ray, const uint32_t *seg_slot, uint32_t k_max, float *Ck, float *Tk,
                                    float *Dk, void *stream)
{
    return mlp_composite_fwd("dg_mlp_composite_fwd", desc, weights, feat, dg::kPlanes, dir_enc, app, S, n_seg, delta, t, seg_ray, seg_slot, k_max, Ck, Tk, Dk,
                             stream);
}

extern "C" int dg_mlp_composite_fwd_rows(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                                         const void *app, uint32_t S, uint32_t n_seg, const float *delta, const float *t,
                                         const uint32_t *seg_ray, const uint32_t *seg_slot, uint32_t k_max, float *Ck, float *Tk,
                                         float *Dk, void *stream)
{
    return mlp_composite_fwd("dg_mlp_composite_fwd_rows", desc, weights, feat, dg::kRows, dir_enc, app, S, n_seg, delta, t, seg_ray, seg_slot, k_max, Ck, Tk,
                             Dk, stream);
}

extern "C" size_t dg_mlp_bwd_workspace_bytes(const dg_mlp_desc *desc, uint64_t N)
{
    return dg_mlp_bwd_app_workspace_bytes(desc, N, 1);
}

extern "C" size_t dg_mlp_bwd_app_workspace_bytes(const dg_mlp_desc *desc, uint64_t N, uint32_t S)
{
    if (!desc || S == 0) return 0;
    const bool ngp = desc->n_feat == 32 && desc->n_hidden_d == 64 && desc->n_geo == 16 && desc->n_dir == 16 &&
                     desc->n_hidden_c == 64 && desc->n_layers_c == 2;
    return ngp ? dg::mlp_mfma_workspace_bytes(N, desc->n_app, S) : dg::mlp_small_workspace_bytes();
}

extern "C" int dg_mlp_bwd(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                          uint32_t S, uint64_t N, const float *dsigma, const float *drgb, float loss_scale,
                          float *dfeat, float *dW, void *ws, size_t ws_bytes, void *stream)
{
    DG_REQUIRE(!desc || desc->n_app == 0, DG_ERR_ARG, "dg_mlp_bwd: a network with appearance inputs needs dg_mlp_bwd_app");
    return dg_mlp_bwd_app(desc, weights, feat, dir_enc, nullptr, S, N, dsigma, drgb, loss_scale, dfeat, dW, ws, ws_bytes, stream);
}

extern "C" int dg_mlp_bwd_app(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                              const void *app, uint32_t S, uint64_t N, const float *dsigma, const float *drgb,
                              float loss_scale, float *dfeat, float *dW, void *ws, size_t ws_bytes, void *stream)
{
    return mlp_bwd("dg_mlp_bwd", desc, weights, feat, dg::kPlanes, 0, dir_enc, app, S, N, dsigma, drgb, loss_scale, dfeat, nullptr, dW, ws, ws_bytes, stream);
}

extern "C" int dg_mlp_bwd_rows(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                               const void *app, uint32_t S, uint64_t N, const float *dsigma, const float *drgb,
                               float loss_scale, uint32_t n_merged, float *dfeat, uint32_t *largest, float *dW, void *ws, size_t ws_bytes,
                               void *stream)
{
    return mlp_bwd("dg_mlp_bwd_rows", desc, weights, feat, dg::kRows, n_merged, dir_enc, app, S, N, dsigma, drgb, loss_scale, dfeat, largest, dW, ws, ws_bytes, stream);
}

extern "C" int dg_mlp_fwd_split(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                                const void *app, uint32_t S, uint64_t N, float *sigma, float *rgb, void *stream)
{
    return mlp_fwd("dg_mlp_fwd_split", desc, weights, feat, dg::kSplit, dir_enc, app, S, N, sigma, rgb, stream);
}

extern "C" int dg_mlp_bwd_split(const dg_mlp_desc *desc, const void *weights, const void *feat, const void *dir_enc,
                                const void *app, uint32_t S, uint64_t N, const float *dsigma, const float *drgb,
                                float loss_scale, uint32_t n_merged, float *dfeat, uint32_t *largest, float *dW, void *ws, size_t ws_bytes,
                                void *stream)
{
    return mlp_bwd("dg_mlp_bwd_split", desc, weights, feat, dg::kSplit, n_merged, dir_enc, app, S, N, dsigma, drgb, loss_scale, dfeat, largest, dW, ws, ws_bytes, stream);
}

namespace {

int occ_evaluate(const char *who, const dg_mlp_desc *desc, const void *weights, const void *feat, dg::FeatureLayout layout, const uint32_t *cell,
                 uint32_t cell_stride, uint64_t M, float *density, uint32_t n_cells, void *stream)
{
    const int net = which_net(desc, who);
    if (net < 0) return net;
    DG_REQUIRE(net == 1, DG_ERR_UNSUPPORTED, "%s: only the 32-64-16 density net has this kernel", who);
    DG_REQUIRE(cell_stride >= 1, DG_ERR_ARG, "%s: cell_stride must be >= 1", who);
    if (M == 0) return DG_OK;
    DG_REQUIRE(weights && feat && cell && density, DG_ERR_ARG, "%s: null pointer", who);
    DG_REQUIRE(dg::aligned(feat, layout != dg::kPlanes ? 16 : 4), DG_ERR_ARG, "%s: feat must be %d-byte aligned", who, layout != dg::kPlanes ? 16 : 4);
    dg::mlp_mfma_density_max(weights, feat, layout, cell, cell_stride, M, density, n_cells, (hipStream_t)stream);
    return dg::launch_status(who);
}

}  // namespace

extern "C" int dg_occ_evaluate(const dg_mlp_desc *desc, const void *weights, const void *feat, uint32_t rows, const uint32_t *cell,
                               uint32_t cell_stride, uint64_t M, float *density, uint32_t n_cells, void *stream)
{
    return occ_evaluate("dg_occ_evaluate", desc, weights, feat, rows ? dg::kRows : dg::kPlanes, cell, cell_stride, M, density, n_cells, stream);
}

extern "C" int dg_occ_evaluate_split(const dg_mlp_desc *desc, const void *weights, const void *feat, const uint32_t *cell,
                                     uint32_t cell_stride, uint64_t M, float *density, uint32_t n_cells, void *stream)
{
    return occ_evaluate("dg_occ_evaluate_split", desc, weights, feat, dg::kSplit, cell, cell_stride, M, density, n_cells, stream);
}
