"""One forward + backward pass of the DistGrid hot path on one GPU: call sequencing only.

`TrainStep` owns the device buffers and issues the library calls in the order of the paper's
training procedure (Sec. 4.4.2, Fig. 2): ray/box segments -> distribution to the resident
sub-models -> per sub-model sampling, encode, MLPs, local compositing -> merge -> loss seeds ->
merge backward (Eq. 7-8) -> per sub-model compositing / MLP / encode backward.  Every arithmetic
step happens inside libdistgrid; this file allocates, slices and calls.
"""
import collections
import contextlib

import torch

from . import binding as B


def split_appearance_columns(w, desc):
    """Packed MLP weights (or their gradient; numpy) with ONE wide first colour layer [n_hidden_c, n_geo + n_dir + n_app]
    -> the library's packing: the matrices without the appearance columns first, those columns
    Wapp [n_hidden_c, n_app] last.  Pure re-arrangement."""
    import numpy as np
    if not desc.n_app:
        return w
    pos = desc.n_hidden_d * desc.n_feat + desc.n_geo * desc.n_hidden_d
    no, ni = desc.n_hidden_c, desc.n_geo + desc.n_dir + desc.n_app
    Wc1 = np.asarray(w[pos:pos + no * ni]).reshape(no, ni)
    return np.concatenate([w[:pos], Wc1[:, :ni - desc.n_app].ravel(), w[pos + no * ni:], Wc1[:, ni - desc.n_app:].ravel()])


class SubModel:
    """Parameters and gradient buffers of one partition's sub-NeRF (hash table + MLP weights)."""

    def __init__(self, grid_desc, mlp_desc, table, weights):
        self.grid, self.mlp = grid_desc, mlp_desc
        self.table, self.weights = table, weights
        # both gradients in one buffer, so that one launch clears them
        buf = torch.zeros((table.numel() + 3) // 4 * 4 + weights.numel(), dtype=torch.float32, device=table.device)
        self.dtable, self.dW = buf[:table.numel()].view(table.shape), buf[buf.numel() - weights.numel():]
        self._grads = (buf, self.dtable, self.dW)
        self.opt = None     # optimiser state, allocated by the first optimiser step

    def _gradients(self):
        """What has to be zeroed to clear both gradients."""
        buf, dtable, dW = self._grads
        return (buf,) if self.dtable is dtable and self.dW is dW else (self.dtable, self.dW)      # the caller may have put buffers of its own there

    def clear_gradients(self, stream=None):
        """Zeroes both gradients, on the current stream or on the raw stream given."""
        for t in self._gradients():
            B.dg_clear(t, stream)

    def optimiser_state(self):
        """Adam moments of the table and of the weights, and the fp32 master copy of the fp16 weights."""
        if self.opt is None:
            self.opt = {"table_m": torch.zeros_like(self.table), "table_v": torch.zeros_like(self.table),
                        "w_master": self.weights.float().reshape(-1).contiguous(), "w_m": torch.zeros_like(self.dW),
                        "w_v": torch.zeros_like(self.dW)}
        return self.opt


class Occupancy:
    """Occupancy grid of one sub-model (Sec. 3.2, Sec. 5.1): geometry, per-cell densities, bit field, marching step."""

    def __init__(self, desc, density, bits, dt, max_steps):
        self.desc, self.density, self.bits, self.dt, self.max_steps = desc, density, bits, float(dt), int(max_steps)
        self.n_set = torch.zeros(1, dtype=torch.int32, device=density.device)


_Rows = collections.namedtuple("_Rows", "start N levels order by_position")     # the first `levels` levels of samples [start, start + N)


class TrainStep:
    def __init__(self, parts, models, resident, R, S, k_max, sh_degree, loss_scale=65536.0, lambda1=0.0, seed=0,
                 device="cuda:0", max_segments=None, binned_backward=True, encode_ws_cap=48 << 30, holes=None,
                 occupancy=None, max_samples=None, appearance=None, foreign_prefilled=False):
        """parts: [P,6] float tensor (device); models: {partition index: SubModel}; resident: partition indices served;
        max_segments: room for the segments of the RESIDENT partitions (default R * k_max);
        foreign_prefilled: the caller keeps the partial slots Ck / Tk of segments in non-resident partitions filled (in a
        deployment the exchange of Fig. 2 step 5 writes them); otherwise a step with non-resident partitions needs a
        `foreign` callable or it raises -- such slots are never silently read as whatever the buffers hold;
        holes: None or [P,6] (device): the box subtracted from each partition (coarse level of the cascade, Sec. 4.2.2);
        occupancy: None (S stratified samples per segment) or {partition index: Occupancy}: occupancy-guided sampling
        (Sec. 3.2, Sec. 5.1), at most max_samples samples per step over all resident partitions (S is then unused);
        appearance: None or (table [n_images, n_app] fp16, image_of_ray [R] int32), both on the device: per-image
        appearance vectors as further colour-net inputs (Sec. 4.4.3; the sub-models' MLP descriptors carry n_app)."""
        self.dev = torch.device(device)
        self.parts, self.models, self.resident, self.holes = parts, models, list(resident), holes
        self.parts_host = parts.cpu().tolist()
        self.P, self.R, self.S, self.k_max, self.deg = parts.shape[0], R, S, k_max, sh_degree
        self.loss_scale, self.lambda1, self.seed = float(loss_scale), float(lambda1), seed
        i32, f32, f16 = torch.int32, torch.float32, torch.float16
        z = lambda *shape, dt=f32: torch.zeros(*shape, dtype=dt, device=self.dev)
        cap = R * k_max if max_segments is None else max_segments
        self.cap = cap
        self.seg_count, self.seg_t, self.seg_part = z(R, dt=i32), z(R, k_max, 2), z(R, k_max, dt=i32)
        self.part_offset = z(self.P + 1, dt=i32)
        self.seg_ray, self.seg_slot = z(R * k_max, dt=i32), z(R * k_max, dt=i32)
        self.ws_seg = z(max(B.dg_segments_workspace_bytes(R, self.P) // 4, 1), dt=i32)
        self.occ = occupancy
        n = cap * S if occupancy is None else int(max_samples)
        self.max_samples = n
        any_model = next(iter(models.values()))
        self.n_feat = any_model.grid.n_levels * any_model.grid.n_features
        self.u, self.delta = z(n, 3), z(n)
        self.dir_enc = z(cap if occupancy is None else n, sh_degree * sh_degree, dt=f16)
        if occupancy is not None:
            self.first = z(R * k_max + self.P + 1, dt=i32)   # per partition: n_seg + 1 sample offsets, at [b + p, e + p]
            self.t, self.sample_ray = z(n), z(n, dt=i32)
            self.ws_march = z(B.dg_march_workspace_bytes(cap) // 4, dt=i32)
            self.samples = {}                               # partition -> (first sample, number of samples) of this step
        self.appearance = appearance
        self.app_rows = None if appearance is None else z(self.dir_enc.shape[0], appearance[0].shape[1], dt=f16)
        self._feat = z(n, self.n_feat, dt=f16)
        self.sigma, self.rgb = z(n), z(n, 3)
        self.dsigma, self.drgb = z(n), z(n, 3)
        self._dfeat = z(n, self.n_feat)
        self.Ck, self.Tk = z(R, k_max, 3), z(R, k_max)
        self.gCk, self.gTk = z(R, k_max, 3), z(R, k_max)
        self.C, self.T, self.gC, self.gT = z(R, 3), z(R), z(R, 3), z(R)
        # the two accumulated words, cleared together at the start of a step
        words = z(2)
        self.loss, self.status = words[:1], words[1:].view(i32)
        self._words = (words, self.loss, self.status)
        self.ws_mlp = z(B.dg_mlp_bwd_app_workspace_bytes(any_model.mlp, n, S if occupancy is None else 1) // 4 + 64)
        # workspace of the binned table-gradient pass, capped (the call batches itself when it is smaller than ideal)
        grids = {(bytes(mm.grid), bytes(mm.mlp)): mm for mm in models.values()}       # sub-models mostly share one
        want = max(self._encode_ws_bytes(mm, n) for mm in grids.values())
        self.ws_enc = torch.zeros(min(want, encode_ws_cap) // 4 + 64, dtype=f32, device=self.dev) if binned_backward else None
        self.foreign_prefilled = bool(foreign_prefilled)
        # The queue sizes of the binned table-gradient pass depend on the sample coordinates alone: for the sub-model whose
        # backward pass comes first they are counted on a second stream as soon as its samples exist, beside the forward
        # pass (which waits for memory and leaves the arithmetic units idle), together with the clearing of its gradient
        # buffers.  One workspace serves all sub-models, so only one count can be ahead.  (Counts ahead for every sub-model,
        # each in a workspace of its own, were measured on four and eight resident sub-models: no gain, 32.5 against 32.3 ms
        # and 40.0 against 40.0 ms per step.)
        self.side = torch.cuda.Stream(device=self.dev) if binned_backward and occupancy is None else None
        self.events = tuple(torch.cuda.Event() for _ in range(3)) if self.side is not None else None
        self.counted = None     # (partition, samples, event) of a count that is ahead
        # Samples in spatial order (large batches): the sorted list of every sub-model and what its bricks hold; the scratch of
        # the sort grows to the largest one asked for.
        order_any = binned_backward and any(n >= self._order_min(mm) for mm in models.values())
        self.ordered = torch.empty(n, 4, dtype=f32, device=self.dev) if order_any else None
        self.pieces, self.ws_order = {}, None
        self.layout = {}        # partition -> (first sample, samples, order or None) of this step
        # What lies in the feature buffers as rows instead of planes: partition -> _Rows.  While an entry of _feat_rows
        # stands, the partition's stretch of `ordered` and its `pieces` are those it was written with.
        self._feat_rows, self._dfeat_rows = {}, {}
        self.offsets = None
        self.local = {}         # resident partition -> index of its first segment among the resident segments (sample buffers)
        self.t_fixed = None
        self.timings = None     # set to {} to collect (start, end) event pairs per entry point

    # -- samples in spatial order ------------------------------------------------------------
    def _order_min(self, m):
        """Samples of a sub-model from which on a training step puts them in spatial order.  The kernels for ordered samples serve
        the 16-level grid with the 32-64-16 / 64-64-3 networks.  The order pays once the samples lie densely enough to share
        table lines and cells: with oblique rays, whose neighbours share less in ray order, earlier than under a camera; the lines lie where views from above
        break even or (T = 2^20 to 2^23) a little earlier.  Whole step, plain / ordered in us, of one box seen from above; oblique rays, and four
        sub-models that they cross, where stated:
        T = 2^17 728 / 771 at 0.91 M samples, 852 / 851 at 1.11 M, 909 / 899 at 1.19 M, oblique 870 / 828 at 1.0 M.  T = 2^18 823 / 842 at 1.03 M, 886 / 885 at 1.14 M,
        953 / 935 at 1.24 M, oblique 802 / 775 at 0.90 M.  T = 2^19 766 / 784 at 0.89 M, 863 / 864 at 1.04 M, 962 / 944 at 1.19 M, 1279 / 1191 at 1.66 M, oblique 906 / 861 at
        1.0 M, 1809 / 1434 at 2.2 M, four sub-models 2392 / 2470 of 0.61 M, 2925 / 2857 of 0.79 M, 4377 / 4036 of 1.28 M, with 48 appearance inputs 1148 / 1111 at 1.20 M.
        T = 2^20 818 / 855 at 0.84 M, 946 / 943 at 1.00 M, 1130 / 1104 at 1.25 M, oblique 920 / 894 at 0.85 M, four sub-models 2071 / 2278 of 0.41 M, 2758 / 2750 of
        0.61 M, 3467 / 3290 of 0.82 M.
        Larger tables, finest level of 2048 cells along the box: T = 2^21 684 / 707 at 0.52 M, 796 / 819 at 0.65 M, 917 / 891 at 0.80 M, oblique 883 / 851 at 0.65 M, four
        sub-models 2463 / 2622 of 0.41 M, 3264 / 3200 of 0.61 M; T = 2^22 698 / 732 at 0.38 M, 832 / 830 at 0.52 M, 941 / 927 at 0.64 M, four 3025 / 3041 of 0.42 M.
        With 8192 cells samples share less: T = 2^21 860 / 874 at 0.60 M, 1001 / 993 at 0.75 M, 1148 / 1125 at 0.91 M; T = 2^22 916 / 925 at 0.46 M, 1083 / 1071 at
        0.62 M, 1261 / 1203 at 0.77 M, oblique 1016 / 1020 at 0.50 M; T = 2^23 1086 / 1138 at 0.40 M, 1348 / 1374 at 0.60 M, 1463 / 1491 at 0.70 M, oblique 1274 / 1303 at
        0.50 M, 1469 / 1413 at 0.64 M; T = 2^24 1397 / 1475 at 0.40 M, 1658 / 1683 at 0.56 M, 1831 / 1831 at 0.65 M, oblique 1590 / 1640 at 0.50 M, 1830 / 1821 at 0.64 M.
        Occupancy-guided samples lie on surfaces, ten times as densely: T = 2^17 604 / 608 at 0.56 M, 1008 / 934 at 1.12 M; T = 2^18 612 / 603 at 0.56 M, 783 / 710 at
        0.78 M; T = 2^19 642 / 630 and 808 / 728; T = 2^20 559 / 560 at 0.39 M, 708 / 672 at 0.56 M; with cells four times as wide T = 2^19 1893 / 1715 at 2.2 M."""
        if m.grid.n_levels != 16 or (m.mlp.n_feat, m.mlp.n_hidden_d, m.mlp.n_layers_c) != (32, 64, 2):
            return 1 << 62
        T = m.grid.log2_T
        if self.occ is not None:
            return 1 << 20 if T < 18 else 3 << 18 if T <= 19 else 1 << 19
        if T <= 20:
            return {17: 9 << 17, 18: 9 << 17, 19: 9 << 17, 20: 3 << 18}.get(T, 1 << 21)
        if not self._fine(m):
            return 1 << 19
        return 3 << 18 if T == 21 else 5 << 17

    @staticmethod
    def _fine(m):
        """The finest level has some 4096 cells or more along the longest side of the box."""
        return max(m.grid.res[m.grid.n_levels - 1]) > 3 << 10

    def _order_factor(self, m, use):
        """How many times as many samples a call needs that has no backward pass to save time in: the gather alone pays for the
        sort and for rows written one by one.  Plain / ordered in ms.
        Rendering: T = 2^17 0.616 / 0.606 at 3.0 M samples; T = 2^18 0.66 / 0.69 at 3.2 M, 1.00 / 0.97 at 5.0 M; T = 2^19 0.59 / 0.70 at 2.4 M, 0.93 / 0.99 at
        4.0 M, 1.10 / 1.13 at 4.8 M, 1.38 / 1.33 at 6.0 M; T = 2^20 0.61 / 0.64 at 1.8 M, 0.75 / 0.74 at 2.2 M.  Finest level of 2048 cells: T = 2^21
        0.35 / 0.36 at 0.68 M, 0.42 / 0.42 at 0.87 M, 0.54 / 0.52 at 1.2 M (oblique rays 1.57 / 1.44 with four sub-models of 0.74 M), T = 2^22 0.26 / 0.27 at 0.40 M,
        0.33 / 0.33 at 0.56 M, 0.39 / 0.37 at 0.72 M; 8192 cells: T = 2^21 1.06 / 1.09 at 1.9 M, 1.53 / 1.52 at 2.8 M, T = 2^22 0.66 / 0.66 at 0.95 M, 0.94 / 0.90 at
        1.4 M, T = 2^23 0.56 / 0.56 at 0.75 M, 0.74 / 0.71 at 1.0 M.
        With occupancy-guided samples from 2^20 on (T = 2^19 0.50 / 0.48 at 1.1 M).
        Occupancy refresh, T = 2^19: 0.36 / 0.38 at 1.05 M candidates, 0.43 / 0.43 at 1.24 M, 0.57 / 0.55 at 1.71 M; T = 2^18 0.33 / 0.31 at 1.05 M."""
        T = m.grid.log2_T
        if use == "step":
            return 1.0
        if self.occ is not None:
            from_2_20 = {18: 4 / 3, 19: 4 / 3, 20: 2.0}.get(T, 1.0)
            return 1.25 * from_2_20 if use == "refresh" and T == 19 else from_2_20
        if T <= 20:
            return {17: 8 / 3, 18: 32 / 9, 19: 4.5, 20: 8 / 3}.get(T, 1.5)
        if self._fine(m):
            return {21: 4.0, 22: 2.25}.get(T, 1.5)
        return 1.5 if T == 21 else 1.0

    def _split(self, m, N, use):
        """Whether the features of samples in spatial order are split: rows of the first levels, planes of the finer ones, which are
        gathered level after level; the rows' merged levels come brick by brick from LDS where that is faster.  Pays where an XCD's L2 holds much of one level's
        table but not of the sixteen that the ordered gather walks at once, and while neighbours share few of the finer levels' lines.  One
        walk / split in us:
        step, T = 2^17 1315 / 1284 at 2.0 M samples, 2260 / 2222 at 4.1 M, 6592 / 6733 at 13.3 M; T = 2^18 2344 / 2272 at 4.1 M, 3594 / 3564 at 6.6 M, 6574 / 6693 at
        13.3 M; T = 2^19 3830 / 3730 at 6.6 M, 5038 / 5020 at 9.2 M, 6737 / 6912 at 13.3 M; T = 2^20 1353 / 1284 at 1.5 M, 2096 / 2016 at 3.1 M, 3972 / 4151 at 6.6 M;
        T = 2^21 1111 / 1092 at 1.0 M, 2236 / 2329 at 3.1 M; T = 2^22 with 2048 cells 4614 / 4825 (four of 1.0 M), with 8192 cells 1257 / 1220 at 0.76 M, 2501 / 2395 at 2.3 M,
        4768 / 4507 at 4.9 M, 8513 / 8501 at 9.8 M, 10 679 / 10 692 at 12.5 M; T = 2^23 11645 / 12166 at 12.8 M; T = 2^24 2395 / 2406 at 1.1 M.  T = 2^21 with 8192 cells 1116 / 1058 at
        0.83 M, 2316 / 2081 at 2.3 M, 4320 / 3992 at 4.9 M.
        Occupancy-guided steps, whose samples share more: T = 2^18 1172 / 1189 at 1.5 M, T = 2^19 1196 / 1229, T = 2^20 1251 / 1363.
        Refresh, pieces of 8.4 M and 2.1 M candidates: T = 2^17 1344 / 1167; T = 2^18 1411 / 1205; T = 2^19 1646 / 1373, 2525 / 1680; T = 2^20 1789 / 1756, 2751 / 2204.
        Tables that are not named (below 2^17) were not measured and keep the one walk."""
        T = m.grid.log2_T
        if use == "refresh":
            return N < {17: 10 << 20, 18: 10 << 20, 19: 10 << 20, 20: 10 << 20}.get(T, 0)
        if use != "step" or self.occ is not None:
            return False
        if T > 20 and self._fine(m):
            return N < {21: 5 << 20, 22: 13 << 20}.get(T, 0)
        return N < {17: 5 << 20, 18: 7 << 20, 19: 9 << 20, 20: 1 << 22, 21: 3 << 19}.get(T, 0)

    def _encode_ws_bytes(self, m, n):
        """Workspace of the table-gradient pass for up to n samples.  In spatial order it holds the unmerged levels only, and
        what it needs grows with the number of samples while the merged levels stay the same and falls where there are more of
        them: besides n, the last size before every such place counts."""
        least = self._order_min(m)
        if n < least:
            return B.dg_hashgrid_encode_bwd_workspace_bytes(m.grid, n)
        orders = {}

        def order(k):
            if k not in orders:
                orders[k] = self._order_desc(m, k)
            return orders[k]

        def need(k):
            q = order(k)
            return B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(m.grid, q, k) if q.n_merged > 0 else B.dg_hashgrid_encode_bwd_workspace_bytes(m.grid, k)

        def last_before_changes(a, b):
            if order(a).n_merged == order(b).n_merged:
                return []
            if b - a == 1:
                return [a]
            mid = (a + b) // 2
            return last_before_changes(a, mid) + last_before_changes(mid, b)

        # a grid of sizes first: a flat box's bricks do not grow evenly
        sizes = sorted({least, n} | {int(least * (n / least) ** (i / 12)) for i in range(1, 12)})
        ends = [k for a, b in zip(sizes, sizes[1:]) for k in last_before_changes(a, b)]
        return max(B.dg_hashgrid_encode_bwd_workspace_bytes(m.grid, least), *(need(k) for k in ends + [n]))

    def _order_of(self, m, N, use="step", full=False):
        """Order descriptor of a batch of N samples for a training step ("step"), a rendering or an occupancy refresh, or None
        where the plain kernels serve it (also where not even the two coarsest levels of a grid fit LDS brick by brick).
        full: occupancy-guided samples that fill the box (_fill_the_box)."""
        if self.ordered is None or N < self._order_min(m) * self._order_factor(m, use):
            return None
        order = self._order_desc(m, N, use, full)
        # fewer merged levels need more room in the table-gradient pass, whose workspace is made for those of thin samples
        if full and use == "step" and B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(m.grid, order, N) > self.ws_enc.numel() * self.ws_enc.element_size():
            order = self._order_desc(m, N, use)
        return order if order.n_merged > 0 else None

    def _fill_the_box(self, p, N, n_seg):
        """Whether N occupancy-guided samples of n_seg segments lie all over partition p's box, as with a grid that has not been thinned out yet,
        and not on surfaces: they take up more than a third of the length that as many chords of the box have on average (four times its volume over
        its surface; a full grid of 512 x 512 x 64 cells under a camera 0.64 of it, one of which half the layers are set 0.32, surfaces 0.05)."""
        ext = [hi - lo for lo, hi in zip(self.parts_host[p][:3], self.parts_host[p][3:])]
        chord = 2.0 / sum(1.0 / e for e in ext)
        return 3.0 * N * self.occ[p].dt > n_seg * chord

    def _order_desc(self, m, N, use="step", full=False):
        """The bricks of a batch of N samples.  Their number, and how many levels are merged brick by brick, follow the number of samples as if these
        filled the box evenly.  Occupancy-guided samples lie on surfaces: bricks that hold some hold several times as many, and are cut as for 3 N
        samples.  Whole step in us at 1, 2, 3, 4 N: T = 2^18 3477, 3458, 3293, 3327 at 5.9 M; T = 2^19 1207, 1130, 1121, 1140 at 1.5 M, 3500, 3448, 3337, 3351 at
        5.9 M, 6727, 6274, 6310, 6319 at 11.7 M; T = 2^22 1401, 1302, 1305, 1319 at 1.5 M; T = 2^24 2213, 2109, 2115, 2101 at 1.9 M; but T = 2^17 1425, 1430,
        1442, 1443 at 2.2 M.  Down from grids of which half the layers are set 3 N is the best or within 0.5 % of it.  Guided samples that fill the box (full) are cut as for
        1.5 N; at 1, 1.5, 3 N: T = 2^18 1437, 1429, 1459 at 2.0 M, 3485, 3484, 3646 at 6.0 M; T = 2^19 1295, 1243, 1254 at 1.6 M, 2055, 2065, 2090 at 3.0 M; T = 2^20
        1550, 1534, 1587 at 2.0 M; T = 2^22 1724, 1713, 1782 at 2.0 M, 2340, 2324, 2402 at 3.0 M; T = 2^24 2329, 2315, 2396 at 2.0 M.  With tables of a few of an XCD's L2 the ninth and tenth level are cheaper merged from fewer samples on: at 1, 1.4, 2 N T = 2^21 1519, 1459, 1450 at
        1.7 M, 2400, 2412, 2394 at 3.3 M; T = 2^22 1625, 1535, 1534 at 1.7 M, 9647, 9688, 9757 with four sub-models of 3.2 M; T = 2^23 3562, 3621, 3602 at 3.3 M; T = 2^19 1915, -, 1967 at 3.3 M."""
        T = m.grid.log2_T
        factor = 1.0
        if self.occ is not None and use != "refresh":
            factor = 1.0 if T < 18 else 1.5 if full else 3.0
        elif use != "refresh" and T in (21, 22):
            factor = max(1.0, min(1.4, (1 << 21) / max(N, 1)))
        return B.dg_order_desc_init(m.grid, int(N * factor))

    def _grown(self, buf, words):
        """buf if it holds that many words, otherwise a larger one.  The old one may have been allocated on another stream
        than the current one, which may still use it."""
        if buf is not None and buf.numel() >= words:
            return buf
        if buf is not None:
            buf.record_stream(torch.cuda.current_stream())
        return torch.empty(words, dtype=torch.int32, device=self.dev)

    def _encode_fwd(self, p, m, order, sl, N, use, ids=None):
        """Features of partition p's samples (their slice of the sample buffers): planes, or rows, of all levels or of the first ones, where
        they are sorted.
        ids: the number that stands beside each sorted sample in place of its index; the features then stay in sorted order."""
        split = order is not None and self._split(m, N, use)
        self._written(self._feat_rows, p, sl.start, N, 0 if order is None else B.SPLIT_LEVELS if split else self.n_feat // 2, order, ids is not None)
        if order is not None:
            self.pieces[p] = self._grown(self.pieces.get(p), B.dg_order_pieces_words(order, N))
            self.ws_order = self._grown(self.ws_order, B.dg_order_workspace_bytes(order) // 4)
            with self._timed("dg_order_samples"):
                B.dg_order_samples(order, self.u[sl], N, self.ordered[sl], self.pieces[p], self.ws_order, ids)
        with self._timed("dg_hashgrid_encode_fwd"):
            if split:
                B.dg_hashgrid_encode_fwd_bricks(m.grid, order, m.table, self.ordered[sl], self.pieces[p], self.u[sl], N, self._feat[sl],
                                                by_position=ids is not None)
            elif order is not None:
                B.dg_hashgrid_encode_fwd_ordered(m.grid, m.table, self.ordered[sl], N, self._feat[sl], by_position=ids is not None)
            else:
                B.dg_hashgrid_encode_fwd(m.grid, m.table, self.u[sl], N, self._feat[sl])

    @staticmethod
    def _written(rows, p, start, N, levels, order=None, by_position=False):
        """Books of a feature buffer: partition p's samples have been written, `levels` levels of them as rows; what lay
        there before is gone."""
        if rows:
            for q in [q for q, r in rows.items() if q == p or (r.start < start + N and start < r.start + r.N)]:
                del rows[q]
        if levels:
            rows[p] = _Rows(start, N, levels, order, by_position)

    def _is_split(self, p):
        return p in self._feat_rows and self._feat_rows[p].levels == B.SPLIT_LEVELS

    def _mlp_fwd(self, p, m, order, sl, dir_enc, app, S, N):
        call = B.dg_mlp_fwd_app if order is None else B.dg_mlp_fwd_split if self._is_split(p) else B.dg_mlp_fwd_rows
        with self._timed("dg_mlp_fwd"):
            call(m.mlp, m.weights, self._feat[sl], dir_enc, app, S, N, self.sigma[sl], self.rgb[sl])

    def _mlp_and_encode_bwd(self, p, m, sl, dir_enc, app, S, N, counted):
        # planes also where the features have been read, replaced or overwritten since the forward pass
        rows = self._feat_rows.get(p)
        order = rows.order if rows is not None and (rows.start, rows.N, rows.by_position) == (sl.start, N, False) else None
        counted = counted and order is self.layout[p][2]        # the counts were those of this order
        self._written(self._dfeat_rows, p, sl.start, N, 0 if order is None else order.n_merged)
        with self._timed("dg_mlp_bwd"):
            if order is None:
                B.dg_mlp_bwd_app(m.mlp, m.weights, self._feat[sl], dir_enc, app, S, N, self.dsigma[sl], self.drgb[sl], self.loss_scale,
                                 self._dfeat[sl], m.dW, self.ws_mlp)
            else:
                largest = self.pieces[p][1:2]
                B.dg_clear(largest)         # the networks only ever raise it, and a forward pass may see several backward passes
                call = B.dg_mlp_bwd_split if rows.levels == B.SPLIT_LEVELS else B.dg_mlp_bwd_rows
                call(m.mlp, m.weights, self._feat[sl], dir_enc, app, S, N, self.dsigma[sl], self.drgb[sl], self.loss_scale,
                     order.n_merged, self._dfeat[sl], largest, m.dW, self.ws_mlp)
        with self._timed("dg_hashgrid_encode_bwd"):
            if order is not None:
                B.dg_hashgrid_encode_bwd_ordered(m.grid, order, self.ordered[sl], self.pieces[p], self.u[sl], self._dfeat[sl], largest, N, m.dtable,
                                                 self.ws_enc, counted)
            elif counted:
                B.dg_hashgrid_encode_bwd_counted(m.grid, self.u[sl], self._dfeat[sl], N, m.dtable, self.ws_enc)
            else:
                B.dg_hashgrid_encode_bwd(m.grid, self.u[sl], self._dfeat[sl], N, m.dtable, self.ws_enc)

    def _as_planes(self, buf, rows):
        """buf, with what lies in it as rows turned into level-major planes, the layout of the plain kernels."""
        for r in rows.values():
            flat = buf[r.start:r.start + r.N].reshape(-1)[:2 * r.levels * r.N]
            planes = flat.view(r.N, r.levels, 2)
            if r.by_position:
                place = self._position_of_candidates(r)
                planes = planes[place]
                rest = buf[r.start:r.start + r.N].reshape(-1)[2 * r.levels * r.N:].view(-1, r.N, 2)
                rest.copy_(rest[:, place])
            flat.copy_(planes.transpose(0, 1).reshape(-1))
        rows.clear()
        return buf

    def _position_of_candidates(self, r):
        """Place in the sorted list of each candidate of the last occupancy refresh.  The list holds cells in place of indices:
        equal (coordinates, cell) are matched up, and candidates equal in all four have equal features."""
        def ranked(*columns):
            at = torch.arange(r.N, device=self.dev)
            for c in columns:
                at = at[torch.sort(c[at], stable=True).indices]
            return at
        bits = self.ordered[r.start:r.start + r.N].view(torch.int32)
        u = self.u[r.start:r.start + r.N].view(torch.int32)
        place = torch.empty(r.N, dtype=torch.int64, device=self.dev)
        place[ranked(u[:, 0], u[:, 1], u[:, 2], self.sample_ray[:r.N])] = ranked(*bits.unbind(1))
        return place

    # The buffers themselves, as level-major planes [L, N, 2] per partition.  Large batches are kept as rows (in part, for the
    # gradient); reading or replacing a buffer ends that, and a backward pass that follows takes the features as they then are.
    @property
    def feat(self):
        """Features of the last forward pass (or occupancy refresh), per partition as level-major planes [L, N, 2]."""
        return self._as_planes(self._feat, self._feat_rows)

    @feat.setter
    def feat(self, buf):
        self._feat = buf
        self._feat_rows.clear()

    @property
    def dfeat(self):
        """Feature gradient of the last backward pass, per partition as level-major planes [L, N, 2]."""
        return self._as_planes(self._dfeat, self._dfeat_rows)

    @dfeat.setter
    def dfeat(self, buf):
        self._dfeat = buf
        self._dfeat_rows.clear()

    @contextlib.contextmanager
    def _timed(self, name):
        """Brackets one library call with events on the stream it is launched on (the current stream)."""
        if self.timings is None:
            yield
            return
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        yield
        b.record()
        self.timings.setdefault(name, []).append((a, b))

    def timing_summary(self):
        """{entry point: (calls, total ms)} from the collected events; synchronises."""
        torch.cuda.synchronize()
        return {k: (len(v), sum(a.elapsed_time(b) for a, b in v)) for k, v in (self.timings or {}).items()}

    # -- forward ---------------------------------------------------------------------------
    def segments(self, o, d, t_min=0.0, clear_loss=False):
        words, loss, status = self._words
        if clear_loss and self.loss is loss and self.status is status:
            B.dg_clear(words)
        else:                                               # the caller may have put tensors of its own there
            for t in (self.status, self.loss) if clear_loss else (self.status,):
                B.dg_clear(t)
        with self._timed("dg_ray_aabb_segments"):
            B.dg_ray_aabb_segments(o, d, self.parts, t_min, self.k_max, self.seg_count, self.seg_t, self.seg_part,
                                   self.status, self.part_offset, self.seg_ray, self.seg_slot, self.ws_seg, holes=self.holes)
        self.offsets = self.part_offset.cpu().tolist()      # P+1 integers: how many segments each sub-model got
        # the sample buffers hold the segments of the resident partitions only, back to back in the order of `resident`
        run = 0
        for p in self.resident:
            self.local[p] = run
            run += self.offsets[p + 1] - self.offsets[p]
        if run > self.cap:
            raise B.DistGridError("segment capacity %d exceeded (%d)" % (self.cap, run))

    def _slices(self, p):
        """Segment range [b, e) of partition p in seg_ray / seg_slot, and the range of its samples in the sample buffers."""
        b, e = self.offsets[p], self.offsets[p + 1]
        first = self.local[p]
        return b, e, slice(first * self.S, (first + e - b) * self.S)

    def _rows(self, p):
        """Rows of partition p in the per-segment tables (direction encoding, appearance rows)."""
        first = self.local[p]
        return slice(first, first + self.offsets[p + 1] - self.offsets[p])

    def forward(self, o, d, Cgt, jitter=None, foreign=None):
        """foreign: optional callable(self) that fills partials of non-resident partitions into Ck/Tk."""
        if foreign is None and not self.foreign_prefilled and len(self.resident) < self.P:
            raise B.DistGridError("partitions %s are not resident: pass `foreign` to fill their partials, or construct with "
                                  "foreign_prefilled=True" % sorted(set(range(self.P)) - set(self.resident)))
        self._partials(o, d, jitter, training=True)
        if foreign is not None:
            foreign(self)
        with self._timed("dg_merge_loss"):
            B.dg_merge_loss(self.Ck, self.Tk, self.seg_count, self.R, self.k_max, Cgt, self.lambda1, self.C, self.T, self.gC, self.gT, self.loss)

    def render(self, o, d, jitter=None, fused=None):
        """Evaluation rendering (Sec. 4.4.2): forward only, every sub-model renders its segments and the partial
        results are merged into the final colour, depth and transmittance.  Returns (C [R,3], D [R], T [R]).
        fused: None = use the fused networks + rendering kernel where it applies; False = the separate entry points."""
        if self.occ is None and self.t_fixed is None:
            self.t_fixed = torch.zeros_like(self.delta)          # sample distances, only evaluation needs them
        Dk = torch.zeros(self.R, self.k_max, device=self.dev)
        D = torch.zeros(self.R, device=self.dev)
        # networks and local rendering in one kernel where the library has one (fixed S <= 64, the 32-64-16 / 64-64-3 nets)
        mlp = next(iter(self.models.values())).mlp
        fused = fused if fused is not None else (self.occ is None and self.S <= 64 and (mlp.n_feat, mlp.n_hidden_d, mlp.n_layers_c) == (32, 64, 2))
        self._partials(o, d, jitter, want_t=True, fused_depth=Dk if fused else None)
        B.dg_merge_segments(self.Ck, self.Tk, self.seg_count, self.R, self.k_max, self.C, self.T)
        if self.occ is not None:
            return self.C, self.depth(), self.T
        for p in () if fused else self.resident:
            b, e, sl = self._slices(p)
            if e > b:
                B.dg_composite_segment_depth(self.sigma[sl], self.delta[sl], self.t_fixed[sl], e - b, self.S, self.seg_ray[b:e],
                                             self.seg_slot[b:e], self.k_max, Dk)
        B.dg_merge_depth(Dk, self.Tk, self.seg_count, self.R, self.k_max, D)
        return self.C, D, self.T

    def _count_ahead(self, p, order, sl, N):
        """Starts the count sweep of sub-model p's table-gradient pass (and clears its gradient buffers) on the second
        stream, behind the work already queued on this one; the backward pass picks it up."""
        m = self.models[p]
        need = (B.dg_hashgrid_encode_bwd_workspace_bytes(m.grid, N) if order is None
                else B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(m.grid, order, N))
        if need > self.ws_enc.numel() * self.ws_enc.element_size():
            return                                  # the workspace would batch: counted with each batch, as usual
        main, side = torch.cuda.current_stream(), self.side
        here, go, done = self.events
        here.record(main)
        side.wait_event(here)
        go.record(side)
        if order is None:
            B.dg_hashgrid_encode_bwd_count(m.grid, self.u[sl], N, self.ws_enc, side.cuda_stream)
        else:
            B.dg_hashgrid_encode_bwd_ordered_count(m.grid, order, self.u[sl], N, self.ws_enc, side.cuda_stream)
        m.clear_gradients(side.cuda_stream)
        done.record(side)
        # this stream goes on once the second one has got that far: the count sweep's few workgroups are then handed out
        # before the forward gather's millions arrive and fill every wavefront slot of the chip
        main.wait_event(go)
        self.counted = (p, N, done)

    def _partials(self, o, d, jitter=None, want_t=False, fused_depth=None, training=False):
        """Segments, and per resident sub-model: samples, encode, MLPs, local compositing into the partial slots.
        fused_depth: None, or Dk [R,k_max]: networks, compositing and depth in one call (evaluation rendering)."""
        self.counted = None
        self.layout = {}
        S = self.S
        self.segments(o, d, clear_loss=training)
        # the sub-model whose backward pass runs first: only its counts may wait in the workspace that all share
        first = next((p for p in self.resident if self.offsets[p + 1] > self.offsets[p]), None)
        use = "step" if training else "render"
        if self.occ is not None:
            self._forward_marched(o, d, use)
        for p in self.resident if self.occ is None else ():
            b, e, sl = self._slices(p)
            n_seg = e - b
            if n_seg == 0:
                continue
            m = self.models[p]
            N = n_seg * S
            jit = None if jitter is None else jitter[sl]
            order = self._order_of(m, N, use)
            if training and jitter is None and self._one_call(order, N):
                self.layout[p] = (sl.start, N, None)
                self._written(self._feat_rows, p, sl.start, N, 0)
                B.dg_field_fwd(self._field(p, m), self.parts_host[p], self.seed, o, d, self.seg_t, m.table, self.Ck, self.Tk)
                continue
            with self._timed("dg_sample_segments"):
                B.dg_sample_segments(o, d, self.seg_t, self.seg_ray[b:e], self.seg_slot[b:e], n_seg, self.k_max,
                                     self.parts_host[p], S, self.seed, jit, self.u[sl], self.delta[sl],
                                     self.t_fixed[sl] if want_t else None)
            rows = self._rows(p)
            if training and self.side is not None and p == first:
                self._count_ahead(p, order, sl, N)
            with self._timed("dg_dir_encode"):
                B.dg_dir_encode(d, self.seg_ray[b:e], n_seg, self.deg, self.dir_enc[rows])
            self.layout[p] = (sl.start, N, order)
            self._encode_fwd(p, m, order, sl, N, use)
            app = self._appearance_rows(self.seg_ray[b:e], n_seg, rows)
            if fused_depth is not None:
                call = B.dg_mlp_composite_fwd if order is None else B.dg_mlp_composite_fwd_rows
                with self._timed("dg_mlp_composite_fwd"):
                    call(m.mlp, m.weights, self._feat[sl], self.dir_enc[rows], app, S, n_seg, self.delta[sl], self.t_fixed[sl], self.seg_ray[b:e],
                         self.seg_slot[b:e], self.k_max, self.Ck, self.Tk, fused_depth)
                continue
            self._mlp_fwd(p, m, order, sl, self.dir_enc[rows], app, S, N)
            with self._timed("dg_composite_segment_fwd"):
                B.dg_composite_segment_fwd(self.sigma[sl], self.rgb[sl], self.delta[sl], n_seg, S, self.seg_ray[b:e],
                                           self.seg_slot[b:e], self.k_max, self.Ck, self.Tk)

    def _one_call(self, order, N):
        """Whether a sub-model's share of a step goes out in one library call each way: samples in ray order, up to 2^21 of them; the count
        sweep of the table gradient then goes with the rest instead of ahead on a stream of its own, whose events cost more than it hides
        up to there.  Not where the single calls are timed.  Whole step, single calls / this, in us: 33 k samples of the small networks
        207 / 101, 29 k 288 / 211, 0.15 M 335 / 297, 0.81 M 755 / 729, 1.6 M 1290 / 1281; four sub-models of 0.1 M 1160 / 1118; eight of 38 k
        2246 / 2175."""
        return order is None and N <= 1 << 21 and self.occ is None and self.appearance is None and self.timings is None

    def _field(self, p, m):
        """The arguments that dg_field_fwd and dg_field_bwd share."""
        b, e = self.offsets[p], self.offsets[p + 1]
        return (m.grid, m.mlp, self.local[p], e - b, self.S, self.deg, b, self.seg_ray, self.seg_slot, self.k_max, m.weights, self.u, self.delta,
                self.dir_enc, self._feat, self.sigma, self.rgb)

    def _appearance_rows(self, index, n, rows):
        """Gathers the appearance vector of each row's ray (rows as for the direction encoding); None without them."""
        if self.appearance is None:
            return None
        with self._timed("dg_appearance_rows"):
            B.dg_appearance_rows(self.appearance[0], self.appearance[1], index, n, self.app_rows[rows])
        return self.app_rows[rows]

    def _forward_marched(self, o, d, use):
        """Per sub-model forward with occupancy-guided sampling (Sec. 3.2, Sec. 5.1): segments of different lengths,
        one direction row per sample."""
        self.samples = {}
        s0 = 0
        for p in self.resident:
            b, e = self.offsets[p], self.offsets[p + 1]
            n_seg = e - b
            if n_seg == 0:
                continue
            m, q = self.models[p], self.occ[p]
            first = self.first[b + p:e + p + 1]
            ray, slot = self.seg_ray[b:e], self.seg_slot[b:e]
            room = self.max_samples - s0
            with self._timed("dg_march_segments"):
                B.dg_march_segments(o, d, self.seg_t, ray, slot, n_seg, self.k_max, self.parts_host[p], q.desc, q.bits, q.dt,
                                    q.max_steps, self.seed, room, first, self.u[s0:], self.delta[s0:], self.t[s0:],
                                    self.sample_ray[s0:], self.status, self.ws_march)
            N = int(first[n_seg].item())                    # the one number the host needs: how many samples were kept
            if N > room:
                raise B.DistGridError("sample capacity %d exceeded (%d more wanted by partition %d)" % (self.max_samples, N - room, p))
            sl = slice(s0, s0 + N)
            self.samples[p] = (s0, N)
            s0 += N
            if N:
                with self._timed("dg_dir_encode"):
                    B.dg_dir_encode(d, self.sample_ray[sl], N, self.deg, self.dir_enc[sl])
                order = self._order_of(m, N, use, self._fill_the_box(p, N, n_seg))
                self.layout[p] = (s0 - N, N, order)
                self._encode_fwd(p, m, order, sl, N, use)
                app = self._appearance_rows(self.sample_ray[sl], N, sl)
                self._mlp_fwd(p, m, order, sl, self.dir_enc[sl], app, 1, N)
            with self._timed("dg_composite_ragged_fwd"):        # also writes C_k = 0, T_k = 1 for segments that saw nothing
                B.dg_composite_ragged_fwd(self.sigma[s0 - N:], self.rgb[s0 - N:], self.delta[s0 - N:], n_seg, first, ray, slot,
                                          self.k_max, self.Ck, self.Tk)

    def depth(self):
        """Depth channel of evaluation rendering (Sec. 4.4.2) for the samples of the last forward pass with
        occupancy-guided sampling; returns D [R]."""
        Dk = torch.zeros(self.R, self.k_max, device=self.dev)
        D = torch.zeros(self.R, device=self.dev)
        for p, (s0, N) in self.samples.items():
            b, e = self.offsets[p], self.offsets[p + 1]
            B.dg_composite_ragged_depth(self.sigma[s0:], self.delta[s0:], self.t[s0:], e - b, self.first[b + p:e + p + 1],
                                        self.seg_ray[b:e], self.seg_slot[b:e], self.k_max, Dk)
        B.dg_merge_depth(Dk, self.Tk, self.seg_count, self.R, self.k_max, D)
        return D

    def _backward_marched(self):
        for p in self.resident:
            m = self.models[p]
            with self._timed("zero_gradients"):
                m.clear_gradients()
            if p not in self.samples or self.samples[p][1] == 0:
                continue
            s0, N = self.samples[p]
            b, e = self.offsets[p], self.offsets[p + 1]
            sl = slice(s0, s0 + N)
            with self._timed("dg_composite_ragged_bwd"):
                B.dg_composite_ragged_bwd(self.sigma[s0:], self.rgb[s0:], self.delta[s0:], e - b, self.first[b + p:e + p + 1],
                                          self.seg_ray[b:e], self.seg_slot[b:e], self.k_max, self.gCk, self.gTk, self.dsigma[s0:],
                                          self.drgb[s0:])
            self._mlp_and_encode_bwd(p, m, sl, self.dir_enc[sl], None if self.app_rows is None else self.app_rows[sl], 1, N, False)

    # -- occupancy refresh (Sec. 5.1; Instant-NGP App. E.2) -------------------------------------
    def refresh_occupancy(self, iteration, tries=32):
        """Decay, candidate cells, the field's density at a random point of each, maximum, new bits -- when the
        schedule asks for it at this iteration.  Candidates are produced in pieces that fit the sample buffers, which
        serve as scratch: call it between training steps, not between a forward and its backward pass."""
        update_now, warmup, decay, threshold = B.dg_occ_schedule(iteration)
        if not update_now:
            return False
        for p in self.resident:
            m, q = self.models[p], self.occ[p]
            n_cells = q.desc.n_cells
            with self._timed("dg_occ_decay"):
                B.dg_occ_decay(q.density, decay)
            M = n_cells if warmup else n_cells // 2
            n_uniform = 0 if warmup else M // 2
            piece = self.max_samples
            density_kernel = (m.mlp.n_feat, m.mlp.n_hidden_d, m.mlp.n_layers_c) == (32, 64, 2)
            for i0 in range(0, M, piece):
                n = min(piece, M - i0)
                cell = self.sample_ray[:n]                      # the step's sample buffers serve as scratch
                with self._timed("dg_occ_candidates"):
                    B.dg_occ_candidates(q.desc, q.bits, n, n_uniform, warmup, self.seed, iteration, tries, cell, self.u[:n], i0=i0)
                order = None if warmup else self._order_of(m, n, "refresh")        # during warm-up the candidates come cell after cell anyway
                self._encode_fwd(p, m, order, slice(0, n), n, "refresh", None if order is None else cell)
                if density_kernel:
                    with self._timed("dg_occ_evaluate"):
                        if order is None:
                            B.dg_occ_evaluate(m.mlp, m.weights, self._feat[:n], False, cell, 1, n, q.density)
                        else:                                   # the cells stand beside the sorted samples
                            cells = self.ordered.view(-1)[3:4 * n].view(torch.int32)
                            if self._is_split(p):
                                B.dg_occ_evaluate_split(m.mlp, m.weights, self._feat[:n], cells, 4, n, q.density)
                            else:
                                B.dg_occ_evaluate(m.mlp, m.weights, self._feat[:n], True, cells, 4, n, q.density)
                    continue
                self.dir_enc[:1].zero_()                        # the density does not depend on the direction: one zero row
                if self.app_rows is not None:
                    self.app_rows[:1].zero_()
                self._mlp_fwd(p, m, order, slice(0, n), self.dir_enc[:1], None if self.app_rows is None else self.app_rows[:1], max(n, 1), n)
                with self._timed("dg_occ_update"):
                    B.dg_occ_update(q.density, cell, self.sigma[:n], n)
            q.n_set.zero_()
            with self._timed("dg_occ_bits"):
                B.dg_occ_bits(q.density, threshold, q.bits, q.n_set)
        return True

    # -- backward --------------------------------------------------------------------------
    def backward(self):
        S = self.S
        with self._timed("dg_merge_segments_bwd"):
            B.dg_merge_segments_bwd(self.Ck, self.Tk, self.seg_count, self.R, self.k_max, self.gC, self.gT, self.gCk,
                                    self.gTk)
        if self.occ is not None:
            return self._backward_marched()
        for p in self.resident:
            b, e, sl = self._slices(p)
            n_seg = e - b
            m = self.models[p]
            ahead = self.counted is not None and self.counted[0] == p
            if n_seg and not ahead and p not in self._feat_rows and self._one_call(None, n_seg * S):
                self._written(self._dfeat_rows, p, sl.start, n_seg * S, 0)
                B.dg_field_bwd(self._field(p, m), self.loss_scale, self.gCk, self.gTk, self.dsigma, self.drgb, self._dfeat, m.dtable, m.dW,
                               m._gradients(), self.ws_mlp, self.ws_enc)
                continue
            if ahead:
                torch.cuda.current_stream().wait_event(self.counted[2])     # queues counted, gradient buffers cleared
                self.counted = None
            else:
                with self._timed("zero_gradients"):
                    m.clear_gradients()
            if n_seg == 0:
                continue
            N = n_seg * S
            with self._timed("dg_composite_segment_bwd"):
                B.dg_composite_segment_bwd(self.sigma[sl], self.rgb[sl], self.delta[sl], n_seg, S, self.seg_ray[b:e],
                                           self.seg_slot[b:e], self.k_max, self.gCk, self.gTk, self.dsigma[sl], self.drgb[sl])
            rows = self._rows(p)
            self._mlp_and_encode_bwd(p, m, sl, self.dir_enc[rows], None if self.app_rows is None else self.app_rows[rows], S, N, ahead)

    def step(self, o, d, Cgt, jitter=None, foreign=None):
        self.forward(o, d, Cgt, jitter, foreign)
        self.backward()

    # -- optimiser (Sec. 5.1) -----------------------------------------------------------------
    def optimiser_step(self, iteration, total_iterations=300000, lr0=0.05, lr1=0.005, l2_weights=1e-6, check_overflow=False):
        """Adam on every resident sub-model, learning rate from the cosine schedule; consumes (clears) the gradients.
        iteration counts from 0.
        check_overflow: the back-propagated deltas are fp16 values times loss_scale; where one overflows, the weight
        gradient (and the table gradient) of that step is not finite.  With this flag the weight gradients are looked
        at first (one small device-to-host read); if any is not finite the step is dropped -- gradients cleared, no
        update, loss_scale halved -- and None is returned."""
        if check_overflow and not all(bool(torch.isfinite(self.models[p].dW).all()) for p in self.resident):
            for p in self.resident:
                self.models[p].dW.zero_()
                self.models[p].dtable.zero_()
            self.loss_scale *= 0.5
            return None
        lr = B.dg_cosine_lr(lr0, lr1, iteration, total_iterations)
        for p in self.resident:
            m = self.models[p]
            st = m.optimiser_state()
            with self._timed("dg_adam_step"):
                B.dg_adam_step(m.table.reshape(-1), m.dtable.reshape(-1), st["table_m"].reshape(-1), st["table_v"].reshape(-1), lr,
                               iteration + 1, skip_zero_grad=True)
                B.dg_adam_step(st["w_master"], m.dW, st["w_m"], st["w_v"], lr, iteration + 1, l2=l2_weights,
                               param_half=m.weights.reshape(-1))
        return lr
