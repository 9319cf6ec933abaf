"""GPU parity of dmt_tower_module_fwd against the CPU oracle."""
import pytest
import torch

import oracle
import workloads as wl
from harness import RTOL, DeviceWorkload, TowerModules, assert_close, nan_behind, to_device, to_f64

pytestmark = pytest.mark.gpu


def check_tm(w, chained=False, guard=False):
    """TM on the oracle's pooled values (rounded to the pooled dtype), then
    optionally also the GPU lookup -> GPU TM chain.  guard: what lies behind the pooled values and
    the weights is NaN."""
    dw = DeviceWorkload(w)
    tm = TowerModules(dw, guard=guard)
    idx, off = wl.lookup_batch(w)
    pooled = oracle.lookup_towered(dw.host_tables, w.table_dtype, w.dims, w.table_to_tower, idx, off, w.batch)
    enc = [oracle.round_to(p, tm.dtype) for p in pooled]
    x_dev = torch.cat([to_device(e, tm.dtype).reshape(-1) for e in enc])
    if guard:
        x_dev = nan_behind(x_dev)
    got = to_f64(tm.run(x_dev))
    x64 = [wl.decode(e, tm.dtype) for e in enc]
    ref = tm.oracle(x64)
    rtol = RTOL[tm.dtype]
    for t, (g, r) in enumerate(zip(dw.split_towers(got, tm.out_widths), ref)):
        if tm.dtype != "f32":
            r = wl.decode(oracle.round_to(r, tm.dtype), tm.dtype)
        assert_close(g, r, rtol, "%s TM tower %d" % (w.name, t))
    if chained:
        pooled_gpu = dw.lookup(idx, off, tm.dtype)
        got2 = to_f64(tm.run(pooled_gpu))
        for t, (g, r) in enumerate(zip(dw.split_towers(got2, tm.out_widths), ref)):
            if tm.dtype != "f32":
                r = wl.decode(oracle.round_to(r, tm.dtype), tm.dtype)
            assert_close(g, r, rtol if tm.dtype != "f32" else 1e-4, "%s lookup+TM tower %d" % (w.name, t))


def test_tiny_linear_relu_f32():
    check_tm(wl.tiny(), chained=True)


def test_mid_scaled_dot_linear_bf16():
    # 2 towers x 8 features x 128: 28 dots | 1024 -> 256 ; B = 301 leaves ragged M tiles
    check_tm(wl.scaled(wl.mid(), max_rows=5000, batch=301, num_tables=16), chained=True)


def test_large_scaled_cross_linear_bf16():
    # 2 towers of 16 x 128 = 2048 wide: two 2048 x 2048 cross layers, then 2048 -> 512
    w = wl.scaled(wl.large(), max_rows=3000, batch=200)
    sel = [f for f in range(256) if w.table_to_tower[f] in (0, 1)]
    w.rows = [w.rows[f] for f in sel]; w.dims = [128] * 32
    w.table_to_tower = [wl.large().table_to_tower[f] for f in sel]
    w.tm_out = [512, 512]
    check_tm(w, chained=True)


@pytest.mark.parametrize("big", ["2", "0"])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_cross_linear_on_interior_tiles(big, dtype, monkeypatch):
    """A batch and widths that are multiples of the 256 x 256 and of the 128 x 128 tile, each in turn;
    two 1024 x 1024 cross layers and a 1024 -> 256 projection on two towers, B = 512."""
    monkeypatch.setenv("DMT_TM_BIG", big)
    w = wl.scaled(wl.large(), max_rows=3000, batch=512)
    sel = [f for f in range(256) if w.table_to_tower[f] in (0, 1)][:16]
    w.rows = [w.rows[f] for f in sel]
    w.dims = [128] * 16
    w.table_to_tower = [f // 8 for f in range(16)]
    w.tm_out = [256, 256]
    w.table_dtype = w.pooled_dtype = w.tm_dtype = dtype
    check_tm(w, chained=True)


def test_imbalanced_scaled_linear_f16():
    # towers of unequal width (mixed 32/64/128 dims), Linear -> 128
    check_tm(wl.scaled(wl.imbalanced(), max_rows=2000, batch=777, num_tables=26), chained=True)


@pytest.mark.parametrize("fuse", ["1", "0"])
def test_dot_linear_odd_feature_count(fuse, monkeypatch):
    # 3 features per tower: ten samples and two idle rows in a Gram tile, in the projection kernel
    # and in the dot kernel
    monkeypatch.setenv("DMT_TM_FUSE", fuse)
    w = wl.scaled(wl.mid(), max_rows=500, batch=50, num_tables=6)
    w.table_to_tower = [0, 0, 0, 1, 1, 1]
    w.tm_out = [40, 24]
    check_tm(w)


def test_dot_linear_f32_and_f16():
    w = wl.scaled(wl.mid(), max_rows=500, batch=70, num_tables=8)
    for dt in ("f32", "f16"):
        w.tm_dtype = dt
        w.pooled_dtype = dt
        check_tm(w)


def test_dot_linear_fused_and_separate_towers_in_one_call():
    """Tower 0 (4 features x 64, 6 dots padded to 8, 300 outputs) takes the GEMM that computes
    its dot terms in-kernel; tower 1 (12 features of 128, 66 terms: more than one K step, 96 outputs)
    the separate dot kernel and a plain GEMM; batch 519 leaves ragged row tiles in both."""
    w = wl.scaled(wl.mid(), max_rows=400, batch=519, num_tables=16)
    w.dims = [64] * 4 + [128] * 12
    w.table_to_tower = [0] * 4 + [1] * 12
    w.tm_out = [300, 96]
    for dt in ("bf16", "f16"):
        w.tm_dtype = dt
        w.pooled_dtype = dt
        check_tm(w)


@pytest.mark.parametrize("big", ["0", "1", "2"])
@pytest.mark.parametrize("out_dim,batch", [(100, 77), (300, 333), (257, 512)])
def test_linear_odd_output_widths_and_ragged_batches(out_dim, batch, big, monkeypatch):
    """Output widths that are no multiple of 8 or of a tile (scalar epilogue, partial
    column tiles) on both tilings of the grouped GEMM and on the one these sizes take (32 x 32)."""
    monkeypatch.setenv("DMT_TM_BIG", big)
    w = wl.scaled(wl.imbalanced(), max_rows=500, batch=batch, num_tables=9)
    w.tm_out = [out_dim] * w.num_towers
    check_tm(w)


def test_cross_with_three_layers_and_narrow_tower():
    w = wl.scaled(wl.large(), max_rows=300, batch=150, num_tables=3)
    w.table_to_tower = [0, 0, 0]
    w.tm_out = [96]
    w.tm_cross_layers = 3
    check_tm(w)                                       # 384-wide cross layers, 96-wide projection


@pytest.mark.parametrize("dt", ["bf16", "f16", "f32"])
def test_dlrm_module_flat_and_shared_per_feature_projection(dt):
    """Listing 1 with c > 0: 2 towers x 8 features x 128, flat 1024 -> 200 next to the shared
    128 -> 24 applied to every feature (200 + 8 * 24 = 392 outputs); batch 301."""
    w = wl.scaled(wl.mid(), max_rows=3000, batch=301, num_tables=16)
    w.tm_kind = wl.TM_DLRM
    w.tm_feat_out = 24
    w.tm_out = [200 + 8 * 24] * 2
    w.tm_dtype = dt
    w.pooled_dtype = dt
    check_tm(w, chained=dt == "bf16")


def test_dlrm_module_odd_widths():
    # 3 features per tower, 20 flat outputs, 5 per feature: nothing is a multiple of 8
    w = wl.scaled(wl.mid(), max_rows=500, batch=77, num_tables=6)
    w.table_to_tower = [0, 0, 0, 1, 1, 1]
    w.tm_kind = wl.TM_DLRM
    w.tm_feat_out = 5
    w.tm_out = [20 + 3 * 5] * 2
    check_tm(w)


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("dim,nf,batch,feat_out,big", [(12, 2, 77, 5, "0"), (12, 4, 301, 24, "2"), (4, 6, 65, 8, "3"),
                                                       (20, 2, 1, 1, "1"), (132, 2, 300, 136, "1")])
def test_dlrm_module_rows_that_end_inside_a_chunk(dim, nf, batch, feat_out, big, dt, monkeypatch):
    """Features of 4 mod 8 columns (float32 tables) under a 16-bit module: a row of the per-feature
    layer's operands ends halfway through a 16-byte piece, whose other half is the next row (behind
    the last one: NaN)."""
    monkeypatch.setenv("DMT_TM_BIG", big)
    w = wl.scaled(wl.mid(), max_rows=300, batch=batch, num_tables=2 * nf)
    w.table_dtype = "f32"
    w.dims = [dim] * (2 * nf)
    w.table_to_tower = [0] * nf + [1] * nf
    w.tm_kind = wl.TM_DLRM
    w.tm_feat_out = feat_out
    w.tm_out = [20 + nf * feat_out, 3 + nf * feat_out]
    w.tm_dtype = w.pooled_dtype = dt
    check_tm(w, guard=True)


@pytest.mark.parametrize("dt,rank", [("bf16", 64), ("bf16", 256), ("f16", 32), ("f32", 5)])
def test_lowrank_cross_module(dt, rank):
    """Two low-rank DCN-v2 cross layers on 512-wide towers, then 512 -> 96; batch 150."""
    w = wl.scaled(wl.large(), max_rows=300, batch=150, num_tables=8)
    w.table_to_tower = [0, 0, 0, 0, 1, 1, 1, 1]
    w.tm_out = [96, 96]
    w.tm_kind = wl.TM_CROSS_LOWRANK_LINEAR
    w.tm_cross_layers = 2
    w.tm_feat_out = rank
    w.tm_dtype = dt
    w.pooled_dtype = dt
    check_tm(w, chained=dt == "bf16" and rank == 64)


@pytest.mark.parametrize("batch,out,dim", [(1, 1, 4), (31, 33, 12), (33, 32, 16), (65, 31, 20), (1100, 64, 64)])
@pytest.mark.parametrize("kind", ["linear_relu", "dot_linear"])
def test_float32_tiles_segments_and_k_splits(kind, batch, out, dim):
    """The float32 contraction at the edges of its 32 x 32 tiles and of its steps of 8 k, with one and
    with several waves per tile; 7 features: 21 dot terms, so a weight row is not 16-byte aligned, and
    dims that are (12, 20) and are not (4) served by the Gram-tile kernel."""
    w = wl.scaled(wl.mid(), max_rows=300, batch=batch, num_tables=9)
    w.table_dtype = "f32"
    w.dims = [dim] * 9
    w.table_to_tower = [0] * 7 + [1] * 2
    w.tm_kind = kind
    w.tm_out = [out, out]
    w.tm_dtype = w.pooled_dtype = "f32"
    check_tm(w)


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("nf", [2, 3, 7, 13, 31, 32, 33])
def test_dot_terms_of_any_feature_count(nf, dt):
    """Feature counts that do and do not divide a 32-row Gram tile, one sample per tile (17 .. 32) and
    more features than a tile has rows (33: one thread per term); dim 24 leaves half of a 16-column
    step empty."""
    w = wl.scaled(wl.mid(), max_rows=100, batch=45, num_tables=nf)
    w.dims = [24] * nf
    w.table_to_tower = [0] * nf
    w.tm_out = [40]
    w.tm_dtype = w.pooled_dtype = dt
    check_tm(w)


@pytest.mark.parametrize("big,fuse", [("0", "1"), ("2", "1"), ("3", "1"), ("0", "0"), ("2", "0")])
@pytest.mark.parametrize("nf", [2, 4, 5, 8, 9, 12])
@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_an_infinite_weight_reaches_only_its_own_products(nf, dt, big, fuse, monkeypatch):
    """The flat weights that stand where a row's dot terms are padded to a whole 16-byte piece: an
    infinite one makes its output infinite, with the sign of the value it multiplies, and no NaN.
    1, 6, 10, 28, 36 and 66 terms; in-kernel terms on all three tilings, and terms of their own."""
    monkeypatch.setenv("DMT_TM_BIG", big)
    monkeypatch.setenv("DMT_TM_FUSE", fuse)
    w = wl.scaled(wl.mid(), max_rows=100, batch=261, num_tables=nf)
    w.dims = [24] * nf
    w.table_to_tower = [0] * nf
    w.tm_out = [264]
    w.tm_dtype = w.pooled_dtype = dt
    dw = DeviceWorkload(w)
    tm = TowerModules(dw)
    np_, pad = nf * (nf - 1) // 2, -(nf * (nf - 1) // 2) % 8
    weights = tm.keep[0]["w_proj"]
    x = torch.randn(w.batch, nf * 24, device="cuda", generator=torch.Generator("cuda").manual_seed(nf)).to(weights.dtype)
    plain = tm.run(x.reshape(-1)).view(w.batch, 264)
    assert torch.isfinite(plain).all()
    planted = {o: j for o, j in zip((0, 31, 130, 263), (0, 1, pad // 2, max(pad - 1, 0)))}
    for o, j in planted.items():
        weights[o, np_ + j] = float("inf")
    got = tm.run(x.reshape(-1)).view(w.batch, 264)
    others = [o for o in range(264) if o not in planted]
    assert torch.equal(got[:, others], plain[:, others])
    for o, j in planted.items():
        assert torch.equal(got[:, o], torch.sign(x[:, j]) * float("inf")), (o, j)


@pytest.mark.parametrize("big", ["0", "2", "3"])
@pytest.mark.parametrize("batch,out", [(129, 130), (255, 264), (256, 256), (257, 129), (520, 513), (31, 33), (1, 7)])
@pytest.mark.parametrize("kind", ["linear_relu", "dot_linear", "cross_linear"])
def test_contraction_tiles_of_both_sizes(kind, batch, out, big, monkeypatch):
    """Rows and columns just below, at and just above a 128 x 128 / 256 x 256 / (3) 32 x 32 tile, K of a whole number of
    steps and with a remainder (4 and 6 features of 72: 288 and 432 columns), widths that do and do not
    split into 16-byte pieces; 6 features: 15 dot terms, repacked weights; 4: 6 terms, read as they
    are."""
    monkeypatch.setenv("DMT_TM_BIG", big)
    w = wl.scaled(wl.mid(), max_rows=300, batch=batch, num_tables=10)
    w.dims = [72] * 10
    w.table_to_tower = [0] * 4 + [1] * 6
    w.tm_kind = kind
    w.tm_out = [out, out]
    w.tm_cross_layers = 1 if kind == "cross_linear" else 0
    check_tm(w)
