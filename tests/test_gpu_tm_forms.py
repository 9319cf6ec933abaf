"""The Tower Module, forward and backward, against float32 torch: plans whose towers have different forms, and
launches that one block per CU works through.

16-bit operands and outputs are rounded once (2^-9 relative per term), in cross towers once a layer: the rms bounds
are a quarter of the elementwise 2e-2 (plain) and 4e-2 (cross) that the other tests allow; float32 sums of up to a
few thousand terms in another order stay within 2e-5 rms.
"""
import pytest
import torch

import paper_2403_00877_amd as dmt

pytestmark = pytest.mark.gpu

DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _tower(kind, nf, dim, out, layers=0, r=0):
    return dict(kind=kind, nf=nf, dim=dim, out=out, layers=layers, r=r)


def _shapes(s):
    """(w_proj, w_cross ..., b_cross ...) shapes of a tower."""
    w = s["nf"] * s["dim"]
    if s["kind"] == "dot_linear":
        return (s["out"], s["nf"] * (s["nf"] - 1) // 2 + w), [], []
    if s["kind"] == "cross_linear":
        return (s["out"], w), [(w, w)] * s["layers"], [w] * s["layers"]
    if s["kind"] == "cross_lowrank_linear":
        return (s["out"], w), [(s["r"], w), (w, s["r"])] * s["layers"], [w] * s["layers"]
    if s["kind"] == "dlrm":
        return (s["out"] - s["nf"] * s["r"], w), [(s["r"], s["dim"])], [s["r"]]
    return (s["out"], w), [], []


def _reference(s, x, p):
    """Float32 torch, from the encoded values."""
    nf, dim = s["nf"], s["dim"]
    h = x
    if s["kind"] == "cross_linear":
        for w, b in zip(p["w_cross"], p["b_cross"]):
            h = x * (h @ w.t() + b) + h
    elif s["kind"] == "cross_lowrank_linear":
        for v, u, b in zip(p["w_cross"][0::2], p["w_cross"][1::2], p["b_cross"]):
            h = x * ((h @ v.t()) @ u.t() + b) + h
    elif s["kind"] == "dot_linear":
        f = x.view(-1, nf, dim)
        i, j = torch.triu_indices(nf, nf, 1, device=x.device)
        h = torch.cat([(f[:, i] * f[:, j]).sum(-1), x], 1)
    y = h @ p["w_proj"].t() + p["b_proj"]
    if s["kind"] == "linear_relu":
        y = torch.relu(y)
    if s["kind"] == "dlrm":
        per = x.reshape(-1, dim) @ p["w_cross"][0].t() + p["b_cross"][0]
        y = torch.cat([y, per.view(x.shape[0], -1)], 1)
    return y


def _check(towers, batch, dtype, keep, backward=True, seed=11):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = DTYPE[dtype]
    rand = lambda scale, *shape: (torch.randn(*shape, generator=g, device="cuda") * scale).to(dt)
    nan = lambda *shape, dtype=torch.float32: torch.full(shape, float("nan"), dtype=dtype, device="cuda")
    dims = [s["dim"] for s in towers for _ in range(s["nf"])]
    tower = [t for t, s in enumerate(towers) for _ in range(s["nf"])]
    plan = dmt.dmt_plan_create([16] * len(dims), dims, dtype, len(towers), tower, batch, 1)
    dmt.dmt_plan_bind(plan, [torch.zeros(16, d, dtype=dt, device="cuda") for d in dims], None)
    xs, params, grads = [], [], []
    for s in towers:
        wp, wc, bc = _shapes(s)
        unit = s["dim"] ** -0.25 if s["kind"] == "dot_linear" else 1.0        # dot terms of unit size
        xs.append(rand(unit, batch, s["nf"] * s["dim"]))
        params.append(dict(kind=s["kind"], out_dim=s["out"], w_proj=rand(wp[1] ** -0.5, *wp), b_proj=rand(0.1, wp[0]),
                           w_cross=[rand(0.5 * w[1] ** -0.5, *w) for w in wc], b_cross=[rand(0.1, n) for n in bc],
                           feat_out=s["r"]))
        grads.append(dict(dw_proj=nan(*wp), db_proj=nan(wp[0]), dw_cross=[nan(*w) for w in wc], db_cross=[nan(n) for n in bc]))
    tp, tg = dmt.make_tm_params(params), dmt.make_tm_grads(grads)
    buf = lambda n: torch.full((max(256, n),), 255, dtype=torch.uint8, device="cuda")
    pooled = torch.cat([x.reshape(-1) for x in xs])
    y = nan(batch * sum(s["out"] for s in towers), dtype=dt)
    ws = buf(dmt.dmt_tm_workspace_bytes(plan, tp, batch))
    kept = None
    if keep:
        nkept = dmt.dmt_tm_kept_bytes(plan, tp, batch, dtype)
        kept = buf(nkept) if nkept else None
        dmt.dmt_tower_module_fwd_keep(plan, tp, pooled, batch, y, kept, ws)
    else:
        dmt.dmt_tower_module_fwd(plan, tp, pooled, batch, y, ws)
    dy, dx = torch.randn(y.numel(), generator=g, device="cuda"), nan(pooled.numel())
    at_y = 0
    for t, s in enumerate(towers):           # (outputs that rounding may switch on or off receive no gradient)
        part = slice(at_y, at_y + batch * s["out"])
        if s["kind"] == "linear_relu":
            dy[part] *= (y[part].float().abs() > 0.02) | (y[part] == 0)
        at_y += batch * s["out"]
    if backward:
        dmt.dmt_tower_module_bwd(plan, tp, pooled, y, batch, dy, dx, tg,
                                 buf(dmt.dmt_tm_bwd_workspace_bytes(plan, tp, batch)), kept=kept)

    def check(got, ref, bound, what):
        err = (got.float() - ref).square().mean().sqrt() / ref.square().mean().sqrt()
        assert err <= bound, "%s: rms error %.2e" % (what, err)               # (NaN fails)

    at_x = at_y = 0
    for t, s in enumerate(towers):
        bound = 2e-5 if dtype == "f32" else 1e-2 if s["layers"] else 5e-3
        leaf = lambda a: a.float().requires_grad_(backward)
        p = {k: [leaf(a) for a in v] if isinstance(v, list) else leaf(v) for k, v in params[t].items()
             if k in ("w_proj", "b_proj", "w_cross", "b_cross")}
        x = leaf(xs[t])
        ny, nx = batch * s["out"], x.numel()
        ref = _reference(s, x, p)
        what = "tower %d (%s) " % (t, s["kind"])
        if s["kind"] == "linear_relu" and backward:
            # as the library does, the output decides which gradients pass
            ref_pre = x @ p["w_proj"].t() + p["b_proj"]
            ref_pre.backward(dy[at_y:at_y + ny].view(batch, -1) * (y[at_y:at_y + ny].view(batch, -1) > 0))
        elif backward:
            ref.backward(dy[at_y:at_y + ny].view(batch, -1))
        check(y[at_y:at_y + ny].view(batch, -1), ref.detach(), bound, what + "output")
        if backward:
            check(dx[at_x:at_x + nx].view(batch, -1), x.grad, bound, what + "grad_pooled")
            check(grads[t]["dw_proj"], p["w_proj"].grad, bound, what + "dw_proj")
            check(grads[t]["db_proj"], p["b_proj"].grad, bound, what + "db_proj")
            for k in ("dw_cross", "db_cross"):
                for l, (a, b) in enumerate(zip(grads[t][k], p["w" + k[2:] if k[1] == "w" else "b" + k[2:]])):
                    check(a, b.grad, bound, what + "%s %d" % (k, l))
        at_x += nx
        at_y += ny


# one tower of every form, cross towers of every depth: the stages' launches mix epilogues (plain ones, cross layers',
# adding ones) and depths, and narrow contractions join flat ones
MIXED = [_tower("cross_linear", 4, 64, 40, layers=3), _tower("linear", 3, 32, 72), _tower("dot_linear", 5, 64, 136),
         _tower("cross_lowrank_linear", 2, 128, 64, layers=2, r=24), _tower("dlrm", 3, 64, 3 * 16 + 40, r=16),
         _tower("cross_linear", 2, 128, 96, layers=1), _tower("linear_relu", 6, 16, 130), _tower("cross_linear", 3, 64, 56, layers=4),
         _tower("dot_linear", 13, 32, 48), _tower("cross_linear", 1, 256, 8, layers=2), _tower("cross_lowrank_linear", 4, 32, 64, layers=1, r=40)]


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("batch,big", [(1, "1"), (77, "1"), (700, "1"), (700, "2"), (300, "0")])
def test_towers_of_every_form_in_one_plan(batch, big, dtype, keep, monkeypatch):
    monkeypatch.setenv("DMT_TM_BIG", big)
    _check(MIXED, batch, dtype, keep)


@pytest.mark.parametrize("keep", [False, True])
def test_wide_towers_of_several_forms_in_one_plan(keep):
    """Large tiles: 512 columns, the launches of a stage big enough for them by themselves."""
    wide = [_tower("cross_linear", 4, 128, 264, layers=3), _tower("linear", 4, 128, 520), _tower("cross_linear", 4, 128, 264, layers=2),
            _tower("cross_lowrank_linear", 4, 128, 264, layers=2, r=136), _tower("dot_linear", 4, 128, 264)]
    _check(wide, 12345, "bf16", keep)


# Blocks that work through several 256 x 256 tiles whose K has two segments, which every tile starts over: dot terms
# beside pooled values (12 features and more) in the forward, a per-feature layer beside the flat one in the backward
# (tests/test_tm_host.py checks that these sizes are such launches).  Ragged rows and columns, a last K step that
# is cut off in either segment.
@pytest.mark.parametrize("nf,dim,out", [(16, 64, 520), (16, 64, 516), (12, 64, 520)])
def test_many_tiles_of_dot_towers(nf, dim, out):
    _check([_tower("dot_linear", nf, dim, out)] * 4, 10233, "bf16", False)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("r", [64, 24])
def test_many_tiles_of_per_feature_layers(r, dtype):
    _check([_tower("dlrm", 4, 256, 4 * r + 264, r=r)] * 4, 10233, dtype, False)


def test_many_tiles_as_wide_as_the_output():
    """Tiles that share no rows of their first operand with another."""
    _check([_tower("linear", 8, 128, 256)] * 4, 32760, "bf16", False)
