"""The output layer and its softmax cross-entropy in one launch (at most 32 classes):
class counts at the edges of its 16 and 32 lane rows, batches that end inside a tile,
contractions shorter than a step and than a wave's share, labels out of range, a batch
whose logits are kept in the workspace and one whose are not; and the chain epilogue's
loss partials on the small tiles."""
import numpy as np
import pytest

import oracle
import paper_1711_03016_amd as dl
from helpers import TOL, assert_close, device, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


def _grad(widths, dtype, batch, seed=5, bad=None):
    import torch
    r = np.random.default_rng([51, seed, batch, *widths])
    acts = ("tanh",) * (len(widths) - 2) + ("none",)
    params = [((r.standard_normal((k, n)) / np.sqrt(k)).astype(np.float32),
               r.uniform(-0.5, 0.5, n).astype(np.float32)) for k, n in zip(widths[:-1], widths[1:])]
    x = r.standard_normal((batch, widths[0])).astype(np.float32)
    y = r.integers(0, widths[-1], batch).astype(np.int32)
    if bad is not None:
        y[bad[0]] = bad[1]
    m = dl.Model(widths, acts, dtype, "softmax_ce", False, batch)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    P = m.pack(params, device(), td)
    ws = torch.full((m.workspace_bytes(batch),), 0xFF, dtype=torch.uint8, device=device())
    loss = torch.full((1,), float("nan"), device=device())
    dP = torch.full((m.param_count(),), float("nan"), device=device())
    m.gradient(P, to_dev(x, dtype), torch.from_numpy(y).to(device()), batch, loss, dP, None, ws)
    torch.cuda.synchronize()
    return m, ws, loss.item(), m.unpack(dP), (widths, acts, x, params, y)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("classes", [1, 2, 10, 16, 17, 24, 25, 32, 33])
@pytest.mark.parametrize("K,batch", [(300, 37), (40, 1030), (520, 9000), (128, 1)])
def test_head_loss(dtype, classes, K, batch, monkeypatch):
    monkeypatch.setenv("DLVM_SMALL_STEP", "0")
    m, ws, loss, grads, (widths, acts, x, params, y) = _grad((24, K, classes), dtype, batch)
    spec = oracle.MlpSpec(widths, acts, "softmax_ce", dtype)
    rl, rg, _ = oracle.mlp_gradient(spec, x, params, y)
    assert m.check(ws) == dl.OK
    # (one class: the loss is exactly zero, and so is its adjoint)
    assert abs(loss - rl) <= 1e-5 * max(abs(rl), 1e-3)
    _, logits = oracle.mlp_forward(spec, x, params, y)
    _, rdz = oracle.softmax_xent(logits, y)
    dz = to_np(m.workspace_tensor(ws, batch, dl.WS_ADJOINT, 2))
    assert (dz[:, classes:] == 0).all()
    if classes > 1:
        assert_close(dz[:, :classes], rdz, TOL[dtype], "dZ_L")
        for (gW, gb), (rW, rb) in zip(grads, rg):
            assert rel_l2(to_np(gW), rW) <= TOL[dtype] and rel_l2(to_np(gb), rb) <= TOL[dtype]
    else:
        assert (dz == 0).all()
    fused = classes <= 32
    names = [e["name"] for e in m.plan(batch)]
    assert (f"gemm_nn_{dtype}_softmax_xent" in names or "head_softmax_xent" in names) == fused
    kept = not {"split_softmax_xent", "head_softmax_xent"} & set(names)
    if kept:
        assert_close(to_np(m.workspace_tensor(ws, batch, dl.WS_LOGITS)), logits, TOL[dtype], "logits")
    else:
        with pytest.raises(dl.DlvmError):
            m.workspace_tensor(ws, batch, dl.WS_LOGITS)


@pytest.mark.parametrize("classes,label", [(10, 10), (10, -1), (20, 20)])
def test_label_out_of_range(classes, label):
    m, ws, loss, _, _ = _grad((24, 600, classes), "f32", 100, bad=(77, label))
    assert m.check(ws) == dl.ERR_LABEL_RANGE
    assert np.isnan(loss)
    dz = to_np(m.workspace_tensor(ws, 100, dl.WS_ADJOINT, 2))[:, :classes]
    assert (dz[77] > 0).all() and ((dz < 0).sum(axis=1) == 1).sum() == 99


@pytest.mark.parametrize("cfg", [6, 7, 8, 9, 20, 21, 22, 23])
@pytest.mark.parametrize("n,batch", [(37, 50), (200, 300)])
def test_chain_in_epilogue_on_every_tile(cfg, n, batch, monkeypatch):
    import torch
    monkeypatch.setenv("DLVM_GEMM_CONFIG", str(cfg))
    r = np.random.default_rng([52, n, batch])
    x = (r.standard_normal((batch, n)) / np.sqrt(n)).astype(np.float32)
    W = (r.standard_normal((n, n)) / np.sqrt(n)).astype(np.float32)
    b = r.uniform(-0.1, 0.1, n).astype(np.float32)
    outs = []
    for epi in (True, False):
        m = dl.Model((n, n), ("none",), "f32", "chain8", True, batch, chain_in_epilogue=epi)
        assert m.plan(batch)[0]["name"].endswith(f"c{cfg}")
        P = m.pack([(W, b)], device(), torch.float32)
        ws = torch.full((m.workspace_bytes(batch),), 0xFF, dtype=torch.uint8, device=device())
        loss, dx = torch.empty(1, device=device()), torch.empty((batch, n), device=device())
        dP = torch.empty(m.param_count(), device=device())
        m.gradient(P, to_dev(x), None, batch, loss, dP, dx, ws)
        torch.cuda.synchronize()
        outs.append((loss.item(), dP, dx))
    assert torch.equal(outs[0][1], outs[1][1]) and torch.equal(outs[0][2], outs[1][2])
    rl, rg, rdx = oracle.mlp_gradient(oracle.MlpSpec((n, n), ("none",), "chain8"), x, [(W, b)], None, wrt_x=True)
    for l, _, _ in outs:
        assert abs(l - rl) <= 1e-5 * abs(rl)
    assert rel_l2(to_np(outs[0][2]), rdx) <= 1e-5
