"""End-to-end GPU parity of the forward, gradient and SGD calls on the five workloads.

Small workloads are compared at full size, element by element. The two large
ones are compared (a) at a reduced batch, element by element, and (b) at their
full batch in the launch configuration the benchmark times, using a batch made
of a few base rows repeated in a seeded order: the mean loss and its gradient
over such a batch equal those over the base rows, and every row's forward value
and input gradient equal those of its base row.
"""
import re

import numpy as np
import pytest

import oracle
import paper_1711_03016_amd as dl
import workloads
from helpers import TOL, assert_close, device, rel_l2, to_dev, to_np, torch_dtype

pytestmark = pytest.mark.gpu


def _run(wl, x, params, y, wrt_x=None, forward=True):
    """Run forward and gradient on the GPU; return host results."""
    import torch
    B = x.shape[0]
    wrt_x = wl.wrt_x if wrt_x is None else wrt_x
    m = dl.Model(wl.widths, wl.acts, wl.dtype, wl.loss, wrt_x, B)
    dev = device()
    P = m.pack(params, dev, torch_dtype(wl.dtype))
    xd = to_dev(x, wl.dtype)
    yd = None if y is None else torch.from_numpy(np.asarray(y, np.int32)).to(dev)
    ws = torch.empty(m.workspace_bytes(B), dtype=torch.uint8, device=dev)
    out = {}
    if forward:
        o = torch.empty((B, wl.widths[-1]), device=dev)
        m.forward(P, xd, B, o, ws)
        out["forward"] = to_np(o)
    loss = torch.empty(1, device=dev)
    dP = torch.full((m.param_count(),), float("nan"), device=dev)
    dx = torch.empty((B, wl.widths[0]), device=dev) if wrt_x else None
    m.gradient(P, xd, yd, B, loss, dP, dx, ws)
    torch.cuda.synchronize()
    out["loss"] = loss.item()
    out["grads"] = [(to_np(a), to_np(b)) for a, b in m.unpack(dP)]
    out["dparams"] = dP
    out["dx"] = None if dx is None else to_np(dx)
    out["status"] = m.check(ws)
    out["model"], out["P"], out["ws"] = m, P, ws
    return out


def _spec(wl):
    return oracle.MlpSpec(wl.widths, wl.acts, wl.loss, wl.dtype)


def _order_tolerances(wl, x, params, y, ref_grads):
    """Per-layer bounds for bf16 networks: max(2e-2, 2 x the oracle's own spread).

    A secondary, end-to-end check: for the deep network these bounds are
    wider than the stated 2e-2 (0.07-0.11 at batch 64). The stated bound is
    applied product by product, row by row, in test_gpu_c5_layers.py.

    The spread is the distance between the oracle's float64-accumulate and
    float32-accumulate evaluations of the same bf16-storage network: the part
    of the gradient that the accumulation order does not determine (ReLU mask
    flips behind bf16 rounding boundaries). Only oracle runs enter it.
    """
    from dataclasses import replace
    if wl.dtype != "bf16":
        return None
    alt = replace(_spec(wl), accumulate="f32")
    _, g32, _ = oracle.mlp_gradient(alt, x, params, y)
    tol = TOL["bf16"]
    return [(max(tol, 2 * rel_l2(a32, a)), max(tol, 2 * rel_l2(b32, b)))
            for (a32, b32), (a, b) in zip(g32, ref_grads)]


def _compare(wl, got, ref_loss, ref_grads, ref_dx=None, ref_out=None, tol=None,
             layer_tols=None, rows=True):
    """Loss, every dW and db, dx and the forward output against the oracle.

    With `rows` every row of a matrix (every element of a vector, against
    the vector's root-mean-square) is held to the same bound as the whole
    tensor, so one wrong row fails. The end-to-end gradients of the deep bf16
    network pass rows=False: their per-layer bounds are widened for the
    accumulation-order ambiguity of the function itself, and its products are
    checked row by row one at a time instead (test_gpu_c5_layers.py). For bf16
    networks dx is checked as a whole tensor only: a row of dx whose path
    crosses a bf16 rounding boundary differs between two valid evaluation
    orders of the oracle itself by several percent (c3: 8e-2).
    """
    tol = TOL[wl.dtype] if tol is None else tol
    assert got["status"] == dl.OK
    assert abs(got["loss"] - ref_loss) <= tol * abs(ref_loss), (got["loss"], ref_loss)
    for l, ((gw, gb), (rw, rb)) in enumerate(zip(got["grads"], ref_grads)):
        tw, tb = (tol, tol) if layer_tols is None else layer_tols[l]
        if rows:
            assert_close(gw, rw, tw, ("dW", l))
            assert_close(gb, rb, tb, ("db", l))
        else:
            ew, eb = rel_l2(gw, rw), rel_l2(gb, rb)
            assert ew <= tw, (l, "dW", ew, tw)
            assert eb <= tb, (l, "db", eb, tb)
    if ref_dx is not None:
        if rows and wl.dtype == "f32":
            assert_close(got["dx"], ref_dx, tol, "dx")
        else:
            assert rel_l2(got["dx"], ref_dx) <= tol
    if ref_out is not None:
        if rows:
            assert_close(got["forward"], ref_out, tol, "forward")
        else:
            assert rel_l2(got["forward"], ref_out) <= tol


@pytest.mark.parametrize("name", ["c1", "c2", "c3"])
def test_workload_full_size(name):
    wl = workloads.WORKLOADS[name]
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    got = _run(wl, x, params, y, wrt_x=True)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), x, params, y, wrt_x=True)
    _, rout = oracle.mlp_forward(_spec(wl), x, params, y)
    _compare(wl, got, rl, rg, rdx, rout)


def test_c2_gradient_then_sgd():
    import torch
    wl = workloads.WORKLOADS["c2"]
    x, params, y = workloads.make_inputs(wl)
    got = _run(wl, x, params, y, forward=False)
    m, P = got["model"], got["P"]
    m.sgd_step(P, None, got["dparams"], wl.lr)
    torch.cuda.synchronize()
    _, rg, _ = oracle.mlp_gradient(_spec(wl), x, params, y)
    for (gW, gb), (W, b), (dW, db) in zip(m.unpack(P), params, rg):
        assert rel_l2(to_np(gW), oracle.sgd_f32(W, dW, wl.lr)) <= 1e-6
        # the biases start at zero, so their new value is the step -lr*db itself
        assert rel_l2(to_np(gb), oracle.sgd_f32(b, db, wl.lr)) <= TOL["f32"]


def test_gradient_is_deterministic():
    import torch
    wl = workloads.WORKLOADS["c2"]
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    a = _run(wl, x, params, y, wrt_x=True)
    m, P, ws = a["model"], a["P"], a["ws"]
    dev = device()
    xd = to_dev(x)
    yd = torch.from_numpy(y).to(dev)
    for _ in range(3):
        loss = torch.empty(1, device=dev)
        dP = torch.empty(m.param_count(), device=dev)
        dx = torch.empty((x.shape[0], wl.widths[0]), device=dev)
        m.gradient(P, xd, yd, x.shape[0], loss, dP, dx, ws)
        torch.cuda.synchronize()
        assert torch.equal(dP, a["dparams"])
        assert loss.item() == a["loss"]
        assert np.array_equal(to_np(dx), a["dx"])


def test_dparams_padding_is_zero():
    wl = workloads.WORKLOADS["c1"]
    x, params, y = workloads.make_inputs(wl)
    got = _run(wl, x, params, y, forward=False)
    dP = to_np(got["dparams"])
    offs, lds = got["model"].param_layout_lds()
    assert lds[-1] == 16 and lds[0] == wl.widths[1]   # 10 classes padded to 16
    live = np.zeros(dP.size, bool)
    for l in range(wl.n_layers):
        K, N, ld = wl.widths[l], wl.widths[l + 1], lds[l]
        for k in range(K):
            live[offs[2 * l] + k * ld:offs[2 * l] + k * ld + N] = True
        live[offs[2 * l + 1]:offs[2 * l + 1] + N] = True
    assert not np.isnan(dP).any()
    assert (dP[~live] == 0).all()     # gaps between tensors and W padding columns


def test_fig3_single_row():
    """Fig. 3's shapes: x <1 x 784>, w <784 x 10>, b <1 x 10>, gradient wrt all."""
    from dataclasses import replace
    wl = replace(workloads.WORKLOADS["c1"], widths=(784, 10), acts=("none",), batch=1)
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    got = _run(wl, x, params, y, wrt_x=True)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), x, params, y, wrt_x=True)
    _, rout = oracle.mlp_forward(_spec(wl), x, params, y)
    _compare(wl, got, rl, rg, rdx, rout)


@pytest.mark.parametrize("batch", [1, 37, 300])
def test_ragged_batches(batch):
    wl = workloads.WORKLOADS["c3"]
    x, params, y = workloads.make_inputs(wl, batch=batch, bias_scale=0.1)
    got = _run(wl, x, params, y, wrt_x=True)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), x, params, y, wrt_x=True)
    _compare(wl, got, rl, rg, rdx, layer_tols=_order_tolerances(wl, x, params, y, rg))


@pytest.mark.parametrize("name,bad", [("c1", 10), ("c2", 10), ("c2", -1)])
def test_label_out_of_range_is_reported(name, bad):
    """c2's output layer is a split product whose slices the loss kernel sums."""
    wl = workloads.WORKLOADS[name]
    x, params, y = workloads.make_inputs(wl)
    y = y.copy()
    y[3] = bad
    got = _run(wl, x, params, y, forward=False)
    assert got["status"] == dl.ERR_LABEL_RANGE
    assert np.isnan(got["loss"])
    y[3] = 2
    good = _run(wl, x, params, y, forward=False)
    assert good["status"] == dl.OK


@pytest.mark.parametrize("name", ["c2", "c3"])
def test_loss_adjoint_labels_are_exact(name):
    """The adjoint of the logits that a full-batch gradient call stores in its
    workspace, (softmax - onehot(y)) / B, read back through
    dlvm_workspace_tensor. The heads of c2 (float32) and c3 (bf16) have ten
    classes: product and loss share a launch whose waves split the contraction,
    so this checks that kernel's label handling bit for bit: every
    row has exactly one negative entry, at its label, and the padding columns
    (10 -> 16) are zero. The values match the oracle's adjoint of its own
    logits."""
    wl = workloads.WORKLOADS[name]
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    got = _run(wl, x, params, y, forward=False)
    m, ws, B, C = got["model"], got["ws"], wl.batch, wl.widths[-1]
    assert any(e["name"] == "head_softmax_xent" for e in m.plan(B))
    with pytest.raises(dl.DlvmError):          # this head never stores its logits
        m.workspace_tensor(ws, B, dl.WS_LOGITS)
    dz = to_np(m.workspace_tensor(ws, B, dl.WS_ADJOINT, m.n_layers))
    assert dz.shape == (B, 16)
    assert (dz[:, C:] == 0).all()
    neg = dz[:, :C] < 0
    assert (neg.sum(axis=1) == 1).all()
    np.testing.assert_array_equal(np.argmax(neg, axis=1), y)
    _, logits = oracle.mlp_forward(_spec(wl), x, params, y)
    _, rdz = oracle.softmax_xent(logits, y)
    assert_close(dz[:, :C], rdz, TOL[wl.dtype], "dZ_L")


def test_non_default_stream():
    import torch
    wl = workloads.WORKLOADS["c2"]
    x, params, y = workloads.make_inputs(wl)
    ref = _run(wl, x, params, y, forward=False)
    m, P, ws = ref["model"], ref["P"], ref["ws"]
    dev = device()
    s = torch.cuda.Stream()
    xd, yd = to_dev(x), torch.from_numpy(y).to(dev)
    loss = torch.empty(1, device=dev)
    dP = torch.empty(m.param_count(), device=dev)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        m.gradient(P, xd, yd, x.shape[0], loss, dP, None, ws, stream=s)
        ev = torch.cuda.Event()
        ev.record(s)
    ev.synchronize()
    assert torch.equal(dP, ref["dparams"])


# ---------------------------------------------------------------------------
# the two large workloads
# ---------------------------------------------------------------------------
def test_c4_reduced_batch():
    wl = workloads.WORKLOADS["c4"]
    x, params, _ = workloads.make_inputs(wl, batch=256, bias_scale=0.05)
    got = _run(wl, x, params, None)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), x, params, None, wrt_x=True)
    _, rout = oracle.mlp_forward(_spec(wl), x, params)
    _compare(wl, got, rl, rg, rdx, rout)


def test_c4_full_batch_repeated_rows():
    wl = workloads.WORKLOADS["c4"]
    base = 128
    xb, params, _ = workloads.make_inputs(wl, batch=base, bias_scale=0.05)
    x, _, idx = workloads.repeat_rows(xb, None, wl.batch)
    got = _run(wl, x, params, None)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), xb, params, None, wrt_x=True)
    _, rout = oracle.mlp_forward(_spec(wl), xb, params)
    _compare(wl, got, rl, rg, rdx[idx] * (base / wl.batch), rout[idx])


def test_c5_reduced_batch():
    wl = workloads.WORKLOADS["c5"]
    x, params, y = workloads.make_inputs(wl, batch=64, bias_scale=0.05)
    got = _run(wl, x, params, y)
    rl, rg, _ = oracle.mlp_gradient(_spec(wl), x, params, y)
    _, rout = oracle.mlp_forward(_spec(wl), x, params, y)
    _compare(wl, got, rl, rg, None, rout, layer_tols=_order_tolerances(wl, x, params, y, rg),
             rows=False)


def test_c5_full_batch_repeated_rows_and_sgd():
    import torch
    wl = workloads.WORKLOADS["c5"]
    base = 64
    xb, params, yb = workloads.make_inputs(wl, batch=base, bias_scale=0.05)
    x, y, idx = workloads.repeat_rows(xb, yb, wl.batch)
    got = _run(wl, x, params, y)
    rl, rg, _ = oracle.mlp_gradient(_spec(wl), xb, params, yb)
    _, rout = oracle.mlp_forward(_spec(wl), xb, params, yb)
    _compare(wl, got, rl, rg, None, rout[idx],
             layer_tols=_order_tolerances(wl, xb, params, yb, rg), rows=False)
    # the fused update over the whole 138M-parameter buffer: master and bf16 shadow
    m, P = got["model"], got["P"]
    master = m.pack(params, device(), torch.float32)
    m.sgd_step(P, master, got["dparams"], wl.lr)
    torch.cuda.synchronize()
    for l, ((gW, gb), (mW, mb)) in enumerate(zip(m.unpack(P), m.unpack(master))):
        (W0, b0), (rdW, rdb) = params[l], rg[l]
        assert rel_l2(to_np(mW), oracle.sgd_f32(W0, rdW, wl.lr)) <= 1e-4
        assert rel_l2(to_np(mb), oracle.sgd_f32(b0, rdb, wl.lr)) <= 1e-3
        # the shadow is the round-to-nearest-even bf16 of the new master
        assert torch.equal(gW, mW.to(torch.bfloat16))
        assert torch.equal(gb, mb.to(torch.bfloat16))


def test_bf16_storage_effect_against_exact_math():
    """bf16 storage of the hidden activations changes the function itself.

    The gate above compares against the network with those storage casts. Here
    the same GPU gradient is compared with the exact function of the rounded
    inputs (no activation casts): the difference is the effect of bf16 storage
    and stays within a few percent on this network.
    """
    wl = workloads.WORKLOADS["c3"]
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    got = _run(wl, x, params, y, forward=False)
    exact = oracle.MlpSpec(wl.widths, wl.acts, wl.loss, wl.dtype, storage_casts=False)
    rl, rg, _ = oracle.mlp_gradient(exact, x, params, y)
    assert abs(got["loss"] - rl) <= 1e-2 * abs(rl)
    for l, ((gw, gb), (rw, rb)) in enumerate(zip(got["grads"], rg)):
        assert rel_l2(gw, rw) <= 0.06, l
        assert rel_l2(gb, rb) <= 0.06, l


@pytest.mark.parametrize("name,batch", [("c2", 256), ("c1", 16), ("c3", 64), ("c4", 32)])
def test_step_graph_replays_match_eager_steps(name, batch):
    """A captured training step replayed K times equals K eager steps, bit for bit.

    Between replays the program does eager work of its own on the same stream
    and synchronises; every replay's loss, gradient and updated parameters are
    checked against the eager sequence (the kernels are deterministic).
    """
    import torch
    from dataclasses import replace
    wl = replace(workloads.WORKLOADS[name], batch=batch)
    x, params, y = workloads.make_inputs(wl, bias_scale=0.05)
    dev = device()
    m = dl.Model(wl.widths, wl.acts, wl.dtype, wl.loss, wl.wrt_x, batch)
    tdt = torch_dtype(wl.dtype)
    update = True
    lr = 0.05

    def fresh():
        P = m.pack(params, dev, tdt)
        master = m.pack(params, dev, torch.float32) if wl.dtype == "bf16" else None
        return P, master

    xd = to_dev(x, wl.dtype)
    yd = None if y is None else torch.from_numpy(np.asarray(y, np.int32)).to(dev)
    ws = torch.empty(m.workspace_bytes(batch), dtype=torch.uint8, device=dev)
    steps = 4
    # eager reference sequence
    P, master = fresh()
    loss = torch.empty(1, device=dev)
    dP = torch.empty(m.param_count(), device=dev)
    dx = torch.empty((batch, wl.widths[0]), device=dev) if wl.wrt_x else None
    ref = []
    for _ in range(steps):
        m.gradient(P, xd, yd, batch, loss, dP, dx, ws)
        m.sgd_step(P, master, dP, lr)
        torch.cuda.synchronize()
        ref.append((loss.clone(), dP.clone(), P.clone(), None if dx is None else dx.clone()))
    # captured step on fresh parameters and fresh output buffers
    P2, master2 = fresh()
    ws2 = torch.empty_like(ws)
    loss2 = torch.empty(1, device=dev)
    dP2 = torch.empty(m.param_count(), device=dev)
    dx2 = torch.empty_like(dx) if dx is not None else None
    g = m.step_graph(P2, master2, xd, yd, batch, loss2, dP2, dx2, ws2, update=update, lr=lr)
    scratch = torch.zeros(1 << 16, device=dev)
    for k in range(steps):
        g.launch()
        scratch.mul_(0.5).add_(float(k))  # eager work between replays
        torch.cuda.synchronize()
        rl, rdp, rp, rdx = ref[k]
        assert torch.equal(loss2, rl), (k, loss2.item(), rl.item())
        assert torch.equal(dP2, rdp), k
        assert torch.equal(P2, rp), k
        if rdx is not None:
            assert torch.equal(dx2, rdx), k
    assert m.check(ws2) == dl.OK
    del g


@pytest.mark.parametrize("dtype,widths,batch", [("f32", (64, 32, 10), 8200), ("bf16", (64, 40, 10), 8200),
                                                ("bf16", (128, 256, 24), 4160)])
def test_split_batch_reduction(dtype, widths, batch):
    """Adjoint products wrt the weights with few output tiles and a long batch
    reduction are computed in k-slices summed in slice order (the plan shows
    the split and its reduction launch); the gradient matches the oracle. The
    batches are not multiples of the slice length, so the last slice is ragged."""
    import torch
    from dataclasses import replace
    wl = replace(workloads.WORKLOADS["c1"], widths=widths, acts=("tanh", "none"), dtype=dtype,
                 batch=batch, x_init=("normal_var", 1.0), w_init=("kaiming_normal",))
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    m = dl.Model(wl.widths, wl.acts, dtype, "softmax_ce", False, batch)
    names = [e["name"] for e in m.plan(batch)]
    assert "splitk_reduce" in names, names
    got = _run(wl, x, params, y, wrt_x=False, forward=False)
    rl, rg, _ = oracle.mlp_gradient(_spec(wl), x, params, y)
    _compare(wl, got, rl, rg)
    # deterministic: a second call gives the same bits
    again = _run(wl, x, params, y, wrt_x=False, forward=False)
    for (a, b), (c, d) in zip(got["grads"], again["grads"]):
        assert np.array_equal(a, c) and np.array_equal(b, d)


@pytest.mark.parametrize("name,batch,wrt_x", [("c1", 16, True), ("c2", 256, False), ("c2", 37, True),
                                              ("c3", 512, False), ("c3", 300, True)])
def test_vjp_against_oracle(name, batch, wrt_x):
    """The seedable gradient of the logits (dlvm_vjp) for a random seed, against
    the oracle's seedable gradient declaration."""
    import torch
    from dataclasses import replace
    wl = replace(workloads.WORKLOADS[name], batch=batch)
    x, params, _ = workloads.make_inputs(wl, bias_scale=0.1)
    seed = (np.random.default_rng([41, batch]).standard_normal((batch, wl.widths[-1])) /
            batch).astype(np.float32)
    dev = device()
    m = dl.Model(wl.widths, wl.acts, wl.dtype, wl.loss, wrt_x, batch)
    P = m.pack(params, dev, torch_dtype(wl.dtype))
    ws = torch.empty(m.workspace_bytes(batch), dtype=torch.uint8, device=dev)
    dP = torch.full((m.param_count(),), float("nan"), device=dev)
    dx = torch.empty((batch, wl.widths[0]), device=dev) if wrt_x else None
    m.vjp(P, to_dev(x, wl.dtype), to_dev(seed), batch, dP, dx, ws)
    torch.cuda.synchronize()
    rg, rdx = oracle.mlp_vjp(_spec(wl), x, params, seed, wrt_x=wrt_x)
    tol = TOL[wl.dtype]
    for (gw, gb), (rw, rb) in zip(m.unpack(dP), rg):
        assert rel_l2(to_np(gw), rw) <= tol
        assert rel_l2(to_np(gb), rb) <= tol
    if wrt_x:
        assert rel_l2(to_np(dx), rdx) <= tol
    # the flat buffer's padding is zero
    offs, lds = m.param_layout_lds()
    used = torch.zeros(m.param_count(), dtype=torch.bool, device=dev)
    for l in range(m.n_layers):
        K, N = wl.widths[l], wl.widths[l + 1]
        used[offs[2 * l]:offs[2 * l] + K * lds[l]] = True
        used[offs[2 * l + 1]:offs[2 * l + 1] + N] = True
    assert torch.count_nonzero(dP[~used]).item() == 0
    pad = [Wp[:, wl.widths[l + 1]:] for l, (Wp, _) in enumerate(m.unpack(dP, padded=True))]
    assert all(torch.count_nonzero(t).item() == 0 for t in pad)


def test_vjp_with_loss_adjoint_matches_gradient():
    """Seeding the logits with the loss adjoint (p - onehot)/B reproduces the
    gradient call's parameter gradient (f32 network)."""
    import torch
    wl = workloads.WORKLOADS["c2"]
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    got = _run(wl, x, params, y)
    z = got["forward"]
    p = np.exp(z - z.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    seed = ((p - np.eye(wl.widths[-1])[y]) / wl.batch).astype(np.float32)
    m, P, ws = got["model"], got["P"], got["ws"]
    dP = torch.empty(m.param_count(), device=device())
    m.vjp(P, to_dev(x), to_dev(seed), wl.batch, dP, None, ws)
    torch.cuda.synchronize()
    for (a, b), (c, d) in zip(m.unpack(dP), got["grads"]):
        assert rel_l2(to_np(a), c) <= 1e-5
        assert rel_l2(to_np(b), d) <= 1e-5


def _grad_with_ckpt(wl, x, params, y, k, wrt_x, seed=None):
    import torch
    B = x.shape[0]
    dev = device()
    m = dl.Model(wl.widths, wl.acts, wl.dtype, wl.loss, wrt_x, B, checkpoint_every=k)
    P = m.pack(params, dev, torch_dtype(wl.dtype))
    ws = torch.full((m.workspace_bytes(B),), 0xFF, dtype=torch.uint8, device=dev)
    dP = torch.full((m.param_count(),), float("nan"), device=dev)
    dx = torch.empty((B, wl.widths[0]), device=dev) if wrt_x else None
    loss = torch.zeros(1, device=dev)  # dlvm_vjp writes no loss
    if seed is None:
        yd = torch.from_numpy(np.asarray(y, np.int32)).to(dev)
        m.gradient(P, to_dev(x, wl.dtype), yd, B, loss, dP, dx, ws)
    else:
        m.vjp(P, to_dev(x, wl.dtype), to_dev(seed), B, dP, dx, ws)
    torch.cuda.synchronize()
    return loss.cpu(), dP.cpu(), None if dx is None else dx.cpu()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("entry", ["gradient", "vjp"])
def test_checkpointing_is_bitwise_neutral(dtype, entry):
    """Checkpointing (section 3.1.3) recomputes dropped layer outputs with the
    same deterministic kernels: loss, parameter and input gradients are bitwise
    those of the keep-everything plan, for every segment length."""
    import torch
    from dataclasses import replace
    wl = replace(workloads.WORKLOADS["c5"], widths=(96,) + (136,) * 8 + (10,), dtype=dtype,
                 batch=300)
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    seed = None
    if entry == "vjp":
        seed = (np.random.default_rng(5).standard_normal((wl.batch, 10)) / wl.batch).astype(np.float32)
    ref = _grad_with_ckpt(wl, x, params, y, 1, True, seed)
    assert not torch.isnan(ref[1]).any()
    for k in (2, 3, 4, 8, 9):
        got = _grad_with_ckpt(wl, x, params, y, k, True, seed)
        for a, b in zip(got, ref):
            assert torch.equal(a, b), k


def test_checkpointing_c5_against_oracle():
    """The c5 network (8 hidden layers of 4096) with only every third hidden
    output kept, against the oracle at a reduced batch."""
    wl = workloads.WORKLOADS["c5"]
    x, params, y = workloads.make_inputs(wl, batch=64, bias_scale=0.05)
    loss, dP, _ = _grad_with_ckpt(wl, x, params, y, 3, False)
    rl, rg, _ = oracle.mlp_gradient(_spec(wl), x, params, y)
    m = dl.Model(wl.widths, wl.acts, wl.dtype, wl.loss, False, 64)
    tols = _order_tolerances(wl, x, params, y, rg)
    assert abs(loss.item() - rl) <= TOL["bf16"] * abs(rl)
    for (gw, gb), (rw, rb), (tw, tb) in zip(m.unpack(dP), rg, tols):
        assert rel_l2(to_np(gw), rw) <= tw
        assert rel_l2(to_np(gb), rb) <= tb


def test_vjp_rejects_chain_models():
    import torch
    wl = workloads.WORKLOADS["c4"]
    m = dl.Model((64, 64), ("none",), "f32", "chain8", True, 8)
    A = torch.zeros(1 << 16, device=device())
    ws = torch.empty(m.workspace_bytes(8), dtype=torch.uint8, device=device())
    with pytest.raises(dl.DlvmError) as e:
        m.vjp(A, A, A, 8, A, A, ws)
    assert e.value.status == dl.ERR_UNSUPPORTED


def _chain_run(wl, x, params, chain_in_epilogue, B):
    import torch
    dev = device()
    m = dl.Model(wl.widths, wl.acts, wl.dtype, wl.loss, True, B,
                 chain_in_epilogue=chain_in_epilogue)
    P = m.pack(params, dev, torch.float32)
    ws = torch.full((m.workspace_bytes(B),), 0xFF, dtype=torch.uint8, device=dev)
    loss = torch.empty(1, device=dev)
    dP = torch.full((m.param_count(),), float("nan"), device=dev)
    dx = torch.full((B, wl.widths[0]), float("nan"), device=dev)
    m.gradient(P, to_dev(x), None, B, loss, dP, dx, ws)
    torch.cuda.synchronize()
    assert m.check(ws) == dl.OK
    return loss.item(), dP.cpu(), dx.cpu(), m


@pytest.mark.parametrize("widths,batch,cfg", [((4096, 4096), 256, None), ((200, 200), 300, None)] +
                         [((200, 200), 300, c) for c in (6, 7, 8, 9, 20, 21, 22, 23)])
def test_chain_in_epilogue(widths, batch, cfg, monkeypatch):
    """The eight-operator chain run in the dense product's epilogue (z never
    stored) against the oracle and, bit for bit in dparams and dx, against the
    standalone chain kernel (same element arithmetic; only the loss partials
    are grouped differently). Every configuration that has the epilogue forced."""
    from dataclasses import replace
    if cfg is not None:
        monkeypatch.setenv("DLVM_GEMM_CONFIG", str(cfg))
    wl = replace(workloads.WORKLOADS["c4"], widths=widths, batch=batch)
    x, params, _ = workloads.make_inputs(wl, bias_scale=0.05)
    l1, g1, d1, m = _chain_run(wl, x, params, True, batch)
    l0, g0, d0, _ = _chain_run(wl, x, params, False, batch)
    assert torch_equal(g1, g0) and torch_equal(d1, d0)
    assert abs(l1 - l0) <= 1e-6 * abs(l0)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), x, params, None, wrt_x=True)
    assert abs(l1 - rl) <= TOL["f32"] * abs(rl)
    (gW, gb), = m.unpack(g1)
    assert rel_l2(to_np(gW), rg[0][0]) <= TOL["f32"]
    assert rel_l2(to_np(gb), rg[0][1]) <= TOL["f32"]
    assert rel_l2(to_np(d1), rdx) <= TOL["f32"]
    names = [p["name"] for p in m.plan(batch)]
    assert any(n.startswith("gemm_nn_chain8") and (cfg is None or n.endswith(f"c{cfg}")) for n in names)
    assert "chain8" not in names


def torch_equal(a, b):
    import torch
    return bool(torch.equal(a, b))



@pytest.mark.parametrize("widths,acts,batch,wrt_x", [
    ((64, 32, 10), ("sigmoid", "none"), 16, False),             # c1
    ((64, 32, 10), ("sigmoid", "none"), 16, True),
    ((37, 50, 23, 10), ("relu", "tanh", "none"), 7, True),      # ragged widths and batch
    ((96, 48, 48, 40, 30), ("tanh", "relu", "sigmoid", "none"), 9, False),
    ((20, 300), ("none",), 5, True),                             # one layer, wide head
    ((6, 3), ("none",), 600, True),                              # a large batch (LDS nearly full)
    ((8, 8, 4), ("relu", "none"), 400, False),
    ((12,) * 8 + (10,), ("tanh",) * 7 + ("none",), 8, True),     # the most layers it takes
    ((1,) * 8 + (2,), ("tanh",) * 7 + ("none",), 840, True),     # rows end to end: padded they do not fit
])
def test_small_network_path(widths, acts, batch, wrt_x, monkeypatch):
    """The one-workgroup gradient of a small float32 network against the
    oracle and against the general multi-launch plan (DLVM_SMALL_STEP=0)."""
    from dataclasses import replace
    wl = replace(workloads.WORKLOADS["c1"], widths=widths, acts=acts, batch=batch, wrt_x=wrt_x)
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    m = dl.Model(wl.widths, wl.acts, wl.dtype, wl.loss, wrt_x, batch)
    assert m.plan(batch)[0]["name"] == "small_step_f32"
    got = _run(wl, x, params, y, wrt_x=wrt_x, forward=False)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), x, params, y, wrt_x=wrt_x)
    _compare(wl, got, rl, rg, rdx if wrt_x else None)
    again = _run(wl, x, params, y, wrt_x=wrt_x, forward=False)   # fixed summation order
    assert again["loss"] == got["loss"]
    assert bool((again["dparams"] == got["dparams"]).all())
    monkeypatch.setenv("DLVM_SMALL_STEP", "0")
    gen = _run(wl, x, params, y, wrt_x=wrt_x, forward=False)
    assert abs(got["loss"] - gen["loss"]) <= 1e-5 * abs(gen["loss"])
    for (a, b), (c, d) in zip(got["grads"], gen["grads"]):
        assert rel_l2(a, c) <= 1e-5 and rel_l2(b, d) <= 1e-5
    # the padding of dparams is zero on both paths
    import torch
    dP = got["dparams"]
    offs, lds = m.param_layout_lds()
    used = torch.zeros(m.param_count(), dtype=torch.bool, device=dP.device)
    for l in range(m.n_layers):
        used[offs[2 * l]:offs[2 * l] + widths[l] * lds[l]] = True
        used[offs[2 * l + 1]:offs[2 * l + 1] + widths[l + 1]] = True
    assert torch.count_nonzero(dP[~used]).item() == 0



@pytest.mark.parametrize("dtype,cfg", [("f32", c) for c in (0, 1, 3, 4, 5)] +
                         [("bf16", c) for c in range(6)])
@pytest.mark.parametrize("batch", [300, 7])
def test_forced_tile_configurations(dtype, cfg, batch, monkeypatch):
    """Every register-staged tile configuration forced on a ragged network,
    against the oracle: in bf16 the forward (NN), the adjoint wrt the input (NT)
    and wrt the weights (TN, paired with NT where the configuration allows), in
    float32 the rectified layer's forward, which alone runs on these tiles. The
    contraction lengths 520, 300, 150, 72 and 10 give odd, even and single
    stage counts (128 k per stage in float32, 256 in bf16 for the 4-segment
    tiles) and K not a multiple of the vector width (150, 10, and a batch of 7
    for the products wrt the weights), where a row's last load starts early or
    goes element by element."""
    from dataclasses import replace
    monkeypatch.setenv("DLVM_GEMM_CONFIG", str(cfg))
    base = workloads.WORKLOADS["c2" if dtype == "f32" else "c3"]
    wl = replace(base, widths=(520, 150, 72, 10), acts=("tanh", "relu", "none"), batch=batch,
                 wrt_x=True)
    m = dl.Model(wl.widths, wl.acts, wl.dtype, wl.loss, True, batch)
    names = [re.sub(r"s\d+$", "", p["name"]) for p in m.plan(batch) if p["name"].startswith("gemm")]
    names = [n for n in names if "xent" not in n]  # (ten classes: the head runs on its own tile)
    forced = [n.split("_")[1] for n in names if n.endswith(f"c{cfg}")]
    if dtype == "f32":                                     # 520-150 is tanh, 150-72 rectified
        assert forced == ["nn"] and names[1].endswith(f"c{cfg}"), names
    elif cfg == 2:                                         # outputs of at most 32 columns
        assert forced == ["tn"], names
    else:
        assert forced == [n.split("_")[1] for n in names], names
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    got = _run(wl, x, params, y, wrt_x=True)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), x, params, y, wrt_x=True)
    _, ref_out = oracle.mlp_forward(_spec(wl), x, params, y)
    _compare(wl, got, rl, rg, rdx, ref_out=ref_out)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("splits", [2, 4])
def test_split_hidden_layer_products(dtype, splits, monkeypatch):
    """The hidden layers' forward products split over k (forced through
    DLVM_GEMM_SPLITS): the slices are summed in slice order and the bias and
    activation applied after the sum; against the oracle, and two runs bitwise
    equal."""
    from dataclasses import replace
    monkeypatch.setenv("DLVM_GEMM_SPLITS", str(splits))
    base = workloads.WORKLOADS["c2" if dtype == "f32" else "c3"]
    wl = replace(base, widths=(1024, 520, 264, 10), acts=("tanh", "relu", "none"), batch=200,
                 wrt_x=True)
    m = dl.Model(wl.widths, wl.acts, wl.dtype, wl.loss, True, wl.batch)
    names = [p["name"] for p in m.plan(wl.batch)]
    assert names[0].startswith("gemm_nn") and names[0].endswith(f"s{splits}")
    assert names[1] == "split_epilogue"
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    got = _run(wl, x, params, y, wrt_x=True)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), x, params, y, wrt_x=True)
    _, rout = oracle.mlp_forward(_spec(wl), x, params, y)
    _compare(wl, got, rl, rg, rdx, ref_out=rout)
    again = _run(wl, x, params, y, wrt_x=True, forward=False)
    assert again["loss"] == got["loss"]
    assert bool((again["dparams"] == got["dparams"]).all())


@pytest.mark.parametrize("seed", range(12))
def test_small_network_random_shapes(seed, monkeypatch):
    """Seeded random small networks (1-4 layers, widths 1-80, batch 1-64,
    random activations, with and without dx) through the one-workgroup
    gradient, against the oracle and the multi-launch plan."""
    from dataclasses import replace
    rng = np.random.default_rng(900 + seed)
    L = int(rng.integers(1, 5))
    widths = tuple(int(v) for v in rng.integers(1, 81, size=L + 1))
    widths = widths[:-1] + (max(widths[-1], 2),)          # at least two classes
    acts = tuple(str(a) for a in rng.choice(["none", "relu", "tanh", "sigmoid"], size=L - 1)) + ("none",)
    batch = int(rng.integers(1, 65))
    wrt_x = bool(rng.integers(0, 2))
    while dl.Model(widths, acts, "f32", "softmax_ce", wrt_x, batch).plan(batch)[0]["name"] \
            != "small_step_f32":
        assert batch > 1, widths
        batch //= 2                                       # until it fits the workgroup's LDS
    wl = replace(workloads.WORKLOADS["c1"], widths=widths, acts=acts, batch=batch, wrt_x=wrt_x)
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    got = _run(wl, x, params, y, wrt_x=wrt_x, forward=False)
    rl, rg, rdx = oracle.mlp_gradient(_spec(wl), x, params, y, wrt_x=wrt_x)
    _compare(wl, got, rl, rg, rdx if wrt_x else None)
    monkeypatch.setenv("DLVM_SMALL_STEP", "0")
    gen = _run(wl, x, params, y, wrt_x=wrt_x, forward=False)
    assert abs(got["loss"] - gen["loss"]) <= 1e-5 * max(abs(gen["loss"]), 1e-30)
    for (a, b), (c, d) in zip(got["grads"], gen["grads"]):
        assert rel_l2(a, c) <= 1e-5 and rel_l2(b, d) <= 1e-5
