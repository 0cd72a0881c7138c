"""The float32 product kernels, every tile configuration forced: the waves that
share the contraction (6-9 and 23, gemm_wave.hpp), the tiles staged in LDS (20-22,
gemm_f32.hpp) and the element-load fallback for leading dimensions beyond their
byte offsets (3), in all three layouts and the two-phase cell product.

Bound: a float32 sum of K products, in any order, differs from the exact sum by at
most about K 2^-24 times the sum of the terms' magnitudes (element by element;
8 more roundings are allowed for the epilogue). A single wrong or missing term is
about 1/K of that sum, far outside for these K.
"""
import re

import numpy as np
import pytest

import oracle
import paper_1711_03016_amd as dl
from helpers import assert_close, assert_forced, device, planned_config, to_dev, to_np

pytestmark = pytest.mark.gpu

CFGS = [6, 7, 8, 9, 20, 21, 22, 23]
# (M, N, K): smaller than one step and one tile, exact tiles, one past a tile in every
# size, sizes that no vector load divides, fewer steps than waves, many k-tiles, two and
# three columns past a tile of 64
SHAPES = [(1, 1, 1), (5, 3, 7), (128, 128, 32), (129, 65, 33), (17, 33, 130), (64, 130, 64),
          (67, 259, 96), (250, 77, 515), (33, 18, 2056), (30, 67, 66), (30, 66, 67)]


def _near(got, ref, magnitude, K, what):
    off = np.abs(np.asarray(got, np.float64) - ref)
    lim = (K + 8) * 2.0 ** -24 * magnitude
    assert got.shape == ref.shape and np.isfinite(got).all(), what
    assert (off <= lim).all(), (what, float((off / lim).max()))


@pytest.fixture(params=CFGS)
def cfg(request, monkeypatch):
    monkeypatch.setenv("DLVM_GEMM_CONFIG", str(request.param))
    return request.param


def _layer(M, N, K):
    import torch
    r = np.random.default_rng([31, M, N, K])
    X = r.standard_normal((M, K)).astype(np.float32)
    W = (r.standard_normal((K, N)) / np.sqrt(K)).astype(np.float32)
    b = r.uniform(-0.5, 0.5, N).astype(np.float32)
    dY = r.standard_normal((M, N)).astype(np.float32)
    R = r.standard_normal((M, K)).astype(np.float32)
    H, dX = (torch.full(s, float("nan"), device=device()) for s in ((M, N), (M, K)))
    dW, db = (torch.full(s, float("nan"), device=device()) for s in ((K, N), (N,)))
    Xd, Wd, bd, dYd = (to_dev(a) for a in (X, W, b, dY))
    dl.dense_forward("f32", "f32", "none", M, N, K, 0.75, Xd, Wd, bd, H)
    dl.dense_backward_data("f32", "f32", "tanh", M, N, K, dYd, Wd, to_dev(np.tanh(X)), to_dev(R), dX)
    dl.dense_backward_params("f32", M, N, K, Xd, dYd, dW, db)
    torch.cuda.synchronize()
    X, W, b, dY, R = (a.astype(np.float64) for a in (X, W, b, dY, R))
    t = np.tanh(X.astype(np.float32)).astype(np.float64)
    aX, aW, aY = np.abs(X), np.abs(W), np.abs(dY)
    _near(to_np(H), 0.75 * (X @ W) + b, aX @ aW + np.abs(b), K, "H")
    _near(to_np(dX), (dY @ W.T) * (1 - t * t) + R, aY @ aW.T + np.abs(R), N, "dX")
    _near(to_np(dW), X.T @ dY, aX.T @ aY, M, "dW")
    _near(to_np(db), dY.sum(0), aY.sum(0), M, "db")


@pytest.mark.parametrize("shape", SHAPES)
def test_layer(cfg, shape):
    assert_forced(cfg, *shape, "f32")
    _layer(*shape)


def _error_of_sums(a, b, parts):
    """Relative error of the dot products of a's rows with b's rows when each is `parts`
    float32 sums, one after the other, that are then added up in pairs."""
    n, K = a.shape
    k = np.concatenate([np.arange(K), np.full(-K % parts, -1)]).reshape(-1, parts)
    acc = np.zeros((n, parts), np.float32)
    for q in k:
        t = a[:, q].astype(np.float64) * b[:, q].astype(np.float64) * (q >= 0)
        acc = (acc + t).astype(np.float32)
    while acc.shape[1] > 1:
        acc = acc[:, ::2] + acc[:, 1::2]
    ref = (a.astype(np.float64) * b).sum(1)
    return np.linalg.norm(acc[:, 0] - ref) / np.linalg.norm(ref)


# Sums that each configuration keeps of one output: its waves or k-groups times its
# accumulators (one network's products may run on any of them, so a longer sum is an error
# that grows from one size to the next).
SUMS = {6: 32, 7: 32, 8: 8, 9: 4, 20: 1, 21: 4, 22: 2, 23: 8}


def test_sums_are_kept_in_parts(cfg):
    """The error of all three products against float64 is that of sums in as many parts as
    the configuration keeps (15% for the sample and for what the order of the parts adds;
    half as many parts are 1.41 times as far off)."""
    import torch
    M = N = K = 1000
    r = np.random.default_rng(34)
    X, W, dY = (r.standard_normal((1000, 1000)).astype(np.float32) for _ in range(3))
    H, dX, dW = (torch.empty((1000, 1000), device=device()) for _ in range(3))
    dl.dense_forward("f32", "f32", "none", M, N, K, 1.0, to_dev(X), to_dev(W), None, H)
    dl.dense_backward_data("f32", "f32", "none", M, N, K, to_dev(dY), to_dev(W), None, None, dX)
    dl.dense_backward_params("f32", M, N, K, to_dev(X), to_dev(dY), dW, None)
    torch.cuda.synchronize()
    want = _error_of_sums(r.standard_normal((4000, 1000)).astype(np.float32),
                          r.standard_normal((4000, 1000)).astype(np.float32), SUMS[cfg])
    X, W, dY = (a.astype(np.float64) for a in (X, W, dY))
    for got, ref, what in ((H, X @ W, "NN"), (dX, dY @ W.T, "NT"), (dW, X.T @ dY, "TN")):
        off = np.linalg.norm(to_np(got) - ref) / np.linalg.norm(ref)
        assert off <= 1.15 * want, (what, off, want)


@pytest.mark.parametrize("shape", [(3, (1 << 22) + 24, 5), (2, 9, (1 << 22) + 4)])
def test_far_leading_dimensions(shape):
    """Rows of more than 2^22 elements: the byte offsets of a step would pass 2^31."""
    _layer(*shape)


@pytest.mark.parametrize("M,Kx,Kh", [(33, 7, 20), (64, 100, 256), (130, 33, 64), (17, 1, 1), (50, 48, 5)])
def test_two_phase_cell(cfg, M, Kx, Kh):
    """Both phases end inside a step; each reads its own operand up to its own end."""
    import torch
    assert planned_config("nn", "f32", M, Kh, Kx + Kh, Kx) == cfg
    r = np.random.default_rng([32, M, Kx, Kh])
    X = r.standard_normal((M, Kx)).astype(np.float32)
    H = r.standard_normal((M, Kh)).astype(np.float32)
    WU = (r.standard_normal((Kx + Kh, Kh)) / np.sqrt(Kx + Kh)).astype(np.float32)
    b = r.uniform(-0.1, 0.1, Kh).astype(np.float32)
    out = torch.full((M, Kh), float("nan"), device=device())
    dl.rnn_cell_forward("f32", "tanh", M, Kx, Kh, Kh, to_dev(X), to_dev(H), to_dev(WU), to_dev(b), out)
    torch.cuda.synchronize()
    XH = np.concatenate([X, H], axis=1).astype(np.float64)
    WU = WU.astype(np.float64)
    _near(to_np(out), np.tanh(XH @ WU + b), np.abs(XH) @ np.abs(WU) + 1, Kx + Kh, "cell")


def test_values_outside_the_operand_are_not_read(cfg):
    """What lies past the last k or row of an operand (here NaN) reaches no output."""
    import torch
    M, N, K = 37, 45, 27
    r = np.random.default_rng(33)
    X = r.standard_normal((M, K)).astype(np.float32)
    W = r.standard_normal((K, N)).astype(np.float32)
    pad = torch.full((8192,), float("nan"), device=device())
    xb, wb = pad.clone(), pad.clone()
    xb[:M * K] = to_dev(X).reshape(-1)
    wb[:K * N] = to_dev(W).reshape(-1)
    H, dW = torch.empty((M, N), device=device()), torch.empty((K, N), device=device())
    dl.dense_forward("f32", "f32", "none", M, N, K, 1.0, xb, wb, None, H)
    yb = pad.clone()
    yb[:M * N] = H.reshape(-1)
    dl.dense_backward_params("f32", M, N, K, xb, yb, dW, None)
    torch.cuda.synchronize()
    X, W, Hn = X.astype(np.float64), W.astype(np.float64), to_np(H)
    _near(Hn, X @ W, np.abs(X) @ np.abs(W), K, "H")
    _near(to_np(dW), X.T @ Hn, np.abs(X.T) @ np.abs(Hn), M, "dW")


@pytest.mark.parametrize("widths,batch", [((130, 70, 33, 20), 77), ((96, 512, 512, 12), 200)])
def test_paired_adjoints(cfg, widths, batch, monkeypatch):
    """A network's gradient with the configuration forced on every product: the
    adjoint pairs share a launch; against the oracle and bit for bit on a second call."""
    import torch
    import workloads
    from dataclasses import replace
    monkeypatch.setenv("DLVM_SMALL_STEP", "0")
    wl = replace(workloads.WORKLOADS["c2"], widths=widths, acts=("tanh", "sigmoid", "none"), batch=batch)
    x, params, y = workloads.make_inputs(wl, bias_scale=0.1)
    m = dl.Model(widths, wl.acts, "f32", "softmax_ce", True, batch)
    names = [p["name"] for p in m.plan(batch)]
    assert any(n.startswith("gemm_pair") for n in names)
    assert all(re.search(rf"c{cfg}(s\d+)?$", n) for n in names if n.startswith("gemm") and "xent" not in n), names
    P = m.pack(params, device(), torch.float32)
    ws = torch.empty(m.workspace_bytes(batch), dtype=torch.uint8, device=device())
    outs = []
    for _ in range(2):
        loss, dx = torch.empty(1, device=device()), torch.empty((batch, widths[0]), device=device())
        dP = torch.full((m.param_count(),), float("nan"), device=device())
        m.gradient(P, to_dev(x), torch.from_numpy(y).to(device()), batch, loss, dP, dx, ws)
        torch.cuda.synchronize()
        outs.append((loss, dP, dx))
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    rl, rg, rdx = oracle.mlp_gradient(oracle.MlpSpec(widths, wl.acts), x, params, y,
                                      wrt_x=True)
    assert abs(outs[0][0].item() - rl) <= 1e-5 * abs(rl)
    assert_close(to_np(outs[0][2]), rdx, 1e-5, "dx", row_tol=1e-4)
    for (gW, gb), (rW, rb) in zip(m.unpack(outs[0][1]), rg):
        assert_close(to_np(gW), rW, 1e-5, "dW", row_tol=1e-4)
        assert_close(to_np(gb), rb, 1e-5, "db", row_tol=1e-4)
