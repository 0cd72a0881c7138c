"""bf16 products whose rows start anywhere: the waves that share the contraction
(6-9 and 23, gemm_wave.hpp) and the register-staged tiles (0-5), each configuration forced,
in all three layouts and the two-phase cell product, at sizes that no 16-byte load
divides (chunks shifted into place at the end of a row, element loads for rows
shorter than a chunk), between NaNs that must reach no output.

Operands are bf16, products and sums float32: the bound of a float32 output is
K 2^-24 times the sum of the terms' magnitudes (any order of the sum, 8 more
roundings for the epilogue), of a bf16 output one rounding (2^-8) of the value more.
"""
import numpy as np
import pytest

import paper_1711_03016_amd as dl
from helpers import assert_forced, device, planned_config, quant, to_np

pytestmark = pytest.mark.gpu

CFGS = [0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 23]
# (M, N, K): one element, rows shorter than a chunk, exactly one, one more; odd sizes past
# one tile of each configuration; sizes that aligned loads take; many steps; two and three
# columns past a tile of 64
SHAPES = [(1, 1, 1), (3, 5, 7), (9, 8, 9), (33, 17, 70), (129, 65, 131), (70, 257, 63), (64, 96, 256),
          (200, 34, 1027), (30, 67, 66), (30, 66, 67)]


@pytest.fixture(params=CFGS)
def cfg(request, monkeypatch):
    monkeypatch.setenv("DLVM_GEMM_CONFIG", str(request.param))
    return request.param


def _between_nans(a, dtype="bf16"):
    """The values of `a` in the storage type, on the device, NaNs right behind them."""
    import torch
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    n = a.size
    buf = torch.full((n + 4096,), float("nan"), dtype=td, device=device())
    buf[:n] = torch.from_numpy(np.ascontiguousarray(a)).reshape(-1).to(device()).to(td)
    return buf


def _near(got, ref, magnitude, K, out_dtype, what):
    lim = (K + 8) * 2.0 ** -24 * magnitude
    if out_dtype == "bf16":
        lim = lim + 2.0 ** -8 * np.abs(ref) * 1.01 + 2.0 ** -8 * lim
    got = np.asarray(got, np.float64)
    assert np.isfinite(got).all(), what
    off = np.abs(got - ref)
    assert (off <= lim).all(), (what, float((off / np.maximum(lim, 1e-300)).max()))


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
def test_layer(cfg, shape, out_dtype):
    import torch
    M, N, K = shape
    assert_forced(cfg, M, N, K, "bf16", lambda layout, n: cfg != 2 or n <= 32)  # (2: narrow outputs)
    r = np.random.default_rng([41, M, N, K])
    X = r.standard_normal((M, K)).astype(np.float32)
    W = (r.standard_normal((K, N)) / np.sqrt(K)).astype(np.float32)
    b = r.uniform(-0.5, 0.5, N).astype(np.float32)
    dY = r.standard_normal((M, N)).astype(np.float32)
    R = r.standard_normal((M, K)).astype(np.float32)
    T = np.tanh(X)
    td = torch.bfloat16 if out_dtype == "bf16" else torch.float32
    H, dX = (torch.full(s, float("nan"), dtype=td, device=device()) for s in ((M, N), (M, K)))
    dW, db = (torch.full(s, float("nan"), device=device()) for s in ((K, N), (N,)))
    Xd, Wd, bd, dYd, Td = (_between_nans(a) for a in (X, W, b, dY, T))
    dl.dense_forward("bf16", out_dtype, "none", M, N, K, 0.75, Xd, Wd, bd, H)
    dl.dense_backward_data("bf16", out_dtype, "tanh", M, N, K, dYd, Wd, Td, _between_nans(R, out_dtype), dX)
    dl.dense_backward_params("bf16", M, N, K, Xd, dYd, dW, db)
    torch.cuda.synchronize()
    X, W, b, dY, T = (quant(a, "bf16") for a in (X, W, b, dY, T))
    R = quant(R, out_dtype)
    aX, aW, aY = np.abs(X), np.abs(W), np.abs(dY)
    _near(to_np(H), 0.75 * (X @ W) + b, aX @ aW + np.abs(b), K, out_dtype, "H")
    _near(to_np(dX), (dY @ W.T) * (1 - T * T) + R, aY @ aW.T + np.abs(R), N, out_dtype, "dX")
    _near(to_np(dW), X.T @ dY, aX.T @ aY, M, "f32", "dW")
    _near(to_np(db), dY.sum(0), aY.sum(0), M, "f32", "db")


@pytest.mark.parametrize("M,Kx,Kh", [(33, 7, 20), (65, 100, 256), (130, 33, 61), (17, 1, 1), (50, 72, 9)])
def test_two_phase_cell(cfg, M, Kx, Kh):
    import torch
    assert (planned_config("nn", "bf16", M, Kh, Kx + Kh, Kx) == cfg) == (cfg != 2 or Kh <= 32)
    r = np.random.default_rng([42, M, Kx, Kh])
    X = r.standard_normal((M, Kx)).astype(np.float32)
    H = r.standard_normal((M, Kh)).astype(np.float32)
    WU = (r.standard_normal((Kx + Kh, Kh)) / np.sqrt(Kx + Kh)).astype(np.float32)
    b = r.uniform(-0.1, 0.1, Kh).astype(np.float32)
    out = torch.full((M, Kh), float("nan"), dtype=torch.bfloat16, device=device())
    dl.rnn_cell_forward("bf16", "tanh", M, Kx, Kh, Kh, *(_between_nans(a) for a in (X, H, WU, b)), out)
    torch.cuda.synchronize()
    XH = np.concatenate([quant(X, "bf16"), quant(H, "bf16")], axis=1)
    WU = quant(WU, "bf16")
    _near(to_np(out), np.tanh(XH @ WU + quant(b, "bf16")), np.abs(XH) @ np.abs(WU) + 1, Kx + Kh, "bf16",
          "cell")
