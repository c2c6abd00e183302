"""Gradient pass and normalisation of the learned escape at the edges of their
tilings: batches below, at and past one chunk of 32 samples and the eight
sample splits, batches with invalid records, record sets below, at and past the
256 chains and the 32,768 records of one round of the normalisation sums."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import mlp
from test_gpu_escape import NORM, NO, NP, _put, _rand_params, _records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 31, 32, 33, 257, 8225])
def test_gradient_of_ragged_batches(gpu_ctx, batch):
    """Mean gradient over the batch, every fifth record invalid (no gradient,
    still counted in the mean), against the bfloat16 emulation: the bounds of
    the full-size check."""
    import torch
    p = _rand_params(21)
    _put(gpu_ctx, p, NORM)
    rng = np.random.default_rng(22)
    nrec = 4000
    rec = _records(rng, nrec)
    rec[4::5, mlp.R_VALID] = 0.0
    idx = rng.integers(0, nrec, batch).astype(np.int32)
    idx[0] = 0
    u = rng.uniform(0, 1, (batch, 4))
    cond = rng.uniform(0, 1, batch) < 0.3
    uq = np.concatenate([u, cond[:, None].astype(np.float64)], axis=1)
    grad = torch.zeros(NP, dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    gpu_ctx.krt_escape_grad(torch.from_numpy(rec.astype(np.float32)).cuda(), torch.from_numpy(idx).cuda(),
                            torch.from_numpy(uq.astype(np.float32)).cuda(), grad, loss)
    g = grad.cpu().numpy().astype(np.float64)
    ok = rec[idx, mlp.R_VALID] > 0.5
    R = rec[idx[ok]].astype(np.float32).astype(np.float64)
    uf = u[ok].astype(np.float32).astype(np.float64)
    l_ref, g_ref = mlp.loss_and_grad(p, mlp.inputs(R, uf, cond[ok]), mlp.targets_normalised(R, NORM, cond[ok]),
                                     mlp.levels(uf, cond[ok]), bf=True, s9=NORM[NO + mlp.O_LOGN])
    share = ok.sum() / batch
    assert np.linalg.norm(g - share * g_ref) <= 2e-2 * share * np.linalg.norm(g_ref)
    assert abs(loss.item() / (share * l_ref) - 1) < 1e-2


@pytest.mark.parametrize("n", [1, 255, 257, 32768, 33001])
def test_normalisation_of_ragged_sets(gpu_ctx, n):
    """Mean and spread of each target over its valid records, and the ranges,
    against NumPy in FP64 (the kernel sums in FP64 and rounds once to FP32, its
    asinh is good to 2^-22 of a value)."""
    import torch
    gpu_ctx.krt_escape_init(1)
    rng = np.random.default_rng(n)
    rec = _records(rng, n).astype(np.float32)
    rec[3::7, mlp.R_VALID] = 0.0
    gpu_ctx.krt_escape_fit_norm(torch.from_numpy(rec).cuda(), n)
    w = torch.zeros(NP + 328, dtype=torch.float32, device="cuda")
    gpu_ctx.krt_escape_get_weights(w)
    norm = w[NP:].cpu().numpy().astype(np.float64)
    R = rec[rec[:, mlp.R_VALID] > 0.5].astype(np.float64)
    t = {mlp.O_LOGN: R[:, mlp.R_LOGN], mlp.O_LOGX2: R[:, mlp.R_LOGX2]}
    for f in range(6):
        t[16 + f] = np.abs(R[R[:, mlp.R_FACE] == f, mlp.R_XOUT])
    for k, col in ((9, mlp.R_YS), (10, mlp.R_YT)):
        t[k] = np.arcsinh(R[:, col])
    t[11], t[12] = R[:, mlp.R_MU] ** 2, R[:, mlp.R_ALPHA]
    for k in range(NO):
        y = t.get(k, np.zeros(0))
        mean, sd = (y.mean(), np.sqrt(max(y.var(), 1e-12))) if len(y) else (0.0, 1.0)
        scale = np.abs(y).max() if len(y) else 0.0
        assert abs(norm[k] - mean) <= 2.0 ** -21 * max(scale, 1e-30), k
        assert abs(norm[NO + k] ** 2 - sd ** 2) <= 2.0 ** -20 * max(scale ** 2, sd ** 2), k
    o = 2 * NO + 256
    assert norm[o] == R[:, 1].min() and norm[o + 1] == R[:, 1].max()
    assert norm[o + 2] == R[:, 0].min() and norm[o + 3] == R[:, 0].max()
    assert norm[o + 4] == R[:, 6].min()


@pytest.mark.parametrize("batch", [33, 257, 8192, 8225, 9001])
@pytest.mark.parametrize("where", ["last", "first chunk", "last chunk", "split end", "split start", "late split"])
def test_gradient_of_one_chunk_alone(gpu_ctx, batch, where):
    """Every row invalid but those of one place (the last sample, the first or
    last chunk of 32, the chunks on both sides of a boundary between the eight
    sample splits): the gradient is theirs alone, so a sample lost or doubled
    there is all of it.  Batches above 8192 take the kernel that shares a
    compute unit.  Bounds of the full-size check, the loss's relative to the
    size of its terms (about one each)."""
    import torch
    p = _rand_params(31)
    _put(gpu_ctx, p, NORM)
    rng = np.random.default_rng(32)
    rec = _records(rng, 1000)
    rec[500:, mlp.R_VALID] = 0.0
    nchunk = (batch + 31) // 32
    chunk = {"last": nchunk - 1, "first chunk": 0, "last chunk": nchunk - 1, "split end": max(nchunk * 3 // 8 - 1, 0),
             "split start": nchunk * 3 // 8, "late split": nchunk * 7 // 8}[where]
    rows = np.arange(32 * chunk, min(batch, 32 * chunk + 32)) if where != "last" else np.array([batch - 1])
    idx = rng.integers(500, 1000, batch).astype(np.int32)
    idx[rows] = rng.integers(0, 500, len(rows))
    u = rng.uniform(0, 1, (batch, 4))
    cond = rng.uniform(0, 1, batch) < 0.4
    uq = np.concatenate([u, cond[:, None].astype(np.float64)], axis=1)
    grad = torch.zeros(NP, dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    gpu_ctx.krt_escape_grad(torch.from_numpy(rec.astype(np.float32)).cuda(), torch.from_numpy(idx).cuda(),
                            torch.from_numpy(uq.astype(np.float32)).cuda(), grad, loss)
    g = grad.cpu().numpy().astype(np.float64)
    R = rec[idx[rows]].astype(np.float32).astype(np.float64)
    uf = u[rows].astype(np.float32).astype(np.float64)
    l_ref, g_ref = mlp.loss_and_grad(p, mlp.inputs(R, uf, cond[rows]), mlp.targets_normalised(R, NORM, cond[rows]),
                                     mlp.levels(uf, cond[rows]), bf=True, s9=NORM[NO + mlp.O_LOGN])
    share = len(rows) / batch
    assert np.linalg.norm(g_ref) > 0
    assert np.linalg.norm(g - share * g_ref) <= 2e-2 * share * np.linalg.norm(g_ref)
    assert abs(loss.item() - share * l_ref) < 1e-2 * share * (abs(l_ref) + 1.0)


def test_gradient_of_large_batches_is_deterministic(gpu_ctx):
    import torch
    _put(gpu_ctx, _rand_params(41), NORM)
    rng = np.random.default_rng(42)
    rec = torch.from_numpy(_records(rng, 5000).astype(np.float32)).cuda()
    batch = 9001
    idx = torch.from_numpy(rng.integers(0, 5000, batch).astype(np.int32)).cuda()
    u = torch.from_numpy(np.concatenate([rng.uniform(0, 1, (batch, 4)), rng.uniform(0, 1, (batch, 1)) < 0.3], axis=1)
                         .astype(np.float32)).cuda()
    g = [torch.zeros(NP, dtype=torch.float32, device="cuda") for _ in range(3)]
    for out in g:
        gpu_ctx.krt_escape_grad(rec, idx, u, out)
    assert torch.equal(g[0], g[1]) and torch.equal(g[0], g[2])
