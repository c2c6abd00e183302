"""Level solve at the edges of its split over workgroups (256 cells each, at
most 2048 workgroups): one cell, a ragged wave, past the last full round."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2608_09340_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solve(ctx, rot, ncoll, ntot, jbar):
    import torch
    from paper_2608_09340_amd import krt
    nl, n = len(rot["E"]), ncoll.numel()
    keep = {k: np.ascontiguousarray(rot[k], dtype=np.float64) for k in ("E", "g", "A", "Cd", "sigma0")}
    pops = torch.full((n * nl + 8,), -1.0, dtype=torch.float64, device="cuda")
    out = [torch.full(((nl - 1) * n + 8,), -1.0, dtype=torch.float32, device="cuda") for _ in range(3)]
    lum = np.zeros(nl - 1)
    d = krt.krt_levels_desc()
    d.n_levels, d.ncell = nl, n
    for k, v in keep.items():
        setattr(d, k, v.ctypes.data)
    d.ncoll_dev, d.ntot_dev, d.pops_dev = ncoll.data_ptr(), ntot.data_ptr(), pops.data_ptr()
    d.k0_out_dev, d.eps_out_dev, d.emis_out_dev = [t.data_ptr() for t in out]
    d.cell_volume, d.lum_out = 1.0, lum.ctypes.data
    ctx.krt_levels_update(d, jbar)
    assert bool((pops[n * nl:] == -1.0).all()) and all(bool((t[(nl - 1) * n:] == -1.0).all()) for t in out)
    return pops[:n * nl].reshape(n, nl), [t[:(nl - 1) * n].reshape(nl - 1, n) for t in out], lum


@pytest.mark.parametrize("nl", [2, 5, 8])
@pytest.mark.parametrize("n", [1, 63, 257, 2048 * 256 + 77])
def test_every_cell_once(gpu_ctx, nl, n):
    """A cell's solution does not depend on where the cell sits: the same cells
    in reverse order give the same bits, nothing is written past the arrays,
    and a line's power is the sum over the cells (FP64: n additions of positive
    terms in either order, within n 2^-53)."""
    import torch
    rot = W.rotor(nl)
    gen = torch.Generator(device="cuda").manual_seed(n)
    ncoll = torch.exp(1.5 * torch.randn(n, generator=gen, device="cuda", dtype=torch.float64))
    ntot = ncoll * (0.5 + torch.rand(n, generator=gen, device="cuda", dtype=torch.float64))
    jbar = 0.2 * torch.rand((nl - 1) * n, generator=gen, device="cuda", dtype=torch.float32)
    p, o, lum = _solve(gpu_ctx, rot, ncoll, ntot, jbar)
    q, r, _ = _solve(gpu_ctx, rot, ncoll.flip(0).contiguous(), ntot.flip(0).contiguous(),
                     jbar.reshape(nl - 1, n).flip(1).contiguous())
    assert torch.equal(p, q.flip(0)) and all(torch.equal(a, b.flip(1)) for a, b in zip(o, r))
    assert bool((torch.abs(p.sum(1) - ntot) <= 1e-10 * ntot).all())
    for l in range(nl - 1):
        want = float((p[:, l + 1] * rot["A"][l + 1][l]).sum())
        assert abs(lum[l] - want) <= max(n, 2) * 2.0 ** -52 * want
