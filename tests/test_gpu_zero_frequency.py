"""A frequency of minus zero is line centre, as zero is: the velocity sampler's
symmetry p(u | -x) = p(-u | x) turns u over for x < 0 only."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2608_09340_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_sampler_at_minus_zero(gpu_ctx):
    import torch
    gpu_ctx.krt_tables_build([(1e-2, 0)])
    u = [torch.zeros(5000, dtype=torch.float32, device="cuda") for _ in range(3)]
    for x, out in zip((0.0, -0.0, -1e-30), u):
        gpu_ctx.krt_debug_upar(0, x, 5, 7, 1, out)
    assert torch.equal(u[0], u[1])
    assert torch.equal(u[0], -u[2])  # the same pieces and quantiles, turned over


@pytest.mark.parametrize("iso", [True, False])
def test_walks_recorded_from_minus_zero(gpu_ctx, iso):
    import torch
    gpu_ctx.krt_tables_build([(1e-2, 0)])
    rec = [torch.zeros((3000, 20), dtype=torch.float32, device="cuda") for _ in range(2)]
    for x, out in zip((0.0, -0.0), rec):
        gpu_ctx.krt_escape_record(0, 3000, 9, 0, 1.0, 2.0, out, x_in=x, q=(0.1, 0.2, 0.7),
                                  n_in=None if iso else (0.0, 0.0, 1.0))
    assert torch.equal(rec[0], rec[1])


def test_source_at_minus_zero(gpu_ctx):
    """Same tallies and log as from zero."""
    from paper_2608_09340_amd import krt
    r = []
    for x0 in (0.0, -0.0):
        p = W.sphere(5, 1.0, 1e-2, phase=1, emis=(16, -12.0, 12.0))
        p["source"]["x0"] = x0
        r.append(krt.Transport(p, ctx=gpu_ctx).run(4000, seed=3, packet_log=True))
    for key in ("spec_raw", "emis_raw", "packet_log"):
        assert np.array_equal(r[0][key], r[1][key])
    assert r[0]["counters"] == r[1]["counters"]
