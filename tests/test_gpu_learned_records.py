"""The learned walk on a moving grid reads its cells from packed records; the
no-allocation entry point reads the fields' own arrays.  Integer tallies, so
the two are compared exactly."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2608_09340_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def network(gpu_ctx):
    """An untrained network: its calls leave cells somewhere, which is all that
    these comparisons need."""
    import torch
    from paper_2608_09340_amd import krt
    gpu_ctx.krt_tables_build([(1e-3, 0)])
    rec = torch.zeros((20000, krt.ESC_NREC), dtype=torch.float32, device="cuda")
    gpu_ctx.krt_escape_record(0, rec.shape[0], 3, 0, 1.5, 3.0, rec)
    gpu_ctx.krt_escape_init(5)
    gpu_ctx.krt_escape_fit_norm(rec, rec.shape[0])
    return gpu_ctx


@pytest.mark.parametrize("n", [1, 5, 6, 9])
def test_learned_cell_records_match_the_fields(network, n):
    """Different opacity and velocity in every cell, packets enough for the
    records (one in eight cells); then the same grid with other fields, which
    records kept from the first runs would not show."""
    from paper_2608_09340_amd import krt
    rng = np.random.default_rng(n)
    nc = n ** 3
    k0 = np.exp(rng.normal(4.5, 1.5, nc)) * n / 2.0
    p = W._problem((n, n, n), (-1.0,) * 3, (1.0,) * 3, (0, 0, 0), k0, 1e-3, vel=rng.normal(0.0, 2.0, (3, nc)),
                   emis=np.ones(nc),
                   source={"kind": W.SRC_VOLUME, "pos": (0.0, 0.0, 0.0), "profile": W.PROF_VOIGT, "x0": 0.0},
                   tally={"spec_nbins": 128, "spec_lo": -24.0, "spec_hi": 24.0, "emis_nch": 16, "ch_lo": -10.0,
                          "ch_hi": 10.0, "n_cam": (0.0, 0.6, 0.8)})
    T = krt.Transport(p, ctx=network)
    kw = dict(seed=5, packet_offset=77, escape_mode=1, esc_cell_tau_min=70.0, packet_log=True)
    seen = []
    for N in (3000, 70000, 70000):
        a, b = T.run(N, **kw), T.run(N, noalloc=True, **kw)
        assert a["rc"] == 0 and b["rc"] == 0
        assert a["counters"] == b["counters"]
        assert a["counters"]["mlp_calls"] > 0 and a["counters"]["scatterings"] > 0
        for key in ("spec_raw", "emis_raw", "packet_log"):
            assert np.array_equal(a[key], b[key]), key
        seen.append(a["counters"]["scatterings"])
        if N > 3000:
            T.k0.mul_(1.3)
            T.vel.mul_(-0.7)
    assert seen[1] != seen[2]
