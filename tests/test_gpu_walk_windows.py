"""The transport's tally windows and start of packets at the sizes where they
can go wrong, against the same walk tallied or split differently: integer
tallies are exact sums, so the comparisons are exact."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2608_09340_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("phase", [0, 1])
@pytest.mark.parametrize("nch", [1, 3, 7, 16, 64])
def test_channel_windows_match_fine_channels(gpu_ctx, phase, nch):
    """A window moves rarely with wide channels and at nearly every scattering
    with 256 narrow ones; the fine channels' sums over each wide channel are
    the wide run's tallies (the edges of the wide channels are edges of the
    fine ones)."""
    from paper_2608_09340_amd import krt
    lo, hi, n = -6.0, 6.0, 20000
    fine = 256 // nch * nch
    T = krt.Transport(W.sphere(7, 200.0, 1e-2, phase=phase, emis=(nch, lo, hi), vmax=2.0), ctx=gpu_ctx)
    a = T.run(n, seed=11)
    F = krt.Transport(W.sphere(7, 200.0, 1e-2, phase=phase, emis=(fine, lo, hi), vmax=2.0), ctx=gpu_ctx)
    b = F.run(n, seed=11)
    assert np.array_equal(a["emis_raw"], b["emis_raw"].reshape(-1, nch, fine // nch).sum(axis=2))
    assert a["counters"] == b["counters"]
    assert a["counters"]["emis_dropped"] > 0
    if phase == 0:  # every scattering tallied once, 2^20 each
        c = a["counters"]
        assert int(a["emis_raw"].sum()) == (c["scatterings"] - c["emis_dropped"]) << 20


def test_windows_hold_long_visits(gpu_ctx):
    """One thick cell and few packets: a lane adds far more scatterings to one
    window than an 8-bit count holds."""
    from paper_2608_09340_amd import krt
    p = W._problem((1, 1, 1), (-1.0,) * 3, (1.0,) * 3, (0, 0, 0), np.array([3000.0]), 1e-2,
                   source={"kind": W.SRC_POINT, "pos": (0.0, 0.0, 0.0), "profile": W.PROF_DELTA, "x0": 0.0},
                   tally={"spec_nbins": 16, "spec_lo": -16.0, "spec_hi": 16.0, "emis_nch": 2, "ch_lo": -64.0,
                          "ch_hi": 64.0, "n_cam": (1.0, 0.0, 0.0)})
    r = krt.Transport(p, ctx=gpu_ctx).run(100, seed=1)
    c = r["counters"]
    assert c["scatterings"] > 100 * 1000 and c["emis_dropped"] == 0
    assert int(r["emis_raw"].sum()) == c["scatterings"] << 20


@pytest.mark.parametrize("ch", [(1e6, 1e6 + 1.0, 64), (-1e-6, 1e-6, 256), (-40.0, 40.0, 1)])
def test_channels_at_the_rounding_of_their_edges(gpu_ctx, ch):
    """Channels narrower than the rounding of their edges, far from zero, or a
    single one: totals and drops still account for every scattering, and the
    beam's own frequency offset puts scatterings inside the first set."""
    from paper_2608_09340_amd import krt
    p = W.thin_moving_slab(tau=5.0, a=1e-2)
    p["tally"].update({"ch_lo": ch[0], "ch_hi": ch[1], "emis_nch": ch[2]})
    if ch[0] > 1e5:
        p["grid"]["vel"][:] = 0.0
        p["grid"]["vel"][2, :] = 1e6
    r = krt.Transport(p, ctx=gpu_ctx).run(5000, seed=3)
    c = r["counters"]
    assert c["scatterings"] > 1000
    assert int(r["emis_raw"].sum()) == (c["scatterings"] - c["emis_dropped"]) << 20
    if ch[0] != -1e-6:
        assert c["emis_dropped"] < c["scatterings"]


@pytest.mark.parametrize("n", [1, 63, 65, 4095, 4097, 70001, 900001])
def test_spread_packets_match_split_range(gpu_ctx, n):
    """Few packets start spread over the waves, more than the lanes come from the
    shared pool in chunks; the same packets as two calls start in other lanes
    and give the same sums."""
    from paper_2608_09340_amd import krt
    T = krt.Transport(W.sphere(5, 30.0, 1e-2, phase=1, emis=(16, -12.0, 12.0)), ctx=gpu_ctx)
    a = T.run(n, seed=3)
    assert a["counters"]["emitted"] == n == a["counters"]["escaped"]
    k = (n + 1) // 3
    parts = [T.run(m, seed=3, packet_offset=o) for m, o in ((k, 0), (n - k, k)) if m]
    for key in ("spec_raw", "emis_raw"):
        assert np.array_equal(a[key], sum(r[key] for r in parts))
    assert a["counters"]["scatterings"] == sum(r["counters"]["scatterings"] for r in parts)


@pytest.mark.parametrize("n", [1, 64, 65, 5000])
def test_records_do_not_depend_on_their_lanes(gpu_ctx, n):
    """Whole-cell walks started together or in two calls, in other lanes and
    with other neighbours, are the same records bit for bit."""
    import torch
    from paper_2608_09340_amd import krt
    krt.Transport(W.sphere(2, 1.0, 1e-2, phase=0, emis=None), ctx=gpu_ctx)
    dev = torch.device("cuda", 0)

    def rec(m, off):
        out = torch.full((m, krt.ESC_NREC), -7.0, device=dev)
        gpu_ctx.krt_escape_record(0, m, 5, off, 1.5, 3.0, out)
        return out.cpu().numpy()

    a, k = rec(n, 40), (n + 1) // 3
    b = np.concatenate([rec(m, 40 + o) for m, o in ((k, 0), (n - k, k)) if m])
    assert np.array_equal(a, b)
    assert np.all(a[:, 18] == 1.0) and np.all(a[:, 19] == 0.0)


@pytest.mark.parametrize("vel", [False, True])
@pytest.mark.parametrize("fields", ["eps", "kabs", "both"])
def test_cell_records_match_the_fields(gpu_ctx, vel, fields):
    """A run that reads its cells from packed records (enough packets per cell)
    and the no-allocation entry point, which reads the fields' own arrays, walk
    the same packets; the fields may change between runs."""
    from paper_2608_09340_amd import krt
    rng = np.random.default_rng(4)
    p = W.sphere(9, 40.0, 1e-2, phase=0, emis=(8, -9.0, 9.0), vmax=3.0 if vel else 0.0, jbar=True)
    nc = 9 ** 3
    if fields != "kabs":
        p["grid"]["eps"] = (0.2 * rng.random(nc)).astype(np.float32)
    if fields != "eps":
        p["grid"]["kabs"] = (2.0 * rng.random(nc)).astype(np.float32)
    T = krt.Transport(p, ctx=gpu_ctx)
    for _ in range(2):
        a, b = T.run(4000, seed=2), T.run(4000, seed=2, noalloc=True)
        assert a["counters"] == b["counters"] and a["counters"]["destroyed"] > 0
        for key in ("spec_raw", "emis_raw", "jbar_raw"):
            assert np.array_equal(a[key], b[key]), key
        T.k0.mul_(0.5)


@pytest.mark.parametrize("nch", [15, 17])
def test_finalised_emissivity_on_both_sides_of_the_cache(gpu_ctx, nch):
    """The pass that checks and scales a tally reads it as a stream past 2^25
    sums: on either side of that the FP32 form is the raw sums times one FP64
    factor, to the last place."""
    import torch
    from paper_2608_09340_amd import krt
    n, N = 128, 4000
    T = krt.Transport(W.sphere(n, 5.0, 1e-2, phase=0, emis=(nch, -9.0, 9.0), source="volume"), ctx=gpu_ctx)
    T.run(N, seed=1, host=False)
    f = 2.0 ** -20 / (4.0 * np.pi * N * (2.0 / n) ** 3 * (18.0 / nch))
    want = T.emis_raw.double() * f
    assert int(torch.count_nonzero(T.emis_raw)) > 1000
    assert bool(((T.emis.double() - want).abs() <= want.abs() * 2.0 ** -23).all())


def test_cell_records_are_given_back(gpu_ctx):
    """The memory of the cell records (32 bytes a cell here) goes back to the
    device when a smaller grid is uploaded; a grid of the same kind and size
    keeps it."""
    import torch
    from paper_2608_09340_amd import krt
    n = 128
    p = W.sphere(n, 5.0, 1e-2, phase=0, emis=None)
    p["grid"]["eps"] = np.full(n ** 3, 0.5, dtype=np.float32)
    T = krt.Transport(p, ctx=gpu_ctx)
    S = W.sphere(5, 5.0, 1e-2, phase=0, emis=None)
    small = torch.from_numpy(S["grid"]["k0"]).cuda()

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    T.run(n ** 3 // 8, seed=1)
    held = free()
    T._bind()
    assert abs(free() - held) < 1 << 20
    T.run(n ** 3 // 8, seed=1)
    assert abs(free() - held) < 1 << 20
    gpu_ctx.krt_grid_upload([5] * 3, [-1.0] * 3, [1.0] * 3, [0] * 3, small)
    assert free() - held >= 32 * n ** 3 - (2 << 20)


def test_dipole_windows_hold_long_visits(gpu_ctx):
    """One thick cell with dipole phase: a lane's sums stay in its window for
    thousands of scatterings; the packets one by one, and without the tail's
    drawn-ahead events, give the same tallies."""
    from paper_2608_09340_amd import krt
    p = W._problem((1, 1, 1), (-1.0,) * 3, (1.0,) * 3, (0, 0, 0), np.array([3000.0]), 1e-2, phase=W.PHASE_DIPOLE,
                   source={"kind": W.SRC_POINT, "pos": (0.0, 0.0, 0.0), "profile": W.PROF_DELTA, "x0": 0.0},
                   tally={"spec_nbins": 16, "spec_lo": -16.0, "spec_hi": 16.0, "emis_nch": 9, "ch_lo": -64.0,
                          "ch_hi": 64.0, "n_cam": (1.0, 0.0, 0.0)})
    T = krt.Transport(p, ctx=gpu_ctx)
    n = 20
    a = T.run(n, seed=1)
    assert a["counters"]["scatterings"] > n * 1000 and a["counters"]["emis_dropped"] == 0
    b = T.run(n, seed=1, tail_lanes=-1)
    one = [T.run(1, seed=1, packet_offset=k)["emis_raw"] for k in range(n)]
    assert np.array_equal(a["emis_raw"], b["emis_raw"]) and np.array_equal(a["emis_raw"], sum(one))
    assert abs(a["emis_raw"].sum() / (a["counters"]["scatterings"] << 20) - 1.0) < 0.05


@pytest.mark.parametrize("phase", [0, 1])
def test_more_workgroups_than_fit(gpu_ctx, phase):
    """Workgroups asked for beyond those a compute unit holds change neither the
    tallies nor, by more than the launch itself, the time: packets given to
    workgroups that wait for others to end would make it a multiple (10 times
    with 64 of 1024 lanes)."""
    from paper_2608_09340_amd import krt
    T = krt.Transport(W.sphere(16, 300.0, 1e-2, phase=phase, emis=(16, -12.0, 12.0)), ctx=gpu_ctx)
    n, ms, ref = 60000, {}, None
    for wg, per in ((0, 0), (1024, 4), (1024, 64), (256, 64)):
        took = []
        for _ in range(3):
            r = T.run(n, seed=3, wg_size=wg, wg_per_cu=per)
            took.append(gpu_ctx.krt_last_transport_ms())
        ms[wg, per] = min(took)
        ref = ref or r
        assert np.array_equal(r["spec_raw"], ref["spec_raw"]) and np.array_equal(r["emis_raw"], ref["emis_raw"])
        assert r["counters"] == ref["counters"]
    print(ms)
    assert ms[1024, 4] < 1.5 * ms[0, 0] and ms[1024, 64] < 1.5 * ms[0, 0], ms
    assert ms[256, 64] < 4.0 * ms[0, 0], ms  # at most two workgroups of 256 lanes: a half or a quarter of the waves
