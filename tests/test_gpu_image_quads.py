"""Images with four channels a lane against one: channel counts that four does
and does not divide, both directions of every axis, with and without each
optional field."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def line_ctx(gpu_ctx):
    gpu_ctx.krt_tables_build([(4.7e-4, 0)])
    return gpu_ctx


def _image(ctx, n, axis, lo, hi, emis, src, kabs):
    import torch
    from paper_2608_09340_amd import krt
    nch = emis.shape[1]
    img = torch.full((n * n * nch + 8,), -1.0, dtype=torch.float32, device="cuda")
    d = krt.krt_image_desc()
    d.line, d.axis, d.nch, d.ch_lo, d.ch_hi = 0, axis, nch, lo, hi
    d.emis_dev, d.image_dev = emis.data_ptr(), img.data_ptr()
    d.src_dev = None if src is None else src.data_ptr()
    d.kabs_dev = None if kabs is None else kabs.data_ptr()
    ctx.krt_image(d)
    assert bool((img[n * n * nch:] == -1.0).all())
    return img[:n * n * nch].reshape(n * n, nch)


@pytest.mark.parametrize("axis,nch,opts", [(0, 64, ""), (1, 63, "v"), (2, 62, "vs"), (3, 61, "a"), (4, 64, "vsa"),
                                           (5, 47, "s")])
def test_quads_equal_single_channels(line_ctx, axis, nch, opts):
    """Three channels of an image (fewer than a quad: one channel a lane) equal
    the same channels of the whole one.  The channel width is a power of two, so
    the centres are the same; the two cut rays into different segments, and
    every term is positive: each of the n cells adds a few roundings of 2^-24,
    bounded by 8 n 2^-24."""
    import torch
    n = 48
    g = torch.Generator(device="cuda").manual_seed(10 * axis + nch)
    r = lambda *s: torch.rand(*s, generator=g, device="cuda", dtype=torch.float32)  # noqa: E731
    nc = n ** 3
    k0 = torch.where(r(nc) < 0.1, torch.zeros((), device="cuda"), torch.exp(8.0 * r(nc) - 2.0))
    vel = 4.0 * (r(3 * nc) - 0.5) if "v" in opts else None
    emis = r(nc, nch)
    src = 0.1 * r(nc, nch) if "s" in opts else None
    kabs = r(nc) if "a" in opts else None
    line_ctx.krt_grid_upload([n] * 3, [-1.0] * 3, [1.0] * 3, [0] * 3, k0, vel)
    w, lo = 0.25, -8.0
    full = _image(line_ctx, n, axis, lo, lo + w * nch, emis, src, kabs)
    for c in (0, nch // 2, nch - 3):
        part = _image(line_ctx, n, axis, lo + w * c, lo + w * (c + 3), emis[:, c:c + 3].contiguous(),
                      None if src is None else src[:, c:c + 3].contiguous(), kabs)
        a, b = full[:, c:c + 3].double(), part.double()
        assert bool((b > 0).all())
        assert float((torch.abs(a - b) / b).max()) <= 8 * n * 2.0 ** -24


# grid, axis, channels: 8, 4, 2 and 1 segments of a ray with four channels a
# lane, rays that segments and chunks of four cells do and do not divide, lanes
# past the last pixel, more than one round of workgroups
@pytest.mark.parametrize("n,axis,nch,opts", [
    ((64, 64, 32), 2, 64, ""), ((64, 64, 29), 5, 64, "v"), ((64, 64, 64), 1, 64, "vsa"), ((64, 64, 37), 2, 64, "a"),
    ((128, 128, 32), 5, 64, "va"), ((128, 128, 11), 2, 64, "s"), ((128, 128, 16), 2, 64, ""), ((127, 129, 18), 5, 64, "vs"),
    ((23, 128, 128), 3, 64, "v"), ((50, 50, 43), 2, 48, "va"), ((72, 60, 104), 1, 48, "v"), ((128, 128, 21), 2, 32, "sa"),
    ((128, 128, 14), 2, 63, "va"), ((127, 129, 18), 5, 61, "vsa"), ((64, 64, 41), 1, 62, "va"), ((31, 90, 90), 0, 37, "va"),
    ((100, 100, 33), 4, 13, "va")])
def test_segments_of_quads_equal_single_channels(line_ctx, n, axis, nch, opts):
    """As above for every segment count, each cell of a ray a few roundings:
    8 cells 2^-24."""
    import torch
    nc, nl = n[0] * n[1] * n[2], n[axis % 3]
    npix = nc // nl
    g = torch.Generator(device="cuda").manual_seed(100 + nc + axis)
    r = lambda *s: torch.rand(*s, generator=g, device="cuda", dtype=torch.float32)  # noqa: E731
    k0 = torch.where(r(nc) < 0.1, torch.zeros((), device="cuda"), torch.exp(8.0 * r(nc) - 2.0))
    vel = 4.0 * (r(3 * nc) - 0.5) if "v" in opts else None
    emis = r(nc, nch)
    src = 0.1 * r(nc, nch) if "s" in opts else None
    kabs = r(nc) if "a" in opts else None
    line_ctx.krt_grid_upload(list(n), [-1.0] * 3, [1.0] * 3, [0] * 3, k0, vel)
    w, lo = 0.25, -8.0
    full = _image_of(line_ctx, npix, axis, lo, lo + w * nch, emis, src, kabs)
    for c in range(0, nch - 2, 5):
        part = _image_of(line_ctx, npix, axis, lo + w * c, lo + w * (c + 3), emis[:, c:c + 3].contiguous(),
                         None if src is None else src[:, c:c + 3].contiguous(), kabs)
        a, b = full[:, c:c + 3].double(), part.double()
        assert bool((b > 0).all())
        assert float((torch.abs(a - b) / b).max()) <= 8 * nl * 2.0 ** -24


def _image_of(ctx, npix, axis, lo, hi, emis, src, kabs):
    import torch
    from paper_2608_09340_amd import krt
    nch = emis.shape[1]
    img = torch.full((npix * nch + 8,), -1.0, dtype=torch.float32, device="cuda")
    d = krt.krt_image_desc()
    d.line, d.axis, d.nch, d.ch_lo, d.ch_hi = 0, axis, nch, lo, hi
    d.emis_dev, d.image_dev = emis.data_ptr(), img.data_ptr()
    d.src_dev = None if src is None else src.data_ptr()
    d.kabs_dev = None if kabs is None else kabs.data_ptr()
    ctx.krt_image(d)
    assert bool((img[npix * nch:] == -1.0).all())
    return img[:npix * nch].reshape(npix, nch)


def test_one_more_channel_costs_no_multiple(line_ctx):
    """Four channels a cell toward +x take about 4/3 of the time of three: their
    lines are shared with the next cell of the ray, so a kernel that reads them
    as a stream fetches them again (four times the time)."""
    import torch
    n = 200
    k0 = torch.rand(n ** 3, device="cuda")
    line_ctx.krt_grid_upload([n] * 3, [-1.0] * 3, [1.0] * 3, [0] * 3, k0)
    ms = {}
    for nch in (3, 4):
        emis = torch.rand(n ** 3, nch, device="cuda")
        took = []
        for _ in range(10):
            _image_of(line_ctx, n * n, 0, -8.0, 8.0, emis, None, None)
            took.append(line_ctx.krt_last_image_ms())
        ms[nch] = min(took)
    assert ms[4] < 2.0 * ms[3], ms
