"""The stream encoding's kernels where their special branches meet the edges
of what a caller may hand over."""
import sys

import numpy as np
import pytest
import torch

import oracle
from tests.helpers import azint, norm_err, oracle_matrix
from tests.test_gpu_2d import oracle2d
from tests.test_gpu_forward import TOL32_F64, TOL64, check

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_gradient_towards_raw_of_masked_pixels(dtype, dev):
    """A norm of zero, of an infinity or below zero, on pixels that feed bins,
    on pixels that feed none, and on whole tiles that feed none: the values and
    signs of the adjoint over the pixel-major entries."""
    say("masked gradient", dtype)
    az = azint()
    h, w, npt = 200, 260, 37
    kw = dict(range=(5e-4, 2e-3), dtype=dtype, device=dev)
    stream, entries = az.Plan(h, w, npt, **kw), az.Plan(h, w, npt, layout="pixel", **kw)
    gen = np.random.default_rng(21)
    flat = gen.uniform(0.9, 1.1, h * w)
    mask = gen.random(h * w) < 0.2
    flat[mask] = gen.choice([0.0, -0.0, -1.5, np.inf, -np.inf, np.nan], mask.sum())
    flat = torch.from_numpy(flat).to(dtype).to(dev)
    x = torch.from_numpy(gen.uniform(0, 1, h * w)).to(dtype).to(dev)
    U = stream.integrate(x)[2]
    g = torch.from_numpy(gen.standard_normal((2, npt))).to(dtype).to(dev)
    out = []
    for p in (stream, entries):
        p.set_corrections(flat=flat)
        out.append(p.backward(U, g[0].contiguous(), g[1].contiguous(), wrt_raw=True))
    a, b = out
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(a), torch.isnan(b))
    keep = ~torch.isnan(b)
    assert torch.equal(a[keep], b[keep])
    assert torch.equal(torch.signbit(a[keep]), torch.signbit(b[keep]))
    assert bool(torch.isnan(a).any())


# Bins as fine as the encoding takes them: most pixels have more than the kernels
# keep in registers
@pytest.mark.parametrize("h,w,npt,dtype,accum", [
    (141, 150, 290, torch.float64, "f64"), (141, 150, 290, torch.float32, "f64"),
    (141, 150, 290, torch.float32, "kahan32"),
    (1740, 1750, 4300, torch.float64, "f64"), (1740, 1750, 4300, torch.float32, "f64")], ids=str)
def test_fine_bins(h, w, npt, dtype, accum, dev):
    say("fine bins", h, w, npt, dtype, accum)
    az = azint()
    npd = np.float64 if dtype == torch.float64 else np.float32
    m = oracle_matrix(h, w, h / 2, w / 2, npt)
    kw = dict(dtype=dtype, accum=accum, device=dev)
    plan, entries = az.Plan(h, w, npt, **kw), az.Plan(h, w, npt, layout="pixel", **kw)
    gen = np.random.default_rng(h)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    x = gen.uniform(0, 1000, h * w).astype(npd)
    tol = TOL64 if dtype == torch.float64 else TOL32_F64
    out = plan.integrate(t(x))
    check(out, m, x.astype(np.float64), tol, what="image")
    raw, flat = gen.integers(60, 1 << 20, h * w).astype(np.int32), gen.uniform(0.9, 1.1, h * w)
    flat, dark = flat.astype(npd), gen.integers(0, 60, h * w).astype(npd)
    plan.set_corrections(dark=t(dark), flat=t(flat))
    check(plan.integrate_raw(t(raw)), m,
          oracle.correct(raw, dark.astype(np.float64), flat.astype(np.float64), None, None), tol,
          what="raw")
    g = [t(gen.standard_normal(npt).astype(npd)) for _ in range(2)]
    a, b = plan.backward(out[2], *g), entries.backward(out[2], *g)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


# Maps that are encoded: h, w, center_y, center_x, npt, npt_azim, split
MAPS = [
    (1420, 1420, 700.3, 680.2, 60, 36, "bbox"),
    (1451, 1453, 725.5, 726.5, 580, 360, "bbox"),    # the beam inside a pixel: it lies in all wedges
    (1409, 1427, -20.0, 600.0, 110, 90, "bbox"),     # the beam off the detector
    (1441, 1390, 700.0, 690.0, 70, 24, "full"),
    (1451, 1453, 725.5, 726.5, 1740, 360, "bbox"),   # the beam's pixel: more runs than a window holds
]
KINDS = [(torch.float64, "f64"), (torch.float32, "f64"), (torch.float32, "kahan32")]


@pytest.fixture(scope="module")
def map_matrix():
    made = {}

    def get(g):
        if g not in made:
            made.clear()
            made[g] = oracle2d(*g[:6], "r_m", g[6])
        return made[g]

    return get


def map_plan(g, dtype, accum, dev, on_device=False):
    az = azint()
    kw = dict(npt_azim=g[5], center=g[2:4], split=g[6], dtype=dtype, accum=accum)
    if on_device:
        return az.Plan.on_device(g[0], g[1], g[4], device=dev, **kw)
    return az.Plan(g[0], g[1], g[4], device=dev, **kw)


@pytest.mark.parametrize("dtype,accum", KINDS, ids=["f64", "f32", "k32"])
@pytest.mark.parametrize("g", MAPS, ids=lambda g: f"{g[0]}x{g[1]}-{g[5]}-{g[6]}")
def test_encoded_map_corrections_and_raw_types(g, dtype, accum, dev, map_matrix):
    """Every raw type, and every kind of correction: dark counts of 16 bits, as
    floats, as doubles; dark or norm alone; neither."""
    say("map", g, dtype, accum)
    m, n = map_matrix(g), g[0] * g[1]
    npd = np.float64 if dtype == torch.float64 else np.float32
    tol = TOL64 if dtype == torch.float64 else TOL32_F64
    plan = map_plan(g, dtype, accum, dev)
    bytes_encoded = plan.device_bytes()
    gen = np.random.default_rng(g[0])
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    flat = gen.uniform(0.9, 1.1, n).astype(npd)
    counts = gen.integers(0, 60, n)
    raws = [gen.integers(60, 30000, n).astype(k) for k in
            (np.int32, np.int16, np.uint16, np.uint32, np.float32, np.float64)]

    def run(raw, dark, flat, what):
        plan.set_corrections(dark=None if dark is None else t(dark),
                             flat=None if flat is None else t(flat))
        out = plan.integrate_raw(t(raw), empty=7.0)
        torch.cuda.synchronize()
        f = lambda a: None if a is None else a.astype(np.float64)
        check(out, m, oracle.correct(raw, f(dark), f(flat), None, None), tol, empty=7.0, what=what)

    for raw in raws:
        run(raw, counts.astype(npd), flat, f"raw {raw.dtype}")
    for add in (0.25, 0.1, 70000.0):
        run(raws[0] + 70000, (counts + add).astype(npd), flat, f"dark + {add}")
    run(raws[0], (counts + 0.1).astype(npd), None, "dark alone")
    run(raws[0], None, flat, "norm alone")
    run(raws[0], None, None, "neither")
    x = raws[5].astype(npd)
    check(plan.integrate(t(x), empty=7.0), m, x.astype(np.float64), tol, empty=7.0, what="image")
    plan.set_tiling(variant=0)  # out of the encoding: the row kernel
    assert plan.device_bytes() < bytes_encoded
    check(plan.integrate(t(x), empty=7.0), m, x.astype(np.float64), tol, empty=7.0, what="rows")


@pytest.mark.parametrize("g", MAPS[:3], ids=lambda g: f"{g[0]}x{g[1]}-{g[5]}")
def test_map_built_on_the_device(g, dev):
    """Encoded from the downloaded positions beside the other copies: the sums
    of the matrix that it exports, the same bits from every build.  (Its azimuths
    are the device's atan2, so a host-built plan's bits may differ.)"""
    say("map on the device", g)
    x = np.random.default_rng(5).integers(0, 1 << 20, g[0] * g[1]).astype(np.int32)
    raw = torch.from_numpy(x).to(dev)
    first = None
    for _ in range(3):
        plan = map_plan(g, torch.float64, "f64", dev, on_device=True)
        out = plan.integrate_raw(raw)
        torch.cuda.synchronize()
        first = first or out
        for u, v in zip(out, first):
            assert torch.equal(u, v)
    data, bins, colptr = plan.export_csc()
    per_pixel = np.repeat(x.astype(np.float64), np.diff(colptr))
    W = np.bincount(bins, weights=data * per_pixel, minlength=plan.npt)
    U = np.bincount(bins, weights=data, minlength=plan.npt)
    assert norm_err(first[1].cpu().numpy(), W, W) <= TOL64
    assert norm_err(first[2].cpu().numpy(), U, U) <= TOL64


def test_encoded_map_keeps_special_values_in_their_bins(dev):
    """NaN and infinite pixels, one of them in several wedges, reach their own
    bins only; so do those of a raw float frame."""
    say("map special values")
    g = MAPS[0]
    plan = map_plan(g, torch.float64, "f64", dev)
    data, bins, colptr = plan.export_csc()
    n = g[0] * g[1]
    x = np.random.default_rng(3).uniform(1, 50, n)
    ref = plan.integrate(torch.from_numpy(x).to(dev))[1].cpu().numpy()
    beam = 700 * g[1] + 680
    many = beam + 5  # a few pixels from the beam: in several wedges
    bad = {7 * g[1] + 13: np.nan, 600 * g[1] + 41: np.inf, many: -np.inf, n - 1: np.nan}
    for p, v in bad.items():
        x[p] = v
    hit = np.zeros(plan.npt, bool)
    for p in bad:
        hit[bins[colptr[p]:colptr[p + 1]]] = True
    xt = torch.from_numpy(x).to(dev)
    for W in (plan.integrate(xt)[1], plan.integrate_raw(xt)[1]):
        W = W.cpu().numpy()
        assert np.all(~np.isfinite(W[hit]))
        assert np.array_equal(W[~hit], ref[~hit])


@pytest.mark.parametrize("n", [2500, 2800])
def test_adjoint_around_its_cache_rule(n, dev):
    """float64 matrices of 147 and 184 MB, the adjoint's words and coefficients
    through the caches and past them: the bits of the entries' adjoint."""
    say("adjoint caches", n)
    az = azint()
    plan = az.Plan.on_device(n, n, n, device=dev)
    gen = torch.Generator(device=dev).manual_seed(n)
    x = torch.rand(n * n, generator=gen, device=dev, dtype=torch.float64)
    g = torch.randn(n, generator=gen, device=dev, dtype=torch.float64)
    U = plan.integrate(x)[2]
    want = plan.backward(U, g, g)
    plan.set_layout("run")
    plan.set_tiling(tile_nnz=0, band=16, grid=0)
    for _ in range(2):
        got = plan.backward(U, g, g)
        torch.cuda.synchronize()
        assert torch.equal(got, want)


@pytest.mark.parametrize("k", [40, 70, 130])
def test_batch_around_its_cache_rule(k, dev):
    """float64 batches of 57, 99 and 184 MB: one launch, the loop and the
    entries' adjoint agree bit for bit."""
    say("batch caches", k)
    az = azint()
    one = az.Plan(250, 250, 250)
    batch = az.Batch([one] * k, device=dev)
    gen = torch.Generator(device=dev).manual_seed(k)
    x = torch.rand(batch.npix, generator=gen, device=dev, dtype=torch.float64)
    g = torch.randn(batch.npt, generator=gen, device=dev, dtype=torch.float64)
    out, loop = batch.forward(x), batch.forward(x, loop=True)
    gx = batch.backward(out[2], g, g)
    torch.cuda.synchronize()
    for a, b in zip(out, loop):
        assert torch.equal(a, b)
    batch.set_tiling(tile_nnz=1024)
    assert torch.equal(batch.backward(out[2], g, g), gx)


def test_float32_map_folds_from_the_same_doubles(dev):
    """Kept from the build on the device, or copied from the host matrix: the
    same folded coefficients, through several changes of corrections."""
    say("float32 fold")
    g = MAPS[0]
    plan = map_plan(g, torch.float32, "f64", dev, on_device=True)
    gen = torch.Generator(device=dev).manual_seed(9)
    n = g[0] * g[1]
    raw = torch.randint(0, 1 << 20, (n,), generator=gen, device=dev, dtype=torch.int32)
    flats = [0.9 + 0.2 * torch.rand(n, generator=gen, device=dev) for _ in range(2)]
    kept = []
    for flat in flats:
        plan.set_corrections(flat=flat)
        kept.append(plan.integrate_raw(raw))
    plan.set_tiling(variant=0)  # out of the encoding, and back
    plan.set_tiling(variant=1)
    for flat, want in list(zip(flats, kept))[::-1]:
        plan.set_corrections(flat=flat)
        got = plan.integrate_raw(raw)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b)


def test_retiling_a_device_built_plan_holds_what_it_reports(dev):
    """A plan built on the device has its arrays cut from shared allocations: a
    change of tiling puts the new band arrays in the old ones' place, and
    device_bytes is what the plan takes from the device."""
    say("retile device built")
    az = azint()
    n = 1500
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info(dev)[0]
    plan = az.Plan.on_device(n, n, n, device=dev)
    x = torch.rand(n * n, device=dev, dtype=torch.float64)
    ref = plan.integrate(x)
    torch.cuda.synchronize()
    slack = 16 << 20
    first = plan.device_bytes()
    held = free - torch.cuda.mem_get_info(dev)[0]
    for tile_nnz in (1024, 4096, 512, 8192, 0):
        plan.set_tiling(tile_nnz=tile_nnz)
        out = plan.integrate(x)
        torch.cuda.synchronize()
        assert abs(plan.device_bytes() - first) < slack, tile_nnz
        assert free - torch.cuda.mem_get_info(dev)[0] < held + slack, tile_nnz
        for a, b in zip(out, ref):
            assert ((a - b).abs() <= 8 * n * 2.0 ** -53 * b.abs()).all()
    assert first < held + slack


@pytest.mark.parametrize("dtype,accum", KINDS, ids=["f64", "f32", "k32"])
@pytest.mark.parametrize("npt", [1, 8, 16, 17])
def test_many_tiles_in_few_bins(npt, dtype, accum, dev):
    """A thousand tiles that all reach the one or two chunks of bins: the
    reduction of the longest lists."""
    say("few bins", npt, dtype, accum)
    az = azint()
    h, w = 1000, 1010
    m = oracle_matrix(h, w, 480.3, 520.7, npt)
    npd = np.float64 if dtype == torch.float64 else np.float32
    plan = az.Plan(h, w, npt, center=(480.3, 520.7), dtype=dtype, accum=accum, device=dev)
    gen = np.random.default_rng(npt)
    x = gen.uniform(0, 1000, h * w).astype(npd)
    tol = TOL64 if dtype == torch.float64 else TOL32_F64
    check(plan.integrate(torch.from_numpy(x).to(dev)), m, x.astype(np.float64), tol, what="image")
    raw = gen.integers(0, 1 << 20, h * w).astype(np.int32)
    check(plan.integrate_raw(torch.from_numpy(raw).to(dev)), m, raw.astype(np.float64), tol,
          what="raw")


def _shifted(t, by):
    """The same values at an address that is `by` elements past an aligned one."""
    room = torch.zeros(t.numel() + by, dtype=t.dtype, device=t.device)
    room[by:] = t
    out = room[by:]
    assert out.is_contiguous() and (out.data_ptr() - room.data_ptr()) == by * t.element_size()
    return out


@pytest.mark.parametrize("g", [(131, 143, 60.2, 70.9, 90, 0, "bbox"), MAPS[0]],
                         ids=["profile", "map"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_frames_aligned_to_one_element(g, dtype, dev):
    """Frames, images and gradients that start one to three elements past an
    aligned address give the bits of the aligned ones, to the last pixel."""
    say("alignment", g, dtype)
    az = azint()
    n = g[0] * g[1]
    kw = dict(center=g[2:4], dtype=dtype, device=dev)
    plan = map_plan(g, dtype, "f64", dev) if g[5] else az.Plan(g[0], g[1], g[4], **kw)
    gen = torch.Generator(device=dev).manual_seed(17)
    counts = torch.randint(0, 30000, (n,), generator=gen, device=dev, dtype=torch.int32)
    flat = 0.9 + 0.2 * torch.rand(n, generator=gen, device=dev, dtype=dtype)
    plan.set_corrections(dark=(counts % 61).to(dtype), flat=flat)
    kinds = [k for k in ("int16", "uint16", "int32", "uint32", "float32", "float64")
             if hasattr(torch, k)]
    for stage in ("fold_sum", "fold", "fuse") if not g[5] else (None,):
        if stage:
            plan.set_tiling(stage=stage)
        for kind in kinds:
            raw = counts.cpu().numpy().astype(kind)
            raw = torch.from_numpy(raw).to(dev)
            want = plan.integrate_raw(raw)
            for by in (1, 2, 3):
                got = plan.integrate_raw(_shifted(raw, by))
                torch.cuda.synchronize()
                for a, b in zip(got, want):
                    assert torch.equal(a, b), (stage, kind, by)
    x = counts.to(dtype)
    want = plan.integrate(x)
    grad = torch.randn(plan.npt, generator=gen, device=dev, dtype=dtype)
    gx = plan.backward(want[2], grad)
    for by in (1, 2, 3):
        got = plan.integrate(_shifted(x, by))
        into = _shifted(torch.zeros(n, dtype=dtype, device=dev), by)
        plan.backward(want[2], _shifted(grad, by), out=into)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b), by
        assert torch.equal(into, gx), by


@pytest.mark.parametrize("dtype,accum", KINDS, ids=["f64", "f32", "k32"])
@pytest.mark.parametrize("band", [16, 32])
def test_balanced_runs_where_the_encoding_is_refused(band, dtype, accum, dev):
    """Bins too fine for the stream encoding, in the library-sized tiling: four
    or eight bands a workgroup over balanced runs, every stage and reduction."""
    say("balanced runs", band, dtype, accum)
    az = azint()
    h, w, npt = 300, 310, 1100
    m = oracle_matrix(h, w, 140.3, 160.7, npt)
    assert m["indices"].size > 4.8 * h * w
    npd = np.float64 if dtype == torch.float64 else np.float32
    tol = TOL64 if dtype == torch.float64 else TOL32_F64
    gen = np.random.default_rng(band)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    raw = gen.integers(60, 1 << 20, h * w).astype(np.int32)
    dark, flat = gen.integers(0, 60, h * w).astype(npd), gen.uniform(0.9, 1.1, h * w).astype(npd)
    plan = az.Plan(h, w, npt, center=(140.3, 160.7), dtype=dtype, accum=accum, device=dev,
                   tile_nnz=0, band=band)
    x = oracle.correct(raw, dark.astype(np.float64), flat.astype(np.float64), None, None)
    for stage in ("fold_sum", "fold", "fuse"):
        plan.set_tiling(stage=stage)
        plan.set_corrections(dark=t(dark), flat=t(flat))
        check(plan.integrate_raw(t(raw), empty=5.0), m, x, tol, empty=5.0, what=stage)
    image = raw.astype(npd)
    check(plan.integrate(t(image), empty=5.0), m, image.astype(np.float64), tol, empty=5.0,
          what="image")
