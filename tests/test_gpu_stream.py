"""The run layout's library-sized tiling (stream encoding: image tiles, one
word per pixel, sums in LDS) at the sizes where it can go wrong, against the
FP64 oracle."""
import sys

import numpy as np
import pytest
import torch

import oracle
from tests.helpers import azint, oracle_matrix
from tests.test_gpu_forward import TOL32_F64, TOL64, check

pytestmark = pytest.mark.gpu

GEOMS = [
    # h, w, center_y, center_x, npt, unit, split
    (1, 4, 0.5, 2.5, 3, "r_m", "bbox"),              # the smallest image that is encoded
    (1, 3, 0.5, 1.5, 2, "r_m", "bbox"),              # one that is not
    (300, 1, 3.5, 0.5, 40, "r_m", "bbox"),
    (37, 63, 10.25, 40.5, 61, "r_m", "bbox"),
    (64, 64, 32.0, 32.0, 64, "r_m", "bbox"),
    (65, 65, 32.5, 32.5, 64, "r_m", "bbox"),
    (129, 67, 64.0, 33.0, 20, "r_m", "bbox"),        # two bins a pixel at most
    (31, 29, 15.5, 14.5, 300, "r_m", "bbox"),        # more bins a pixel than are unrolled
    (200, 200, 100.0, 100.0, 3000, "r_m", "bbox"),
    (300, 280, 150.2, 139.7, 1, "r_m", "bbox"),
    (141, 138, 20.6, 18.2, 150, "q_nm", "full"),
]
RAWS = {"int16": np.int16, "uint16": np.uint16, "int32": np.int32, "uint32": np.uint32,
        "float32": np.float32, "float64": np.float64}


@pytest.mark.parametrize("dtype,accum", [(torch.float64, "f64"), (torch.float32, "f64"),
                                         (torch.float32, "kahan32")], ids=["f64", "f32", "k32"])
@pytest.mark.parametrize("g", GEOMS, ids=lambda g: f"{g[0]}x{g[1]}-{g[4]}-{g[6]}")
def test_stream_shapes(g, dtype, accum, dev):
    h, w, cy, cx, npt, unit, split = g
    print("stream", g, dtype, accum, flush=True)
    sys.stdout.flush()
    az = azint()
    npd = np.float64 if dtype == torch.float64 else np.float32
    tol = TOL64 if dtype == torch.float64 else TOL32_F64
    rng = np.random.default_rng(h * 1000 + w)
    flat = rng.uniform(0.9, 1.1, h * w).astype(npd)
    dark = rng.integers(0, 60, h * w).astype(npd)
    m = oracle_matrix(h, w, cy, cx, npt, 1e-4, 1e-4, unit, split)
    t = lambda a: torch.from_numpy(a).to(dev)
    for name, raw_type in RAWS.items():
        if not hasattr(torch, name):
            continue
        raw = rng.integers(60, 30000, h * w).astype(raw_type)
        # the frame ends where its buffer ends: the last pixels' loads stay inside
        plan = az.Plan(h, w, npt, center=(cy, cx), unit=unit, split=split, dtype=dtype,
                       accum=accum, device=dev)
        check(plan.integrate_raw(t(raw), empty=7.0), m, raw.astype(np.float64), tol, empty=7.0,
              what=f"{name}")
        for stage in ("fold_sum", "fold", "fuse"):
            plan.set_tiling(stage=stage)
            plan.set_corrections(dark=t(dark), flat=t(flat))
            x = oracle.correct(raw, dark.astype(np.float64), flat.astype(np.float64), None, None)
            check(plan.integrate_raw(t(raw), empty=7.0), m, x, tol, empty=7.0,
                  what=f"{name} {stage}")


def test_stream_range_leaves_pixels_out(dev):
    """A narrow range: tiles whose pixels feed no bin."""
    az = azint()
    rng = (5e-4, 2e-3)
    plan = az.Plan(200, 260, 37, range=rng, device=dev)
    m = oracle_matrix(200, 260, 100.0, 130.0, 37, 1e-4, 1e-4, "r_m", "bbox", rng)
    x = np.random.default_rng(4).uniform(-1, 50, 200 * 260)
    check(plan.integrate(torch.from_numpy(x).to(dev)), m, x, TOL64, what="range")


def test_stream_keeps_special_values_in_their_bins(dev):
    """A NaN and an infinite pixel reach their own bins only."""
    az = azint()
    h = w = 96
    plan = az.Plan(h, w, 80, device=dev)
    data, bins, colptr = plan.export_csc()
    x = np.random.default_rng(3).uniform(1, 50, h * w)
    ref = plan.integrate(torch.from_numpy(x).to(dev))[1].cpu().numpy()
    bad = {5 * w + 7: np.nan, 60 * w + 41: np.inf}
    for p, v in bad.items():
        x[p] = v
    W = plan.integrate(torch.from_numpy(x).to(dev))[1].cpu().numpy()
    hit = np.zeros(80, bool)
    for p in bad:
        hit[bins[colptr[p]:colptr[p + 1]]] = True
    assert np.all(~np.isfinite(W[hit]))
    assert np.array_equal(W[~hit], ref[~hit])


def test_stream_batch_equals_loop_and_oracle(dev):
    """Instances from one pixel short of a block to several tiles, in one
    launch and one by one, and after leaving the encoding and coming back."""
    az = azint()
    geoms = [(1, 4, 3), (16, 16, 12), (15, 17, 9), (64, 33, 50), (130, 141, 100), (70, 300, 200)]
    plans = [az.Plan(h, w, n) for h, w, n in geoms]
    batch = az.Batch(plans, device=dev)
    x = np.random.default_rng(8).uniform(-1, 50, batch.npix)
    xt = torch.from_numpy(x).to(dev)
    first = [o.clone() for o in batch.forward(xt)]
    for kw in (dict(), dict(tile_nnz=1024), dict(tile_nnz=0, grid=64), dict(grid=0)):
        batch.set_tiling(**kw)
        out, loop = batch.forward(xt), batch.forward(xt, loop=True)
        raw = batch.forward_raw(xt)
        torch.cuda.synchronize()
        for a, b, c in zip(out, loop, raw):
            assert torch.equal(a, b) and torch.equal(a, c), kw
        po, bo = batch.pix_off, batch.bin_off
        for k, (h, w, n) in enumerate(geoms):
            m = oracle_matrix(h, w, h / 2, w / 2, n)
            check([o[bo[k]:bo[k + 1]] for o in out], m, x[po[k]:po[k + 1]], TOL64, what=f"{k} {kw}")
    for a, b in zip(first, out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("g", GEOMS + [(200, 260, 100.0, 130.0, 37, "r_m", "bbox")],
                         ids=lambda g: f"{g[0]}x{g[1]}-{g[4]}-{g[6]}")
def test_stream_adjoint_bits_equal_entry_adjoint(g, dtype, dev):
    """The adjoint over the stream encoding gives the bits of the adjoint over
    the pixel-major entries (same products, same order), with either gradient
    absent, towards the raw counts too, and zero for pixels that feed no bin."""
    h, w, cy, cx, npt, unit, split = g
    print("stream adjoint", g, dtype, flush=True)
    az = azint()
    npd = np.float64 if dtype == torch.float64 else np.float32
    rng = np.random.default_rng(h + 7 * w)
    t = lambda a: torch.from_numpy(a.astype(npd)).to(dev)
    flat, x = t(rng.uniform(0.9, 1.1, h * w)), t(rng.uniform(0, 1, h * w))
    gI, gW = t(rng.standard_normal(npt)), t(rng.standard_normal(npt))
    kw = dict(center=(cy, cx), unit=unit, split=split, dtype=dtype, device=dev)
    if (h, w) == (200, 260):
        kw["range"] = (5e-4, 2e-3)
    stream, entries = az.Plan(h, w, npt, **kw), az.Plan(h, w, npt, layout="pixel", **kw)
    U = stream.integrate(x)[2]
    for p in (stream, entries):
        p.set_corrections(flat=flat)
    for grads in ((gI, gW), (gI, None), (None, gW), (None, None)):
        for wrt_raw in (False, True):
            out = [torch.full((h * w,), float("nan"), dtype=dtype, device=dev) for _ in range(2)]
            a = stream.backward(U, *grads, wrt_raw=wrt_raw, out=out[0])
            b = entries.backward(U, *grads, wrt_raw=wrt_raw, out=out[1])
            torch.cuda.synchronize()
            assert torch.equal(a, b), (grads[0] is None, grads[1] is None, wrt_raw)


@pytest.mark.parametrize("dim", ["1d-fold_sum", "1d-fuse", "2d"])
def test_stream_graph_replays(dim, dev):
    """A captured frame pass replays on what its buffers hold now: with eager
    work between, on other streams, from another thread, and recorded into a
    torch graph; each replay gives the eager bits."""
    import threading
    az = azint()
    h, w, npt = 130, 141, 100
    kw = dict(npt_azim=12) if dim == "2d" else {}
    plan = az.Plan(h, w, npt, device=dev, **kw)
    rng = np.random.default_rng(11)
    t = lambda a: torch.from_numpy(a).to(dev)
    if dim != "2d":
        plan.set_tiling(stage=dim[3:])
    plan.set_corrections(dark=t(rng.integers(0, 60, h * w).astype(np.float64)),
                         flat=t(rng.uniform(0.9, 1.1, h * w)))
    frames = [t(rng.integers(60, 30000, h * w).astype(np.int32)) for _ in range(5)]
    want = [[o.clone() for o in plan.integrate_raw(f, empty=7.0)] for f in frames]
    raw, outs = frames[0].clone(), [torch.empty_like(o) for o in want[0]]
    graph = plan.graph(raw, *outs, empty=7.0)
    side = torch.cuda.Stream()

    def replay(k, how):
        raw.copy_(frames[k])
        for o in outs:
            o.zero_()
        torch.cuda.synchronize()
        how()
        torch.cuda.synchronize()
        for a, b in zip(outs, want[k]):
            assert torch.equal(a, b), (k, how)

    def thread():
        worker = threading.Thread(target=graph.launch)
        worker.start()
        worker.join()

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        graph.launch()
    for k, how in enumerate((graph.launch, lambda: graph.launch(side), thread, g.replay, g.replay)):
        replay(k, how)
        _ = (raw * 2).sum().item()
    with pytest.raises(az.AzintError):
        plan.graph(raw, None)


@pytest.mark.parametrize("n,dtype", [(1650, torch.float64), (1750, torch.float64),
                                     (2300, torch.float64), (3000, torch.float32),
                                     (3600, torch.float32)], ids=str)
def test_stream_sizes_around_the_cache_rule(n, dtype, dev):
    """Matrices read through the caches and past them (64 MiB in float64, 160
    in float32): the sums of the run encoding to rounding, the adjoint of the
    entries bit for bit."""
    az = azint()
    plan = az.Plan.on_device(n, n, n, device=dev, dtype=dtype)
    gen = torch.Generator().manual_seed(n)
    x = torch.rand(n * n, generator=gen, dtype=torch.float64).to(dtype).to(dev)
    g = torch.randn(n, generator=gen, dtype=torch.float64).to(dtype).to(dev)
    band = plan.integrate(x)
    gx0 = plan.backward(band[2], g)
    plan.set_layout("run")
    plan.set_tiling(tile_nnz=0, band=16, grid=0)
    out = plan.integrate(x)
    gx = plan.backward(band[2], g)
    # float64 sums of positive terms: a bin of n terms is off by n/2^53 at most
    # either way; float32 outputs are rounded once more
    tol = 2 * 4 * n * 2.0 ** -53 + (0.0 if dtype == torch.float64 else 2.0 ** -22)
    for a, b in zip(out, band):
        assert ((a - b).abs() <= tol * b.abs()).all()
    assert torch.equal(gx, gx0)
