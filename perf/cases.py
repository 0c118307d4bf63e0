"""Performance cases of azimuthal integration: what one call of a user's program costs.

A case is one pass through the package's public entry points (a frame integrated, a
training step, a batch, a plan built and used).  The kinds of pass:

  frame  Plan.integrate_raw: raw detector frame -> I, W, U with the four corrections
  image  Plan.integrate: an image that is corrected already -> I, W, U
  graph  Graph.launch: the frame pass captured once and replayed on fixed buffers
  grad   Integrate1d forward and its backward: I, W, U and the image's gradient
  batch  Batch.forward, or forward + backward, of uneven images in one launch
  build  Plan.on_device + Plan.integrate: a new geometry at every pass

Sizes are those of the repository's benchmark and tests and of the paper (1043 x 981
Pilatus 1M, 2048 x 2048, 3162 x 3163), or odd ones between them.  Raw values are detector
counts of 12 to 20 bits; the corrections are drawn in the ranges of the synthetic workloads.

exact() computes every output in float64 with plain torch from the definitions: the bin
shares of a pixel's bounding box, or of its corner quadrilateral.
"""
import math

import torch

import paper_1412_6367_amd as az

DEV = "cuda:0"
PIXEL, DIST, WAVELENGTH = 1e-4, 0.1, 1e-10
DTYPES = {"f64": torch.float64, "f32": torch.float32}
RAWS = {"int32": (torch.int32, 4, 20), "uint16": (torch.uint16, 2, 16)}


def _case(name, kind, h, w, npt, dtype, **kw):
    c = dict(name=name, kind=kind, h=h, w=w, npt=npt, azim=0, dtype=dtype, accum="f64",
             raw="int32", unit="r_m", split="bbox", cy=0.5, cx=0.5)
    c.update(kw)
    return c


def _batch(name, images, lo, hi, dtype, backward):
    return dict(name=name, kind="batch", images=images, lo=lo, hi=hi, dtype=dtype,
                backward=backward, mix=1)


def listed():
    return [
        # the smallest frame a program integrates by itself: launches and host work
        _case("frame_100_f64", "frame", 100, 100, 100, "f64"),
        # a small fast detector in a serving loop that replays a captured graph
        _case("graph_512_f32", "graph", 512, 512, 512, "f32"),
        # the paper's profiled frame (Pilatus 1M), its unit and its Kahan float sums
        _case("frame_pilatus1m_kahan", "frame", 1043, 981, 1000, "f32", accum="kahan32",
              unit="2th_deg"),
        # the paper's 2048 x 2048 test detector, 16-bit counts, beam off the middle
        _case("frame_4m_u16_f32", "frame", 2048, 2048, 2048, "f32", raw="uint16", cy=0.41,
              cx=0.63),
        # the benchmark frame in double
        _case("frame_10m_f64", "frame", 3162, 3163, 3162, "f64"),
        # the same detector in single precision reduced to the usual 1000 bins
        _case("frame_10m_f32_1000", "frame", 3162, 3163, 1000, "f32"),
        # full pixel splitting in q of an image the program has corrected itself
        _case("image_4m_full_q_f64", "image", 1967, 2011, 1500, "f64", unit="q_nm",
              split="full"),
        # radius x azimuth map of the benchmark frame (texture, calibration)
        _case("map_10m_f64", "frame", 3162, 3163, 1000, "f64", azim=360),
        # one fitting step through the integration: forward and gradient of the image
        _case("grad_1m_f64", "grad", 1000, 1000, 1000, "f64"),
        # many small regions or modules at once, doubles
        _batch("batch_512_f64", 512, 1e2, 1e5, "f64", False),
        # uneven detectors in a training step, single precision, forward and backward
        _batch("batch_64_f32_grad", 64, 1e3, 1e6, "f32", True),
        # geometry refinement: every step builds the matrix of a new geometry and uses it
        _case("build_1m_f64", "build", 1043, 981, 1000, "f64"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "map", "image", "graph", "grad", "batch",
                       "build"])
    dtype = rng.choice(["f64", "f32"])
    if kind == "batch":
        c = _batch("", int(_log(rng, 8, 512)), 1e2, 1e5, dtype, rng.random() < 0.5)
        if c["backward"] and dtype == "f64":
            c["images"] = max(8, c["images"] // 2)
        if c["images"] < 64:
            c["lo"], c["hi"] = 1e3, 6e5
        c["mix"] = rng.randrange(1, 1 << 20)
        del c["name"]
        return c
    most = {"frame": 9.9e6, "map": 8e6, "image": 4e6, "graph": 1e6, "grad": 4e6, "build": 1e6}[kind]
    n = _log(rng, 1e4, most)
    aspect = math.exp(rng.uniform(-0.5, 0.5))
    h = max(16, int(math.sqrt(n * aspect)))
    w = max(16, int(n / h))
    npt = max(8, int(math.sqrt(n) * _log(rng, 0.2, 1.5)))
    c = _case("", "frame" if kind == "map" else kind, h, w, npt, dtype)
    if dtype == "f32" and kind != "map":
        c["accum"] = rng.choice(["f64", "f64", "kahan32"])
    if kind == "map":
        c["azim"] = rng.choice([36, 90, 180, 360])
        c["npt"] = max(8, npt // 3)
    if kind in ("frame", "map", "graph"):
        c["raw"] = rng.choice(["int32", "uint16"])
    c["unit"] = rng.choice(["r_m", "r_mm", "2th_deg", "q_nm"])
    if kind in ("frame", "image", "grad") and not c["azim"]:
        c["split"] = rng.choice(["bbox", "bbox", "full"])
    c["cy"], c["cx"] = round(rng.uniform(0.3, 0.7), 4), round(rng.uniform(0.3, 0.7), 4)
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _uniform(g, n, lo, hi, dtype):
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64).mul_(hi - lo).add_(lo).to(dtype)


def _frame(case, g, n):
    kind, _, bits = RAWS[case["raw"]]
    return torch.randint(0, 1 << bits, (n,), generator=g, device=DEV, dtype=torch.int32).to(kind)


def _corrections(g, n, dtype):
    dark = torch.randint(0, 64, (n,), generator=g, device=DEV, dtype=torch.int32).to(dtype)
    return (dark, _uniform(g, n, 0.95, 1.05, dtype), _uniform(g, n, 0.90, 1.00, dtype),
            _uniform(g, n, 0.95, 1.00, dtype))


def _centre(case, seed=None):
    cy, cx = case["cy"] * case["h"], case["cx"] * case["w"]
    if seed is not None:  # the geometry a refinement step proposes
        cy, cx = cy + (seed % 977) * 1e-3, cx - (seed % 953) * 1e-3
    return cy, cx


def _plan(case, **kw):
    return az.Plan(case["h"], case["w"], case["npt"], center=_centre(case), dist=DIST,
                   wavelength=WAVELENGTH, pixel=PIXEL, unit=case["unit"], split=case["split"],
                   dtype=DTYPES[case["dtype"]], accum=case["accum"], device=DEV, **kw)


def _on_device(case, centre):
    return az.Plan.on_device(case["h"], case["w"], case["npt"], device=DEV,
                             npt_azim=case["azim"] or None, center=centre, dist=DIST,
                             wavelength=WAVELENGTH, pixel=PIXEL, unit=case["unit"],
                             split=case["split"], dtype=DTYPES[case["dtype"]],
                             accum=case["accum"])


def _batch_shapes(case):
    """(h, w, npt) of every image: pixel counts spread evenly over the logarithm of
    [lo, hi], in an order mixed by case["mix"]."""
    k, n = case["images"], []
    for i in range(k):
        n.append(case["lo"] * (case["hi"] / case["lo"]) ** ((i + 0.5) / k))
    order = sorted(range(k), key=lambda i: ((i + 1) * (2 * case["mix"] + 7919) * 2654435761) % (1 << 32))
    shapes = []
    for i in order:
        h = max(1, round(math.sqrt(n[i])))
        w = max(1, round(n[i] / h))
        shapes.append((h, w, max(1, round(math.sqrt(h * w)))))
    return shapes


def _batch_inputs(case, seed):
    g, dtype = _gen(seed), DTYPES[case["dtype"]]
    shapes = _batch_shapes(case)
    n, bins = sum(h * w for h, w, _ in shapes), sum(b for _, _, b in shapes)
    x = torch.randint(0, 1 << 20, (n,), generator=g, device=DEV, dtype=torch.int32).to(dtype)
    gI = torch.randn(bins, generator=g, device=DEV, dtype=dtype)
    gW = torch.randn(bins, generator=g, device=DEV, dtype=dtype)
    return shapes, x, gI, gW


def prepare(case, seed):
    if case["kind"] == "batch":
        shapes, x, gI, gW = _batch_inputs(case, seed)
        plans = [az.Plan(h, w, b, dtype=DTYPES[case["dtype"]]) for h, w, b in shapes]
        return dict(kind="batch", batch=az.Batch(plans, device=DEV), x=x,
                    gI=gI if case["backward"] else None, gW=gW)
    g, n, dtype = _gen(seed), case["h"] * case["w"], DTYPES[case["dtype"]]
    s = dict(kind=case["kind"])
    if case["kind"] == "build":
        s.update(case=case, centre=_centre(case, seed), x=_frame(case, g, n).to(dtype))
        return s
    s["plan"] = plan = _on_device(case, _centre(case)) if case["azim"] else _plan(case)
    if case["kind"] in ("frame", "graph"):
        s["raw"] = _frame(case, g, n)
        plan.set_corrections(*_corrections(g, n, dtype))
        if case["kind"] == "graph":
            s["out"] = tuple(torch.empty(plan.npt, dtype=dtype, device=DEV) for _ in range(3))
            s["graph"] = plan.graph(s["raw"], *s["out"])
    elif case["kind"] == "image":
        s["x"] = _frame(case, g, n).to(dtype)
    else:
        s["x"] = _frame(case, g, n).to(dtype).mul_(2.0 ** -20).requires_grad_()
        s["gI"] = torch.randn(plan.npt, generator=g, device=DEV, dtype=dtype)
        s["gW"] = torch.randn(plan.npt, generator=g, device=DEV, dtype=dtype)
    return s


def run(state):
    kind = state["kind"]
    if kind == "frame":
        return state["plan"].integrate_raw(state["raw"])
    if kind == "image":
        return state["plan"].integrate(state["x"])
    if kind == "graph":
        state["graph"].launch()
        return state["out"]
    if kind == "grad":
        I, W, U = az.Integrate1d.apply(state["x"], state["plan"], 0.0)
        (gx,) = torch.autograd.grad((I, W), state["x"], (state["gI"], state["gW"]))
        return I.detach(), W.detach(), U, gx
    if kind == "batch":
        I, W, U = state["batch"].forward(state["x"])
        if state["gI"] is None:
            return I, W, U
        return I, W, U, state["batch"].backward(U, state["gI"], state["gW"])
    return _on_device(state["case"], state["centre"]).integrate(state["x"])


# ---------------------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------------------


def _entries(h, w, npt, azim=0, cy=0.5, cx=0.5):
    """About how many nonzeros the matrix has: a pixel of side 1 spans 4 / pi of a pixel
    along the radius on average, the bins divide the way to the farthest corner."""
    far = math.hypot(max(cy, 1 - cy) * h, max(cx, 1 - cx) * w)
    n = h * w * (1 + 4 / math.pi * npt / far)
    if azim:
        n *= 1 + 4 / math.pi * 3.53 / math.sqrt(h * w) * azim / (2 * math.pi)
    return n


def work(case):
    s = 8 if case["dtype"] == "f64" else 4
    if case["kind"] == "batch":
        shapes = _batch_shapes(case)
        npix, bins = sum(h * w for h, w, _ in shapes), sum(b for _, _, b in shapes)
        nnz = sum(_entries(*sh) for sh in shapes)
        both = 2 if case["backward"] else 1
        return {"bytes": both * (nnz + npix) * s + (3 + 2 * both) * bins * s, "flops": 2 * both * nnz}
    npix = case["h"] * case["w"]
    bins = case["npt"] * max(1, case["azim"])
    nnz = _entries(case["h"], case["w"], case["npt"], case["azim"], case["cy"], case["cx"])
    image = RAWS[case["raw"]][1] if case["kind"] in ("frame", "graph") else s
    got = {"bytes": nnz * s + npix * image + 3 * bins * s, "flops": 2 * nnz}
    if case["kind"] == "grad":
        got["bytes"] += nnz * s + npix * s + 2 * bins * s
        got["flops"] *= 2
    elif case["kind"] == "build":
        got["bytes"] += nnz * (s + 4)
        got["flops"] += 40 * npix
    return got


# ---------------------------------------------------------------------------------------
# Every output in float64
# ---------------------------------------------------------------------------------------


def _to_unit(r, unit):
    if unit == "r_m":
        return r
    if unit == "r_mm":
        return r * 1e3
    tth = torch.atan(r / DIST)
    if unit == "2th_deg":
        return tth * (180.0 / math.pi)
    return 4.0 * math.pi * torch.sin(tth / 2.0) / (WAVELENGTH * 1e9)


def _corners(h, w, cy, cx):
    """y of the upper and lower, x of the left and right pixel edges, in metres."""
    y = torch.arange(h + 1, device=DEV, dtype=torch.float64).sub_(cy).mul_(PIXEL)
    x = torch.arange(w + 1, device=DEV, dtype=torch.float64).sub_(cx).mul_(PIXEL)
    lo = lambda v: v[:-1]
    hi = lambda v: v[1:]
    e = lambda a, b: torch.stack((a[:, None].expand(h, w), b[None, :].expand(h, w))).reshape(2, -1)
    return e(lo(y), lo(x)), e(lo(y), hi(x)), e(hi(y), hi(x)), e(hi(y), lo(x))


def _turn(chi, ref):
    """chi moved by whole turns to within half a turn of ref."""
    return torch.where(chi - ref > math.pi, chi - 2 * math.pi,
                       torch.where(chi - ref < -math.pi, chi + 2 * math.pi, chi))


def _shares(lo, hi, first, n):
    """Yields (pixels, bin, share) for boxes [lo, hi] over bins of width 1, bin by bin."""
    p = torch.arange(lo.numel(), device=DEV)
    k = 0
    while p.numel():
        b = first[p] + k
        share = (torch.minimum(hi[p], b + 1.0) - torch.maximum(lo[p], b.double())).clamp_(min=0) \
            / (hi[p] - lo[p])
        ok = (b >= 0) & (b < n) & (share > 0)
        yield p[ok], b[ok], share[ok]
        k += 1
        p = p[(first[p] + k).double() < hi[p]]


def _full_shares(u, chi, lo, hi, first, n):
    """The same for the quadrilaterals with corners (u[k], chi[k]): the share of the area
    below t is the sum over the edges of the integral of chi(u) up to t."""
    def below(p, t):
        a = torch.zeros_like(t)
        for k in range(4):
            u0, u1, c0, c1 = u[k][p], u[(k + 1) % 4][p], chi[k][p], chi[(k + 1) % 4][p]
            v0, v1 = torch.minimum(u0, t), torch.minimum(u1, t)
            slope = torch.where(u1 != u0, (c1 - c0) / (u1 - u0), torch.zeros_like(t))
            mid = c0 + slope * ((v0 + v1) / 2 - u0)
            a += torch.where(u1 != u0, mid * (v1 - v0), torch.zeros_like(t))
        return a
    p = torch.arange(lo.numel(), device=DEV)
    whole = below(p, hi + 1.0)
    k = 0
    while p.numel():
        b = first[p] + k
        share = (below(p, torch.minimum(b + 1.0, hi[p])) - below(p, torch.maximum(b.double(), lo[p]))) / whole[p]
        ok = (b >= 0) & (b < n) & (share > 0)
        yield p[ok], b[ok], share[ok]
        k += 1
        p = p[(first[p] + k).double() < hi[p]]


def _matrix(h, w, npt, cy, cx, unit="r_m", split="bbox", azim=0):
    """Yields (pixels, rows, coefficients) that together are the matrix."""
    cs = _corners(h, w, cy, cx)
    y0, x0, y1, x1 = cs[0][0], cs[0][1], cs[2][0], cs[2][1]
    zero = torch.zeros((), device=DEV, dtype=torch.float64)
    ny = torch.where(y0 > 0, y0, torch.where(y1 < 0, y1, zero))
    nx = torch.where(x0 > 0, x0, torch.where(x1 < 0, x1, zero))
    fy, fx = torch.maximum(y0.abs(), y1.abs()), torch.maximum(x0.abs(), x1.abs())
    near = torch.sqrt(ny * ny + nx * nx)
    lo, hi = _to_unit(near, unit), _to_unit(torch.sqrt(fy * fy + fx * fx), unit)
    bottom, top = lo.min(), hi.max()
    scale = lambda v: (v - bottom) / ((top - bottom) / npt)
    lo, hi = scale(lo), scale(hi)
    first = lo.floor().long()
    holds = near == 0
    if not azim and split == "bbox":
        yield from _shares(lo, hi, first, npt)
        return
    chi0 = torch.atan2(cs[0][0], cs[0][1])
    chi = [chi0] + [_turn(torch.atan2(c[0], c[1]), chi0) for c in cs[1:]]
    if not azim:
        out = (~holds).nonzero()[:, 0]
        u = [scale(_to_unit(torch.sqrt(c[0] * c[0] + c[1] * c[1]), unit))[out] for c in cs]
        for p, b, s in _full_shares(u, [c[out] for c in chi], lo[out], hi[out], first[out], npt):
            yield out[p], b, s
        inn = holds.nonzero()[:, 0]
        for p, b, s in _shares(lo[inn], hi[inn], first[inn], npt):
            yield inn[p], b, s
        return
    wedge = 2 * math.pi / azim
    chi = torch.stack(chi)
    clo, chi_hi = (chi.amin(0) + math.pi) / wedge, (chi.amax(0) + math.pi) / wedge
    clo, chi_hi = torch.where(holds, zero, clo), torch.where(holds, zero + azim, chi_hi)
    cfirst = clo.floor().long()
    for p, b, s in _shares(lo, hi, first, npt):
        # wedges from half a turn below to half a turn above: numbered from 0 by a shift
        for q, c, t in _shares(clo[p] + azim, chi_hi[p] + azim, cfirst[p] + azim, 3 * azim):
            yield p[q], (c % azim) * npt + b[q], s[q] * t


def _integrated(entries, x, bins):
    W = torch.zeros(bins, device=DEV, dtype=torch.float64)
    U = torch.zeros_like(W)
    for p, b, c in entries:
        W.index_add_(0, b, c * x[p])
        U.index_add_(0, b, c)
    return torch.where(U != 0, W / U, torch.zeros_like(W)), W, U


def _gradient(entries, U, gI, gW, npix):
    v = torch.where(U != 0, gI / U, torch.zeros_like(U)) + gW
    gx = torch.zeros(npix, device=DEV, dtype=torch.float64)
    for p, b, c in entries:
        gx.index_add_(0, p, c * v[b])
    return gx


def exact(case, seed):
    if case["kind"] == "batch":
        shapes, x, gI, gW = _batch_inputs(case, seed)
        parts, p, b = [], 0, 0
        for h, w, npt in shapes:
            pix, bins = slice(p, p + h * w), slice(b, b + npt)
            m = list(_matrix(h, w, npt, h / 2.0, w / 2.0))
            got = _integrated(m, x[pix].double(), npt)
            if case["backward"]:
                got += (_gradient(m, got[2], gI[bins].double(), gW[bins].double(), h * w),)
            parts.append(got)
            p, b = p + h * w, b + npt
        return tuple(torch.cat(v) for v in zip(*parts))
    g, n, dtype = _gen(seed), case["h"] * case["w"], DTYPES[case["dtype"]]
    x = _frame(case, g, n).to(dtype)
    if case["kind"] in ("frame", "graph"):
        dark, flat, solid, polar = (c.double() for c in _corrections(g, n, dtype))
        x = (x.double() - dark) / (flat * solid * polar)
    elif case["kind"] == "grad":
        x = x.mul_(2.0 ** -20)
    cy, cx = _centre(case, seed if case["kind"] == "build" else None)
    bins = case["npt"] * max(1, case["azim"])
    matrix = lambda: _matrix(case["h"], case["w"], case["npt"], cy, cx, case["unit"], case["split"],
                             case["azim"])
    got = _integrated(matrix(), x.double(), bins)
    if case["kind"] == "grad":
        gI = torch.randn(bins, generator=g, device=DEV, dtype=dtype).double()
        gW = torch.randn(bins, generator=g, device=DEV, dtype=dtype).double()
        got += (_gradient(matrix(), got[2], gI, gW, n),)
    return got
