"""Timed cases: the work that users of this library have it do, through the
public Python entry points, from single small signals to 4096 x 4096 images.

A case is a dict of plain values; `kind` selects the workload:
  signal_cg       CG filter of one 1D signal on a kept BF operator (the 1D
                  filter study: a call of some tens of microseconds per step,
                  where launches and latency count)
  signal_lobpcg   block LOBPCG filter of one 1D signal on a kept BF operator
  experiment      the image experiment: the 5-point operator (normalized by
                  diag L) of a new image, then CG and LOBPCG (m = 1) of it
  colour          a new colour image: sRGB -> CIE-Lab, the three-channel BF
                  operator, the RGB block filtered by block CG
  reguided        re-guided (non-linear) filters: the graph follows the iterate
  joint           a new image: operator build, then CG and LOBPCG side by side
                  (the step that the benchmark times)
  filter          CG or power filter of one image on a kept BF or GF operator
  lobpcg          block LOBPCG filter of one image on a kept BF or GF operator
  batch           an uneven batch of images and signals (BF and GF, CG and
                  LOBPCG mixed), planned once and replayed on new contents
  net_grad        learned preconditioner, training: loss and weight gradient
                  of one mini-batch of residual / target pairs
  precond         learned preconditioner, inference: T(R) of an n x m block

Inputs are seeded synthetic images, signals and weights of the kinds the
benchmark and the tests use, made on the GPU.  `exact` evaluates the same
filters with plain torch in FP64.
"""
import math
import random

import numpy as np
import torch

import paper_1509_02468_amd as gsf

PREC = {"f32": gsf.F32, "f64": gsf.F64}
DTYPE = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # the smallest call of the 1D study: 500 samples, 20 CG steps, noiseless guidance
        dict(name="signal_cg_500", kind="signal_cg", n=500, radius=1, sigma_d=1.0, sigma_r=0.1, prec="f64", steps=20),
        # one signal through block LOBPCG: every step a chain of small launches
        dict(name="signal_lobpcg_4096", kind="signal_lobpcg", n=4096, radius=5, sigma_d=3.0, sigma_r=0.2, prec="f64",
             m=3, steps=30, constraint=False),
        # the image experiment at its size: 5-point lattice, noise variance 0.01, 20 steps of each filter
        dict(name="experiment_1024", kind="experiment", rows=1024, cols=1024, steps=20),
        # a colour photograph denoised: Lab guidance, 11 x 11 window, 10 CG steps on three channels
        dict(name="colour_1024", kind="colour", rows=1024, cols=1024, radius=5, sigma_d=2.0, sigma_r=5.0, steps=10),
        # non-linear filtering: 20 CG steps, the 11 x 11 graph rebuilt from every iterate
        dict(name="reguided_1024", kind="reguided", graph="bf", method="cg", rows=1024, cols=1024, radius=5,
             prec="f32", steps=20),
        # the benchmark's step: build, CG 50 and LOBPCG (m = 4) 50 of a 1024 x 1024 image, 11 x 11 window
        dict(name="joint_1024", kind="joint", rows=1024, cols=1024, radius=5, m=4, prec="f32", steps=50),
        # a large image on the guided-filter operator: 20 CG steps at 4096 x 4096, radius 8
        dict(name="filter_gf_4096", kind="filter", graph="gf", method="cg", rows=4096, cols=4096, radius=8,
             prec="f32", steps=20),
        # a wide block on a large image: LOBPCG m = 8 at 4096 x 4096, 7 x 7 window (10 of its steps)
        dict(name="lobpcg_bf_4096", kind="lobpcg", graph="bf", rows=4096, cols=4096, radius=3, m=8, prec="f32",
             steps=10, constraint=False),
        # the same filter on the guided-filter operator, all in FP64, on a ragged grid, with the constraint
        dict(name="lobpcg_gf_1531x2047", kind="lobpcg", graph="gf", rows=1531, cols=2047, radius=8, m=8, prec="f64",
             steps=10, constraint=True),
        # a server's mixed batch: 18 images and 6 signals of uneven sizes, replayed
        dict(name="batch_24", kind="batch", images=18, signals=6, largest=512, recipe=4, steps=20),
        # one training mini-batch of the preconditioner network: 16 pairs of 512 x 512
        dict(name="net_grad_16x512", kind="net_grad", batch=16, rows=512, cols=512),
        # the network applied to the four residual columns of a 2048 x 2048 LOBPCG step
        dict(name="precond_2048", kind="precond", rows=2048, cols=2048, m=4, prec="f32"),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["signal_cg", "signal_lobpcg", "experiment", "colour", "reguided", "joint", "filter", "lobpcg",
                       "batch", "net_grad", "precond"])
    c = dict(kind=kind)
    if kind == "signal_cg":
        c.update(n=size(300, 200000), radius=rng.choice([1, 2, 5]), sigma_d=rng.choice([1.0, 3.0]),
                 sigma_r=rng.choice([0.1, 0.2]), prec=rng.choice(["f64", "f32"]), steps=rng.randint(10, 30))
    elif kind == "signal_lobpcg":
        c.update(n=size(1000, 200000), radius=rng.choice([1, 3, 5]), sigma_d=3.0, sigma_r=0.2, prec="f64",
                 m=rng.randint(1, 4), steps=rng.randint(10, 30), constraint=rng.random() < 0.5)
    elif kind == "experiment":
        c.update(rows=size(200, 1200), cols=size(200, 1200), steps=rng.randint(10, 20))
    elif kind == "colour":
        c.update(rows=size(200, 1200), cols=size(200, 1200), radius=rng.randint(2, 5), sigma_d=2.0, sigma_r=5.0,
                 steps=rng.randint(5, 10))
    elif kind == "reguided":
        c.update(graph=rng.choice(["bf", "gf"]), method=rng.choice(["cg", "power"]), rows=size(128, 1200),
                 cols=size(128, 1200), radius=rng.randint(1, 5), prec=rng.choice(["f32", "f32", "f64"]),
                 steps=rng.randint(5, 20))
    elif kind == "joint":
        c.update(rows=size(200, 1024), cols=size(200, 1024), radius=rng.randint(2, 5), m=rng.choice([1, 3, 4, 4]),
                 prec="f32", steps=rng.randint(10, 40))
    elif kind == "filter":
        graph = rng.choice(["bf", "gf"])
        c.update(graph=graph, method=rng.choice(["cg", "cg", "power"]), rows=size(256, 4096), cols=size(256, 4096),
                 radius=rng.randint(1, 4) if graph == "bf" else rng.randint(1, 8),
                 prec=rng.choice(["f32", "f32", "f64"]), steps=rng.randint(5, 20))
    elif kind == "lobpcg":
        graph = rng.choice(["bf", "gf"])
        c.update(graph=graph, rows=size(256, 2048), cols=size(256, 2048),
                 radius=rng.randint(1, 4) if graph == "bf" else rng.randint(1, 8), m=rng.randint(1, 8),
                 prec=rng.choice(["f32", "f64"]), steps=rng.randint(5, 10), constraint=rng.random() < 0.5)
    elif kind == "batch":
        c.update(images=rng.randint(4, 18), signals=rng.randint(2, 6), largest=size(128, 512),
                 recipe=rng.randint(1, 1000), steps=rng.randint(10, 20))
    elif kind == "net_grad":
        c.update(batch=rng.randint(1, 16), rows=size(64, 512), cols=size(64, 512))
    else:
        c.update(rows=size(128, 2048), cols=size(128, 2048), m=rng.randint(1, 4), prec=rng.choice(["f32", "f32", "f64"]))
    return c


# ---- inputs ------------------------------------------------------------------
def _signal(n, sigma, seed, steep=False):
    """(clean, noisy) 1D signal, FP64 on the GPU: nine constant pieces, or
    (steep) piecewise linear with steep ascents and descents."""
    rng = np.random.default_rng(seed)
    cuts = np.sort(rng.choice(np.arange(8, n - 8, 8), size=8, replace=False))
    if steep:
        kx, ky = [0.0], [rng.uniform()]
        for k in cuts[::2]:
            up = rng.uniform(0.3, 0.7)
            kx += [float(k), float(k) + 4.0]
            ky += [ky[-1], ky[-1] + (up if ky[-1] < 0.5 else -up)]
        kx.append(float(n))
        ky.append(ky[-1] + 0.2)
        clean = np.interp(np.arange(n), kx, ky)
    else:
        clean = np.repeat(rng.uniform(0.0, 1.0, 9), np.diff(np.concatenate(([0], cuts, [n]))))
    noisy = clean + sigma * rng.standard_normal(n)
    return torch.from_numpy(clean).cuda(), torch.from_numpy(noisy).cuda()


def _scene(rows, cols, sigma, seed, channels=1):
    """Noisy scene (rows x cols x channels, FP64 on the GPU): a linear
    gradient background, 40 rectangles and discs, Gaussian noise."""
    rng = random.Random(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    y = torch.arange(rows, device="cuda", dtype=torch.float32)[:, None] + 0.5
    x = torch.arange(cols, device="cuda", dtype=torch.float32)[None, :] + 0.5
    side = float(max(rows, cols))
    level = lambda: torch.tensor([rng.random() for _ in range(channels)], device="cuda", dtype=torch.float64)  # noqa: E731
    phi = rng.uniform(0.0, 2.0 * math.pi)
    t = (math.cos(phi) * x + math.sin(phi) * y).double()
    t = (t - t.min()) / (t.max() - t.min())
    c0, c1 = level(), level()
    img = c0 + (c1 - c0) * t[..., None]
    for _ in range(40):
        cy, cx = rng.uniform(0.0, rows), rng.uniform(0.0, cols)
        if rng.random() < 0.5:
            hy, hx = rng.uniform(0.02, 0.15) * side, rng.uniform(0.02, 0.15) * side
            mask = ((y - cy).abs() <= hy) & ((x - cx).abs() <= hx)
        else:
            rad = rng.uniform(0.02, 0.15) * side
            mask = (y - cy) ** 2 + (x - cx) ** 2 <= rad * rad
        img = torch.where(mask[..., None], level(), img)
    return img + sigma * torch.randn(img.shape, generator=gen, device="cuda", dtype=torch.float64)


def _image(case, seed, sigma, dtype):
    return _scene(case["rows"], case["cols"], sigma, seed)[..., 0].reshape(-1).to(dtype)


def _graph_args(graph, radius):
    """Parameters of the two operators as the large-image workloads set them."""
    return dict(radius=radius, sigma_d=2.0, sigma_r=0.15) if graph == "bf" else dict(radius=radius, eps=1e-2)


def _batch_recipe(case):
    """The items' shapes and parameters (the same for every seed of the inputs)."""
    rng = random.Random(case["recipe"])
    items = []
    for i in range(case["images"] + case["signals"]):
        if i < case["images"]:
            s = int(round(math.exp(rng.uniform(math.log(64), math.log(case["largest"])))))
            shape = (s, s)
        else:
            shape = (int(round(math.exp(rng.uniform(math.log(2 ** 10), math.log(2 ** 18))))),)
        it = dict(shape=shape, sigma=rng.uniform(0.03, 0.1))
        if rng.random() < 0.5:
            it.update(kind="bf", radius=rng.randint(1, 5), sigma_d=rng.uniform(1.0, 3.0), sigma_r=rng.uniform(0.05, 0.3))
        else:
            it.update(kind="gf", radius=rng.randint(1, 8), eps=math.exp(rng.uniform(math.log(1e-3), math.log(1e-1))))
        lob = rng.random() < 0.5
        it.update(method="lobpcg" if lob else "cg", m=4 if lob else 1, kmax=case["steps"], tol=0.0)
        items.append(it)
    return items


def _batch_inputs(case, seed):
    return [(_scene(*it["shape"], it["sigma"], 1000 * seed + i)[..., 0].reshape(-1) if len(it["shape"]) == 2
             else _signal(it["shape"][0], it["sigma"], 1000 * seed + i)[1]).float()
            for i, it in enumerate(_batch_recipe(case))]


def _weights(seed):
    """He-scaled initial weights of the network (2736 values)."""
    rng = np.random.default_rng(seed)
    return np.concatenate([rng.standard_normal(288) * math.sqrt(2 / 18), rng.standard_normal(2304) * math.sqrt(2 / 144),
                           rng.standard_normal(144) * math.sqrt(1 / 144)]).astype(np.float32)


def _pairs(case, seed):
    """Training pairs: residual columns of unit RMS beside their guidance, and
    smoother, larger targets; and the mini-batch's sample indices."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rows, cols, count = case["rows"], case["cols"], case["batch"] + 4
    inputs = torch.empty((count, rows * cols, 2), device="cuda")
    targets = torch.empty((count, rows * cols), device="cuda")
    for s in range(count):
        r = torch.randn((rows, cols), generator=gen, device="cuda")
        g = _scene(rows, cols, 0.05, 100 * seed + s)[..., 0].float()
        r = r * (0.2 + (g - 0.5).abs())
        r = r / r.square().mean().sqrt()
        smooth = r
        for _ in range(3):
            smooth = (smooth + smooth.roll(1, 0) + smooth.roll(1, 1) + smooth.roll((1, 1), (0, 1))) * 0.5
        inputs[s, :, 0], inputs[s, :, 1], targets[s] = r.reshape(-1), g.reshape(-1), smooth.reshape(-1) * 4.0
    idx = torch.randperm(count, generator=gen, device="cuda")[:case["batch"]].to(torch.int32)
    return inputs, targets, idx


def _signal_pair(case, seed):
    clean, noisy = _signal(case["n"], 0.1, seed, steep=True)
    d = DTYPE[case["prec"]]
    return clean.to(d), noisy.to(d)


def _residual_block(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    d = DTYPE[case["prec"]]
    g = _image(case, seed, 0.05, d)
    R = torch.randn((g.numel(), case["m"]), generator=gen, device="cuda", dtype=torch.float64)
    R = R * (1e-3 * (0.2 + (g.double() - 0.5).abs()))[:, None]
    return g, R.to(d)


# ---- the calls -----------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("signal_cg", "signal_lobpcg"):
        clean, noisy = _signal_pair(case, seed)
        op = gsf.Operator("bf", (case["n"],), clean if kind == "signal_cg" else noisy, case["radius"], case["sigma_d"],
                          case["sigma_r"], prec=PREC[case["prec"]])
        ws = op.workspace(gsf.METHOD_CG) if kind == "signal_cg" else op.workspace(gsf.METHOD_LOBPCG, case["m"])
        s.update(op=op, x0=noisy, out=torch.empty_like(noisy), ws=ws)
    elif kind == "experiment":
        x0 = _image(case, seed, 0.1, torch.float32)
        op = _experiment_operator(case, x0)
        s.update(x0=x0, op_ws=op.ws, out=(torch.empty_like(x0), torch.empty_like(x0)),
                 ws=(op.workspace(gsf.METHOD_CG), op.workspace(gsf.METHOD_LOBPCG, 1)))
    elif kind == "colour":
        rgb = _scene(case["rows"], case["cols"], 0.05, seed, 3).reshape(-1, 3).float()
        op = _colour_operator(case, torch.empty_like(rgb).fill_(50.0))
        s.update(rgb=rgb, lab=torch.empty_like(rgb), op_ws=op.ws, out=torch.empty_like(rgb),
                 ws=op.workspace(gsf.METHOD_CG, 3))
    elif kind == "reguided":
        x0 = _image(case, seed, 0.05, DTYPE[case["prec"]])
        method = gsf.METHOD_CG if case["method"] == "cg" else gsf.METHOD_POWER
        par = _graph_args(case["graph"], case["radius"])
        shape = (case["rows"], case["cols"])
        s.update(x0=x0, out=torch.empty_like(x0), method=method, shape=shape, par=par,
                 ws=gsf.reguided_workspace(case["graph"], shape, method, prec=PREC[case["prec"]], **par))
    elif kind == "joint":
        x0 = _image(case, seed, 0.05, DTYPE[case["prec"]])
        op = _joint_operator(case, x0)
        s.update(x0=x0, op_ws=op.ws, ws=op.joint_workspace(case["m"]), out=(torch.empty_like(x0), torch.empty_like(x0)))
    elif kind in ("filter", "lobpcg"):
        x0 = _image(case, seed, 0.08, DTYPE[case["prec"]])
        op = gsf.Operator(case["graph"], (case["rows"], case["cols"]), x0, prec=PREC[case["prec"]],
                          **_graph_args(case["graph"], case["radius"]))
        if kind == "lobpcg":
            ws = op.workspace(gsf.METHOD_LOBPCG, case["m"])
        else:
            ws = op.workspace(gsf.METHOD_CG if case["method"] == "cg" else gsf.METHOD_POWER)
        s.update(op=op, x0=x0, out=torch.empty_like(x0), ws=ws)
    elif kind == "batch":
        items = [dict(it, guidance=x, x0=x) for it, x in zip(_batch_recipe(case), _batch_inputs(case, seed))]
        s.update(items=items, batch=gsf.Batch(items, gsf.F32, autotune=False, graphs=True))
    elif kind == "net_grad":
        inputs, targets, idx = _pairs(case, seed)
        s.update(inputs=inputs, targets=targets, idx=idx,
                 trainer=gsf.NetTrainer(_weights(seed), case["batch"], case["rows"], case["cols"]))
    else:
        g, R = _residual_block(case, seed)
        op = gsf.Operator("bf", (case["rows"], case["cols"]), g, 1, 2.0, 0.1, prec=PREC[case["prec"]])
        w = torch.from_numpy(_weights(seed)).cuda().bfloat16()
        s.update(T=gsf.Precond(op, g, w), R=R, out=torch.empty_like(R))
    return s


def _experiment_operator(case, x0, ws=None):
    return gsf.Operator("bf", (case["rows"], case["cols"]), x0, 1, 1.0, 0.1, stencil="cross", norm="diagl", ws=ws)


def _colour_operator(case, lab, ws=None):
    return gsf.Operator("bf", (case["rows"], case["cols"]), lab, case["radius"], case["sigma_d"], case["sigma_r"],
                        channels=3, ws=ws)


def _joint_operator(case, x0, ws=None):
    return gsf.Operator("bf", (case["rows"], case["cols"]), x0, case["radius"], 2.0, 0.1, prec=PREC[case["prec"]], ws=ws)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "signal_cg":
        return s["op"].cg_filter(s["x0"], case["steps"], out=s["out"], ws=s["ws"], info=False)[0]
    if kind in ("signal_lobpcg", "lobpcg"):
        return s["op"].lobpcg_filter(s["x0"], case["m"], case["steps"], constraint=case["constraint"], out=s["out"],
                                     ws=s["ws"], info=False)[0]
    if kind == "experiment":
        op = _experiment_operator(case, s["x0"], s["op_ws"])
        a, _ = op.cg_filter(s["x0"], case["steps"], out=s["out"][0], ws=s["ws"][0], info=False)
        b, _ = op.lobpcg_filter(s["x0"], 1, case["steps"], out=s["out"][1], ws=s["ws"][1], info=False)
        return a, b
    if kind == "colour":
        lab = gsf.srgb_to_lab(s["rgb"], out=s["lab"])
        op = _colour_operator(case, lab, s["op_ws"])
        y, _ = op.cg_filter_block(s["rgb"], case["steps"], out=s["out"], ws=s["ws"], info=False)
        return lab, y
    if kind == "reguided":
        return gsf.reguided_filter(case["graph"], s["shape"], s["x0"], s["method"], case["steps"],
                                   prec=PREC[case["prec"]], out=s["out"], ws=s["ws"], info=False, **s["par"])[0]
    if kind == "joint":
        op = _joint_operator(case, s["x0"], s["op_ws"])
        a, b, _, _ = op.joint_filter(s["x0"], case["steps"], s["x0"], case["m"], case["steps"], out_cg=s["out"][0],
                                     out_lob=s["out"][1], ws=s["ws"], info=False)
        return a, b
    if kind == "filter":
        if case["method"] == "power":
            return s["op"].power_filter(s["x0"], case["steps"], out=s["out"], ws=s["ws"])
        return s["op"].cg_filter(s["x0"], case["steps"], out=s["out"], ws=s["ws"], info=False)[0]
    if kind == "batch":
        s["batch"].run()
        return [it["out"] for it in s["items"]]
    if kind == "net_grad":
        return s["trainer"].loss_grad(s["idx"], s["inputs"], s["targets"])
    return s["T"].apply(s["R"], out=s["out"])


# ---- what a pass cannot do without -----------------------------------------------
def _apply_work(graph, n, radius, ndim, elem, m, stencil="square"):
    """(bytes, flops) of one operator apply: the operator's stored data once, the block in and out."""
    if graph == "gf":
        return n * elem * (3 + 2 * m), n * m * 40
    planes = 2 * radius if stencil == "cross" else ((2 * radius + 1) ** ndim - 1) // 2
    return n * elem * (planes + 1 + 2 * m), n * m * 6 * planes


def _cg_work(graph, n, radius, ndim, elem, m, steps, stencil="square"):
    b, f = _apply_work(graph, n, radius, ndim, elem, m, stencil)
    return (steps + 1) * (b + 6 * n * m * elem), (steps + 1) * (f + 10 * n * m)


def _lobpcg_work(graph, n, radius, ndim, elem, m, steps, stencil="square"):
    b, f = _apply_work(graph, n, radius, ndim, elem, m, stencil)
    return (steps + 1) * (b + 11 * n * m * elem), (steps + 1) * (f + n * m * m * (27 + 12))


def _build_work(n, planes, elem, channels=1):
    return n * elem * (channels + planes + 2), n * planes * (3 * channels + 4)


def work(case):
    kind = case["kind"]
    elem = 8 if case.get("prec") == "f64" else 4
    n = case["n"] if "n" in case else case.get("rows", 0) * case.get("cols", 0)
    if kind == "signal_cg":
        parts = [_cg_work("bf", n, case["radius"], 1, elem, 1, case["steps"])]
    elif kind == "signal_lobpcg":
        parts = [_lobpcg_work("bf", n, case["radius"], 1, elem, case["m"], case["steps"])]
    elif kind == "experiment":
        parts = [_build_work(n, 2, 4), _cg_work("bf", n, 1, 2, 4, 1, case["steps"], "cross"),
                 _lobpcg_work("bf", n, 1, 2, 4, 1, case["steps"], "cross")]
    elif kind == "colour":
        planes = ((2 * case["radius"] + 1) ** 2 - 1) // 2
        parts = [(n * 24, n * 100), _build_work(n, planes, 4, 3),
                 _cg_work("bf", n, case["radius"], 2, 4, 3, case["steps"])]
    elif kind == "reguided":
        window = (2 * case["radius"] + 1) ** 2 if case["graph"] == "bf" else 8
        vectors = 8 if case["method"] == "cg" else 2
        parts = [(case["steps"] * n * elem * vectors, case["steps"] * n * window * 8)]
    elif kind == "joint":
        planes = ((2 * case["radius"] + 1) ** 2 - 1) // 2
        b, f = _apply_work("bf", n, case["radius"], 2, elem, case["m"] + 1)
        steps = case["steps"] + 1
        parts = [_build_work(n, planes, elem),
                 (steps * (b + n * elem * (6 + 11 * case["m"])), steps * (f + n * (10 + 39 * case["m"] ** 2)))]
    elif kind == "filter":
        if case["method"] == "power":
            b, f = _apply_work(case["graph"], n, case["radius"], 2, elem, 1)
            parts = [(case["steps"] * b, case["steps"] * f)]
        else:
            parts = [_cg_work(case["graph"], n, case["radius"], 2, elem, 1, case["steps"])]
    elif kind == "lobpcg":
        parts = [_lobpcg_work(case["graph"], n, case["radius"], 2, elem, case["m"], case["steps"])]
    elif kind == "batch":
        parts = []
        for it in _batch_recipe(case):
            size, ndim = int(np.prod(it["shape"])), len(it["shape"])
            planes = ((2 * it["radius"] + 1) ** ndim - 1) // 2 if it["kind"] == "bf" else 3
            step = _cg_work if it["method"] == "cg" else _lobpcg_work
            parts += [_build_work(size, planes, 4), step(it["kind"], size, it["radius"], ndim, 4, it["m"], it["kmax"])]
    elif kind == "net_grad":
        pixels = case["batch"] * n
        parts = [(pixels * 12, pixels * 2 * 2736 * 3)]
    else:
        parts = [(n * elem * (2 * case["m"] + 1), n * case["m"] * 2 * 2736)]
    return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}


# ---- the same filters in FP64, plain torch ------------------------------------------
class _Bf:
    """BF graph of eq. (2): L u summed over the half window's edges."""

    def __init__(self, g, shape, radius, sigma_d, sigma_r, stencil="square", norm="d"):
        self.shape = shape if len(shape) == 2 else (1,) + tuple(shape)
        g = g.double().reshape(self.shape + (-1,))
        r, two_d = radius, len(shape) == 2
        offs = [(0, k) for k in range(1, r + 1)]
        if two_d:
            offs += [(k, 0) for k in range(1, r + 1)] if stencil == "cross" else \
                [(dy, dx) for dy in range(1, r + 1) for dx in range(-r, r + 1)]
        self.edges = []
        d = torch.zeros(self.shape, device=g.device, dtype=torch.float64)
        for dy, dx in offs:
            a, b = self._ends(dy, dx)
            if a is None:
                continue
            w = torch.exp(-(dy * dy + dx * dx) / (2.0 * sigma_d ** 2) - (g[a] - g[b]).square().sum(-1) / (2.0 * sigma_r ** 2))
            self.edges.append((a, b, w))
            d[a] += w
            d[b] += w
        if norm == "d":
            d += 1.0
        else:
            d[d == 0.0] = 1.0
        self.d = d.reshape(-1)
        self.sq = self.d.sqrt()

    def _ends(self, dy, dx):
        H, W = self.shape
        if dy >= H or abs(dx) >= W:
            return None, None
        xa, xb = (slice(0, W - dx), slice(dx, W)) if dx >= 0 else (slice(-dx, W), slice(0, W + dx))
        return (slice(0, H - dy), xa), (slice(dy, H), xb)

    def lap(self, u):
        v = u.reshape(self.shape + (-1,))
        y = torch.zeros_like(v)
        for a, b, w in self.edges:
            t = (v[a] - v[b]) * w[..., None]
            y[a] += t
            y[b] -= t
        return y.reshape(u.shape)


class _Gf:
    """GF graph of Algorithm 1: D u - GF(u) with truncated windows."""

    def __init__(self, g, shape, radius, eps):
        self.shape, self.r = tuple(shape), radius
        self.g = g.double().reshape(self.shape + (1,))
        self.count = self._box(torch.ones_like(self.g))
        self.full = float((2 * radius + 1) ** len(shape))
        self.mu = self._box(self.g) / self.count
        # centred about the image mean: the window variances lose fewer digits
        c = self.g - self.g.mean()
        mc = self._box(c) / self.count
        self.inv = 1.0 / (self._box(c * c) / self.count - mc * mc + eps)
        self.d = (self.count / self.full).reshape(-1)
        self.sq = self.d.sqrt()

    def _box(self, v):
        for axis, n in enumerate(self.shape):
            c = torch.cumsum(v, axis)
            i = torch.arange(n, device=v.device)
            hi = c.index_select(axis, (i + self.r).clamp(max=n - 1))
            lo = c.index_select(axis, (i - self.r - 1).clamp(min=0))
            mask = (i - self.r - 1 >= 0).double().reshape([-1 if k == axis else 1 for k in range(v.dim())])
            v = hi - lo * mask
        return v

    def lap(self, u):
        if u.dim() == 2:  # column by column
            return torch.stack([self.lap(u[:, j].contiguous()) for j in range(u.shape[1])], 1)
        v = u.reshape(self.shape + (1,))
        mean = self._box(v) / self.count
        a = (self._box(self.g * v) / self.count - self.mu * mean) * self.inv
        y = (self._box(a) * self.g + self._box(mean - a * self.mu)) / self.full
        return (self.d.reshape(self.shape + (1,)) * v - y).reshape(u.shape)


def _lsym(op, z):
    s = op.sq if z.dim() == 1 else op.sq[:, None]
    return op.lap(z / s) / s


def _cg(op, x0, steps):
    z = op.sq * x0.double()
    r = -_lsym(op, z)
    p, rho = r, torch.dot(r, r)
    for _ in range(steps):
        q = _lsym(op, p)
        alpha = rho / torch.dot(p, q)
        z = z + alpha * p
        r_new = r - alpha * q
        beta = torch.dot(r_new, r_new - r) / rho
        r = r_new
        rho = torch.dot(r, r)
        p = r + beta * p
    return z / op.sq


def _power(op, x0, steps):
    x = x0.double()
    for _ in range(steps):
        x = x - op.lap(x) / op.d
    return x


def _start_block(shape, z0, m):
    from numpy.polynomial import legendre
    if len(shape) == 1:
        degs = [(j,) for j in range(m)]
    else:
        degs = [(a, t - a) for t in range(m) for a in range(t + 1)][:m]
    cols = []
    for dg in degs:
        phi = None
        for n, k in zip(shape, dg):
            t = 2.0 * (np.arange(n) + 0.5) / n - 1.0
            v = torch.from_numpy(legendre.legval(t, np.eye(k + 1)[k])).to(z0.device)
            phi = v if phi is None else phi[:, None] * v[None, :]
        cols.append(z0 * phi.reshape(-1))
    return torch.stack(cols, 1)


def _rayleigh_ritz(GA, GB, m, drop, zero):
    GA, GB = 0.5 * (GA + GA.T), 0.5 * (GB + GB.T)
    k = len(GA)
    diag = np.diag(GB)
    good = diag > zero * zero * max(diag.max(), 0.0)
    delta = np.where(good, 1.0 / np.sqrt(np.where(good, diag, 1.0)), 0.0)
    A, B = delta[:, None] * GA * delta, delta[:, None] * GB * delta
    idx, L = [], np.zeros((k, k))
    for j in range(k):
        if not good[j]:
            continue
        t = len(idx)
        c = np.zeros(t)
        for i in range(t):
            c[i] = (B[j, idx[i]] - L[i, :i] @ c[:i]) / L[i, i]
        piv = B[j, j] - c @ c
        if piv > drop:
            L[t, :t], L[t, t] = c, np.sqrt(piv)
            idx.append(j)
    L = L[:len(idx), :len(idx)]
    Li = np.linalg.inv(L)
    M = Li @ A[np.ix_(idx, idx)] @ Li.T
    th, Z = np.linalg.eigh(0.5 * (M + M.T))
    C = np.zeros((k, m))
    C[idx] = delta[idx, None] * (Li.T @ Z[:, :m])
    return th[:m], C


def _gram(a, b):
    """a^T b, summed over slices of the rows."""
    return sum((x.T @ y).cpu().numpy() for x, y in zip(a.split(1 << 20), b.split(1 << 20)))


def _lobpcg(op, shape, x0, m, steps, constraint, prec):
    drop, zero = (1e-6, 1e-6) if prec == "f32" else (1e-10, 1e-13)
    z0 = op.sq * x0.double()
    Y = op.sq / op.sq.norm()
    free = (lambda V: V - Y[:, None] * (Y[:, None] * V).sum(0)) if constraint else (lambda V: V)
    X = free(_start_block(shape, z0, m))
    S, AS = [X], [_lsym(op, X)]
    for k in range(steps + 1):
        if k > 0:
            W = free(AX - X * theta)
            S, AS = [X, W] + ([P] if k > 1 else []), [AX, _lsym(op, W)] + ([AP] if k > 1 else [])
        T, AT = torch.cat(S, 1), torch.cat(AS, 1)
        th, C = _rayleigh_ritz(_gram(T, AT), _gram(T, T), m, drop, zero)
        theta, C = torch.from_numpy(th).to(X.device), torch.from_numpy(C).to(X.device)
        if k > 0:
            P, AP = T[:, m:] @ C[m:], AT[:, m:] @ C[m:]
        X, AX = T @ C, AT @ C
    y = (X * (X * z0[:, None]).sum(0)).sum(1)
    if constraint:
        y = y + Y * (Y * z0).sum()
    return y / op.sq


def _graph(graph, g, shape, par):
    return _Bf(g, shape, **par) if graph == "bf" else _Gf(g, shape, **par)


def _reguided(case, x0, shape, par):
    x = x0.double()
    if case["method"] == "power":
        for _ in range(case["steps"]):
            x = _power(_graph(case["graph"], x, shape, par), x, 1)
        return x
    op = _graph(case["graph"], x, shape, par)
    r = -op.lap(x)
    p = r_old = rho_old = None
    for k in range(case["steps"]):
        if k > 0:
            op = _graph(case["graph"], x, shape, par)
        s = r / op.d
        rho = torch.dot(s, r)
        p = s if k == 0 else s + torch.dot(s, r - r_old) / rho_old * p
        rho_old = rho
        q = op.lap(p)
        alpha = rho / torch.dot(p, q)
        x = x + alpha * p
        r_old = r
        r = r - alpha * q
    return x


def _lab(rgb):
    def xyz(x, y):
        return np.array([x / y, 1.0, (1.0 - x - y) / y])

    P = np.column_stack([xyz(0.64, 0.33), xyz(0.30, 0.60), xyz(0.15, 0.06)])
    M = P * np.linalg.solve(P, xyz(0.3127, 0.3290))
    c = rgb.double()
    lin = torch.where(c <= 0.04045, c / 12.92, ((c.clamp(min=0.04045) + 0.055) / 1.055) ** 2.4)
    t = (lin @ torch.from_numpy(M.T.copy()).to(c.device)) / torch.from_numpy(M.sum(1)).to(c.device)
    k = 6.0 / 29.0
    f = torch.where(t > k ** 3, t.clamp(min=k ** 3) ** (1.0 / 3.0), t / (3 * k * k) + 4.0 / 29.0)
    return torch.stack([116 * f[:, 1] - 16, 500 * (f[:, 0] - f[:, 1]), 200 * (f[:, 1] - f[:, 2])], 1)


def _round(v):
    """To BF16 values, the gradient passed through."""
    return v + (v.detach().float().bfloat16().double() - v.detach())


def _net(x, w):
    """The network on x (channels x samples x rows x cols) with BF16-rounded input and hidden activations."""
    def conv(v, W):
        p = torch.nn.functional.pad(v, (1, 1, 1, 1))
        H, Wd = v.shape[-2:]
        y = 0.0
        for t in range(9):
            tap = p[..., t // 3:t // 3 + H, t % 3:t % 3 + Wd].reshape(v.shape[0], -1)
            y = y + W[:, :, t] @ tap
        return y.reshape((W.shape[0],) + v.shape[1:])

    W1, W2, W3 = w[:288].reshape(16, 2, 9), w[288:2592].reshape(16, 16, 9), w[2592:].reshape(1, 16, 9)
    a1 = _round(torch.relu(conv(_round(x), W1)))
    a2 = _round(torch.relu(conv(a1, W2)))
    return conv(a2, W3)[0]


def exact(case, seed):
    kind = case["kind"]
    shape = (case["n"],) if "n" in case else (case.get("rows"), case.get("cols"))
    if kind in ("signal_cg", "signal_lobpcg"):
        clean, noisy = _signal_pair(case, seed)
        op = _Bf(clean if kind == "signal_cg" else noisy, shape, case["radius"], case["sigma_d"], case["sigma_r"])
        if kind == "signal_cg":
            return _cg(op, noisy, case["steps"])
        return _lobpcg(op, shape, noisy, case["m"], case["steps"], case["constraint"], case["prec"])
    if kind == "experiment":
        x0 = _image(case, seed, 0.1, torch.float32)
        op = _Bf(x0, shape, 1, 1.0, 0.1, "cross", "diagl")
        return _cg(op, x0, case["steps"]), _lobpcg(op, shape, x0, 1, case["steps"], False, "f32")
    if kind == "colour":
        rgb = _scene(case["rows"], case["cols"], 0.05, seed, 3).reshape(-1, 3).float()
        lab = _lab(rgb)
        op = _Bf(lab, shape, case["radius"], case["sigma_d"], case["sigma_r"])
        return lab, torch.stack([_cg(op, rgb[:, c], case["steps"]) for c in range(3)], 1)
    if kind == "reguided":
        x0 = _image(case, seed, 0.05, DTYPE[case["prec"]])
        return _reguided(case, x0, shape, _graph_args(case["graph"], case["radius"]))
    if kind == "joint":
        x0 = _image(case, seed, 0.05, DTYPE[case["prec"]])
        op = _Bf(x0, shape, case["radius"], 2.0, 0.1)
        return _cg(op, x0, case["steps"]), _lobpcg(op, shape, x0, case["m"], case["steps"], False, case["prec"])
    if kind in ("filter", "lobpcg"):
        x0 = _image(case, seed, 0.08, DTYPE[case["prec"]])
        op = _graph(case["graph"], x0, shape, _graph_args(case["graph"], case["radius"]))
        if kind == "lobpcg":
            return _lobpcg(op, shape, x0, case["m"], case["steps"], case["constraint"], case["prec"])
        return (_cg if case["method"] == "cg" else _power)(op, x0, case["steps"])
    if kind == "batch":
        got = []
        for it, x in zip(_batch_recipe(case), _batch_inputs(case, seed)):
            par = {k: it[k] for k in ("radius", "sigma_d", "sigma_r", "eps") if k in it}
            op = _graph(it["kind"], x, it["shape"], par)
            got.append(_cg(op, x, it["kmax"]) if it["method"] == "cg" else
                       _lobpcg(op, it["shape"], x, it["m"], it["kmax"], False, "f32"))
        return got
    w = torch.from_numpy(_weights(seed)).cuda().bfloat16().double()
    if kind == "net_grad":
        inputs, targets, idx = _pairs(case, seed)
        w.requires_grad_(True)
        loss, count = 0.0, case["batch"] * shape[0] * shape[1]
        for i in idx.tolist():  # sample by sample: the gradients add up
            x = inputs[i].double().T.reshape((2, 1) + shape)
            e = (_net(x, w)[0] - targets[i].double().reshape(shape)).square().sum() / count
            e.backward()
            loss = loss + e.detach()
        return loss.reshape(1), w.grad
    g, R = _residual_block(case, seed)
    got = []
    for j in range(case["m"]):
        r = R[:, j].double()
        rms = r.square().mean().sqrt()
        x = torch.stack([r / rms, g.double()]).reshape((2, 1) + shape)
        got.append(rms * _net(x, w).reshape(-1))
    return torch.stack(got, 1)
