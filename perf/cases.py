"""The workloads this framework is timed on, through its public entry points.

listed() names the work a user of the framework has it do: training steps from
a toy grid to a batch of 2^20 on a 16-level model, gradients through autograd
and through the separate layers, point queries, one rendered image, a batch of
served requests, and the preprocessing of a volume (coreset selection and index
build).  draw() takes more of the same from the ranges those stand for.

Volumes are seeded blobs advected through time (scalar float32 in [0, 1], sparse
moving features); the feature is the gradient magnitude above its 80th
percentile, dilated by 2 voxels, as in the benchmark's workloads.  exact() works
each result out again in 64 bits with plain torch, index and sampler included.
"""
import math

import numpy as np
import torch

DEV = "cuda"

# ------------------------------------------------------------------ the cases


def listed():
    return [
        # one step of the toy grid of the parity tests: launches and latency count
        dict(name="step tiny", kind="step", x=32, y=32, z=32, t=8, levels=4, features=2,
             rmin=4, rmin_t=2, hidden=32, layers=2, batch=4096, precision="fp32", lazy=False),
        # a small volume, four features per level, a ragged batch, dense Adam
        dict(name="step ragged f4", kind="step", x=121, y=90, z=61, t=20, levels=8, features=4,
             rmin=16, rmin_t=4, hidden=64, layers=3, batch=20011, precision="fp32", lazy=False),
        # the FP32 training recipe (16 levels, 32-64-64-1, deferred Adam, sorted
        # batches of 2^18) on the 480x720x120x100 volume at half resolution
        dict(name="step fp32 2^18", kind="step", x=240, y=360, z=60, t=50, levels=16, features=2,
             rmin=16, rmin_t=4, hidden=64, layers=2, batch=1 << 18, precision="fp32", lazy=True),
        # the mixed-precision recipe (32-64-64-64-1 FP16 decoder, batch 2^20) on
        # the 432^3x60 volume at two thirds of its resolution
        dict(name="step mixed 2^20", kind="step", x=288, y=288, z=288, t=40, levels=16, features=2,
             rmin=16, rmin_t=4, hidden=64, layers=3, batch=1 << 20, precision="mixed", lazy=True),
        # a custom loss through autograd on a dense feature-box model (fold
        # policy, one feature per level), points in draw order
        dict(name="autograd dense f1", kind="autograd", x=120, y=180, z=30, t=10, fold=2,
             features=1, hidden=64, layers=2, batch=65537),
        # the separate layers, forward and backward, at the feature count that
        # only they take
        dict(name="layers f8", kind="layers", x=97, y=80, z=64, t=16, levels=8, features=8,
             rmin=8, rmin_t=4, hidden=64, layers=2, batch=100003),
        # a probe of a trained model at a few points
        dict(name="points 1000", kind="points", x=121, y=90, z=61, t=20, levels=16, features=2,
             rmin=16, rmin_t=4, hidden=64, layers=2, batch=1000, table="f32"),
        # a large point query against a served model (FP16 table and decoder)
        dict(name="points 2^20", kind="points", x=288, y=288, z=288, t=40, levels=16, features=2,
             rmin=16, rmin_t=4, hidden=64, layers=3, batch=1 << 20, table="f16"),
        # one image, as an interactive viewer asks for it
        dict(name="render 200x150", kind="render", x=121, y=90, z=61, t=20, levels=16, features=2,
             rmin=16, rmin_t=4, hidden=64, layers=2, width=200, height=150, table="f32"),
        # renders and point queries served together from one resident model
        dict(name="serve", kind="serve", x=216, y=216, z=216, t=30, levels=16, features=2,
             rmin=16, rmin_t=4, hidden=64, layers=3, side=512, renders=4, queries=3,
             points=1 << 18, table="f16"),
        # a new volume: 24 timesteps of 480x720x120 through coreset selection
        dict(name="coreset 480x720x120x24", kind="coreset", x=480, y=720, z=120, t=24,
             feature="interval", radius=2),
        # and the index of the 16-level model over it
        dict(name="index 480x720x120x24", kind="index", x=480, y=720, z=120, t=24, levels=16,
             features=2, rmin=16, rmin_t=4, layout="rows"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_volume(rng, lo, hi, voxels):
    while True:
        x = _log_int(rng, lo, hi)
        d = dict(x=x, y=max(8, int(x * rng.uniform(0.4, 1.5))),
                 z=max(8, int(x * rng.uniform(0.3, 1.0))), t=rng.randint(4, 40))
        if d["x"] * d["y"] * d["z"] * d["t"] <= voxels:
            return d


def draw(rng):
    kind = rng.choice(["step", "step", "step", "autograd", "layers", "points", "points", "render",
                       "serve", "coreset", "index"])
    c = dict(kind=kind)
    if kind in ("coreset", "index"):
        c.update(_draw_volume(rng, 40, 500, 900_000_000))
        if kind == "coreset":
            c.update(feature=rng.choice(["interval", "isosurface"]), radius=rng.randint(1, 4))
        else:
            c.update(levels=rng.randint(4, 16), features=rng.choice([1, 2, 4]), rmin=8, rmin_t=2,
                     layout=rng.choice(["rows", "rows", "bricks"]))
        return c
    if kind == "autograd":
        c.update(_draw_volume(rng, 40, 200, 8_000_000), fold=rng.choice([2, 3, 4]),
                 features=rng.choice([1, 2]), hidden=rng.choice([32, 64]),
                 layers=rng.randint(1, 3), batch=_log_int(rng, 1000, 200_000))
        return c
    c.update(_draw_volume(rng, 24, 280, 250_000_000), rmin=rng.choice([4, 8, 16]),
             rmin_t=rng.choice([2, 4]), hidden=rng.choice([32, 64]), layers=rng.randint(1, 3))
    if kind == "layers":
        c.update(features=rng.choice([1, 2, 4, 8]), levels=rng.randint(3, 8),
                 batch=_log_int(rng, 1000, 200_000))
        return c
    if kind == "step":
        c.update(precision=rng.choice(["fp32", "fp32", "mixed"]), lazy=rng.random() < 0.5,
                 batch=_log_int(rng, 1000, 600_000))
        c["features"] = 2 if c["precision"] == "mixed" else rng.choice([1, 2, 2, 4])
    else:
        c.update(features=2, table=rng.choice(["f32", "f16"]))
        if kind == "points":
            c["batch"] = _log_int(rng, 100, 900_000)
        elif kind == "render":
            c.update(width=_log_int(rng, 64, 512), height=_log_int(rng, 64, 512))
        else:
            c.update(side=_log_int(rng, 96, 512), renders=rng.randint(1, 4),
                     queries=rng.randint(0, 4), points=_log_int(rng, 500, 200_000))
    c["levels"] = rng.randint(3, 32 // c["features"] if c["features"] > 1 else 16)
    return c


# ------------------------------------------------------------------ inputs


def _dims(c):
    return [c["x"], c["y"], c["z"], c["t"]]


def _cpu(seed, salt):
    g = torch.Generator()
    g.manual_seed((int(seed) * 1000003 + salt) % (1 << 62))
    return g


def _gpu(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) % (1 << 62))
    return g


def _field(dims, seed):
    """Advected Gaussian blobs in [0, 1], float32 [T][Sz][Sy][Sx].  A seed mirrors
    the axes, so that every seed has a volume of its own with as many voxels in
    the feature and as many active vertices as any other."""
    Sx, Sy, Sz, T = dims
    n = 8 if max(dims[:3]) <= 40 else 48
    u = torch.rand(n, 8, generator=_cpu(17, 1), dtype=torch.float64)
    wide = n == 8
    sig = (0.05 + 0.10 * u[:, 3]) if wide else (0.02 + 0.06 * u[:, 3])
    amp = 0.5 + 0.5 * u[:, 4]
    vel = (u[:, 5:8] - 0.5) * (0.10 if wide else 0.008)
    f = torch.zeros(T, Sz, Sy, Sx, dtype=torch.float32, device=DEV)
    for b in range(n):
        g = []
        for d, S in enumerate((Sx, Sy, Sz)):
            at = u[b, d] + vel[b, d] * torch.arange(T, dtype=torch.float64)[:, None]
            r = (torch.arange(S, dtype=torch.float64)[None, :] / (S - 1) - at) / sig[b]
            g.append(torch.exp(-0.5 * r * r).float().to(DEV))
        zy = (float(amp[b]) * g[2])[:, :, None] * g[1][:, None, :]
        f.addcmul_(zy[..., None], g[0][:, None, None, :])
    flip = [d for d in range(4) if (int(seed) >> d) & 1]
    f.clamp_(0.0, 1.0)
    return f.flip(flip) if flip else f


def _attribute(f, seed):
    """Gradient magnitude inside each frame (central differences, clamped at the
    faces) and its 80th percentile over a regular subsample (of the volume as it
    was before the seed's mirroring)."""
    a = torch.zeros_like(f)
    for d in (1, 2, 3):
        n = f.shape[d]
        g = torch.empty_like(f)
        g.narrow(d, 1, n - 2).copy_(f.narrow(d, 2, n - 2)).sub_(f.narrow(d, 0, n - 2)).mul_(0.5)
        g.narrow(d, 0, 1).copy_(f.narrow(d, 1, 1)).sub_(f.narrow(d, 0, 1))
        g.narrow(d, n - 1, 1).copy_(f.narrow(d, n - 1, 1)).sub_(f.narrow(d, n - 2, 1))
        a.addcmul_(g, g)
        del g
    a.sqrt_()
    flip = [d for d in range(4) if (int(seed) >> d) & 1]
    flat = (a.flip(flip) if flip else a).view(-1)
    s = flat[:: max(1, flat.numel() // 500_000)].sort().values
    return a, float(s[int(0.8 * (s.numel() - 1))])


RADIUS = 2  # dilation of the models' feature, in voxels


def _resolutions(c):
    """R_l = floor(Rmin b^l + 1/2) up to the volume's own size, clamped to it."""
    L, dims, out = c["levels"], _dims(c), []
    for l in range(L):
        r = []
        for d in range(4):
            top = max(dims[0], dims[1], dims[2]) if d < 3 else dims[3]
            lo = min(c["rmin"] if d < 3 else c["rmin_t"], top)
            v = lo if L == 1 else lo * (top / lo) ** (l / (L - 1))
            r.append(max(2, min(int(math.floor(v + 0.5)), dims[d])))
        out.append(r)
    return out


def _fold(c):
    """Level resolutions of the dense feature box by the fold policy."""
    size, fold = _dims(c), c["fold"]
    L = max(next(k for k in range(1, 25) if fold ** k >= s) for s in size)
    rows = [list(size)]
    while len(rows) < L:
        rows.append([-(-r // fold) if r > fold else 2 for r in rows[-1]])
    return rows[::-1]


def _width(c, L):
    return [L * c["features"]] + [c["hidden"]] * c["layers"] + [1]


def _decoder(width, seed, trained):
    """Packed decoder parameters: nn.Linear's own initialisation, or the larger
    weights and the mid-range output of a trained model."""
    g = _cpu(seed, 2)
    parts = []
    for k in range(len(width) - 1):
        b = (2.0 if trained and k + 2 < len(width) else 1.0) / math.sqrt(width[k])
        parts.append((torch.rand(width[k + 1] * width[k], generator=g) * 2 - 1) * b)
        bias = (torch.rand(width[k + 1], generator=g) * 2 - 1) * b
        parts.append(bias * 0 + 0.35 if trained and k + 2 == len(width) else bias)
    return torch.cat(parts).float()


def _table(rows, F, seed, trained):
    s = 0.4 if trained else 1e-4
    return torch.empty(rows * F, device=DEV).uniform_(-s, s, generator=_gpu(seed, 3))


def _points(n, seed, salt=4):
    return torch.rand(n, 4, device=DEV, generator=_gpu(seed, salt))


def _view(c, seed, W, H, k=0):
    """Orbit camera: eye, fwd, right, up, tan(fovy / 2), aspect (float32)."""
    u = torch.rand(2, generator=_cpu(seed, 50 + k), dtype=torch.float64).tolist()
    az, el = 2 * math.pi * u[0], (u[1] - 0.5) * 2 * math.pi / 3
    ctr = np.array([(s - 1) / 2 for s in _dims(c)[:3]])
    r = 2.0 * float(np.linalg.norm(ctr))
    eye = ctr + r * np.array([math.cos(el) * math.cos(az), math.cos(el) * math.sin(az),
                              math.sin(el)])
    fwd = (ctr - eye) / np.linalg.norm(ctr - eye)
    right = np.cross(fwd, [0.0, 0.0, 1.0])
    right = right / np.linalg.norm(right)
    up = np.cross(right, fwd)
    return np.concatenate([eye, fwd, right, up, [math.tan(math.radians(22.5)), W / H]]).astype(
        np.float32)


def _time(c, seed, k=0):
    return float(np.float32(torch.rand(1, generator=_cpu(seed, 70 + k)).item() * (c["t"] - 1)))


def _transfer():
    """Warm colour ramp, transparent below 0.15, opacity 0.4 at 1."""
    v = np.arange(256) / 255.0
    rgba = [np.clip(1.5 * v, 0, 1), np.clip(1.5 * v - 0.5, 0, 1), np.clip(0.6 - v, 0, 1),
            np.clip((v - 0.15) / 0.85, 0, 1) * 0.4]
    return torch.from_numpy(np.stack(rgba, axis=1).astype(np.float32)).to(DEV)


def _requests(c, seed):
    """(kind, side or points, request number) of the served mix."""
    out = [("render", max(32, c["side"] >> (k & 1)), k) for k in range(c["renders"])]
    return out + [("points", max(1, c["points"] >> (3 * k)), k) for k in range(c["queries"])]


def _prepare_model(c, seed, trained):
    """Mask and index over the volume, table and decoder."""
    from paper_2507_03836_amd import _lib as fl
    from paper_2507_03836_amd import volume
    dims = _dims(c)
    f = _field(dims, seed)
    a, thr = _attribute(f, seed)
    del f
    bits = volume.select_coreset(a, dims, thr, radius=RADIUS)["bits"]
    del a
    res = _resolutions(c)
    grid = fl.grid_desc(res, c["features"])
    index, _, dirs, _ = fl.fhash_build_index(grid, bits, dims)
    rows = int(index.slot_offset[len(res)])
    dt = {"f32": fl.F32, "f16": fl.F16}[c.get("table", "f32")]
    width = _width(c, len(res))
    s = dict(c=c, fl=fl, dims=dims, bits=bits, index=index, dir=dirs, rows=rows,
             mlp=fl.mlp_desc(width, dt), params=_decoder(width, seed, trained).to(DEV),
             table=_table(rows, c["features"], seed, trained))
    if dt == fl.F16:
        s["table"] = s["table"].half()
    return s


def prepare(case, seed):
    from paper_2507_03836_amd import _lib as fl
    c, kind, dims = case, case["kind"], _dims(case)
    if kind == "step":
        from paper_2507_03836_amd import volume
        from paper_2507_03836_amd.model import FHashConfig, FHashModel
        f = _field(dims, seed)
        a, thr = _attribute(f, seed)
        sel = volume.select_coreset(a, dims, thr, radius=RADIUS)
        del a
        res = _resolutions(c)
        cfg = FHashConfig(res=res, n_features=c["features"], hidden=c["hidden"],
                          n_hidden=c["layers"])
        mixed = c["precision"] == "mixed"
        # the deferred recipe of the benchmark: moments beside the parameters,
        # FP32 table reads and an FP16 decoder under mixed precision; else the
        # model's own defaults
        kw = dict(lazy=True, moments_with_params=True) if c["lazy"] else {}
        if mixed and c["lazy"]:
            kw.update(table_reads="f32", decoder="f16")
        g = _gpu(seed, 3)
        width = _width(c, len(res))
        m = FHashModel(cfg, sel["bits"], dims, precision=c["precision"],
                       init_seed=int(g.initial_seed() % (1 << 31)),
                       mlp_init=_decoder(width, seed, False), **kw)
        m.coarse_lds = c["lazy"]
        n = c["batch"]
        return dict(c=c, fl=fl, dims=dims, model=m, field=f, sel=sel, seed=int(seed) + 2000, k=0,
                    pos=torch.empty(n, 4, device=DEV), target=torch.empty(n, device=DEV), ws=None)
    if kind == "autograd":
        res = _fold(c)
        index, _ = fl.fhash_dense_index(fl.grid_desc(res, c["features"]))
        rows = int(index.slot_offset[len(res)])
        width = _width(c, len(res))
        s = dict(c=c, index=index, mlp=fl.mlp_desc(width), pos=_points(c["batch"], seed),
                 target=torch.rand(c["batch"], device=DEV, generator=_gpu(seed, 5)),
                 table=_table(rows, c["features"], seed, True).view(rows, -1).requires_grad_(),
                 params=_decoder(width, seed, True).to(DEV).requires_grad_())
        return s
    if kind in ("coreset", "index"):
        a, thr = _attribute(_field(dims, seed), seed)
        if kind == "coreset":  # the frames in another order, too
            return dict(c=c, fl=fl, dims=dims, attr=a.roll(int(seed) // 16 % c["t"], 0), thr=thr)
        from paper_2507_03836_amd import volume
        lay = fl.LAYOUT_BRICKS if c["layout"] == "bricks" else fl.LAYOUT_ROWS
        return dict(c=c, fl=fl, dims=dims, grid=fl.grid_desc(_resolutions(c), c["features"], lay),
                    bits=volume.select_coreset(a, dims, thr, radius=RADIUS)["bits"])
    s = _prepare_model(c, seed, True)
    if kind == "layers":
        n = c["batch"]
        s.update(pos=_points(n, seed), target=torch.rand(n, device=DEV, generator=_gpu(seed, 5)),
                 enc=torch.empty(n, c["levels"] * c["features"], device=DEV),
                 y=torch.empty(n, device=DEV), dy=torch.empty(n, device=DEV),
                 dx=torch.empty(n, c["levels"] * c["features"], device=DEV),
                 d_table=torch.zeros_like(s["table"]), d_params=torch.zeros_like(s["params"]),
                 ws=None)
    elif kind == "points":
        s.update(pos=_points(c["batch"], seed))
    elif kind == "render":
        W, H = c["width"], c["height"]
        s.update(tf=_transfer(), view=fl.view_struct(_view(c, seed, W, H)), time=_time(c, seed),
                 opts=fl.render_opts(), rgba=torch.empty(H, W, 4, device=DEV), ws=None)
    elif kind == "serve":
        from paper_2507_03836_amd.serving import GpuExecutor, ResidentModel
        ex = GpuExecutor(sample_budget=1 << 21)
        ex.add_model("m", ResidentModel(index=s["index"], mlp=s["mlp"], table=s["table"],
                                        params=s["params"], mask_bits=s["bits"], dims=dims,
                                        tf=_transfer(), keep=(s["dir"],),
                                        occ=fl.fhash_occupancy_grid(s["bits"], dims)))
        s.update(ex=ex, asked=[
            (k, v, _view(c, seed, v, v, i) if k == "render" else _points(v, seed, 10 + i),
             _time(c, seed, i)) for k, v, i in _requests(c, seed)])
    return s


# ------------------------------------------------------------------ one pass


def _run_step(s):
    c, fl, m, n = s["c"], s["fl"], s["model"], s["c"]["batch"]
    s["k"] += 1
    m.loss_sum.zero_()
    fl.fhash_sample(s["seed"], s["k"], n, s["sel"]["coreset"], s["sel"]["M"], s["dims"],
                    s["field"], s["pos"], s["target"])
    if c["lazy"]:
        s["ws"] = fl.fhash_sort_samples(s["pos"], s["target"], n, s["ws"])
    m.train_step(s["pos"], s["target"])
    out = dict(loss=m.loss_sum.float())
    if c["lazy"]:  # parameters with m, gradients with v, and the decoder's arrays
        out.update(params=m.pm, grads=m.gv, decoder=m.mlp_p)
    else:
        out.update(params=m.params, m=m.m, v=m.v)
    return out


def _run_autograd(s):
    from paper_2507_03836_amd.autograd import fhash_apply
    s["table"].grad = s["params"].grad = None
    y = fhash_apply(s["pos"], s["table"], s["params"], s["index"], s["mlp"])
    loss = torch.nn.functional.smooth_l1_loss(y, s["target"])
    loss.backward()
    return dict(y=y.detach(), loss=loss.detach(), d_table=s["table"].grad,
                d_params=s["params"].grad)


def _run_layers(s):
    fl, n = s["fl"], s["c"]["batch"]
    s["d_table"].zero_()
    s["d_params"].zero_()
    fl.fhash_encode_fwd(s["index"], s["pos"], n, s["table"], s["enc"])
    fl.fhash_mlp_fwd(s["mlp"], s["params"], s["enc"], n, s["y"])
    fl.fhash_mse_grad(s["y"], s["target"], n, s["dy"])
    s["ws"] = fl.fhash_mlp_bwd(s["mlp"], s["params"], s["enc"], s["dy"], n, s["d_params"],
                               dx=s["dx"], ws=s["ws"])
    fl.fhash_encode_bwd(s["index"], s["pos"], n, s["dx"], s["d_table"])
    return dict(enc=s["enc"], y=s["y"], dx=s["dx"], d_table=s["d_table"],
                d_params=s["d_params"])


def _run_serve(s):
    from paper_2507_03836_amd.serving import Request, Scheduler
    sch = Scheduler(s["ex"], sample_budget=1 << 21)
    reqs = [Request(model="m", kind=k, view=x, t=t, W=v, H=v) if k == "render"
            else Request(model="m", kind=k, pos=x, n=v) for k, v, x, t in s["asked"]]
    sch.run(reqs, realtime=False)
    return [r.result for r in reqs]


def run(state):
    s, kind = state, state["c"]["kind"]
    if kind == "step":
        return _run_step(s)
    if kind == "autograd":
        return _run_autograd(s)
    if kind == "layers":
        return _run_layers(s)
    if kind == "serve":
        return _run_serve(s)
    fl, c = s["fl"], s["c"]
    if kind == "points":
        y = torch.empty(c["batch"], device=DEV)
        fl.fhash_fused_fwd(s["index"], s["mlp"], s["pos"], c["batch"], s["table"], s["params"], y)
        return y
    if kind == "render":
        _, s["ws"] = fl.fhash_render(s["index"], s["mlp"], s["table"], s["params"], s["bits"],
                                     s["dims"], s["view"], s["time"], s["tf"], c["width"],
                                     c["height"], s["opts"], s["rgba"], s["ws"])
        return s["rgba"]
    if kind == "coreset":
        from paper_2507_03836_amd import volume
        iso = c["feature"] == "isosurface"
        r = volume.select_coreset(s["attr"], s["dims"], s["thr"], radius=c["radius"],
                                  kind=fl.FEATURE_ISOSURFACE if iso else fl.FEATURE_INTERVAL)
        return dict(bits=r["bits"], ids=r["coreset"], box=fl.fhash_feature_boxes(r["bits"], s["dims"]),
                    occ=fl.fhash_occupancy_grid(r["bits"], s["dims"]))
    _, slots, dirs, _ = fl.fhash_build_index(s["grid"], s["bits"], s["dims"])
    return dict(slots=slots, dir=dirs)


# ------------------------------------------------------------------ what it cannot do without


def _macs(width):
    return sum(width[k] * width[k + 1] for k in range(len(width) - 1))


def work(case):
    c, kind = case, case["kind"]
    vox = c["x"] * c["y"] * c["z"] * c["t"]
    mask = vox / 8
    if kind in ("coreset", "index"):
        if kind == "coreset":  # field in; mask, occupancy bits and about 0.35 of the voxel ids out
            return dict(bytes=vox * 4 + 2 * mask + 0.35 * vox * 8, flops=0)
        box = sum(math.prod(r) for r in _resolutions(c))
        return dict(bytes=mask + box / 64 * 16, flops=0)
    res = _fold(c) if kind == "autograd" else _resolutions(c)
    F, width = c["features"], _width(c, len(res))
    live = 1.0 if kind == "autograd" else 0.5  # active vertices, about
    rows = [live * math.prod(r) for r in res]
    if kind in ("render", "serve"):
        # about a fifth of the lattice samples of every ray that meets the
        # volume are decoded; their table rows once, the image once
        diag = math.sqrt(c["x"] ** 2 + c["y"] ** 2 + c["z"] ** 2)
        px = c["width"] * c["height"] if kind == "render" else sum(
            v * v for k, v, _ in _requests(c, 0) if k == "render")
        n = px * 0.3 * diag * 0.2
        n += sum(v for k, v, _ in _requests(c, 0) if k == "points") if kind == "serve" else 0
        size = 2 if c["table"] == "f16" else 4
        return dict(bytes=sum(min(16 * n, r) for r in rows) * F * size + px * 16 + n * 4,
                    flops=n * (2 * _macs(width) + 64 * width[0]))
    n = c["batch"]
    touched = sum(min(16 * n, r) for r in rows) * F
    fwd = 2 * _macs(width) + 64 * width[0]
    if kind == "points":
        return dict(bytes=n * 20 + touched * (2 if c["table"] == "f16" else 4), flops=n * fwd)
    if kind == "step":
        # draw the batch; every touched parameter and its moments read and
        # written once, and every parameter of a dense update
        every = touched if c["lazy"] else sum(rows) * F
        return dict(bytes=n * 52 + every * 24, flops=n * 3 * fwd)
    return dict(bytes=n * 28 + touched * 4 + sum(rows) * F * 4, flops=n * 3 * fwd)


# ------------------------------------------------------------------ in 64 bits


def _ranges(S, R):
    """Voxels that share a cell with vertex v: lo..hi along one axis."""
    lo = [max(0, -((-(v - 1) * (S - 1)) // (R - 1))) for v in range(R)]
    hi = [min(S - 1, ((v + 1) * (S - 1)) // (R - 1)) for v in range(R)]
    return lo, hi


def _dilated(m, r):
    for d in (1, 2, 3):
        out = m.clone()
        for k in range(1, min(r, m.shape[d] - 1) + 1):
            n = m.shape[d] - k
            out.narrow(d, k, n).logical_or_(m.narrow(d, 0, n))
            out.narrow(d, 0, n).logical_or_(m.narrow(d, k, n))
        m = out
    return m


def _slots(mask, dims, res):
    """Row of every vertex of a level in the F-Hash order (-1: inactive), rows."""
    m = mask
    for d, (S, R) in enumerate(((dims[3], res[3]), (dims[2], res[2]), (dims[1], res[1]))):
        lo, hi = _ranges(S, R)
        m = torch.stack([m.narrow(d, lo[v], hi[v] - lo[v] + 1).any(d) for v in range(R)], d)
    lo, hi = (torch.tensor(v, device=DEV) for v in _ranges(dims[0], res[0]))
    s = torch.zeros(*m.shape[:3], dims[0] + 1, dtype=torch.int16, device=DEV)
    torch.cumsum(m, 3, dtype=torch.int16, out=s[..., 1:])
    act = (s[..., hi + 1] > s[..., lo]).reshape(-1)
    del s, m
    n = torch.cumsum(act, 0, dtype=torch.int32)
    rows = int(n[-1])
    n -= 1
    n[~act] = -1
    return n, rows


class _Model:
    """The encoding and the decoder in 64 bits."""

    def __init__(self, c, seed, trained, mask=None):
        dims = _dims(c)
        self.c, self.F = c, c["features"]
        self.res = _fold(c) if mask is None else _resolutions(c)
        self.off, self.slot = [0], []
        for r in self.res:
            if mask is None:
                self.slot.append(None)
                self.off.append(self.off[-1] + math.prod(r))
            else:
                s, rows = _slots(mask, dims, r)
                self.slot.append(s)
                self.off.append(self.off[-1] + rows)
        self.rows = self.off[-1]
        self.width = _width(c, len(self.res))
        self.params = _decoder(self.width, seed, trained).to(DEV).double()

    def corners(self, pos, l):
        """(rows [n][16], weights [n][16]) of level l; inactive corners weigh 0."""
        R = self.res[l]
        p = pos.clamp(0.0, 1.0)
        cell, frac = [], []
        for d in range(4):
            u = p[:, d] * float(R[d] - 1)
            i = u.floor().clamp(max=R[d] - 2)
            cell.append(i.long())
            frac.append((u - i).double())
        rows, w = [], []
        for k in range(16):
            o = [(k >> d) & 1 for d in range(4)]
            lin = ((cell[3] + o[3]) * R[2] + cell[2] + o[2]) * R[1] + cell[1] + o[1]
            lin = lin * R[0] + cell[0] + o[0]
            wk = torch.ones_like(frac[0])
            for d in range(4):
                wk = wk * (frac[d] if o[d] else 1.0 - frac[d])
            s = lin if self.slot[l] is None else self.slot[l][lin].long()
            rows.append(s.clamp(min=0) + self.off[l])
            w.append(wk * (s >= 0))
        return torch.stack(rows, 1), torch.stack(w, 1)

    def encode(self, pos, table):
        out = []
        for l in range(len(self.res)):
            rows, w = self.corners(pos, l)
            out.append((table[rows].double() * w[..., None]).sum(1))
        return torch.cat(out, 1)

    def scatter(self, pos, d_enc, d_table):
        for l in range(len(self.res)):
            rows, w = self.corners(pos, l)
            g = d_enc[:, l * self.F:(l + 1) * self.F]
            d_table.index_add_(0, rows.reshape(-1),
                               (w[..., None] * g[:, None, :]).reshape(-1, self.F))

    def decode(self, x, params):
        at = 0
        for k in range(len(self.width) - 1):
            i, o = self.width[k], self.width[k + 1]
            W = params[at:at + i * o].view(o, i)
            x = x @ W.t() + params[at + i * o:at + i * o + o]
            at += i * o + o
            if k + 2 < len(self.width):
                x = x.relu()
        return x[:, 0]

    def forward(self, pos, table):
        return torch.cat([self.decode(self.encode(q, table), self.params)
                          for q in pos.split(1 << 18)])

    def both(self, pos, target, table, loss):
        """y, sum of the losses, encoding gradient pieces and the gradients."""
        d_table = torch.zeros(self.rows, self.F, dtype=torch.float64, device=DEV)
        params = self.params.clone().requires_grad_()
        ys, total, encs, dxs = [], 0.0, [], []
        for q, v in zip(pos.split(1 << 18), target.split(1 << 18)):
            enc = self.encode(q, table).requires_grad_()
            y = self.decode(enc, params)
            part = loss(y, v.double())
            part.backward()
            self.scatter(q, enc.grad, d_table)
            ys.append(y.detach())
            encs.append(enc.detach())
            dxs.append(enc.grad)
            total = total + part.detach()
        return torch.cat(ys), total, torch.cat(encs), torch.cat(dxs), d_table, params.grad


def _philox(i, step, seed):
    """The 64-bit words of Philox4x32-10 for counters (i, step), as (hi, lo)."""
    m32 = 0xFFFFFFFF

    def mul(a, b):  # 32-bit constant x int64 tensor below 2^32 -> (high, low) words
        return _hi(a, b), ((b & 0xFFFF) * a + (((b >> 16) * (a & 0xFFFF)) << 16)) & m32

    def _hi(a, b):
        al, ah, bl, bh = a & 0xFFFF, a >> 16, b & 0xFFFF, b >> 16
        t = bl * al
        u = bh * al + (t >> 16)
        v = bl * ah + (u & 0xFFFF)
        return bh * ah + (u >> 16) + (v >> 16)

    x, y = i & m32, i >> 32
    z, w = torch.full_like(i, step & m32), torch.full_like(i, step >> 32)
    k0, k1 = seed & m32, (seed >> 32) & m32
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, x)
        h1, l1 = mul(0xCD9E8D57, z)
        x, y, z, w = h1 ^ y ^ k0, l1, h0 ^ w ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return y, x


def _sampled(n, step, seed, field, ids):
    """Positions and labels of a training batch drawn from the coreset."""
    hi, lo = _philox(torch.arange(n, device=DEV), step, seed)
    M = ids.numel()
    at = ids[(hi * M + ((lo * M) >> 32)) >> 32]
    T, Sz, Sy, Sx = field.shape
    p = torch.stack([at % Sx, at // Sx % Sy, at // (Sx * Sy) % Sz, at // (Sx * Sy * Sz)], 1)
    ext = torch.tensor([Sx - 1, Sy - 1, Sz - 1, T - 1], device=DEV)
    return p.float() / ext.float(), field.view(-1)[at]


def _adam1(p, g):
    """Step 1 of Adam from m = v = 0: (p, m, v)."""
    return p - 0.01 * g / (g.abs() + 1e-8), 0.1 * g, 0.001 * g * g


def _exact_step(c, seed):
    dims = _dims(c)
    f = _field(dims, seed)
    a, thr = _attribute(f, seed)
    mask = _dilated(a > thr, RADIUS)
    del a
    M = _Model(c, seed, False, mask)
    # linear ids of the masked voxels (the mask is searched in parts: a part
    # fits nonzero's 32-bit count)
    flat = mask.view(-1)
    ids = torch.cat([q.nonzero()[:, 0] + k * (1 << 28) for k, q in enumerate(flat.split(1 << 28))])
    pos, target = _sampled(c["batch"], 1, int(seed) + 2000, f, ids)
    del f, ids, flat, mask
    g = _gpu(seed, 3)
    ti = torch.Generator(device=DEV)
    ti.manual_seed(int(g.initial_seed() % (1 << 31)))
    nt = M.rows * M.F
    table = torch.empty(nt, device=DEV).uniform_(-1e-4, 1e-4, generator=ti).view(M.rows, M.F)
    n = c["batch"]
    _, sse, _, _, dt, dp = M.both(pos, target, table, lambda y, v: ((y - v) ** 2).sum())
    dt, dp = dt.view(-1) / n, dp / n
    M.slot = None
    off, nm = (nt + 3) // 4 * 4, dp.numel()
    loss = sse.reshape(1)
    if not c["lazy"]:
        p = torch.zeros((off + nm + 3) // 4 * 4, dtype=torch.float64, device=DEV)
        gr = torch.zeros_like(p)
        p[:nt], p[off:off + nm] = table.view(-1), M.params
        gr[:nt], gr[off:off + nm] = dt, dp
        p, m, v = _adam1(p, gr)
        return dict(loss=loss, params=p, m=m, v=v)
    # deferred: the levels of 2^21 segments of 16 floats or more keep their
    # parameters and hold the step's (scaled) gradient; all before them is stepped
    scale = 2.0 ** 16 if c["precision"] == "mixed" else 1.0
    first = next((l for l in range(len(M.res))
                  if (M.off[l + 1] - M.off[l]) * M.F // 16 >= (1 << 21)), None)
    begin = 0 if first is None else M.off[first] * M.F // 16 * 16
    nv = (off + 15) // 16 * 16
    pm = torch.zeros(nv // 16, 2, 16, dtype=torch.float64, device=DEV)
    gv = torch.zeros_like(pm)
    p = torch.zeros(nv, dtype=torch.float64, device=DEV)
    gr = torch.zeros_like(p)
    p[:nt] = table.view(-1)
    gr[:nt] = dt
    del dt
    q, m, v = _adam1(p[:begin], gr[:begin])
    p[:begin] = q
    gr[:begin] = 0
    gr *= scale
    pm[:, 0], gv[:, 0] = p.view(-1, 16), gr.view(-1, 16)
    pm[: begin // 16, 1], gv[: begin // 16, 1] = m.view(-1, 16), v.view(-1, 16)
    dec = torch.zeros((nm + 3) // 4 * 4, dtype=torch.float64, device=DEV)
    dec[:nm] = _adam1(M.params, dp)[0]
    return dict(loss=loss, params=pm.view(-1), grads=gv.view(-1), decoder=dec)


def _model_inputs(c, seed):
    a, thr = _attribute(_field(_dims(c), seed), seed)
    mask = _dilated(a > thr, RADIUS)
    del a
    M = _Model(c, seed, True, mask)
    t = _table(M.rows, c["features"], seed, True)
    if c.get("table") == "f16":
        t = t.half()
    return M, t.view(M.rows, c["features"]), mask


def _exact_image(c, M, table, mask, view, t, W, H):
    """The image, every ray's occupied lattice samples decoded in 64 bits; the
    geometry in FP32 as it is specified."""
    dims = _dims(c)
    v = torch.from_numpy(view).to(DEV)
    eye, fwd, right, up, tan, asp = v[0:3], v[3:6], v[6:9], v[9:12], v[12], v[13]
    r = torch.arange(W * H, device=DEV)
    u = (2.0 * ((r % W).float() + 0.5) / float(W) - 1.0) * tan * asp
    w = (1.0 - 2.0 * ((r // W).float() + 0.5) / float(H)) * tan
    d = (fwd + u[:, None] * right) + w[:, None] * up
    d = d / torch.sqrt((d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2])[:, None]
    top = torch.tensor([float(s - 1) for s in dims[:3]], device=DEV)
    a, b = (0.0 - eye) / d, (top - eye) / d
    s0 = torch.minimum(a, b).amax(1).clamp(min=0.0)
    s1 = torch.maximum(a, b).amin(1)
    t0, t1 = int(math.floor(t)), int(math.ceil(t))
    occ = mask[t0] | mask[t1]
    for k in range(3):
        n = occ.shape[k] - 1
        occ = occ.narrow(k, 0, n) | occ.narrow(k, 1, n)
    tau = float(np.float32(t) / np.float32(dims[3] - 1))
    steps = int(math.ceil(float(((s1 - s0).clamp(min=0).max()) / 0.5))) + 1
    tf = _transfer().double()
    out = torch.zeros(W * H, 4, dtype=torch.float64, device=DEV)
    lim = torch.tensor([s - 2 for s in dims[:3]], device=DEV)

    def fma(x, y, z):  # one FP32 rounding of x y + z (the product is exact in 64 bits)
        return (x.double() * y.double() + z.double()).float()

    per = max(1, (1 << 23) // steps)
    half = torch.tensor(0.5, device=DEV)
    for q in r.split(per):
        k = torch.arange(steps, device=DEV).float() + 0.5
        sk = fma(k[None, :], half, s0[q][:, None])
        p = fma(sk[..., None], d[q][:, None, :], eye[None, None, :])
        cell = torch.minimum(p.floor().long().clamp(min=0), lim)
        live = (sk < s1[q][:, None]) & occ[cell[..., 2], cell[..., 1], cell[..., 0]]
        pos = torch.cat([p[live] / top, torch.full((int(live.sum()), 1), tau, device=DEV)], 1)
        rgba = torch.zeros(q.numel(), steps, 4, dtype=torch.float64, device=DEV)
        if pos.shape[0]:
            x = M.forward(pos, table).clamp(0.0, 1.0) * 255.0
            i = x.floor().clamp(max=254).long()
            fr = (x - i)[:, None]
            rgba[live] = (1 - fr) * tf[i] + fr * tf[i + 1]
        through = torch.cumprod(1 - rgba[..., 3], 1)  # 1 - A after each sample
        before = torch.cat([torch.ones_like(through[:, :1]), through[:, :-1]], 1)
        stop = float(np.float32(0.99))
        w8 = torch.where(1 - before < stop, before * rgba[..., 3], torch.zeros_like(before))
        out[q, :3] = (w8[..., None] * rgba[..., :3]).sum(1)
        out[q, 3] = w8.sum(1)
    return out.view(H, W, 4)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("coreset", "index"):
        return None  # whole numbers throughout
    if kind == "step":
        return _exact_step(c, seed)
    if kind == "autograd":
        M = _Model(c, seed, True)
        t = _table(M.rows, c["features"], seed, True).view(M.rows, -1)
        n = c["batch"]
        y, loss, _, _, dt, dp = M.both(
            _points(n, seed), torch.rand(n, device=DEV, generator=_gpu(seed, 5)), t,
            lambda p, v: torch.nn.functional.smooth_l1_loss(p, v, reduction="sum") / n)
        return dict(y=y, loss=loss, d_table=dt, d_params=dp)
    M, table, mask = _model_inputs(c, seed)
    if kind == "points":
        return M.forward(_points(c["batch"], seed), table)
    if kind == "layers":
        n = c["batch"]
        y, _, enc, dx, dt, dp = M.both(
            _points(n, seed), torch.rand(n, device=DEV, generator=_gpu(seed, 5)), table,
            lambda p, v: ((p - v) ** 2).sum() / n)
        return dict(enc=enc, y=y, dx=dx, d_table=dt.view(-1), d_params=dp)
    if kind == "render":
        W, H = c["width"], c["height"]
        if W * H > 40_000:
            return None
        return _exact_image(c, M, table, mask, _view(c, seed, W, H), _time(c, seed), W, H)
    # served: the point queries; of the images the small ones
    return [M.forward(_points(v, seed, 10 + i), table) if k == "points" else
            _exact_image(c, M, table, mask, _view(c, seed, v, v, i), _time(c, seed, i), v, v)
            if v * v <= 40_000 else None for k, v, i in _requests(c, seed)]
