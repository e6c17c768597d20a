"""The workloads whose speed is tracked, through the package's public entry points.

Five kinds, over the sizes that a program meets from a unit test's column to
the benchmark's largest bed:

  step     a scene stepped `steps` times and its state read back
  mlp      the learned start's network on device buffers (forward)
  train    one minibatch of its training: loss, gradient, Adam
  voxels   the mesoscale step on a voxel grid: cut, advection, deposit, surface
  fields   coarse-grained density, momentum and velocity of a bed

Beds start as dense packings that rest on their floor (a cubic lattice at
contact distance with small scatter in radius and position, about three
contacts per sphere as in a settled bed), so that nothing has to settle first.
"""
import math
import random

import numpy as np
import torch

from paper_2011_00459_amd import terrain as T

DT = 1.0 / 60.0
G = 9.81
PI = math.pi


def _step(name, n, n_max=None, envs=1, sweeps=100, tol=0.0, warm="prev", mu_r=0.0, shape="bed", tool="none",
          mode="default", steps=1):
    case = dict(kind="step", envs=envs, n_min=n, n_max=n_max or n, sweeps=sweeps, tol=tol, warm=warm, mu_r=mu_r,
                shape=shape, tool=tool, mode=mode, steps=steps)
    return dict(case, name=name) if name else case


def listed():
    return [
        # a unit test's or a demo's column: latency and launches, not throughput
        _step("column_300", 300, sweeps=50, warm="cold", shape="column"),
        # a small problem solved to a residual tolerance from a cold start
        _step("column_1000_to_1e-3", 1000, sweeps=5000, tol=1e-3, warm="cold", shape="column"),
        # eight columns of a rolling-resistance soil (dirt), as a calibration sweep steps them
        _step("columns_8x1000_rolling", 1000, envs=8, mu_r=0.1, shape="column"),
        # training environments with the network's warm start, sizes as they come
        _step("beds_24_learned", 700, n_max=6000, envs=24, warm="learned", tool="blade", steps=2),
        # the bulldozing bed under the default schedule, tool force and zone read every step
        _step("bed_50000", 50000, sweeps=150, tool="blade"),
        # the batch of independent beds, observed every eight steps
        _step("beds_256", 500, n_max=20000, envs=256, tool="mixed", steps=8),
        # the excavation with a bucket on the schedule tuned for one large scene, drawn every four steps
        _step("excavation_500000", 500000, sweeps=200, shape="wide", tool="bucket", mode="spread", steps=4),
        # inference over a recorded data set, BF16 on the matrix cores
        dict(name="mlp_bf16_4194304", kind="mlp", batch=1 << 22, bf16=True),
        # a minibatch as the training driver takes it
        dict(name="train_4096", kind="train", batch=4096),
        # the dig site's grid, fluid advected and converted once a step
        dict(name="voxels_256x256x128", kind="voxels", nx=256, ny=256, nz=128),
        # fields of the bulldozing bed on its own grid, smooth kernel
        dict(name="fields_50000_gauss", kind="fields", n=50000, smooth=True, cell=0.06),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["column", "columns", "bed", "beds", "learned", "large", "mlp", "train", "voxels", "fields"])
    if kind == "column":
        tol = rng.choice([0.0, 0.0, 1e-3])
        return _step(None, size(100, 3000), sweeps=2000 if tol else rng.randint(10, 200), tol=tol, shape="column",
                     warm=rng.choice(["cold", "prev"]), mu_r=rng.choice([0.0, 0.1]))
    if kind == "columns":
        return _step(None, size(200, 1500), envs=rng.randint(2, 12), sweeps=rng.randint(20, 150), shape="column",
                     mu_r=rng.choice([0.0, 0.02, 0.3]))
    if kind == "bed":
        return _step(None, size(3000, 70000), sweeps=rng.randint(10, 150), tool=rng.choice(["blade", "bucket"]),
                     mode=rng.choice(["default", "default", "spread"]))
    if kind == "beds":
        lo = size(300, 3000)
        return _step(None, lo, n_max=lo * rng.randint(1, 8), envs=rng.randint(9, 200), sweeps=rng.randint(20, 100),
                     tool="mixed", mu_r=rng.choice([0.0, 0.0, 0.1]), steps=4)
    if kind == "learned":
        lo = size(500, 3000)
        return _step(None, lo, n_max=3 * lo, envs=rng.randint(1, 40), warm="learned", tool="blade", steps=2)
    if kind == "large":
        return _step(None, size(120000, 450000), sweeps=rng.randint(20, 150), shape="wide", tool="bucket",
                     mode="spread", steps=2)
    if kind == "mlp":
        return dict(kind="mlp", batch=size(1000, 4_000_000), bf16=rng.random() < 0.7)
    if kind == "train":
        return dict(kind="train", batch=size(256, 65536))
    if kind == "voxels":
        return dict(kind="voxels", nx=rng.randint(24, 256), ny=rng.randint(24, 256), nz=rng.randint(16, 150))
    return dict(kind="fields", n=size(1000, 200000), smooth=rng.random() < 0.5, cell=rng.uniform(0.05, 0.12))


# --------------------------------------------------------------------------
# scenes
# --------------------------------------------------------------------------
ASPECT = {"column": (1.0, 1.0, 1.0), "bed": (4.0, 2.0, 1.0), "wide": (8.0, 4.0, 1.0)}


def _sizes(case):
    """Spheres of each env: evenly spread in the logarithm, in a fixed shuffled order."""
    e, lo, hi = case["envs"], case["n_min"], case["n_max"]
    n = [int(round(lo * (hi / lo) ** ((k + 0.5) / e))) for k in range(e)]
    random.Random(e).shuffle(n)
    return n


def _plane(n, d):
    return dict(type="plane", n=n, d=d)


def _box(half, off):
    return dict(type="box", half=half, off=off)


def _body(pos, shapes, vx=0.0, zone=None):
    b = dict(pos=pos, quat=(1.0, 0.0, 0.0, 0.0), linvel=(vx, 0.0, 0.0), angvel=(0.0, 0.0, 0.0), shapes=shapes)
    if zone is not None:
        b["zone_planes"] = zone
    return b


def _zone(edge_x, edge_z, width, top, mu):
    """The wedge in front of a vertical cutting face: (n, d) with n . y <= d."""
    th = 0.5 * PI - 0.5 * (math.atan(mu) + 0.5 * PI)
    s, c = math.sin(th), math.cos(th)
    return [[-1.0, 0.0, 0.0, -edge_x], [s, 0.0, -c, s * edge_x - c * edge_z], [0.0, 0.0, 1.0, top],
            [0.0, 1.0, 0.0, 0.5 * width], [0.0, -1.0, 0.0, 0.5 * width]]


def _tool(kind, lx, ly, top, speed, mu, zone):
    if kind == "blade":
        h = 0.5 * top + 0.15
        w, depth, t = 0.75 * ly, 0.15 * top, 0.025
        pos = (-0.3 * lx, 0.0, top - depth + h)
        z = _zone(t, -h, w, depth - h + 0.3, mu) if zone else None
        return _body(pos, [_box((t, 0.5 * w, h), (0.0, 0.0, 0.0))], speed, z)
    hl, hw, hh, p = 0.0625 * lx, 0.15 * ly, 0.4 * top, 0.01
    depth = 0.3 * top
    pos = (-0.3 * lx, 0.0, top - depth + hh)
    shapes = [_box((hl, hw, p), (0.0, 0.0, p - hh)), _box((p, hw, hh), (p - hl, 0.0, 0.0)),
              _box((hl, p, hh), (0.0, p - hw, 0.0)), _box((hl, p, hh), (0.0, hw - p, 0.0))]
    return _body(pos, shapes, speed, _zone(hl, -hh, 2 * hw, depth - hh + 0.3, mu) if zone else None)


def _specs(case, seed):
    """One scene description per env, its inputs drawn from the seed."""
    specs = []
    ax, ay, az = ASPECT[case["shape"]]
    column = case["shape"] == "column"
    mu, c = (0.6, 1000.0) if column else (0.7, 2000.0)
    if case["mu_r"] > 0.0:
        mu, c = 0.4, 2500.0
    mat = dict(mu_t=mu, mu_r=case["mu_r"], c_p=c, rho=2000.0)
    for e, n in enumerate(_sizes(case)):
        rng = np.random.default_rng([seed, e])
        k = (n * az * az / (ax * ay)) ** (1.0 / 3.0)
        nx, ny = max(1, round(k * ax / az)), max(1, round(k * ay / az))
        # one scene keeps its sphere size, the beds of a batch their width
        r0 = 1.5 / nx if case["envs"] > 1 and not column else {"column": 0.05, "bed": 0.03, "wide": 0.02}[case["shape"]]
        i = np.arange(n)
        x = np.stack([(i % nx - 0.5 * (nx - 1)), (i // nx % ny - 0.5 * (ny - 1)), i // (nx * ny) + 0.5], 1) * (2.0 * r0)
        x += rng.uniform(-0.005, 0.005, x.shape) * r0
        r = r0 * rng.uniform(0.99, 1.01, n)
        v = rng.normal(0.0, 0.02, x.shape)
        lx, ly, top = 2.0 * r0 * nx, 2.0 * r0 * ny, 2.0 * r0 * (-(-n // (nx * ny)))
        w = 0.5 * lx + 0.02 * r0, 0.5 * ly + 0.02 * r0
        bodies = [_body((0.0, 0.0, 0.0), [_plane((0.0, 0.0, 1.0), 0.0), _plane((1.0, 0.0, 0.0), -w[0]),
                                          _plane((-1.0, 0.0, 0.0), -w[0]), _plane((0.0, 1.0, 0.0), -w[1]),
                                          _plane((0.0, -1.0, 0.0), -w[1])])]
        tool = case["tool"]
        if tool == "mixed":
            tool = "blade" if rng.uniform() < 0.5 else "bucket"
        if tool != "none":
            speed = rng.uniform(0.2, 0.5)
            bodies.append(_tool(tool, lx, ly, top, speed, mu, case["envs"] == 1))
        f32 = lambda a: np.asarray(a, np.float32).astype(np.float64)  # noqa: E731
        specs.append(dict(x=f32(x), r=f32(r), v=f32(v), bodies=bodies, material=mat, dt=DT, gravity=(0.0, 0.0, -G),
                          max_sweeps=case["sweeps"], tol=case["tol"], warm_start=case["warm"], r_ref=r0,
                          grid_lo=(-0.5 * lx - 4 * r0, -0.5 * ly - 4 * r0, -4 * r0),
                          grid_hi=(0.5 * lx + 4 * r0, 0.5 * ly + 4 * r0, top + 0.5)))
    return specs


def _weights(seed):
    """Weights of the size a training run leaves: small corrections."""
    rng = np.random.default_rng([seed, 77])
    shapes = [(64, 12), (64,), (64, 64), (64,), (3, 64), (3,)]
    scale = [0.28, 0.05, 0.21, 0.05, 0.02, 0.005]
    w = [rng.uniform(-a, a, s).ravel() for s, a in zip(shapes, scale)]
    return np.concatenate(w + [rng.uniform(0.2, 1.0, 12)]).astype(np.float32)


def _prepare_step(case, seed):
    specs = _specs(case, seed)
    n = [len(s["x"]) for s in specs]
    sc = T.scene_from_specs(specs, cap_contacts=(16 if case["envs"] == 1 else 8) * max(n))
    if case["mode"] != "default":
        sc.set_solver_config(mode=case["mode"])
    if case["warm"] == "learned":
        sc.set_mlp_weights(_weights(seed))
    return dict(case=case, scene=sc, n=n, obs=np.zeros((sum(n), 9), np.float32),
                tool=len(specs[0]["bodies"]) > 1, zone="zone_planes" in specs[0]["bodies"][-1])


def _run_step(s):
    sc = s["scene"]
    st = sc.step(s["case"]["steps"])
    obs, o = s["obs"], 0
    for e, n in enumerate(s["n"]):
        p = sc.get_particles(e)
        for k, f in enumerate(("x", "v", "w")):
            obs[o:o + n, 3 * k:3 * k + 3] = p[f]
        o += n
    out = dict(obs=obs)
    for key in ("contacts", "pair_contacts", "colours", "sweeps"):
        out[key] = np.array([x[key] for x in st], np.int64)
    out["residual"] = np.array([x["residual"] for x in st], np.float32)
    if s["case"]["warm"] == "learned":
        out["fallback"] = np.array([x["fallback_used"] for x in st], np.int64)
    if s["tool"]:
        out["force"] = np.array([np.concatenate(sc.get_contact_forces(e, 1)) for e in range(len(s["n"]))], np.float32)
    if s["zone"]:
        a = sc.get_aggregates(0)[0]
        out["zone_n"] = int(a["n_particles"])
        out["zone"] = np.concatenate([[a["M"]], a["x"], a["v"], a["I"]])
    return out


# --------------------------------------------------------------------------
# the other kinds
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _samples(n, seed):
    """Inputs of the network as contacts give them: the radii positive, the flags 0 or 1, the rest centred."""
    f = torch.randn((n, 12), generator=_gen(seed), device="cuda")
    f[:, 8:10] = f[:, 8:10].abs() * 0.1 + 1.0
    f[:, 10:] = (f[:, 10:] > 0).float()
    return f


def _prepare_mlp(case, seed):
    return dict(case=case, w=torch.from_numpy(_weights(seed)).cuda(), f=_samples(case["batch"], seed),
                out=torch.empty((case["batch"], 3), device="cuda"))


def _run_mlp(s):
    T.mlp_forward(s["w"].data_ptr(), s["f"].data_ptr(), s["case"]["batch"], s["out"].data_ptr(), bf16=s["case"]["bf16"])
    return s["out"]


def _prepare_train(case, seed):
    b = case["batch"]
    z = lambda n: torch.zeros(n, device="cuda")  # noqa: E731
    ns = T.mlp_grad_scratch_floats(b)
    return dict(b=b, w=torch.from_numpy(_weights(seed)).cuda(), f=_samples(b, seed),
                lab=torch.randn((b, 3), generator=_gen(seed + 1), device="cuda"), g=z(T.MLP_TRAINABLE),
                loss=z(1), m=z(T.MLP_TRAINABLE), v=z(T.MLP_TRAINABLE), ns=ns, scratch=z(ns), t=0)


def _run_train(s):
    s["t"] += 1
    T.mlp_loss_grad(s["w"].data_ptr(), s["f"].data_ptr(), s["lab"].data_ptr(), s["b"], s["g"].data_ptr(),
                    s["loss"].data_ptr(), s["scratch"].data_ptr(), s["ns"])
    T.mlp_adam_step(s["w"].data_ptr(), s["g"].data_ptr(), s["m"].data_ptr(), s["v"].data_ptr(), 1e-3, s["t"])
    return dict(grad=s["g"], loss=s["loss"], w=s["w"], m=s["m"], v=s["v"])


L0, RHO_B, W_DEP = 0.05, 1800.0, 0.85


def _voxel_inputs(case, seed):
    """Rolling terrain, loose fluid above it and an ellipsoid of fluid ahead of the tool, a swirl velocity."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    g = _gen(seed)
    d = dict(device="cuda", dtype=torch.float64)
    rand = lambda *s: torch.rand(*s, generator=g, **d)  # noqa: E731
    z, y, x = torch.meshgrid(*[(torch.arange(m, **d) + 0.5) / m for m in (nz, ny, nx)], indexing="ij")
    top = nz * L0
    h = 0.55 + 0.12 * torch.exp(-((x[0] - 0.6) ** 2 + (y[0] - 0.4) ** 2) / 0.05)
    h = top * (h + 0.04 * torch.sin(9 * x[0]) * torch.cos(7 * y[0])) + 0.2 * L0 * (rand(ny, nx) - 0.5)
    h = h.clamp(0.4 * top, 0.75 * top)
    phi = ((h - (z * nz - 0.5) * L0) / L0).clamp(0.0, 1.0)
    wc = 0.85 + 0.15 * rand(nz, ny, nx)
    mf = torch.where((phi == 0) & (rand(nz, ny, nx) < 0.05), 0.25 * rand(nz, ny, nx), 0.0)
    q = ((x - 0.5) / 0.3) ** 2 + ((y - 0.5) / 0.2) ** 2 + ((z - 0.3) / 0.25) ** 2
    mf += 1600.0 * L0 ** 3 * (1.2 * rand(nz, ny, nx)).clamp(max=1.0) * (q < 1)
    rho_p = ((mf > 0) & (rand(nz, ny, nx) < 0.3)).double()
    u = torch.stack([0.7 - y, x - 0.5, 0.3 * torch.sin(2 * PI * x)], -1) + 0.2 * (rand(nz, ny, nx, 3) - 0.5)
    u *= 0.4 * L0 / DT / u.abs().max()
    # eight lateral wedges of a blade: in front of its face, above the failure plane, below the top
    ex, ez, th = 0.45 * nx * L0, 0.45 * top, 0.45
    wedges = []
    for k in range(8):
        y0, y1 = (0.2 + 0.075 * k) * ny * L0, (0.275 + 0.075 * k) * ny * L0
        s, c = math.sin(th + 0.01 * k), math.cos(th + 0.01 * k)
        wedges.append([[-1.0, 0.0, 0.0, -ex], [s, 0.0, -c, s * ex - c * ez], [0.0, 0.0, 1.0, 0.8 * top],
                       [0.0, -1.0, 0.0, -y0], [0.0, 1.0, 0.0, y1]])
    return phi, wc, mf, rho_p, u.contiguous(), wedges


def _prepare_voxels(case, seed):
    phi, wc, mf, rho_p, u, wedges = _voxel_inputs(case, seed)
    b = _body((0.0, 0.0, 0.0), [_plane((0.0, 0.0, 1.0), 0.0)])
    sc = T.scene_from_specs(dict(x=np.ones((1, 3)), r=np.full(1, 0.2), v=np.zeros((1, 3)), bodies=[b],
                                 material=dict(c_p=0.0), dt=DT, gravity=(0.0, 0.0, 0.0), max_sweeps=0,
                                 grid_lo=(0.0, 0.0, 0.0), grid_hi=(2.0, 2.0, 2.0)))
    sc.step(1)
    dims = (case["nx"], case["ny"], case["nz"])
    return dict(scene=sc, grid=((0.0, 0.0, 0.0), L0, dims), phi=phi, wc=wc, mf=[mf, torch.empty_like(mf)],
                rho_p=rho_p, u=u, wedges=wedges, h=torch.empty(dims[1], dims[0], device="cuda", dtype=torch.float64))


def _run_voxels(s):
    sc, g, (a, b) = s["scene"], s["grid"], s["mf"]
    phi, wc = s["phi"].data_ptr(), s["wc"].data_ptr()
    sc.convert_cut(0, *g, RHO_B, phi, wc, a.data_ptr(), wedges=s["wedges"], sync=False)
    sc.advect_fluid(*g, DT, s["u"].data_ptr(), a.data_ptr(), b.data_ptr(), sync=False)
    sc.convert_deposit(0, *g, RHO_B, W_DEP, s["rho_p"].data_ptr(), phi, wc, b.data_ptr(), wedges=s["wedges"],
                       sync=False)
    sc.terrain_from_voxels(0, *g, phi, s["h"].data_ptr())
    s["mf"] = [b, a]
    return dict(phi=s["phi"], wc=s["wc"], mf=b, h=s["h"])


def _field_specs(case, seed):
    spec = _specs(_step(None, case["n"], sweeps=0, warm="cold"), seed)[0]
    lo = [-0.5 * case["cell"] + min(spec["x"][:, k]) for k in range(3)]
    dims = [int((max(spec["x"][:, k]) - lo[k]) / case["cell"]) + 2 for k in range(3)]
    return spec, (lo, case["cell"], dims)


def _prepare_fields(case, seed):
    spec, grid = _field_specs(case, seed)
    sc = T.scene_from_specs(dict(spec, v=None, gravity=(0.0, 0.0, 0.0)))  # at rest: its one step moves nothing
    sc.step(1)
    sc.set_particles(0, v=spec["v"])
    nv = int(np.prod(grid[2]))
    z = lambda *s: torch.empty(*s, device="cuda", dtype=torch.float64)  # noqa: E731
    return dict(case=case, scene=sc, grid=grid, rho=z(nv), mom=z(nv, 3), u=z(nv, 3))


def _run_fields(s):
    c = s["case"]
    s["scene"].coarse_grain(0, *s["grid"], s["rho"].data_ptr(), s["mom"].data_ptr(), s["u"].data_ptr(),
                            kernel="gauss" if c["smooth"] else "heaviside", R=c["cell"] if c["smooth"] else 0.0)
    return dict(rho=s["rho"], mom=s["mom"], u=s["u"])


PREPARE = dict(step=_prepare_step, mlp=_prepare_mlp, train=_prepare_train, voxels=_prepare_voxels,
               fields=_prepare_fields)
RUN = dict(step=_run_step, mlp=_run_mlp, train=_run_train, voxels=_run_voxels, fields=_run_fields)


def prepare(case, seed):
    return dict(kind=case["kind"], state=PREPARE[case["kind"]](case, int(seed)))


def run(state):
    return RUN[state["kind"]](state["state"])


def work(case):
    """A bed: its state in and out once a step and at the read-back, and the arithmetic of its sweeps (about 150
    operations a contact and sweep; a solve to a tolerance from a cold start takes about 1,000 sweeps)."""
    kind = case["kind"]
    if kind == "step":
        n = sum(_sizes(case))
        sweeps = 1000 if case["tol"] else case["sweeps"]
        return dict(bytes=n * (case["steps"] * 104 + 72), flops=3.0 * n * case["steps"] * (sweeps * 150 + 300))
    if kind == "mlp":
        return dict(bytes=case["batch"] * 60 + 5199 * 4, flops=2.0 * case["batch"] * (12 * 64 + 64 * 64 + 3 * 64))
    if kind == "train":
        return dict(bytes=case["batch"] * 60 + 5199 * 4 * 8, flops=6.0 * case["batch"] * (12 * 64 + 64 * 64 + 3 * 64))
    if kind == "voxels":
        nv = case["nx"] * case["ny"] * case["nz"]
        # the columns' occupancy, compaction, fluid and particles read, the fluid and what changed written
        return dict(bytes=nv * (4 + 3 + 1 + 0.5) * 8, flops=nv * 40)
    nv = case["n"] * (2 * 0.03 / case["cell"]) ** 3
    return dict(bytes=case["n"] * 52 + nv * 56, flops=case["n"] * (113 * 40 if case["smooth"] else 30))


# --------------------------------------------------------------------------
# the same results in 64 bits, from the equations alone
# --------------------------------------------------------------------------
def exact(case, seed):
    if case["kind"] == "step":
        n = sum(_sizes(case))
        # several steps of a bed multiply any difference; a network's start is rounded to BF16 by definition
        if case["steps"] > 1 or case["warm"] == "learned" or n * case["sweeps"] > 2e7:
            return None
        return _exact_step(case, seed)
    if case["kind"] in ("mlp", "train"):
        return _exact_network(case, seed)
    return _exact_voxels(case, seed) if case["kind"] == "voxels" else _exact_fields(case, seed)


def _splitmix64(x):
    z = x + np.uint64(0x9E3779B97F4A7C15)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _pairs(x, r, kappa):
    """All pairs i < j with |x_j - x_i| < (1 + kappa) (r_i + r_j), through a cell list."""
    h = 2.0 * r.max() * (1.0 + kappa) * 1.001
    c = np.floor((x - x.min(0)) / h).astype(np.int64) + 1
    d = c.max(0) + 2
    key = (c[:, 2] * d[1] + c[:, 1]) * d[0] + c[:, 0]
    order = np.argsort(key, kind="stable")
    sk = key[order]
    out = []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                k = key + (dz * d[1] + dy) * d[0] + dx
                beg, end = np.searchsorted(sk, k, "left"), np.searchsorted(sk, k, "right")
                for t in range(int((end - beg).max())):
                    i = np.nonzero(beg + t < end)[0]
                    j = order[beg[i] + t]
                    keep = i < j
                    i, j = i[keep], j[keep]
                    e = x[j] - x[i]
                    rs = r[i] + r[j]
                    R = rs + kappa * rs
                    hit = (e[:, 0] * e[:, 0] + e[:, 1] * e[:, 1]) + e[:, 2] * e[:, 2] < R * R
                    out.append(np.stack([i[hit], j[hit]], 1))
    return np.concatenate(out)


def _touch(s, b, x, r, kappa):
    """Spheres in contact with a boundary shape: indices, overlaps and normals."""
    R = r + kappa * (2.0 * r)
    if s["type"] == "plane":
        n = np.array(s["n"])
        sd = x @ n - s["d"]
        i = np.nonzero((sd < 0) | (sd * sd < R * R))[0]
        return i, r[i] - sd[i], np.repeat(n[None], len(i), 0)
    half = np.array(s["half"])
    loc = x - (np.array(b["pos"]) + np.array(s["off"]))
    q = np.clip(loc, -half, half)
    e = loc - q
    d2 = (e * e).sum(1)
    inside = (np.abs(loc) <= half).all(1)
    i = np.nonzero(inside | (d2 < R * R))[0]
    loc, e, dist, inside = loc[i], e[i], np.sqrt(d2[i]), inside[i]
    pen = half - np.abs(loc)
    kb = np.argmin(pen, 1)
    nin = np.zeros_like(loc)
    nin[np.arange(len(i)), kb] = np.where(loc[np.arange(len(i)), kb] >= 0, 1.0, -1.0)
    nout = e / np.where(dist > 0, dist, 1.0)[:, None]
    delta = np.where(inside, r[i] + pen.min(1), r[i] - dist)
    return i, delta, np.where(inside[:, None], nin, nout)


def _cross(a, b):
    return np.stack([a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]])


def _exact_env(case, spec, id_base):
    """One step of an env from rest impulses: detection, rows, colouring, sweeps, integration."""
    m_ = spec["material"]
    mu, mu_r, c_p, E, nu, kappa, kmin = m_["mu_t"], m_["mu_r"], m_["c_p"], 1e9, 0.15, 0.025, 1e-4
    x, r, n = spec["x"], spec["r"], len(spec["x"])
    p = _pairs(x, r, kappa)
    e = x[p[:, 1]] - x[p[:, 0]]
    d = np.sqrt((e * e).sum(1))
    A, B = [p[:, 0]], [p[:, 1]]
    N, delta = [e / d[:, None]], [(r[p[:, 0]] + r[p[:, 1]]) - d]
    key = [((p[:, 0] + id_base).astype(np.uint64) << np.uint64(32)) | (p[:, 1] + id_base).astype(np.uint64)]
    owner, shape = [np.full(len(p), -1)], 0
    for bi, b in enumerate(spec["bodies"]):
        for s in b["shapes"]:
            i, dl, nn = _touch(s, b, x, r, kappa)
            A.append(np.full(len(i), n))
            B.append(i)
            N.append(nn)
            delta.append(dl)
            key.append(((i + id_base).astype(np.uint64) << np.uint64(32)) | np.uint64(0x80000000 | shape))
            owner.append(np.full(len(i), bi))
            shape += 1
    A, B, N, delta, key, owner = (np.concatenate(a) for a in (A, B, N, delta, key, owner))
    pair = A < n
    # rows
    re = np.append(r, 0.0)
    mass = spec["material"]["rho"] * 4.0 / 3.0 * PI * r ** 3
    im, iI = np.append(1.0 / mass, 0.0), np.append(1.0 / (0.4 * mass * r * r), 0.0)
    r1, r2 = np.where(pair, re[A], r[B]), r[B]
    l1, l2 = np.where(pair, r1 - 0.5 * delta, 0.0), r2 - 0.5 * delta
    vel = np.concatenate([spec["v"].T, np.zeros((3, 1))], 1)
    vk = np.zeros((3, len(A)))
    for bi, b in enumerate(spec["bodies"]):
        vk[:, owner == bi] = np.array(b["linvel"])[:, None]
    un = (N.T * (vel[:, B] - np.where(pair, vel[:, A], vk))).sum(0)
    kn = E / (2 * (1 - nu * nu)) * np.sqrt(1 / (1 / (2 * r1) + 1 / (2 * r2)) * np.where(pair, 1.0, 2.0)) / 3
    eps = 4 / (5 * kn * np.sqrt(np.maximum(delta, kmin * (r1 + r2))))
    ups = 1.0 / 9.0  # 1 / (1 + 4 tau / dt) with tau = 2 dt
    sig = 4 / DT ** 2 * ups * eps
    q = 4 / DT * ups * 0.8 * delta + ups * un
    iDn = 1 / (im[A] + im[B] + sig)
    iDt = 1 / (im[A] + im[B] + l1 * l1 * iI[A] + l2 * l2 * iI[B])
    rmin = np.minimum(r1, r2)
    lo = -c_p * PI * DT * rmin * rmin
    iWr = 1 / (iI[A] + iI[B])
    # greedy colouring in decreasing (hash, key) order
    order = np.lexsort((key, _splitmix64(key)))[::-1]
    used, colour = [0] * (n + 1), np.zeros(len(A), np.int64)
    for c, a, b in zip(order.tolist(), A[order].tolist(), B[order].tolist()):
        u = used[b] | (used[a] if a < n else 0)
        bit = ~u & (u + 1)
        colour[c] = bit.bit_length() - 1
        used[b] |= bit
        used[a] |= bit
    classes = []
    for k in range(int(colour.max()) + 1 if len(A) else 0):
        c = np.nonzero(colour == k)[0]
        classes.append((c, A[c], B[c], pair[c], N[c].T.copy(), vk[:, c], l1[c], l2[c], sig[c], q[c], iDn[c], iDt[c],
                        lo[c], im[A[c]], im[B[c]], iI[A[c]], iI[B[c]], iWr[c], rmin[c] * mu_r))
    v, w = vel.copy(), np.zeros_like(vel)
    v[2, :n] -= DT * G
    ln, lt, lr = np.zeros(len(A)), np.zeros((3, len(A))), np.zeros((3, len(A)))
    done, R = 0, 0.0
    for done in range(1, case["sweeps"] + 1):
        num = den = 0.0
        for c, a, b, pr, nn, vkc, e1, e2, sg, qq, dn_, dt_, lw, ma, mb, ia, ib, wr, rl in classes:
            va, vb, wa, wb = np.where(pr, v[:, a], vkc), v[:, b], np.where(pr, w[:, a], 0.0), w[:, b]
            l0, t0 = ln[c], lt[:, c]
            u = (nn * (vb - va)).sum(0)
            l = np.maximum(lw, l0 - (u + sg * l0 - qq) * dn_)
            dl = (l - l0) * nn
            vb, va = vb + dl * mb, va - dl * ma
            u = (vb - va) - _cross(e2 * wb + e1 * wa, nn)
            u -= (u * nn).sum(0) * nn
            t = t0 - u * dt_
            lim, size = mu * np.abs(l), np.sqrt((t * t).sum(0))
            t = t * np.where(size > lim, lim / np.where(size > 0, size, 1.0), 1.0)
            dt = t - t0
            cx = _cross(nn, dt)
            vb, va = vb + dt * mb, va - dt * ma
            wb, wa = wb - e2 * ib * cx, wa - e1 * ia * cx
            num += ((l - l0) ** 2 / dn_).sum() + ((dt * dt).sum(0) / dt_).sum()
            den += (l * l / dn_).sum() + ((t * t).sum(0) / dt_).sum()
            if mu_r > 0.0:
                s0 = lr[:, c]
                s = s0 - (wb - wa) * wr
                lim, size = rl * np.abs(l), np.sqrt((s * s).sum(0))
                s = s * np.where(size > lim, lim / np.where(size > 0, size, 1.0), 1.0)
                wb, wa = wb + ib * (s - s0), wa - ia * (s - s0)
                num += (((s - s0) ** 2).sum(0) / wr).sum()
                den += ((s * s).sum(0) / wr).sum()
                lr[:, c] = s
            ln[c], lt[:, c] = l, t
            v[:, b], w[:, b] = vb, wb
            v[:, a[pr]], w[:, a[pr]] = va[:, pr], wa[:, pr]
        R = math.sqrt(num / den) if den > 0 else float(num > 0)
        if case["tol"] > 0 and R <= case["tol"]:
            break
    v, w = v[:, :n].T, w[:, :n].T
    xe = x + DT * v
    out = dict(obs=np.concatenate([xe, v, w], 1), contacts=len(A), pair_contacts=int(pair.sum()), colours=len(classes),
               sweeps=done, residual=R)
    if len(spec["bodies"]) > 1:
        c = np.nonzero(owner == 1)[0]
        f = -(ln[c] * N[c].T + lt[:, c]) / DT
        arm = (x[B[c]] - l2[c][:, None] * N[c] - np.array(spec["bodies"][1]["pos"])).T
        out["force"] = np.concatenate([f.sum(1), (_cross(arm, f) - lr[:, c] / DT).sum(1)])
    if "zone_planes" in spec["bodies"][-1]:
        b = spec["bodies"][-1]
        y = xe - (np.array(b["pos"]) + DT * np.array(b["linvel"]))
        k = np.all([y @ np.array(pl[:3]) <= pl[3] for pl in b["zone_planes"]], axis=0)
        m, xz, vz, rz = mass[k], xe[k], v[k], r[k]
        M = m.sum()
        xc = (m[:, None] * xz).sum(0) / M
        s = xz - xc
        own = (0.4 * m * rz * rz).sum()
        C = (m[:, None, None] * s[:, :, None] * s[:, None, :]).sum(0)
        I = (own + np.trace(C)) * np.eye(3) - C
        out["zone_n"] = int(k.sum())
        out["zone"] = np.concatenate([[M], xc, (m[:, None] * vz).sum(0) / M, [I[0, 0], I[1, 1], I[2, 2], I[0, 1],
                                                                              I[0, 2], I[1, 2]]])
    return out


def _exact_step(case, seed):
    specs = _specs(case, seed)
    cap = max(len(s["x"]) for s in specs)
    envs = [_exact_env(case, s, e * cap) for e, s in enumerate(specs)]
    out = dict(obs=np.concatenate([o["obs"] for o in envs]))
    for key in ("contacts", "pair_contacts", "colours", "sweeps"):
        out[key] = np.array([o[key] for o in envs], np.int64)
    out["residual"] = np.array([o["residual"] for o in envs])
    if "force" in envs[0]:
        out["force"] = np.array([o["force"] for o in envs])
    if "zone" in envs[0]:
        out["zone_n"], out["zone"] = envs[0]["zone_n"], envs[0]["zone"]
    return out


def _exact_network(case, seed):
    w = torch.from_numpy(_weights(seed)).cuda().double()
    f = _samples(case["batch"], seed).double()
    sizes = [768, 64, 4096, 64, 192, 3, 12]
    w1, b1, w2, b2, w3, b3, scale = torch.split(w, sizes)
    par = [w1.reshape(64, 12), b1, w2.reshape(64, 64), b2, w3.reshape(3, 64), b3]
    if case["kind"] == "train":
        par = [t.clone().requires_grad_(True) for t in par]
    h = torch.nn.functional.silu(torch.nn.functional.linear(f * scale, par[0], par[1]))
    h = torch.nn.functional.silu(torch.nn.functional.linear(h, par[2], par[3]))
    y = torch.nn.functional.linear(h, par[4], par[5])
    if case["kind"] == "mlp":
        return y
    lab = torch.randn((case["batch"], 3), generator=_gen(seed + 1), device="cuda").double()
    loss = 0.5 * ((y - lab) ** 2).sum(1).mean()
    g = torch.cat([t.reshape(-1) for t in torch.autograd.grad(loss, par)])
    new = w.clone()
    new[:5187] -= 1e-3 * g / (g.abs() + 1e-8)
    return dict(grad=g, loss=loss.detach().reshape(1), w=new, m=0.1 * g, v=1e-3 * g * g)


def _exact_voxels(case, seed):
    phi, wc, mf, rho_p, u, wedges = _voxel_inputs(case, seed)
    nz, ny, nx = phi.shape
    V0 = L0 ** 3
    d = dict(device="cuda", dtype=torch.float64)
    z, y, x = torch.meshgrid(*[(torch.arange(m, **d) + 0.5) * L0 for m in (nz, ny, nx)], indexing="ij")
    inf = float("inf")
    # cut: the lowest of the wedges' bottoms over each column's centre
    cut = torch.full((ny, nx), inf, **d)
    inside = torch.zeros_like(phi, dtype=torch.bool)
    for W in wedges:
        lo, hi, ok = torch.full((ny, nx), -inf, **d), torch.full((ny, nx), inf, **d), torch.ones_like(cut).bool()
        here = torch.ones_like(inside)
        for a, b, c, e in W:
            rest = e - a * x[0] - b * y[0]
            if c > 0:
                hi = torch.minimum(hi, rest / c)
            elif c < 0:
                lo = torch.maximum(lo, rest / c)
            else:
                ok &= rest >= 0
            here &= a * x + b * y + c * z - e <= 0
        inside |= here
        cut = torch.where(ok & (lo <= hi), torch.minimum(cut, lo), cut)
    t = ((cut - (z - 0.5 * L0)) / L0).clamp(0.0, 1.0)
    t = torch.where(torch.isinf(cut), torch.ones_like(t), t)
    moved = phi > t
    mf = torch.where(moved, mf + wc * RHO_B * V0 * (phi - t), mf)
    phi = torch.where(moved, t, phi)
    # advection: the donor's mass through each interior face
    out = mf.clone()
    for k, dim in ((2, 0), (1, 1), (0, 2)):
        m = phi.shape[dim]
        ua, ub = u[..., k].narrow(dim, 0, m - 1), u[..., k].narrow(dim, 1, m - 1)
        uf = 0.5 * (ua + ub)
        flux = DT * uf * torch.where(uf > 0, mf.narrow(dim, 0, m - 1), mf.narrow(dim, 1, m - 1)) / L0
        out.narrow(dim, 0, m - 1).sub_(flux)
        out.narrow(dim, 1, m - 1).add_(flux)
    mf = out
    # deposit: upwards, each voxel's fluid onto its column's surface
    fp, fw = phi.reshape(nz, -1).clone(), wc.reshape(nz, -1).clone()
    fm = mf.reshape(nz, -1)
    falls = ((mf > 0) & (rho_p == 0) & ~inside).reshape(nz, -1)
    full = W_DEP * RHO_B * V0
    col = torch.arange(ny * nx, device="cuda")
    top = torch.where(fp < 1, torch.arange(nz, device="cuda")[:, None], nz).min(0).values  # first voxel not full
    for k in range(nz):
        m = torch.where(falls[k], fm[k], torch.zeros_like(fm[k]))
        while True:
            c = col[(m > 0) & (top < nz)]
            if not len(c):
                break
            kk = top[c]
            f0, w0 = fp[kk, c], fw[kk, c]
            room = (1.0 - f0) * full
            take = torch.minimum(m[c], room)
            f = torch.where(take == room, 1.0, f0 + take / full)
            fw[kk, c] = torch.where(f0 > 0, (w0 * RHO_B * V0 * f0 + take) / (RHO_B * V0 * f), W_DEP)
            fp[kk, c] = f
            m[c] -= take
            top[c] = torch.where(f >= 1.0, kk + 1, kk)
        fm[k] = torch.where(falls[k], m, fm[k])
    solid = fp > 0
    k = torch.where(solid, torch.arange(nz, device="cuda")[:, None], -1).max(0).values
    h = (k.double() + 0.5) * L0 + (fp[k.clamp(min=0), col] - 0.5) * L0
    h = torch.where(k >= 0, h, torch.zeros_like(h))
    shape = phi.shape
    return dict(phi=fp.reshape(shape), wc=fw.reshape(shape), mf=fm.reshape(shape), h=h.reshape(ny, nx))


def _exact_fields(case, seed):
    spec, (lo, l0, dims) = _field_specs(case, seed)
    x, v = (torch.from_numpy(spec[k]).cuda() for k in ("x", "v"))
    m = torch.from_numpy(2000.0 * 4.0 / 3.0 * PI * spec["r"] ** 3).cuda()
    lo, dim = torch.tensor(lo, dtype=torch.float64, device="cuda"), torch.tensor(dims, device="cuda")
    nv = int(np.prod(dims))
    rho, mom = torch.zeros(nv, dtype=torch.float64, device="cuda"), torch.zeros((nv, 3), dtype=torch.float64, device="cuda")
    cell = torch.floor((x - lo) / l0).long()
    reach = range(-4, 5) if case["smooth"] else range(1)
    for dz in reach:
        for dy in reach:
            for dx in reach:
                c = cell + torch.tensor([dx, dy, dz], device="cuda")
                ok = ((c >= 0) & (c < dim)).all(1)
                if case["smooth"]:
                    d2 = ((lo + (c.double() + 0.5) * l0 - x) ** 2).sum(1)
                    ok &= d2 <= 9 * l0 * l0
                    z = torch.exp(-d2 / (2 * l0 * l0)) / (math.sqrt(2 * PI) * l0) ** 3
                else:
                    z = torch.full_like(m, 1 / l0 ** 3)
                at = ((c[:, 2] * dims[1] + c[:, 1]) * dims[0] + c[:, 0])[ok]
                rho.index_add_(0, at, (m * z)[ok])
                mom.index_add_(0, at, ((m * z)[:, None] * v)[ok])
    u = torch.where(rho[:, None] > 0, mom / rho[:, None].clamp(min=1e-300), torch.zeros_like(mom))
    return dict(rho=rho, mom=mom, u=u)
