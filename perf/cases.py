"""The work that users of this library have it do, as cases to be timed: time steps of single
lattices and of batches with the read-back that belongs to them, and the surrogate's
prediction, training step and convolution layers.

Kinds of cases
  steps   a lattice on the GPU advanced by `steps` steps; then `read` says what the program
          takes from it: "state" (phi and u / u_scale of every cell, on the device), "phi"
          (the phi field on the host, kept in single precision) or "diagnostics" (masses, mean
          pressures and the largest speed).
  sweep   a batch of uneven jets advanced together, then every case's 4^3 block means on the
          device, as the surrogate takes them.
  predict one forward pass of the surrogate on device-resident coarse states.
  train   one training step of the surrogate (forward, backward, Adam).
  conv    one 3x3x3 convolution layer: forward with ReLU, data gradient behind a ReLU mask (where
          the layer has one: cin a multiple of 32), weight and bias gradient.
"""
import ctypes
import math

import numpy as np
import torch

from paper_1705_03141_amd import lbm
from paper_1705_03141_amd import surrogate as S
from paper_1705_03141_amd import workloads as W

VALUE_BYTES = {"f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # the smallest lattice in use, the 32^3 droplet of the smoke run and the quick checks: a few
        # steps, where launches and the length of one step's dependency chain count
        dict(name="droplet_32", kind="steps", flow="droplet", nx=32, ny=32, nz=32, storage="f32", steps=10,
             read="state"),
        # the oscillation test, 41^3: some steps, then the phi field to track the interface
        dict(name="oscillation_41", kind="steps", flow="droplet", nx=41, ny=41, nz=41, storage="f32", steps=20,
             read="phi"),
        # the Laplace-law test, 85^3 (tens of thousands of steps), with its pressure-jump diagnostics
        dict(name="laplace_85", kind="steps", flow="droplet", nx=85, ny=85, nz=85, storage="f32", steps=50,
             read="diagnostics"),
        # Rayleigh-Taylor at the size of the benchmark's second workload: walls in z, body force
        dict(name="rt_128x512", kind="steps", flow="rt", nx=128, ny=128, nz=512, storage="f32", steps=10,
             read="state"),
        # the same with 16-bit storage
        dict(name="rt_128x512_bf16", kind="steps", flow="rt", nx=128, ny=128, nz=512, storage="bf16", steps=10,
             read="state"),
        # the benchmark's jet: the largest lattice in regular use
        dict(name="jet_256x1024", kind="steps", flow="jet", nx=256, ny=256, nz=1024, storage="f32", steps=4,
             read="state", walls=False),
        # the reference jet between free-slip lateral walls, 8D x 8D x 20D with D = 25
        dict(name="walls_200x500", kind="steps", flow="jet", nx=200, ny=200, nz=500, storage="f32", steps=5,
             read="state", walls=True),
        # the varicose jet (D = 15) between walls, with 16-bit storage
        dict(name="walls_120x300_f16", kind="steps", flow="jet", nx=120, ny=120, nz=300, storage="f16", steps=10,
             read="state", walls=True),
        # uneven jets of a regime map advanced together, FP16 storage, snapshots for the surrogate
        dict(name="sweep_6_f16", kind="sweep", cases=6, small=96, large=112, storage="f16", steps=5),
        # the surrogate on its padded box: one network's prediction
        dict(name="predict_256x64x64", kind="predict", n=1, d=256, h=64, w=64),
        # and one training step on it
        dict(name="train_256x64x64", kind="train", n=1, d=256, h=64, w=64),
        # one layer at half resolution (the encoder's widening layer), forward and backward
        dict(name="conv_32_64", kind="conv", n=1, d=128, h=32, w=32, cin=32, cout=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["droplet", "droplet", "rt", "jet", "jet", "jet_walls", "jet_walls", "sweep", "predict", "train",
                       "conv", "conv"])
    storage = rng.choice(["f32", "f32", "f16", "bf16"])
    if kind == "droplet":
        nx, ny, nz = (_log_int(rng, 20, 160) for _ in range(3))
        return dict(kind="steps", flow="droplet", nx=nx, ny=ny, nz=nz, storage=storage, steps=rng.randint(4, 30),
                    read=rng.choice(["state", "phi", "diagnostics"]))
    if kind == "rt":
        w = _log_int(rng, 16, 144)
        return dict(kind="steps", flow="rt", nx=w, ny=w, nz=rng.randint(2 * w, 4 * w), storage=storage,
                    steps=rng.randint(4, 12), read=rng.choice(["state", "diagnostics"]))
    if kind in ("jet", "jet_walls"):
        w = _log_int(rng, 24, 256)
        return dict(kind="steps", flow="jet", nx=w, ny=w + rng.randint(-4, 4), nz=int(w * rng.uniform(1.5, 2.5)),
                    storage=storage, steps=rng.randint(3, 7), read="state", walls=kind == "jet_walls")
    if kind == "sweep":
        small = 4 * rng.randint(12, 26)
        return dict(kind="sweep", cases=rng.randint(2, 6), small=small, large=small + 4 * rng.randint(1, 5),
                    storage=storage, steps=rng.randint(3, 8))
    if kind in ("predict", "train"):
        return dict(kind=kind, n=rng.randint(1, 3), d=4 * rng.randint(6, 48), h=4 * rng.randint(4, 17),
                    w=4 * rng.randint(4, 17))
    return dict(kind="conv", n=rng.randint(1, 2), d=_log_int(rng, 3, 128), h=_log_int(rng, 5, 70),
                w=_log_int(rng, 5, 90), cin=rng.choice([8, 16, 32, 32, 64, 128]), cout=rng.choice([32, 64]))


# ---------------------------------------------------------------- lattices

def _flow(case):
    """The physics of a lattice case: a workloads.Problem without fields, and its velocity scale."""
    nx, ny, nz, flow = case["nx"], case["ny"], case["nz"], case["flow"]
    if flow == "droplet":
        return W.Problem(name="droplet", nx=nx, ny=ny, nz=nz, rho_r0=1.5, rho_b0=1.0, nu_r=1e-3, nu_b=1e-3, A=1e-2,
                         beta=0.7), 0.02
    if flow == "rt":
        g = 1e-5
        nu = math.sqrt(nx * g) * nx / 256.0
        return W.Problem(name="rt", nx=nx, ny=ny, nz=nz, rho_r0=3.0, rho_b0=1.0, nu_r=nu, nu_b=nu, A=0.0, beta=0.7,
                         faces=(W.PERIODIC,) * 4 + (W.BOUNCEBACK,) * 2, force_model=1, g=(0.0, 0.0, g),
                         rho_ref=2.0), 0.02
    walls = case["walls"]
    pb = W.jet(nx=nx, ny=ny, nz=nz, diameter=max(6.0, nx / (8.0 if walls else 16.0)), eta=4.2 if walls else 1.0,
               fields=False, lateral=W.FREESLIP if walls else W.PERIODIC)
    return pb, pb.u_in


def _fields(case, pb, seed):
    """Initial (rho_r, rho_b, u) in FP64 on the GPU: the flow's interface with a tanh profile of
    width 4, seeded noise of 1e-4 on the densities and a smooth velocity of a few per cent."""
    dev, f64 = "cuda", torch.float64
    gen = torch.Generator(device=dev).manual_seed(1000003 * int(seed) + 17)
    nx, ny, nz = pb.nx, pb.ny, pb.nz
    x = torch.arange(nx, device=dev, dtype=f64).view(1, 1, nx)
    y = torch.arange(ny, device=dev, dtype=f64).view(1, ny, 1)
    z = torch.arange(nz, device=dev, dtype=f64).view(nz, 1, 1)
    p = torch.rand(6, generator=gen, device=dev, dtype=f64)
    tau = 2 * math.pi
    u = torch.zeros((3, nz, ny, nx), device=dev, dtype=f64)
    if case["flow"] == "droplet":
        r = torch.sqrt((x - (nx - 1) / 2 - p[0]) ** 2 + (y - (ny - 1) / 2 - p[1]) ** 2 + (z - (nz - 1) / 2 - p[2]) ** 2)
        t = torch.tanh((r - 0.35 * min(nx, ny, nz)) / 2.0)
        u[0] = 0.01 * torch.sin(tau * (y / ny + p[3]))
        u[1] = 0.01 * torch.sin(tau * (z / nz + p[4]))
        u[2] = 0.01 * torch.sin(tau * (x / nx + p[5]))
    elif case["flow"] == "rt":
        zi = (nz - 1) / 2 + 0.05 * nx * (torch.cos(tau * (x / nx + p[0])) + torch.cos(tau * (y / ny + p[1])))
        t = torch.tanh((z - zi) / 2.0)
        wall = torch.sin(math.pi * (z + 0.5) / nz)
        u[0] = 0.01 * torch.sin(tau * (y / ny + p[2])) * wall
        u[2] = 0.01 * torch.sin(tau * (x / nx + p[3])) * wall
    else:
        r = torch.sqrt((x - pb.xc - p[0] + 0.5) ** 2 + (y - pb.yc - p[1] + 0.5) ** 2)
        radius = 0.5 * pb.diameter * (1.0 + 0.1 * torch.sin(tau * (4 * z / nz + p[2])))
        t = torch.maximum(torch.tanh((r - radius) / 2.0), torch.tanh((z - (0.5 + 0.3 * p[3]) * nz) / 2.0))
        u[2] = 0.5 * pb.u_in * (1.0 - torch.tanh((r - radius) / 2.0)) + 0.05 * pb.u_in
    rho_r, rho_b = 0.5 * pb.rho_r0 * (1.0 - t), 0.5 * pb.rho_b0 * (1.0 + t)
    noise = lambda: 1.0 + 1e-4 * (2.0 * torch.rand((nz, ny, nx), generator=gen, device=dev) - 1.0)  # noqa: E731
    return rho_r * noise(), rho_b * noise(), u


def _sweep_problems(case, seed):
    pbs = W.regime_sweep(ncases=case["cases"], seed=11, sizes=(case["small"], case["large"]))
    for k, pb in enumerate(pbs):
        pb.seed = 1000 * seed + k
    return pbs


def _host(t):
    return np.ascontiguousarray(t.cpu().numpy())


# ---------------------------------------------------------------- the surrogate's inputs

def _coarse_fields(case, seed):
    """Coarse states as the sweep gives them: phi of a wavy jet column and u / u_in around it,
    zeros beyond the case's own lattice in the padded box; (n, d, h, w, 4) FP32."""
    gen = torch.Generator(device="cuda").manual_seed(7919 * int(seed) + 5)
    n, d, h, w = case["n"], case["d"], case["h"], case["w"]
    z = torch.arange(d, device="cuda").view(1, d, 1, 1) / d
    y = torch.arange(h, device="cuda").view(1, 1, h, 1) / h
    x = torch.arange(w, device="cuda").view(1, 1, 1, w) / w
    p = torch.rand((4, n, 1, 1, 1), generator=gen, device="cuda")
    wave = 0.03 * torch.sin(2 * math.pi * (5 * z + p[0]))
    r = torch.sqrt((x - 0.3 - wave) ** 2 + (y - 0.3) ** 2)
    phi = torch.maximum(torch.tanh(20 * (r - 0.08)), torch.tanh(20 * (z - 0.3 - 0.4 * p[1])))
    uz = 0.5 * (1 - phi) + 0.1 * torch.sin(2 * math.pi * (2 * x + 3 * z + p[2]))
    ux = 0.1 * torch.sin(2 * math.pi * (3 * y + 4 * z + p[3]))
    state = torch.stack([-phi, ux.expand_as(phi), 0.5 * ux.expand_as(phi), uz], dim=-1)
    state = state + 0.02 * torch.randn(state.shape, generator=gen, device="cuda")
    inside = (z < 0.9) & (y < 0.75) & (x < 0.75)
    return torch.where(inside.unsqueeze(-1), state, torch.zeros_like(state)).float().contiguous()


def _bf16(shape, gen, scale=1.0):
    return (scale * torch.randn(shape, generator=gen, device="cuda")).to(torch.bfloat16)


def _conv_inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(104729 * int(seed) + 3)
    dims, cin, cout = (case["n"], case["d"], case["h"], case["w"]), case["cin"], case["cout"]
    x = torch.relu(_bf16(dims + (cin,), gen))  # the layer's input is the ReLU output of the one before
    wt = _bf16((27, cout, cin), gen, math.sqrt(2.0 / (27 * cin)))
    b = 0.1 * torch.randn(cout, generator=gen, device="cuda")
    dout = _bf16(dims + (cout,), gen, 1e-2) * (_bf16(dims + (cout,), gen) > 0)
    return x, wt, b, dout


# ---------------------------------------------------------------- prepare and run

def prepare(case, seed):
    kind = case["kind"]
    if kind == "steps":
        pb, u_scale = _flow(case)
        rr, rb, u = _fields(case, pb, seed)
        pb.rho_r, pb.rho_b, pb.u = _host(rr), _host(rb), _host(u)
        pb.seed = int(seed)
        lat = lbm.Lattice(pb, storage=case["storage"])
        pb.rho_r = pb.rho_b = pb.u = None
        st = dict(case=case, lat=lat, u_scale=u_scale)
        if case["read"] == "state":
            st["out"] = torch.empty(lat.shape + (4,), dtype=torch.float32, device="cuda")
        return st
    if kind == "sweep":
        pbs = _sweep_problems(case, seed)
        batch = lbm.Batch(pbs, storage=case["storage"], init=False)
        for k, (pb, c) in enumerate(zip(pbs, batch.cases)):
            rr, rb, u = _fields(dict(flow="jet"), pb, 100 * seed + k)
            c.init_fields(_host(rr), _host(rb), _host(u))
        outs = [torch.empty(S.coarse_extent(pb) + (4,), dtype=torch.float32, device="cuda") for pb in pbs]
        return dict(case=case, batch=batch, outs=outs, u_scale=pbs[0].u_in)
    if kind in ("predict", "train"):
        net = S.Network(case["n"], case["d"], case["h"], case["w"], seed=int(seed) % 100003)
        x = _coarse_fields(case, seed)
        st = dict(case=case, net=net, x=x)
        if kind == "train":
            st["target"] = (_coarse_fields(case, seed + 1) - x).contiguous()
        return st
    x, wt, b, dout = _conv_inputs(case, seed)
    dims, cin, cout = (case["n"], case["d"], case["h"], case["w"]), case["cin"], case["cout"]
    L = S._lib()
    i16 = torch.int16
    st = dict(case=case, L=L, x=x.view(i16), w=wt.view(i16), b=b, dout=dout.view(i16),
              out=torch.empty(dims + (cout,), dtype=i16, device="cuda"),
              dw=torch.empty((27, cout, cin), device="cuda"), db=torch.empty(cout, device="cuda"),
              scratch=torch.empty(int(L.surr_conv3d_wgrad_scratch_bytes(*dims, cin, cout)) // 4 + 1, device="cuda"))
    if cin % 32 == 0:
        st["w_t"] = torch.empty((27, cin, cout), dtype=i16, device="cuda")
        st["din"] = torch.empty(dims + (cin,), dtype=i16, device="cuda")
        S._ok(L.surr_conv3d_flip_weights(S._p(st["w"]), S._p(st["w_t"]), cin, cout, None), "flip")
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "steps":
        lat = state["lat"]
        lat.step(case["steps"])
        if case["read"] == "state":
            lat.coarse_state_into(state["out"], 1, state["u_scale"])
            return state["out"]
        if case["read"] == "phi":
            return lat.field("phi").astype(np.float32)
        d = lat.diagnostics(**_diag_query(case))
        return {k: d[k] for k in ("mass_r", "mass_b", "umax", "p_in", "p_out", "n_in", "n_out", "nan_cells")}
    if kind == "sweep":
        state["batch"].step(case["steps"])
        for c, out in zip(state["batch"].cases, state["outs"]):
            c.coarse_state_into(out, 4, state["u_scale"])
        return state["outs"]
    if kind == "predict":
        net, x = state["net"], state["x"]
        net.set_input(x)
        return x + net.forward()[..., :S.FIELDS]
    if kind == "train":
        net = state["net"]
        net.train_step(state["x"], state["target"], sync_loss=False)
        # the network works in BF16: its refreshed working weights, and the gradients in the same type
        return {"w": {k: v.view(torch.bfloat16) for k, v in net.wbf.items()},
                "g": {k: v.to(torch.bfloat16) for k, v in net.gw.items()},
                "gb": {k: v.to(torch.bfloat16) for k, v in net.gb.items()}}
    L, p = state["L"], S._p
    dims, cin, cout = (case["n"], case["d"], case["h"], case["w"]), case["cin"], case["cout"]
    S._ok(L.surr_conv3d_fwd(p(state["x"]), p(state["w"]), p(state["b"]), p(state["out"]), None, *dims, cin, cout, 1,
                            None), "forward")
    S._ok(L.surr_conv3d_wgrad(p(state["x"]), p(state["dout"]), p(state["dw"]), p(state["db"]), p(state["scratch"]),
                              *dims, cin, cout, None), "weight gradient")
    res = {"out": state["out"].view(torch.bfloat16), "dw": state["dw"], "db": state["db"]}
    if "din" in state:
        S._ok(L.surr_conv3d_dgrad(p(state["dout"]), p(state["w_t"]), p(state["x"]), p(state["din"]), *dims, cin, cout,
                                  None), "data gradient")
        res["din"] = state["din"].view(torch.bfloat16)
    return res


def _diag_query(case):
    n = min(case["nx"], case["ny"], case["nz"])
    return dict(center=tuple((case[k] - 1) / 2 for k in ("nx", "ny", "nz")), r_in=0.2 * n, r_out=0.45 * n)


# ---------------------------------------------------------------- what a pass cannot do without

def _layer_flops(nv):
    """Forward FLOPs of the surrogate's layers for nv full-resolution voxels; the last layer's
    four fields."""
    per = {"e1a": 8 * 32, "e1b": 32 * 32, "e2": 32 * 64 / 8, "bt": 64 * 64 / 64, "d2": 64 * 32 / 8, "d1": 32 * 32,
           "out": 32 * 4}
    return {k: 54.0 * v * nv for k, v in per.items()}


def work(case):
    kind = case["kind"]
    if kind == "steps":
        n = case["nx"] * case["ny"] * case["nz"]
        cell = 2 * (27 * VALUE_BYTES[case["storage"]] + 20)  # the 32-value state read and written
        out = {"state": 16, "phi": 4, "diagnostics": 0}[case["read"]]
        return {"bytes": n * (case["steps"] * cell + out), "flops": n * case["steps"] * 1000.0}
    if kind == "sweep":
        n = sum(pb.ncells for pb in _sweep_problems(case, 0))
        cell = 2 * (27 * VALUE_BYTES[case["storage"]] + 20)
        return {"bytes": n * (case["steps"] * cell + 0.25), "flops": n * case["steps"] * 1000.0}
    nv = case["n"] * case["d"] * case["h"] * case["w"]
    if kind in ("predict", "train"):
        f = _layer_flops(nv)
        if kind == "predict":
            return {"bytes": nv * 16.0 * 2, "flops": sum(f.values())}
        # the first layer has no data gradient
        return {"bytes": nv * 16.0 * 2, "flops": 3 * sum(f.values()) - f["e1a"]}
    cin, cout = case["cin"], case["cout"]
    one, back = 54.0 * nv * cin * cout, cin % 32 == 0
    values = nv * ((2 * cin if back else cin) + 2 * cout) + 27 * cin * cout * 2
    return {"bytes": 2.0 * values + 4.0 * 27 * cin * cout, "flops": one * (3 if back else 2)}


# ---------------------------------------------------------------- FP64 references in plain torch

_V = np.array([(x, y, z) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1)])
_SHELL = (_V ** 2).sum(1)
_WT = np.array([8 / 27, 2 / 27, 1 / 54, 1 / 216])[_SHELL]
_BI = np.array([-10 / 27, 2 / 27, 1 / 54, 1 / 216])[_SHELL]
_QI = np.array([0.0, 2 / 19, 1 / 38, 1 / 152])[_SHELL]
_INDEX = {tuple(v): i for i, v in enumerate(_V)}


def _moments():
    """The orthogonal moment set of the method, each row with its relaxation rate (None: the
    local shear rate): tensor products of 1, c and t = 3 c^2 - 2."""
    x, y, z = (_V[:, k].astype(float) for k in range(3))
    a, b, c = (3 * v * v - 2 for v in (x, y, z))
    rows = [(np.ones(27), 0.0), (x, 0.0), (y, 0.0), (z, 0.0), ((a + b + c) / 3, 1.5)]
    rows += [((2 * a - b - c) / 3, None), ((b - c) / 3, None), (x * y, None), (y * z, None), (x * z, None)]
    rows += [(x * (b + c), 1.5), (y * (a + c), 1.5), (z * (a + b), 1.5)]
    rows += [(x * b * c, 1.83), (y * a * c, 1.83), (z * a * b, 1.83)]
    rows += [((a * b + a * c + b * c) / 3, 1.4), (a * b * c, 1.61)]
    rows += [((a * b + a * c - 2 * b * c) / 3, 1.98), ((a * b - a * c) / 3, 1.98)]
    rows += [(x * y * c, 1.98), (y * z * a, 1.98), (x * z * b, 1.98)]
    rows += [(x * (b - c), 1.74), (y * (c - a), 1.74), (z * (a - b), 1.74), (x * y * z, 1.74)]
    return np.stack([r for r, _ in rows]), [s for _, s in rows]


class _Exact:
    """The method of the paper in FP64 with dense moment matrices, two colours of 27 populations."""

    def __init__(self, pb, A, rr, rb, u):
        self.pb, self.A = pb, A
        t = lambda v: torch.tensor(v, device="cuda", dtype=torch.float64)  # noqa: E731
        self.w, self.B, self.q, self.c = t(_WT), t(_BI), t(_QI), t(_V.astype(float))
        M, self.rates = _moments()
        self.M, self.Mi = t(M), t(np.linalg.inv(M))
        self.ab = 8 / 27
        self.ar = 1 - (1 - self.ab) * pb.rho_b0 / pb.rho_r0
        self.step_no = 0
        if pb.inflow:
            y, x = np.mgrid[0:pb.ny, 0:pb.nx]
            self.sites = np.flatnonzero((x - pb.xc) ** 2 + (y - pb.yc) ** 2 < 0.25 * pb.diameter ** 2)
            self.at = torch.tensor(self.sites, device="cuda")
        self.f = [self.colour(rr, self.ar, u), self.colour(rb, self.ab, u)]
        if pb.inflow:
            self.hold_inflow()
        self.outlet = [f[:, -1].clone() for f in self.f]

    def phi_i(self, alpha):
        return (1 - alpha) * self.q + alpha * (self.q == 0).double()

    def colour(self, rho, alpha, u):
        cu = torch.tensordot(self.c, u, 1)
        shape = (27,) + (1,) * rho.dim()
        return rho * (self.phi_i(alpha).view(shape) +
                      self.w.view(shape) * (3 * cu + 4.5 * cu * cu - 1.5 * (u * u).sum(0)))

    def inflow_speed(self):
        pb = self.pb
        xi = W.splitmix64_uniform(pb.seed, self.step_no * pb.ncells + self.sites) if pb.noise_rel else 0 * self.sites
        return torch.tensor(pb.u_in * (1 + pb.noise_rel * xi), device="cuda", dtype=torch.float64)

    def hold_inflow(self):
        v = self.inflow_speed()
        u = torch.stack([torch.zeros_like(v), torch.zeros_like(v), v])
        self.f[0][:, 0] = self.f[0][:, 0].reshape(27, -1).index_copy(
            1, self.at, self.colour(torch.full_like(v, self.pb.rho_r0), self.ar, u)).view_as(self.f[0][:, 0])
        self.f[1][:, 0] = self.f[1][:, 0].reshape(27, -1).index_fill(1, self.at, 0.0).view_as(self.f[1][:, 0])

    def index(self, axis, c):
        """Source index along an axis for velocity component c, and where a wall is crossed."""
        n = (self.pb.nz, self.pb.ny, self.pb.nx)[axis]
        faces = self.pb.faces[2 * (2 - axis):2 * (2 - axis) + 2]
        s = np.arange(n) - c
        face = faces[0] if c > 0 else faces[1]
        wall = face != W.PERIODIC and c != 0
        edge = (0 if c > 0 else n - 1) if wall else None
        return torch.tensor(np.clip(s, 0, n - 1) if wall else s % n, device="cuda"), edge, face

    def gradient(self, fld):
        g = [torch.zeros_like(fld) for _ in range(3)]
        for v, wt in zip(_V, _WT):
            s = fld
            for axis, c in zip((0, 1, 2), (v[2], v[1], v[0])):
                if c:
                    s = s.index_select(axis, self.index(axis, -c)[0])
            for d in range(3):
                if v[d]:
                    g[d] += 3 * wt * v[d] * s
        return torch.stack(g)

    def macro(self):
        rr, rb = self.f[0].sum(0), self.f[1].sum(0)
        j = torch.tensordot(self.c.T, self.f[0] + self.f[1], 1)
        rho = rr + rb
        F = torch.zeros_like(j)
        if self.pb.force_model:
            for d in range(3):
                F[d] = (rho - self.pb.rho_ref) * self.pb.g[d]
        return rr, rb, rho, (j + 0.5 * F) / rho, F

    def step(self):
        pb = self.pb
        rr, rb, rho, u, F = self.macro()
        phi = (rr - rb) / rho
        gp, gr = self.gradient(phi), self.gradient(rho)
        a = rr / rho
        nu = a * pb.nu_r + (1 - a) * pb.nu_b
        shp = (27, 1, 1, 1)
        cu = torch.tensordot(self.c, u, 1)
        f = self.f[0] + self.f[1]
        # equilibrium with the velocity-gradient correction, and the forcing, in velocity space
        ug = (u * gr).sum(0)
        cg = torch.tensordot(self.c, gr, 1)
        coef = torch.tensor(np.array([0.0, 16.0, 4.0, 1.0])[_SHELL], device="cuda", dtype=torch.float64).view(shp)
        abar = a * self.ar + (1 - a) * self.ab
        feq = rho * ((1 - abar) * self.q.view(shp) + self.w.view(shp) * (3 * cu + 4.5 * cu * cu - 1.5 * (u * u).sum(0)))
        feq += coef * nu * 2 * cu * cg / 48
        feq[13] += rho * abar - 3 * nu * ug
        del cg
        m = torch.tensordot(self.M, f, 1)
        feq = torch.tensordot(self.M, feq, 1)
        Fp = None
        if pb.force_model:
            cF = torch.tensordot(self.c, F, 1)
            Fp = torch.tensordot(self.M, self.w.view(shp) * (3 * (cF - (u * F).sum(0)) + 9 * cu * cF), 1)
            del cF
        del cu
        snu = 1 / (3 * nu + 0.5)
        for j, s in enumerate(self.rates):
            s = snu if s is None else s
            m[j] -= s * (m[j] - feq[j])
            if Fp is not None:
                m[j] += (1 - 0.5 * s) * Fp[j]
        del feq, Fp
        f = torch.tensordot(self.Mi, m, 1)
        del m
        # perturbation and recolouring with the interface normal
        mag = torch.sqrt((gp * gp).sum(0))
        n = torch.where(mag > 1e-12, gp / mag.clamp(min=1e-300), torch.zeros_like(gp))
        mag = torch.where(mag > 1e-12, mag, torch.zeros_like(mag))
        cn = torch.tensordot(self.c, n, 1)
        f += self.A * mag * (self.w.view(shp) * cn * cn - self.B.view(shp))
        length = torch.tensor(np.sqrt(np.maximum(_SHELL, 1)), device="cuda", dtype=torch.float64).view(shp)
        seg = pb.beta * rr * rb / rho * (1 - abar) * self.q.view(shp) * cn / length
        del cn
        post = [a * f + seg, (1 - a) * f - seg]
        del f, seg
        if pb.inflow:  # the disk is not collided: it emits what it holds
            for k in range(2):
                held = self.f[k][:, 0].reshape(27, -1).index_select(1, self.at)
                post[k][:, 0] = post[k][:, 0].reshape(27, -1).index_copy(1, self.at, held).view_as(post[k][:, 0])
        self.f = [self.stream(p) for p in post]
        del post
        self.step_no += 1
        if pb.faces[5] == W.OUTFLOW:
            below = [x[:, -2] for x in self.f]
            r = below[0].sum(0) + below[1].sum(0)
            jz = torch.tensordot(self.c[:, 2], below[0] + below[1], 1)
            Fz = (r - pb.rho_ref) * pb.g[2] if pb.force_model else 0.0
            lam = ((jz + 0.5 * Fz) / r).clamp(min=0.0)
            for k in range(2):
                self.outlet[k] = (self.outlet[k] + lam * below[k]) / (1 + lam)
                self.f[k][:, -1] = self.outlet[k]
        if pb.inflow:
            self.hold_inflow()

    def stream(self, post):
        out = torch.empty_like(post)
        for i, v in enumerate(_V):
            c = (int(v[2]), int(v[1]), int(v[0]))  # by axis
            idx, edge, face = zip(*(self.index(a, c[a]) for a in range(3)))
            slip = [a for a in range(3) if edge[a] is not None and face[a] == W.FREESLIP]
            for bits in range(1 << len(slip)):
                cut = [a for k, a in enumerate(slip) if bits >> k & 1]
                d = [(-c[a] if a in cut else c[a]) for a in range(3)]
                src, dst = post[_INDEX[(d[2], d[1], d[0])]], out[i]
                for a in range(3):
                    if a in cut:
                        src, dst = src.narrow(a, edge[a], 1), dst.narrow(a, edge[a], 1)
                    elif c[a]:
                        src = src.index_select(a, idx[a])
                dst.copy_(src)
            if edge[0] is not None and face[0] != W.FREESLIP:  # bounce-back on a z face
                out[i][edge[0]] = post[_INDEX[(-int(v[0]), -int(v[1]), -int(v[2]))]][edge[0]]
        return out

    def state(self, u_scale):
        rr, rb, rho, u, _ = self.macro()
        phi = (rr - rb) / rho
        if self.pb.inflow:
            v = self.inflow_speed()
            phi[0].view(-1)[self.at] = 1.0
            for d in range(3):
                u[d, 0].view(-1)[self.at] = v if d == 2 else 0.0
        return torch.cat([phi.unsqueeze(-1), (u / u_scale).permute(1, 2, 3, 0)], dim=-1)


def _exact_lattice(pb, u_scale, fields, steps):
    A = pb.A if pb.A is not None else 9 * pb.sigma / (4 * (3 * pb.nu_b + 0.5))
    e = _Exact(pb, A, *fields)
    for _ in range(steps):
        e.step()
    return e, e.state(u_scale)


def _conv64(x, wt, b=None):
    """x (n, d, h, w, cin), wt (27, cout, cin), zero padding, FP64."""
    n, d, h, w, _ = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    y = 0 if b is None else b
    for k in range(27):
        dz, dy, dx = k // 9, k // 3 % 3, k % 3
        y = y + p[:, dz:dz + d, dy:dy + h, dx:dx + w] @ wt[k].T
    return y


def _net64(x, P):
    """The encoder-decoder on x (n, d, h, w, 4): the change of the four fields."""
    def pool(t):
        n, d, h, w, c = t.shape
        return t.view(n, d // 2, 2, h // 2, 2, w // 2, 2, c).mean(dim=(2, 4, 6))

    def up(t):
        return t.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)

    conv = lambda t, k: _conv64(t, *P[k])  # noqa: E731
    x = torch.nn.functional.pad(x, (0, 4))
    e1 = torch.relu(conv(torch.relu(conv(x, "e1a")), "e1b"))
    e2 = torch.relu(conv(pool(e1), "e2"))
    bt = torch.relu(conv(pool(e2), "bt"))
    d2 = torch.relu(conv(up(bt) + e2, "d2"))
    return conv(torch.relu(conv(up(d2) + e1, "d1")), "out")[..., :4]


def exact(case, seed):
    kind = case["kind"]
    if kind == "steps":
        if case["nx"] * case["ny"] * case["nz"] * case["steps"] > 150e6:
            return None
        pb, u_scale = _flow(case)
        pb.seed = int(seed)
        e, st = _exact_lattice(pb, u_scale, _fields(case, pb, seed), case["steps"])
        if case["read"] == "state":
            return st
        if case["read"] == "phi":
            return st[..., 0].contiguous()
        q = _diag_query(case)
        rr, rb, _, u, _ = e.macro()
        z, y, x = torch.meshgrid(*(torch.arange(k, device="cuda", dtype=torch.float64) for k in rr.shape), indexing="ij")
        r = torch.sqrt((x - q["center"][0]) ** 2 + (y - q["center"][1]) ** 2 + (z - q["center"][2]) ** 2)
        p = rr * 9 * (1 - e.ar) / 19 + rb * 9 * (1 - e.ab) / 19
        s = lambda v: float(v)  # noqa: E731
        return {"mass_r": s(rr.sum()), "mass_b": s(rb.sum()), "umax": s(torch.sqrt((u * u).sum(0)).max()),
                "p_in": s(p[r <= q["r_in"]].mean()), "p_out": s(p[r >= q["r_out"]].mean()),
                "n_in": int((r <= q["r_in"]).sum()), "n_out": int((r >= q["r_out"]).sum()), "nan_cells": 0}
    if kind == "sweep":
        pbs = _sweep_problems(case, seed)
        if sum(pb.ncells for pb in pbs) * case["steps"] > 150e6:
            return None
        res = []
        for k, pb in enumerate(pbs):
            st = _exact_lattice(pb, pbs[0].u_in, _fields(dict(flow="jet"), pb, 100 * seed + k), case["steps"])[1]
            d, h, w = S.coarse_extent(pb)
            res.append(st.view(d, 4, h, 4, w, 4, 4).mean(dim=(1, 3, 5)))
        return res
    if kind in ("predict", "train"):
        net = S.Network(case["n"], case["d"], case["h"], case["w"], seed=int(seed) % 100003)  # its initial weights
        P = {k: [torch.from_numpy(v).cuda().double().requires_grad_(kind == "train") for v in wb]
             for k, wb in net.get_params().items()}
        lr = net.lr
        del net
        x = _coarse_fields(case, seed).double()
        if kind == "predict":
            return x + _net64(x, P)
        target = _coarse_fields(case, seed + 1).double() - x
        ((_net64(x, P) - target) ** 2).mean().backward()
        adam = lambda p: (p - lr * p.grad / (p.grad.abs() + 1e-8)).detach()  # noqa: E731
        return {"w": {k: adam(p[0]) for k, p in P.items()}, "g": {k: p[0].grad for k, p in P.items()},
                "gb": {k: p[1].grad for k, p in P.items()}}
    x, wt, b, dout = (t.double() for t in _conv_inputs(case, seed))
    res = {"out": torch.relu(_conv64(x, wt, b)), "db": dout.sum(dim=(0, 1, 2, 3))}
    n, d, h, w, cin = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    g = dout.reshape(-1, case["cout"]).T
    res["dw"] = torch.stack([g @ p[:, k // 9:k // 9 + d, k // 3 % 3:k // 3 % 3 + h, k % 3:k % 3 + w].reshape(-1, cin)
                             for k in range(27)])
    if cin % 32 == 0:
        res["din"] = torch.where(x > 0, _conv64(dout, wt.flip(0).transpose(1, 2)), 0.0)
    return res
