"""The work that this library's performance is measured on.

Every case is one pass through the public entry points as a program that uses
the library makes them, in one of seven kinds:

  run        a box from its initial fields: init, time steps, then the moments
             (FP64 storage) or the checkpoint state (FP32 storage)
  ensemble   a batch of boxes of different sizes restarted from checkpoints,
             advanced by captured graphs, and checkpointed again
  snapshot   the statistics and the fields of a state, as a run writes them
             every so many steps
  pair       one training pair of the corrector: the box-filtered fine fields
             and the coarse fields as network planes, then the coarse state set
             to the filtered fields
  forward    the corrector network's forward pass alone
  train      one mini-batch of the corrector's training: weights in, forward,
             loss and backward per sample, Adam step, gradients out
  corrected  a coarse run with the corrector applied every four steps

Inputs are made on the GPU from the seed alone: a shock tube, a standing shock
with a vortex, and solenoidal random velocity of a given turbulent Mach number,
as in this repository's tests and benchmark.
"""
import math

import numpy as np
import torch

from paper_2102_09512_amd import lbm

GAMMA = 1.4
FP64, FP32 = "fp64", "fp32"


# ---- the cases ----------------------------------------------------------------

def _run_case(flow, dims, precision, steps, zero_grad="", deriv="upwind", visc_exp=0.0, caloric=False):
    return {"kind": "run", "flow": flow, "nx": dims[0], "ny": dims[1], "nz": dims[2] if len(dims) > 2 else 0,
            "precision": precision, "steps": steps, "zero_grad": zero_grad, "deriv": deriv, "visc_exp": visc_exp,
            "caloric": caloric}


def listed():
    return [
        # the smallest box anyone runs, the paper's shock tube: launches and latency are all there is
        {"name": "sod_800x4_fp64", **_run_case("sod", (800, 4), FP64, 200, zero_grad="x")},
        # the two-dimensional benchmark box
        {"name": "shock_vortex_1024_fp32", **_run_case("shock_vortex", (1024, 1024), FP32, 40, zero_grad="x")},
        # the corrector's coarse grid, and the first of the paper's turbulence grids
        {"name": "turbulence_64_fp32", **_run_case("turbulence", (64, 64, 64), FP32, 32, visc_exp=0.76)},
        # the headline grid
        {"name": "turbulence_256_fp32", **_run_case("turbulence", (256, 256, 256), FP32, 10, visc_exp=0.76)},
        # double precision on a box of no round size, with the other difference scheme and an open axis
        {"name": "channel_190x131x110_fp64", **_run_case("turbulence", (190, 131, 110), FP64, 10, zero_grad="z",
                                                         deriv="central", visc_exp=0.76)},
        # a parameter study: 64 independent boxes of 64 to 512 nodes a side
        {"name": "ensemble_64_fp32", "kind": "ensemble", "count": 64, "smallest": 64, "largest": 512,
         "precision": FP32, "steps": 50, "graph_steps": 50},
        # statistics and fields of the headline grid
        {"name": "snapshot_256_fp32", "kind": "snapshot", "nx": 256, "ny": 256, "nz": 256, "precision": FP32,
         "noalloc": False},
        # a watch on a two-dimensional run from code that may not allocate
        {"name": "watch_1000x700_fp64", "kind": "snapshot", "nx": 1000, "ny": 700, "nz": 0, "precision": FP64,
         "noalloc": True},
        # the corrector's data generation
        {"name": "pair_256_to_64", "kind": "pair", "nx": 64, "ny": 64, "nz": 64, "factor": 4},
        # the network at a larger grid than it was trained on
        {"name": "forward_128x96x64", "kind": "forward", "nx": 128, "ny": 96, "nz": 64, "hidden": 3, "outputs": 3},
        # the corrector's training
        {"name": "train_64_batch4", "kind": "train", "nx": 64, "ny": 64, "nz": 64, "hidden": 3, "outputs": 3,
         "batch": 4},
        # the corrector at work
        {"name": "corrected_64", "kind": "corrected", "nx": 64, "ny": 64, "nz": 64, "hidden": 3, "outputs": 3,
         "windows": 4},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "run", "ensemble", "snapshot", "pair", "forward", "train", "corrected"])
    precision = rng.choice([FP64, FP32])
    if kind in ("run", "snapshot"):
        three = rng.random() < 0.5
        if three:
            dims = [_log_uniform(rng, 12, 220) for _ in range(3)]
            while math.prod(dims) > 160 ** 3:
                dims[dims.index(max(dims))] //= 2
        else:
            dims = [_log_uniform(rng, 32, 2200), _log_uniform(rng, 4, 1600)]
    if kind == "run":
        flow = "turbulence" if three else rng.choice(["sod", "shock_vortex", "turbulence"])
        if flow == "shock_vortex":  # the vortex has to fit
            dims = [max(d, 96) for d in dims]
        axes = "xyz" if three else "xy"
        zero_grad = "x" if flow != "turbulence" else "".join(a for a in axes if rng.random() < 0.25)
        steps = max(3, min(150, int(2e9 / (math.prod(dims) * 3 ** len(dims) * 16)), _log_uniform(rng, 4, 150)))
        return _run_case(flow, dims, precision, steps, zero_grad, rng.choice(["upwind", "upwind", "central"]),
                         0.76 if flow == "turbulence" else 0.0, rng.random() < 0.15)
    if kind == "ensemble":
        lo = rng.randrange(32, 129)
        return {"kind": kind, "count": _log_uniform(rng, 3, 48), "smallest": lo, "largest": lo + rng.randrange(32, 300),
                "precision": precision, "steps": rng.randrange(10, 50), "graph_steps": rng.choice([0, 10, 25])}
    if kind == "snapshot":
        return {"kind": kind, "nx": dims[0], "ny": dims[1], "nz": dims[2] if three else 0, "precision": precision,
                "noalloc": rng.random() < 0.3}
    grid = {"nx": 32 * rng.randrange(1, 4), "ny": 4 * rng.randrange(2, 22), "nz": 4 * rng.randrange(2, 22)}
    if kind == "pair":
        return {"kind": kind, **grid, "factor": rng.choice([2, 3])}
    net = {"kind": kind, **grid, "hidden": rng.choice([1, 2, 3, 4]), "outputs": rng.choice([3, 3, 5])}
    if kind == "train":
        return {**net, "batch": rng.randrange(1, 5)}
    if kind == "corrected":
        return {**net, "windows": rng.randrange(1, 5)}
    return net


# ---- inputs -------------------------------------------------------------------

def _lattice(case):
    return 3 if case["nz"] else 2


def _dims(case):
    return (case["nx"], case["ny"], case["nz"]) if case["nz"] else (case["nx"], case["ny"])


def _dev(*a, **k):
    return torch.tensor(*a, dtype=torch.float64, device="cuda", **k)


def _turbulence(dims, seed, Ma=0.3, T0=0.15, mean=0.0, wobble=0.0, waves=24):
    """rho, u, T of `waves` random solenoidal waves of up to six periods a
    side, scaled to sqrt(<u.u>) = Ma sqrt(gamma T0), plus a mean velocity;
    wobble: relative amplitude of one wave in rho and T."""
    D = len(dims)
    rng = np.random.default_rng(seed)
    shape = tuple(reversed(tuple(dims) + (1,) * (3 - D)))
    u = torch.zeros((D,) + shape, dtype=torch.float64, device="cuda")

    def phase(k):
        p = _dev(rng.uniform(0, 2 * math.pi)).reshape(1, 1, 1)
        for a in range(D):
            axis = torch.arange(dims[a], dtype=torch.float64, device="cuda") * (2 * math.pi * float(k[a]) / dims[a])
            p = p + axis.reshape((1,) * (2 - a) + (dims[a],) + (1,) * a)
        return p

    for _ in range(waves):
        k = rng.integers(-6, 7, D)
        while not 2 <= math.sqrt((k * k).sum()) <= 6.5:
            k = rng.integers(-6, 7, D)
        kp = k / np.asarray(dims)
        a = rng.standard_normal(D)
        a -= kp * (a @ kp) / (kp @ kp)
        wave = torch.cos(phase(k))
        for c in range(D):
            u[c] += float(a[c]) * wave
    u *= Ma * math.sqrt(GAMMA * T0) / u.square().sum(0).mean().sqrt()
    for c in range(D):
        u[c] += mean * (1.0, -0.8, 0.6)[c]
    w1, w2 = torch.cos(phase(np.ones(D))), torch.cos(phase(np.ones(D)))
    rho = (1.0 + wobble * w1).expand(shape).contiguous()
    T = (T0 * (1.0 + wobble * w2)).expand(shape).contiguous()
    return rho, u, T


def _sod(nx, ny, seed):
    r = np.random.default_rng(seed)
    shape = (1, ny, nx)
    left = (torch.arange(nx, device="cuda") < nx // 2).expand(shape)
    T_l = 0.15 * float(r.uniform(0.97, 1.03))
    rho = torch.where(left, _dev(1.0), _dev(0.125)).contiguous()
    p = torch.where(left, _dev(T_l), _dev(0.1 * T_l))
    return rho, torch.zeros((2,) + shape, dtype=torch.float64, device="cuda"), (p / rho).contiguous()


def _free_stream(T_l=0.05, Ma=1.2):
    return Ma * math.sqrt(GAMMA * T_l)


def _shock_vortex(nx, ny, seed, T_l=0.05, Ma=1.2, Ma_v=0.25):
    r = np.random.default_rng(seed)
    r_v, x_s = max(8.0, nx / 32), nx // 2
    x_v, y_v = x_s - r_v * float(r.uniform(1.8, 2.2)), ny * float(r.uniform(0.45, 0.55))
    u1 = _free_stream(T_l, Ma)
    ratio = (GAMMA + 1) * Ma * Ma / ((GAMMA - 1) * Ma * Ma + 2)
    p_ratio = 1 + 2 * GAMMA / (GAMMA + 1) * (Ma * Ma - 1)
    x = torch.arange(nx, dtype=torch.float64, device="cuda")[None, None, :]
    y = torch.arange(ny, dtype=torch.float64, device="cuda")[None, :, None]
    up = (x < x_s).expand(1, ny, nx)
    rho = torch.where(up, _dev(1.0), _dev(ratio))
    p = torch.where(up, _dev(T_l), _dev(T_l * p_ratio))
    r2 = ((x - x_v) ** 2 + (y - y_v) ** 2) / r_v ** 2
    b = 1 - 0.5 * (GAMMA - 1) * Ma_v ** 2 * torch.exp(1 - r2)
    rho, p = rho * b ** (1 / (GAMMA - 1)), p * b ** (GAMMA / (GAMMA - 1))
    a = math.sqrt(GAMMA * T_l) * Ma_v * torch.exp(0.5 * (1 - r2)) / r_v
    u = torch.stack([torch.where(up, _dev(u1), _dev(u1 / ratio)) + a * (y - y_v), -a * (x - x_v)])
    return rho.contiguous(), u.contiguous(), (p / rho).contiguous()


def _viscosity(n, Ma, T0=0.15, Re=72.0):
    return Ma * math.sqrt(GAMMA * T0) / math.sqrt(3) * 2 / (4 * 2 * math.pi / n) / Re


class _Box:
    """The physics of one box and its initial fields."""

    def __init__(self, dims, precision, fields, *, mu, Pr, T_ref, rho_ref=1.0, u_ref=(0.0, 0.0, 0.0), zero_grad="",
                 deriv="upwind", visc_exp=0.0, caloric=False):
        self.D, self.dims, self.precision, self.fields = len(dims), tuple(dims), precision, fields
        self.mu, self.Pr, self.T_ref, self.rho_ref, self.u_ref = mu, Pr, T_ref, rho_ref, tuple(u_ref)
        self.clamp = tuple(a in zero_grad for a in "xyz")
        self.deriv, self.visc_exp = deriv, visc_exp
        self.cv = (2.5, 0.4, 0.2) if caloric else None  # C_v(T) rising with T

    def handle(self):
        h = lbm.lbm_create(self.D, self.dims, GAMMA, self.Pr, self.mu,
                           precision=lbm.LBM_FP32_DEV if self.precision == FP32 else lbm.LBM_FP64,
                           bc=[int(c) for c in self.clamp], visc_exponent=self.visc_exp, T_ref=self.T_ref,
                           rho_ref=self.rho_ref, u_ref=self.u_ref, cv_poly=self.cv,
                           deriv_scheme=lbm.LBM_DERIV_CENTRAL if self.deriv == "central" else lbm.LBM_DERIV_UPWIND)
        lbm.lbm_set_stream(h, torch.cuda.current_stream())
        return h

    def state(self):
        """An empty checkpoint."""
        return torch.empty((2 * 3 ** self.D, math.prod(self.dims)), device="cuda",
                           dtype=torch.float32 if self.precision == FP32 else torch.float64)

    def moments(self):
        return [torch.empty_like(f) for f in self.fields]


def _turbulent_box(dims, seed, precision=FP32, Ma=0.3, mean=0.0, wobble=0.0, visc_exp=0.76, **kw):
    return _Box(dims, precision, _turbulence(dims, seed, Ma, mean=mean, wobble=wobble), mu=_viscosity(min(dims), Ma)
                if min(dims) >= 24 else 0.01, Pr=0.7, T_ref=0.15, visc_exp=visc_exp, **kw)


def _run_box(case, seed):
    dims = _dims(case)
    kw = dict(zero_grad=case["zero_grad"], deriv=case["deriv"], visc_exp=case["visc_exp"], caloric=case["caloric"])
    if case["flow"] == "sod":
        return _Box(dims, case["precision"], _sod(*dims, seed), mu=0.015, Pr=0.71, T_ref=0.12, rho_ref=0.125, **kw)
    if case["flow"] == "shock_vortex":
        return _Box(dims, case["precision"], _shock_vortex(*dims, seed), mu=0.0198, Pr=0.75, T_ref=0.05,
                    u_ref=(_free_stream(), 0.0), **kw)
    return _turbulent_box(dims, seed, case["precision"], **kw)


def _snapshot_box(case, seed):
    return _turbulent_box(_dims(case), seed, case["precision"], mean=0.05, wobble=0.02)


def _ensemble_boxes(case, seed):
    sizes = np.random.default_rng(case["count"]).integers(case["smallest"], case["largest"] + 1, (case["count"], 2))
    return [_turbulent_box((int(nx), int(ny)), seed * 1000 + k, case["precision"], Ma=0.1 + 0.2 * k / case["count"])
            for k, (nx, ny) in enumerate(sizes)]


class _Net:
    """Weights, scaling and samples of a corrector network."""

    def __init__(self, case, seed):
        self.grid = (case["nx"], case["ny"], case["nz"])
        self.ch = [5] + [32] * case["hidden"] + [case["outputs"]]
        self.offset = 1 if case["outputs"] == 3 else 0
        r = np.random.default_rng(seed)
        p = []
        for l, (i, o) in enumerate(zip(self.ch, self.ch[1:])):
            p += [r.normal(0, (0.5 if l + 2 == len(self.ch) else 1.0) * math.sqrt(2 / (27 * i)), 27 * i * o),
                  r.normal(0, 0.02, o)]
        self.params = torch.tensor(np.concatenate(p).astype(np.float32), device="cuda")
        u = 0.3 * math.sqrt(GAMMA * 0.15 / 3)
        self.mean, self.std = np.array([1, 0, 0, 0, 0.15]), np.array([0.02, u, u, u, 0.003])
        self.out_std = 0.02 * self.std[self.offset: self.offset + case["outputs"]]

    def handle(self):
        n = lbm.lbm_nn_create(self.ch, self.grid)
        lbm.lbm_nn_set_stream(n, torch.cuda.current_stream())
        lbm.lbm_nn_set_params(n, self.params)
        lbm.lbm_nn_set_scaling(n, self.mean, self.std, self.out_std)
        lbm.lbm_nn_set_output_offset(n, self.offset)
        lbm.lbm_nn_set_correction_limit(n, 2.0)
        return n

    def sample(self, seed, noise=0.0):
        """Planes of a turbulent field, and with noise of a nearby one."""
        planes = torch.cat([f.reshape(-1, math.prod(self.grid))
                            for f in _turbulence(self.grid, seed, wobble=0.02)]).float()
        if not noise:
            return planes
        other = torch.cat([f.reshape(-1, math.prod(self.grid)) for f in _turbulence(self.grid, seed + 7, wobble=0.02)])
        return planes, (planes + noise * (other - planes.double())).float()


# ---- a pass -------------------------------------------------------------------

class _State(dict):
    """What a program holds; it gives the library's handles back when it goes."""

    def __del__(self):
        for destroy, handles in ((lbm.lbm_batch_destroy, "batches"), (lbm.lbm_nn_destroy, "nets"),
                                 (lbm.lbm_destroy, "handles")):
            for h in self.get(handles, ()):
                destroy(h)


def prepare(case, seed):
    s = _State(case=dict(case))
    kind = case["kind"]
    if kind == "run":
        box = _run_box(case, seed)
        s.update(handles=[box.handle()], fields=box.fields,
                 out=box.state() if case["precision"] == FP32 else box.moments())
    elif kind == "snapshot":
        box = _snapshot_box(case, seed)
        s.update(handles=[box.handle()], out=box.moments())
        lbm.lbm_init_fields(s["handles"][0], *box.fields)
    elif kind == "ensemble":
        boxes = _ensemble_boxes(case, seed)
        sizes = [b.state().numel() for b in boxes]
        flat = torch.empty(sum(sizes), dtype=boxes[0].state().dtype, device="cuda")
        s.update(handles=[b.handle() for b in boxes], start=flat.split(sizes), out=torch.empty_like(flat))
        s["parts"] = s["out"].split(sizes)
        for h, b, part in zip(s["handles"], boxes, s["start"]):
            lbm.lbm_init_fields(h, *b.fields)
            lbm.lbm_get_state(h, part)
        s["batches"] = [lbm.lbm_batch_create(s["handles"])]
    elif kind == "pair":
        coarse, fine = _pair_boxes(case, seed)
        s.update(handles=[coarse.handle(), fine.handle()], coarse=coarse.moments(), filtered=coarse.moments(),
                 x=torch.empty((5, math.prod(coarse.dims)), dtype=torch.float32, device="cuda"), out=coarse.state())
        s["t"] = torch.empty_like(s["x"])
        for h, b in zip(s["handles"], (coarse, fine)):
            lbm.lbm_init_fields(h, *b.fields)
    elif kind == "forward":
        net = _Net(case, seed)
        s.update(nets=[net.handle()], x=net.sample(seed))
        s["out"] = torch.empty((case["outputs"], s["x"].shape[1]), dtype=torch.float32, device="cuda")
    elif kind == "train":
        net = _Net(case, seed)
        s.update(nets=[net.handle()], params=net.params, step=0,
                 samples=[net.sample(seed * 100 + k, 0.01) for k in range(case["batch"])])
    else:
        net, box = _Net(case, seed), _corrected_box(case, seed)
        s.update(nets=[net.handle()], handles=[box.handle()], fields=box.fields, out=box.state())
    return s


def _pair_boxes(case, seed):
    f = case["factor"]
    return (_turbulent_box(_dims(case), seed + 1, wobble=0.02),
            _turbulent_box(tuple(f * n for n in _dims(case)), seed, wobble=0.02))


def _corrected_box(case, seed):
    return _turbulent_box(_dims(case), seed, wobble=0.02)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "run":
        h = s["handles"][0]
        lbm.lbm_init_fields(h, *s["fields"])
        lbm.lbm_step(h, case["steps"])
        if case["precision"] == FP32:
            lbm.lbm_get_state(h, s["out"])
        else:
            lbm.lbm_moments(h, *s["out"])
        return s["out"]
    if kind == "snapshot":
        h = s["handles"][0]
        d = (lbm.lbm_diagnostics_noalloc if case["noalloc"] else lbm.lbm_diagnostics)(h)
        if case["noalloc"]:
            return d
        lbm.lbm_moments(h, *s["out"])
        return [d, *s["out"]]
    if kind == "ensemble":
        for h, part in zip(s["handles"], s["start"]):
            lbm.lbm_set_state(h, part)
        lbm.lbm_batch_step(s["batches"][0], case["steps"], case["graph_steps"])
        for h, part in zip(s["handles"], s["parts"]):
            lbm.lbm_get_state(h, part)
        return s["out"]
    if kind == "pair":
        coarse, fine = s["handles"]
        lbm.lbm_filter_moments(fine, case["factor"], *s["filtered"])
        lbm.lbm_moments(coarse, *s["coarse"])
        stream = torch.cuda.current_stream()
        lbm.lbm_nn_fields_to_planes(3, *s["coarse"], s["x"], stream)
        lbm.lbm_nn_fields_to_planes(3, *s["filtered"], s["t"], stream)
        lbm.lbm_fields_set(coarse, *s["filtered"])
        lbm.lbm_get_state(coarse, s["out"])
        return [*s["filtered"], s["x"], s["t"], s["out"]]
    if kind == "forward":
        lbm.lbm_nn_forward(s["nets"][0], s["x"], s["out"])
        return s["out"]
    if kind == "train":
        n = s["nets"][0]
        s["step"] += 1
        lbm.lbm_nn_set_params(n, s["params"])  # the weights as a data-parallel trainer broadcasts them
        lbm.lbm_nn_zero_grad(n)
        for x, t in s["samples"]:
            lbm.lbm_nn_loss_backward(n, x, t, sync=False)
        lbm.lbm_nn_adam_step(n, 1e-3, grad_scale=1.0 / case["batch"], t=s["step"])
        total, count = lbm.lbm_nn_take_loss(n)
        return [np.float32(total / count), lbm.lbm_nn_get_grads(n)]
    n, h = s["nets"][0], s["handles"][0]
    lbm.lbm_init_fields(h, *s["fields"])
    for _ in range(case["windows"]):
        lbm.lbm_step(h, 4)
        lbm.lbm_nn_correct(n, h)
    lbm.lbm_get_state(h, s["out"])
    return s["out"]


# ---- what a pass cannot do without -----------------------------------------------

def _conv_flops(case):
    ch = [5] + [32] * case["hidden"] + [case["outputs"]]
    return [2 * 27 * i * o for i, o in zip(ch, ch[1:])]


def _node_flops(D):
    return 35 * 3 ** D  # sums, equilibria and relaxation of both populations


def work(case):
    kind = case["kind"]
    word = 8 if case.get("precision", FP32) == FP64 else 4
    if kind == "ensemble":
        sizes = np.random.default_rng(case["count"]).integers(case["smallest"], case["largest"] + 1, (case["count"], 2))
        N = int((sizes[:, 0] * sizes[:, 1]).sum())
        return {"bytes": N * 36 * word * (case["steps"] + 2), "flops": N * _node_flops(2) * case["steps"]}
    D, N = _lattice(case), math.prod(_dims(case))
    pops, fields = 2 * 3 ** D * word, 8 * (D + 2)
    if kind == "run":
        last = 2 * pops if case["precision"] == FP32 else pops + fields
        return {"bytes": N * (fields + pops + 2 * pops * case["steps"] + last), "flops": N * _node_flops(D) * case["steps"]}
    if kind == "snapshot":
        return {"bytes": N * (pops + (0 if case["noalloc"] else fields)), "flops": N * 8 * 3 ** D}
    if kind == "pair":
        fine = case["factor"] ** 3
        return {"bytes": N * (fine * pops + pops + fields + 2 * 20 + 2 * pops + 2 * pops), "flops": N * (fine + 1) * 8 * 27}
    flops = _conv_flops(case)
    planes = 4 * (5 + case["outputs"])
    if kind == "forward":
        return {"bytes": N * planes, "flops": N * sum(flops)}
    if kind == "train":  # per sample: forward, weight gradients, and data gradients of all layers but the first
        acts = 2 * 2 * 32 * case["hidden"]
        return {"bytes": case["batch"] * N * (40 + acts), "flops": case["batch"] * N * (3 * sum(flops) - flops[0])}
    steps = 4 * case["windows"]
    return {"bytes": N * (fields + pops + 2 * pops * steps + case["windows"] * 3 * pops + 2 * pops),
            "flops": N * (_node_flops(3) * steps + case["windows"] * sum(flops))}


# ---- the same in 64 bits, in plain torch ---------------------------------------------

def _velocities(D):
    return [(i % 3 - 1, i // 3 % 3 - 1, i // 9 % 3 - 1 if D == 3 else 0) for i in range(3 ** D)]


def _f32(x):
    return float(np.float32(x))


class _Exact:
    """The method on whole fields in 64 bits.  Populations f, g: [Q][nz][ny][nx]."""

    def __init__(self, box):
        self.b, self.c = box, _velocities(box.D)
        cv = box.cv or (1 / (GAMMA - 1), 0.0, 0.0)
        self.cv = tuple(_f32(v) for v in cv) if box.precision == FP32 and box.cv else cv
        self.f = self.g = None

    def _shift(self, a, axis, by):
        """a(x + by) along a space axis (0 x, 1 y, 2 z) of the last three, by the box's boundary rule."""
        if not by:
            return a
        n = a.shape[-1 - axis]
        k = torch.arange(n, device=a.device) + by
        k = k.clamp(0, n - 1) if self.b.clamp[axis] else k % n
        return a.index_select(a.dim() - 1 - axis, k)

    def U(self, T):
        c0, c1, c2 = self.cv
        return T * (c0 + T * (c1 / 2 + T * (c2 / 3)))

    def T_of(self, U):
        c0, c1, c2 = self.cv
        T = U / c0
        if c1 or c2:
            for _ in range(30):
                T = T - (self.U(T) - U) / (c0 + T * (c1 + T * c2))
        return T

    @staticmethod
    def _psi(u, P):
        return 0.5 * (P - u), 1 - P, 0.5 * (P + u)

    def feq(self, rho, u, T, d=None, corr=None):
        F = [self._psi(u[a], T + u[a] ** 2 + (corr * d[a] if d is not None else 0)) for a in range(self.b.D)]
        for c in self.c:
            v = rho
            for a in range(self.b.D):
                v = v * F[a][c[a] + 1]
            yield v

    def geq(self, rho, u, T):
        D = self.b.D
        A = [self._psi(u[a], T + u[a] ** 2) for a in range(D)]
        B = []
        for a in range(D):
            B1 = u[a] * (u[a] ** 2 + 2 * T) / 2
            B2 = (u[a] ** 4 + 5 * u[a] ** 2 * T + 2 * T * T) / 2
            B.append((0.5 * (B2 - B1), u[a] ** 2 / 2 - B2, 0.5 * (B2 + B1)))
        U = self.U(T)
        for c in self.c:
            v = U
            for a in range(D):
                v = v * A[a][c[a] + 1]
            for a in range(D):
                w = B[a][c[a] + 1]
                for e in range(D):
                    if e != a:
                        w = w * A[e][c[e] + 1]
                v = v + w
            yield rho * v

    def init(self, rho, u, T):
        self.f, self.g = torch.stack(list(self.feq(rho, u, T))), torch.stack(list(self.geq(rho, u, T)))

    def sums(self, f, g):
        D = self.b.D
        rho, E = f.sum(0), g.sum(0)
        j = [sum(c[a] * f[i] for i, c in enumerate(self.c) if c[a]) for a in range(D)]
        u = [x / rho for x in j]
        T = self.T_of(E / rho - 0.5 * sum(x * x for x in u))
        return rho, u, T

    def moments(self):
        rho, u, T = self.sums(self.f, self.g)
        return rho, torch.stack(u), T

    def step(self):
        b, D = self.b, self.b.D
        for p in (self.f, self.g):
            for i, c in enumerate(self.c):
                for a in range(D):
                    if c[a]:
                        p[i] = self._shift(p[i], a, -c[a])
        f, g = self.f, self.g
        rho, u, T = self.sums(f, g)
        nu = b.mu * (T / b.T_ref) ** b.visc_exp / (rho * T)
        om, om1 = 1 / (nu + 0.5), 1 / (nu / b.Pr + 0.5)
        d = []
        for a in range(D):
            q = rho * u[a] * (1 - 3 * T - u[a] ** 2)
            qm, qp = self._shift(q, a, -1), self._shift(q, a, 1)
            d.append(0.5 * (qp - qm) if b.deriv == "central" else torch.where(u[a] > 0, q - qm, qp - q))
        dq = []
        for a in range(D):
            v = 0.5 * u[a] * d[a]
            for e in range(D):
                P = sum(c[a] * c[e] * f[i] for i, c in enumerate(self.c) if c[a] * c[e])
                v = v + u[e] * (P - rho * u[a] * u[e] - (rho * T if a == e else 0))
            dq.append(v)
        for i, (c, fe, ge) in enumerate(zip(self.c, self.feq(rho, u, T, d, nu / rho), self.geq(rho, u, T))):
            f[i] += om * (fe - f[i])
            g[i] += om1 * (ge - g[i])
            if sum(abs(x) for x in c) == 1:
                a = next(k for k in range(D) if c[k])
                g[i] -= 0.5 * (om - om1) * c[a] * dq[a]

    def set_moments(self, rho, u, T):
        r0, u0, T0 = self.moments()
        for p, eq in ((self.f, self.feq), (self.g, self.geq)):
            for i, (new, old) in enumerate(zip(eq(rho, u, T), eq(r0, u0, T0))):
                p[i] += new - old

    def state(self):
        """The checkpoint: FP32 storage keeps the deviations from the reference state."""
        s = torch.cat([self.f, self.g]).reshape(2 * len(self.c), -1)
        if self.b.precision == FP32:
            rho, T = _dev(_f32(self.b.rho_ref)), _dev(_f32(self.b.T_ref))
            u = [_dev(_f32(v)) for v in self.b.u_ref]
            s -= torch.stack(list(self.feq(rho, u, T)) + list(self.geq(rho, u, T)))[:, None]
        return s


def _stack_planes(fields):
    return torch.cat([f.reshape(-1, fields[0].numel()) for f in fields])


def _forward(net, params, planes):
    """The network's outputs [c][V] in 64 bits; planes [5][V], params as one vector."""
    nx, ny, nz = net.grid
    a = ((planes.double() - _dev(net.mean)[:, None]) / _dev(net.std)[:, None]).t()
    at = 0
    for l, (i, o) in enumerate(zip(net.ch, net.ch[1:])):
        W = params[at: at + 27 * i * o].reshape(27, i, o)
        at += 27 * i * o
        field = a.reshape(nz, ny, nx, i)
        y = params[at: at + o].expand(a.shape[0], o)
        at += o
        for t in range(27):
            s = (t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1)
            y = y + torch.roll(field, (-s[0], -s[1], -s[2]), (0, 1, 2)).reshape(-1, i) @ W[t]
        a = torch.relu(y) if l + 2 < len(net.ch) else y
    return a.t()


def exact(case, seed):
    with torch.enable_grad() if case["kind"] == "train" else torch.no_grad():
        return _exact_of(case, seed)


def _exact_of(case, seed):
    kind = case["kind"]
    if kind == "run":
        e = _Exact(_run_box(case, seed))
        e.init(*e.b.fields)
        for _ in range(case["steps"]):
            e.step()
        return e.state() if case["precision"] == FP32 else list(e.moments())
    if kind == "ensemble":
        parts = []
        for b in _ensemble_boxes(case, seed):
            e = _Exact(b)
            e.init(*b.fields)
            for _ in range(case["steps"]):
                e.step()
            parts.append(e.state().reshape(-1))
        return torch.cat(parts)
    if kind == "snapshot":
        b = _snapshot_box(case, seed)
        d = _exact_statistics(b)
        return d if case["noalloc"] else [d, *b.fields]
    if kind == "pair":
        cb, fb = _pair_boxes(case, seed)
        k, (nx, ny, nz) = case["factor"], cb.dims

        def mean(a):
            return a.reshape(nz, k, ny, k, nx, k).mean((1, 3, 5))

        rho, u, T = fb.fields
        r = mean(rho)
        v = torch.stack([mean(rho * u[a]) / r for a in range(3)])
        t = mean(rho * (T / (GAMMA - 1) + 0.5 * u.square().sum(0))) / r
        t = (t - 0.5 * v.square().sum(0)) * (GAMMA - 1)
        e = _Exact(cb)
        e.init(*cb.fields)
        e.set_moments(r, v, t)
        return [r, v, t, _stack_planes(cb.fields), _stack_planes((r, v, t)), e.state()]
    if kind == "forward":
        net = _Net(case, seed)
        return _forward(net, net.params.double(), net.sample(seed))
    if kind == "train":
        net = _Net(case, seed)
        p = net.params.double().requires_grad_()
        total = 0.0
        for k in range(case["batch"]):
            x, t = net.sample(seed * 100 + k, 0.01)
            f = slice(net.offset, net.offset + case["outputs"])
            r = _forward(net, p, x) + (x - t)[f].double() / _dev(net.out_std)[:, None]
            loss = r.square().mean()
            loss.backward()
            total += float(loss.detach())
        return [_dev(total / case["batch"]), p.grad]
    net, box = _Net(case, seed), _corrected_box(case, seed)
    e = _Exact(box)
    e.init(*box.fields)
    for _ in range(case["windows"]):
        for _ in range(4):
            e.step()
        fields = _stack_planes(e.moments())
        y = _forward(net, net.params.double(), fields).clamp(-2.0, 2.0) * _dev(net.out_std)[:, None]
        fields[net.offset: net.offset + case["outputs"]] += y
        shape = box.fields[0].shape
        e.set_moments(fields[0].reshape(shape), fields[1:4].reshape((3,) + shape), fields[4].reshape(shape))
    return e.state()


def _exact_statistics(b):
    rho, u, T = b.fields
    e = _Exact(b)

    def diff(q, a):
        return 0.5 * (e._shift(q, a, 1) - e._shift(q, a, -1))

    D = b.D
    grad = [[diff(u[c], a) for a in range(D)] for c in range(D)]  # grad[c][a] = d_a u_c
    curl = [grad[1][0] - grad[0][1]]
    if D == 3:
        curl += [grad[2][1] - grad[1][2], grad[0][2] - grad[2][0]]
    vort2, uu = sum(w * w for w in curl), u.square().sum(0)

    def total(q):
        return float(q.sum())

    def axes(qs):
        return [total(q) for q in qs] + [0.0] * (3 - D)

    return {"step": None, "nodes": None, "nonfinite": None, "nonpositive": None,
            "mass": total(rho), "momentum": axes([rho * u[a] for a in range(D)]),
            "energy": total(rho * (e.U(T) + 0.5 * uu)), "kinetic_energy": total(0.5 * rho * uu),
            "dilatation_sq_sum": total(sum(grad[a][a] for a in range(D)).square()), "u2_sum": total(uu),
            "cs_sum": total((GAMMA * T).sqrt()), "rho2_sum": total(rho * rho), "vorticity_sq_sum": total(vort2),
            "dissipation_sum": total(b.mu * (T / b.T_ref) ** b.visc_exp * vort2),
            "u_axis_sq_sum": axes([u[a] ** 2 for a in range(D)]),
            "du_axis_sq_sum": axes([grad[a][a] ** 2 for a in range(D)])}
