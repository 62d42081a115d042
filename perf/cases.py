"""The work that users of this framework have it do, as cases that can be timed.

    listed()            the cases by name
    draw(rng)           one more case of the same ranges
    prepare(case, seed) what a program holds before the call: lattices set up and their launch chosen,
                        an ensemble, a trainer with its samples
    run(state)          one pass through the public entry points, and its outputs
    work(case)          the bytes and operations one pass cannot do without
    exact(case, seed)   the outputs in 64 bits, by plain torch

Kinds of case:
    lattice     one D2Q9 lattice advanced `steps` steps, then its moments read
    reflection  a test lattice and its 4x reference with the energy of their difference every few steps
    ensemble    many uneven lattices advanced by one graph launch, then every member's moments or, with
                `log_every`, the closure's training samples
    lattice3d   one D3Q19 or D3Q27 lattice
    train       one Adam step of the closure network on a minibatch
    dataset     a data round made ready: normalisation fitted, samples packed, the network evaluated on all
                of them, and the loss's gradients on a batch

`plan` says how a lattice's launch was chosen: "default" (nothing asked for), "tuned" (the library's
autotuners, or their cached choice for the sizes in tuning/tiles.json).
"""
import itertools
import math

import numpy as np
import torch

from paper_2005_08674_amd import autotune, closure, lbm
from paper_2005_08674_amd import workloads as W
from paper_2005_08674_amd.ensemble import Ensemble, member_params
from paper_2005_08674_amd.lattice import Lattice
from paper_2005_08674_amd.lattice3d import Lattice3D
from paper_2005_08674_amd.reflection import ReflectionRun

DEV = "cuda"
EDGES = {"nsbc": (1, 1, 1, 1), "channel": (1, 1, 0, 0), "inlet": (2, 1, 0, 0), "periodic": (0, 0, 0, 0)}
FACES = {"nsbc": (1,) * 6, "channel": (1, 1, 0, 0, 0, 0), "periodic": (0,) * 6}
ESIZE = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
REPS = 3           # timed runs per candidate when a launch is tuned
LR = 2e-3          # the trainer's starting learning rate
GAMMA = 0.6
MAX_BATCH = 65536  # the trainer's largest batch


def listed():
    return [
        # the paper's 128^2 acoustic test at parity precision, a few steps between looks at the field:
        # the smallest call, nearly all launches
        {"name": "pulse128_f64", "kind": "lattice", "nx": 128, "ny": 128, "store": "f64", "edges": "nsbc",
         "flow": "pulse", "coll": "bgk", "tau": 0.6, "steps": 10, "plan": "default", "closure": False},
        # its reflection measurement: a 512^2 reference beside it, the fp64 energy every 5 steps
        {"name": "reflection128_f64", "kind": "reflection", "n": 128, "scale": 4, "store": "f64", "tau": 0.6,
         "steps": 100, "every": 5},
        # the paper's convected vortex: velocity inlet, MRT collision, 50 steps between energies
        {"name": "inlet128_mrt_f32", "kind": "lattice", "nx": 128, "ny": 128, "store": "f32", "edges": "inlet",
         "flow": "vortex", "coll": "mrt", "tau": 0.5384, "steps": 50, "plan": "default", "closure": False},
        # a channel of ordinary, odd size: NSBC at both ends, periodic across, launched as it comes
        {"name": "channel1501x701_f32", "kind": "lattice", "nx": 1501, "ny": 701, "store": "f32",
         "edges": "channel", "flow": "vortex", "coll": "bgk", "tau": 0.55, "steps": 50, "plan": "default",
         "closure": False},
        # the large acoustic lattice the benchmark runs, on its cached launch
        {"name": "pulses4096_f32", "kind": "lattice", "nx": 4096, "ny": 4096, "store": "f32", "edges": "nsbc",
         "flow": "pulse", "coll": "bgk", "tau": 0.51, "steps": 60, "plan": "tuned", "closure": False},
        # 16-bit storage on a ragged lattice with a mean flow
        {"name": "vortex3001x2047_f16", "kind": "lattice", "nx": 3001, "ny": 2047, "store": "f16",
         "edges": "nsbc", "flow": "vortex", "coll": "bgk", "tau": 0.55, "steps": 60, "plan": "tuned",
         "closure": False},
        # the learned closure on the 2048^2 vortex case, 50 steps between energies
        {"name": "closure2048_f32", "kind": "lattice", "nx": 2048, "ny": 2048, "store": "f32", "edges": "nsbc",
         "flow": "vortex", "coll": "bgk", "tau": 0.55, "steps": 50, "plan": "tuned", "closure": True},
        # the batched ensemble that training data comes from
        {"name": "ensemble256_f32", "kind": "ensemble", "count": 256, "lo": 64, "hi": 512, "store": "f32",
         "steps": 200, "log_every": 0},
        # three dimensions, the size the benchmark runs
        {"name": "d3q19_256_f32", "kind": "lattice3d", "q": 19, "nx": 256, "ny": 256, "nz": 256, "store": "f32",
         "edges": "nsbc", "tau": 0.55, "steps": 20, "plan": "tuned"},
        # and a small, odd one as it comes
        {"name": "d3q27_97x80x65_bf16", "kind": "lattice3d", "q": 27, "nx": 97, "ny": 80, "nz": 65,
         "store": "bf16", "edges": "nsbc", "tau": 0.58, "steps": 20, "plan": "default"},
        # one minibatch of the closure's training at the batch it is trained with
        {"name": "train4096", "kind": "train", "batch": 4096, "samples": 131072},
        # a round of samples made ready, and the held-out evaluation over them
        {"name": "dataset300007", "kind": "dataset", "samples": 300007, "batch": 65536},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("lattice", "reflection", "ensemble", "lattice3d", "train", "dataset"), (6, 1, 2, 3, 2, 2))[0]
    if kind == "lattice":
        edges = rng.choices(("nsbc", "channel", "inlet", "periodic"), (5, 1, 1, 1))[0]
        nx, ny = _log_int(rng, 64, 4096), _log_int(rng, 64, 4096)
        flow = "vortex" if edges == "inlet" else rng.choice(("pulse", "vortex"))
        return {"kind": kind, "nx": nx, "ny": ny, "store": rng.choice(("f64", "f32", "f16", "bf16")), "edges": edges,
                "flow": flow, "coll": rng.choices(("bgk", "mrt"), (3, 1))[0], "tau": round(rng.uniform(0.52, 0.8), 4),
                "steps": rng.randint(5, 60), "plan": rng.choice(("default", "tuned")),
                "closure": edges == "nsbc" and flow == "vortex" and rng.random() < 0.3}
    if kind == "reflection":
        return {"kind": kind, "n": _log_int(rng, 64, 512), "scale": rng.choice((2, 3, 4)),
                "store": rng.choice(("f64", "f32")), "tau": round(rng.uniform(0.52, 0.8), 4),
                "steps": rng.randint(20, 100), "every": rng.choice((5, 10, 20))}
    if kind == "ensemble":
        log_every = rng.choice((0, 0, 10))
        return {"kind": kind, "count": _log_int(rng, 4, 64 if log_every else 200), "lo": 64,
                "hi": _log_int(rng, 128, 256 if log_every else 512), "store": rng.choice(("f64", "f32", "f16", "bf16")),
                "steps": rng.randint(20, 100), "log_every": log_every}
    if kind == "lattice3d":
        q = rng.choice((19, 27))
        return {"kind": kind, "q": q, "nx": _log_int(rng, 24, 220), "ny": _log_int(rng, 24, 220),
                "nz": _log_int(rng, 24, 220), "store": rng.choice(("f64", "f32", "f16", "bf16")),
                "edges": rng.choices(("nsbc", "channel", "periodic"), (4, 1, 1))[0],
                "tau": round(rng.uniform(0.52, 0.8), 4), "steps": rng.randint(5, 20),
                "plan": rng.choice(("default", "tuned"))}
    if kind == "train":
        return {"kind": kind, "batch": _log_int(rng, 200, MAX_BATCH), "samples": rng.randint(70000, 140000)}
    return {"kind": kind, "samples": _log_int(rng, 10000, 300000), "batch": _log_int(rng, 200, 9000)}


# ---------------------------------------------------------------- inputs


def _rng(seed, salt):
    return np.random.default_rng([int(seed), salt])


def _grid(*shape):
    """Node coordinates (x, y[, z]) of an array [z][y][x], float64 on the device."""
    axes = [torch.arange(n, dtype=torch.float64, device=DEV) for n in shape]
    return torch.meshgrid(*axes, indexing="ij")[::-1]


def _pulse_sum(coords, pulses):
    dr = torch.zeros_like(coords[0])
    for a, w, *centre in pulses:
        d2 = sum((x - c) ** 2 for x, c in zip(coords, centre))
        dr += a * torch.exp(-math.log(2.0) * d2 / (w * w))
    return dr


def _seeded_pulses(r, sides):
    """Eight pulses of the benchmark's amplitudes and widths, anywhere but in the outer sixteenth."""
    wide = min(16.0, max(4.5, min(sides) / 12.0))
    return [(r.uniform(1e-4, 1e-3), r.uniform(4.0, wide)) + tuple(r.uniform(n / 16, n - n / 16) for n in sides)
            for _ in range(8)]


def _vortex(coords, xc, yc, rc, uv, u0):
    x, y = coords
    d2 = (x - xc) ** 2 + (y - yc) ** 2
    e = torch.exp(-d2 / (2.0 * rc * rc))
    return -1.5 * uv * uv * e * e, u0[0] - uv * (y - yc) / rc * e, u0[1] + uv * (x - xc) / rc * e


def _lattice_inputs(case, seed):
    """(fields, m0, base velocity, inlet velocity): pulses at rest, or a vortex carried towards the right edge
    that it is about to cross."""
    r = _rng(seed, 1)
    nx, ny = case["nx"], case["ny"]
    coords = _grid(ny, nx)
    if case["flow"] == "pulse":
        dr = _pulse_sum(coords, _seeded_pulses(r, (nx, ny)))
        return (dr, torch.zeros_like(dr), torch.zeros_like(dr)), (1.0, 0.0, 0.0), (0.0, 0.0), None
    u0 = (0.1, 0.0)
    rc = min(12.0, min(nx, ny) / 10.0)
    xc, yc = nx - 1 - r.uniform(0.5, 4.0) * rc, ny / 2.0 + r.uniform(-0.2, 0.2) * ny
    uv = W.swirl_amplitude(r.uniform(0.01, 0.02))
    fields = _vortex(coords, xc, yc, rc, uv, u0)
    return fields, (1.0, *u0), u0, (u0 if case["edges"] == "inlet" else None)


def _fields3(case, seed):
    r = _rng(seed, 2)
    dr = _pulse_sum(_grid(case["nz"], case["ny"], case["nx"]), _seeded_pulses(r, (case["nx"], case["ny"], case["nz"])))
    z = torch.zeros_like(dr)
    return dr, z, z, z


def _ensemble_members(case, seed):
    """(members, fields, m0 of each, base velocities): pulses and convected vortices, half each, their sizes and
    places those of the workload's seed, their strengths and directions this one's.  With samples logged every
    member has a twin padded by half its size on each side, after all the members."""
    r = _rng(seed, 4)
    ms = W.ensemble_members(case["count"], seed=4, lo=case["lo"], hi=case["hi"])
    for m in ms:
        if m.kind == "pulse":
            m.params["a"] = r.uniform(1e-4, 1e-3)
        else:
            speed, turn = r.uniform(0.05, 0.1), r.uniform(0.0, 2.0 * math.pi)
            m.params.update(u0=(speed * math.cos(turn), speed * math.sin(turn)),
                            uv=W.swirl_amplitude(r.uniform(0.005, 0.02)))
    members, fields, m0s, ubs = [], [], [], []
    for pad in (0, 1) if case["log_every"] else (0,):
        for m in ms:
            px, py = pad * (m.nx // 2), pad * (m.ny // 2)
            nx, ny, p = m.nx + 2 * px, m.ny + 2 * py, m.params
            coords = _grid(ny, nx)
            ub = p["u0"] if m.kind == "vortex" else (0.0, 0.0)
            if m.kind == "pulse":
                dr = _pulse_sum(coords, [(p["a"], p["w"], p["xc"] + px, p["yc"] + py)])
                f = (dr, torch.zeros_like(dr), torch.zeros_like(dr))
            else:
                f = _vortex(coords, p["xc"] + px, p["yc"] + py, p["rc"], p["uv"], p["u0"])
            members.append((nx, ny, m.tau))
            fields.append(f)
            m0s.append(W.member_m0(m))
            ubs.append(ub)
    return ms, members, fields, m0s, ubs


def _reflection_pulse(case, seed):
    """A pulse about to reach the left edge of the test lattice."""
    r = _rng(seed, 3)
    n = case["n"]
    return 1e-3, 4.0, r.uniform(8.0, n / 4.0), r.uniform(0.3, 0.7) * n


def _mlp_samples(case, seed):
    """Raw inputs [n][96] and residual targets [n][3] of the closure, with the spreads they have in earnest: every
    strip moment has a scale of its own, the targets follow the inputs, and some noise.  Inputs 87..95 are zero."""
    g = torch.Generator(device=DEV).manual_seed(int(seed) % (1 << 31))
    n = case["samples"]
    feat = torch.randn((n, 96), device=DEV, generator=g)
    kind = torch.tensor([1.0, 1.0, 1.0, 0.1, 0.1, 0.1, 0.02, 0.02, 0.01], device=DEV)
    feat[:, :81] *= kind.repeat(9)
    feat[:, 81] = 1.25 + 0.3 * torch.rand(n, device=DEV, generator=g)
    feat[:, 85:87] *= 0.1
    feat[:, 87:] = 0.0
    mix = torch.randn((87, 3), device=DEV, generator=g) / 9.0
    resid = torch.tanh(feat[:, :87] @ mix) + 0.2 * torch.randn((n, 3), device=DEV, generator=g)
    return feat, resid.contiguous()


def _train_inputs(case, seed):
    """Packed samples as the trainer keeps them, and the rows of one shuffled minibatch."""
    g = torch.Generator(device=DEV).manual_seed(int(seed) % (1 << 31))
    x = torch.randn((case["samples"], 96), device=DEV, generator=g).to(torch.bfloat16)
    x[:, 87:] = 0
    t = torch.randn((case["samples"], 3), device=DEV, generator=g)
    rows = torch.randperm(case["samples"], device=DEV, generator=g)[:case["batch"]].to(torch.int32)
    return x, t, rows


def _net_params(seed):
    return closure.xavier_params(int(seed) % (1 << 31))


# ---------------------------------------------------------------- prepare and run


def _tune(lat, store):
    """The launch a program settles on: the cached choice for the size, else the faster of the tuners' two."""
    if autotune.apply(lat, store) is None:
        autotune.tune(lat, store, reps=REPS, path=None)


def _committed_net():
    tr = closure.Trainer.load(closure.__file__.rsplit("/", 1)[0] + "/data/closure_c4.npz")
    blob = tr.export()
    tr.close()
    return blob


def _prepare_lattice(case, seed):
    fields, m0, ub, uw = _lattice_inputs(case, seed)
    mrt = (1.4, 1.4, 1.2) if case["coll"] == "mrt" else None
    lat = Lattice(case["nx"], case["ny"], case["tau"], fields, bc=EDGES[case["edges"]], gamma=GAMMA,
                  store=case["store"], m0=m0, ubase=ub, mrt=mrt, uw=uw)
    net = None
    if case["closure"]:
        net = _committed_net()
        lbm.lbm_set_closure(lat.ctx, net.data_ptr(), 1)
    if case["plan"] == "tuned":
        _tune(lat, case["store"])
    return {"lat": lat, "net": net}


def _run_lattice(s):
    lat, case = s["lat"], s["case"]
    lat.step(case["steps"])
    return lat.moments(f64=case["store"] == "f64")


def _prepare_reflection(case, seed):
    a, w, xc, yc = _reflection_pulse(case, seed)
    rr = ReflectionRun(lambda x, y: W.gaussian_pulses_xy(x, y, [(a, w, xc, yc)]), case["n"], case["n"], case["tau"],
                       scale=case["scale"], store=case["store"])
    return {"rr": rr}


def _run_reflection(s):
    case, rr = s["case"], s["rr"]
    series = rr.run(case["steps"], case["every"], respect_clean_time=False)["series"]
    return {"series": series, "moments": rr.test.moments(f64=case["store"] == "f64")}


def _prepare_ensemble(case, seed):
    ms, members, fields, m0s, ubs = _ensemble_members(case, seed)
    ens = Ensemble([member_params(nx, ny, tau, gamma=GAMMA, store=case["store"], ubase=ub)
                    for (nx, ny, tau), ub in zip(members, ubs)],
                   [tuple(c.cpu().numpy() for c in f) for f in fields])
    for k, m0 in enumerate(m0s):
        ens.set_farfield(k, 0.0, *m0)
    if case["log_every"]:
        own, twin = [], []
        for k, m in enumerate(ms):
            e = closure.edge_sites(m.nx, m.ny, 4)
            own.append(np.concatenate([np.full((len(e), 1), k, np.int32), e], 1))
            twin.append(own[-1] + np.array([len(ms), m.nx // 2, m.ny // 2, 0], np.int32))
        ens.set_log_sites(*(torch.from_numpy(np.concatenate(v)).to(DEV) for v in (own, twin)))
        return {"ens": ens}
    best, times = ens.autotune(REPS)
    b2, t2 = ens.autotune_two_step(REPS)
    if not 0 < t2[b2] < times[best]:
        ens.set_two_step(-1)
    return {"ens": ens, "nodes": sum(nx * ny for nx, ny, _ in members)}


def _run_ensemble(s):
    case, ens = s["case"], s["ens"]
    if case["log_every"]:
        return ens.step_graph_logged(case["steps"], case["log_every"])
    ens.step_graph(case["steps"])
    f64 = case["store"] == "f64"
    out = torch.empty((3, s["nodes"]), dtype=torch.float64 if f64 else torch.float32, device=DEV)
    at, step = [out[c].data_ptr() for c in range(3)], out.element_size()
    for k, p in enumerate(ens.members):
        lbm.lbm_ens_moments(ens.ens, k, *at, f64, True)
        at = [a + step * p.nx * p.ny for a in at]
    return out


def _prepare_lattice3d(case, seed):
    lat = Lattice3D(case["nx"], case["ny"], case["nz"], case["tau"], _fields3(case, seed), bc=FACES[case["edges"]],
                    gamma=GAMMA, store=case["store"], q=case["q"])
    if case["plan"] == "tuned":
        lat.autotune(REPS)
    return {"lat": lat}


def _run_lattice3d(s):
    lat, case = s["lat"], s["case"]
    lat.step(case["steps"])
    out = torch.empty((4,) + lat.shape, dtype=torch.float64, device=DEV)
    lbm.lbm3d_moments(lat.ctx, out.data_ptr())
    return out if case["store"] == "f64" else out.float()  # fields of a 32-bit run are kept in 32 bits


def _prepare_train(case, seed):
    x, t, rows = _train_inputs(case, seed)
    tr = closure.Trainer(params=_net_params(seed), max_batch=-(-case["batch"] // 64) * 64)
    return {"tr": tr, "x": x, "t": t, "rows": rows}


def _run_train(s):
    tr = s["tr"]
    loss = tr.train_step(s["x"], s["t"], LR, rows=s["rows"])
    params = torch.empty(closure.NPARAM, dtype=torch.float32, device=DEV)
    lbm.lbm_mlp_params(tr.m, params.data_ptr())
    return {"loss": loss, "params": params}


def _prepare_dataset(case, seed):
    feat, resid = _mlp_samples(case, seed)
    return {"feat": feat, "resid": resid,
            "tr": closure.Trainer(params=_net_params(seed), max_batch=-(-case["batch"] // 64) * 64)}


def _run_dataset(s):
    tr, batch = s["tr"], s["case"]["batch"]
    tr.fit_normalization(s["feat"], s["resid"])
    x, t = tr.pack(s["feat"], s["resid"])
    y = tr.forward(x)
    grads, loss = tr.grads(x[:batch], t[:batch])
    mean, inv, scale = tr.normalization()
    return {"x": x, "t": t, "y": y, "grads": grads, "loss": loss, "mean": mean, "inv_std": inv, "scale": scale}


_PREPARE = {"lattice": _prepare_lattice, "reflection": _prepare_reflection, "ensemble": _prepare_ensemble,
            "lattice3d": _prepare_lattice3d, "train": _prepare_train, "dataset": _prepare_dataset}
_RUN = {"lattice": _run_lattice, "reflection": _run_reflection, "ensemble": _run_ensemble,
        "lattice3d": _run_lattice3d, "train": _run_train, "dataset": _run_dataset}


def prepare(case, seed):
    return dict(_PREPARE[case["kind"]](case, seed), case=case)


def run(state):
    return _RUN[state["case"]["kind"]](state)


# ---------------------------------------------------------------- work

# operations of one node update: moments, equilibrium and relaxation (2-D BGK 120, MRT 80 more; per direction in 3-D)
FLOPS_2D, FLOPS_MRT, FLOPS_3D_DIR = 120, 200, 14
# of one sample of the network 96 -> 64 -> 64 -> 3: forward, and forward with all gradients
FLOPS_FWD = 2 * (96 * 64 + 64 * 64 + 64 * 3)
FLOPS_GRAD = 2 * FLOPS_FWD + 2 * (64 * 64 + 64 * 3)


def _state_work(nodes, q, esize, out_bytes, steps, flops):
    """One read and one write of the populations, however many steps lie between, and the moments written."""
    return {"bytes": nodes * (2 * q * esize + out_bytes), "flops": nodes * steps * flops}


def work(case):
    kind = case["kind"]
    if kind == "lattice":
        out = 3 * (8 if case["store"] == "f64" else 4)
        return _state_work(case["nx"] * case["ny"], 9, ESIZE[case["store"]], out, case["steps"],
                           FLOPS_MRT if case["coll"] == "mrt" else FLOPS_2D)
    if kind == "reflection":
        n, s = case["n"] ** 2, ESIZE[case["store"]]
        steps = case["steps"] // case["every"] * case["every"]
        return _state_work(n * (1 + case["scale"] ** 2), 9, s, 0, steps, FLOPS_2D)
    if kind == "ensemble":
        # the mean member (sides uniform in [lo, hi]); the twins have four times the nodes and are not read out
        nodes = case["count"] * ((case["lo"] + case["hi"]) / 2) ** 2
        if case["log_every"]:
            sites = case["count"] * (case["lo"] + case["hi"]) / 2  # every 4th node of four edges
            w = _state_work(5 * nodes, 9, ESIZE[case["store"]], 0, case["steps"], FLOPS_2D)
            w["bytes"] += -(-case["steps"] // case["log_every"]) * sites * 4 * lbm.LBM_ENS_LOG_FLOATS
            return w
        return _state_work(nodes, 9, ESIZE[case["store"]], 3 * (8 if case["store"] == "f64" else 4), case["steps"],
                           FLOPS_2D)
    if kind == "lattice3d":
        return _state_work(case["nx"] * case["ny"] * case["nz"], case["q"], ESIZE[case["store"]],
                           4 * (8 if case["store"] == "f64" else 4), case["steps"], FLOPS_3D_DIR * case["q"])
    if kind == "train":
        # rows, inputs and targets; parameters and both Adam moments read and written, parameters handed out
        return {"bytes": case["batch"] * (4 + 192 + 12) + closure.NPARAM * 4 * 7, "flops": case["batch"] * FLOPS_GRAD}
    n, b = case["samples"], min(case["batch"], case["samples"])
    # inputs and targets read, packed inputs and targets written, outputs written
    return {"bytes": n * (384 + 12 + 192 + 12 + 12) + closure.NPARAM * 8, "flops": n * FLOPS_FWD + b * FLOPS_GRAD}


# ---------------------------------------------------------------- 64-bit values

def _velocities(d, q):
    c = [v for v in itertools.product((-1, 0, 1), repeat=d) if q != 19 or sum(map(abs, v)) <= 2]
    by_speed = {9: (4 / 9, 1 / 9, 1 / 36), 19: (1 / 3, 1 / 18, 1 / 36), 27: (8 / 27, 2 / 27, 1 / 54, 1 / 216)}[q]
    w = [by_speed[sum(map(abs, v))] for v in c]
    return c, w, [c.index(tuple(-a for a in v)) for v in c]


def _mrt_matrix(c, tau, rates):
    """M^-1 S M of the moments 1, |c|^2, |c|^4, c_x, c_x|c|^2, c_y, c_y|c|^2, c_x^2 - c_y^2, c_x c_y, made orthogonal
    one after the other."""
    cc = torch.tensor(c, dtype=torch.float64, device=DEV)
    x, y = cc[:, 0], cc[:, 1]
    s = x * x + y * y
    rows = []
    for v in (torch.ones_like(x), s, s * s, x, x * s, y, y * s, x * x - y * y, x * y):
        for r in rows:
            v = v - (v @ r) / (r @ r) * r
        rows.append(v)
    m = torch.stack(rows)
    e, eps, qf = rates
    k = torch.tensor([0, e, eps, 0, qf, 0, qf, 1 / tau, 1 / tau], dtype=torch.float64, device=DEV)
    return torch.linalg.inv(m) @ (k[:, None] * m)


class _Exact:
    """Stream, boundary, collide in float64 on arrays [z][y][x]; faces (low, high) per axis x, y, z: 0 periodic,
    1 NSBC, 2 the velocity uw."""

    def __init__(self, fields, tau, faces, q, uw=None, mrt=None):
        self.d = len(fields) - 1
        self.c, self.w, self.opp = _velocities(self.d, q)
        self.tau, self.faces, self.uw = tau, faces, uw
        self.relax = _mrt_matrix(self.c, tau, mrt) if mrt else None
        rho, u = 1.0 + fields[0], list(fields[1:])
        self.f = torch.stack([self.eq(i, rho, u) for i in range(q)])

    def eq(self, i, rho, u):
        cu = sum(a * v for a, v in zip(self.c[i], u) if a)
        uu = sum(v * v for v in u)
        return self.w[i] * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * uu)

    def moments(self, f):
        rho = sum(f)
        return rho, [sum(v[a] * g for v, g in zip(self.c, f) if v[a]) / rho for a in range(self.d)]

    def region(self, side, inward=None):
        """Index of the nodes on the faces `side` names per axis (-1 low, 1 high, 0 neither), or of their neighbours
        one node inward along axis `inward`."""
        at = []
        for a in range(self.d):
            k = 1 if a == inward else 0
            if side[a]:
                at.append(slice(k, k + 1) if side[a] < 0 else slice(-1 - k, -k or None))
            else:
                at.append(slice(1, -1) if self.faces[2 * a] else slice(None))
        return tuple(at[::-1])

    def boundary(self, side, rho, u, f):
        """Rebuilds the streamed populations f of the nodes on the faces `side`."""
        at = self.region(side)
        here = [g[at] for g in f]
        unknown = {i for i, v in enumerate(self.c) if any(s and v[a] * s < 0 for a, s in enumerate(side))}
        axes = [a for a in range(self.d) if side[a]]
        a = axes[0]
        if len(axes) == 1 and self.faces[2 * a + (side[a] > 0)] == 2:
            mass = sum((1 if v[a] == 0 else 2) * g for v, g in zip(self.c, here) if v[a] * side[a] >= 0)
            rc = mass / (1 + self.uw[a] * side[a])
            uc = [torch.full_like(rc, v) for v in self.uw]
        else:
            m = [rho[at]] + [v[at] for v in u]
            k = GAMMA / math.sqrt(len(axes))
            inner = [[rho[j]] + [v[j] for v in u] for j in (self.region(side, b) for b in axes)]
            rc, *uc = [v - k * sum(v - n[x] for n in inner) for x, v in enumerate(m)]
        new = list(here)
        for i in unknown:
            o = self.opp[i]
            new[i] = self.eq(i, rc, uc) + (0 if o in unknown else here[o] - self.eq(o, rc, uc))
        r1 = rc - sum(new)
        j1 = [rc * uc[b] - sum(v[b] * g for v, g in zip(self.c, new) if v[b]) for b in range(self.d)]
        for i, v in enumerate(self.c):
            f[i][at] = new[i] + self.w[i] * (r1 + 3 * sum(v[b] * j1[b] for b in range(self.d)))

    def step(self, n):
        sides = [(0,) + ((-1, 1) if self.faces[2 * a] else ()) for a in range(self.d)]
        for _ in range(n):
            rho, u = self.moments(self.f)
            s = torch.stack([torch.roll(self.f[i], v[::-1], tuple(range(self.d))) for i, v in enumerate(self.c)])
            copy = [g.clone() for g in s] if any(self.faces) else None
            for side in itertools.product(*sides):
                if any(side):
                    self.boundary(side, rho, u, copy)
            if copy is not None:
                s = torch.stack(copy)
            rho, u = self.moments(s)
            if self.relax is not None:
                e = torch.stack([self.eq(i, rho, u) for i in range(len(self.c))])
                self.f = s - torch.tensordot(self.relax, s - e, 1)
            else:
                for i in range(len(self.c)):
                    s[i] += (self.eq(i, rho, u) - s[i]) / self.tau
                self.f = s

    def out(self):
        rho, u = self.moments(self.f)
        return [rho - 1.0, *u]


def _exact_lattice(case, seed):
    if case["closure"]:
        return None
    fields, _, _, uw = _lattice_inputs(case, seed)
    e = _Exact(fields, case["tau"], EDGES[case["edges"]], 9, uw, (1.4, 1.4, 1.2) if case["coll"] == "mrt" else None)
    e.step(case["steps"])
    return tuple(e.out())


def _exact_reflection(case, seed):
    a, w, xc, yc = _reflection_pulse(case, seed)
    n, s = case["n"], case["scale"]
    off = (s * n - n) // 2
    both = []
    for side, o in ((n, 0), (s * n, off)):
        x, y = _grid(side, side)
        dr = _pulse_sum((x - o, y - o), [(a, w, xc, yc)])
        both.append(_Exact((dr, torch.zeros_like(dr), torch.zeros_like(dr)), case["tau"], EDGES["nsbc"], 9))
    test, ref = both
    win = (slice(off, off + n),) * 2
    energy = lambda m: float(0.5 * (m[0] ** 2 / 3.0 + m[1] ** 2 + m[2] ** 2).sum())  # noqa: E731
    e0, series = energy(test.out()), []
    for k in range(case["steps"] // case["every"] + 1):
        if k:
            test.step(case["every"])
            ref.step(case["every"])
        series.append(energy([p - q[win] for p, q in zip(test.out(), ref.out())]) / e0)
    return {"series": np.array(series), "moments": tuple(test.out())}


def _exact_ensemble(case, seed):
    if case["log_every"] or case["count"] * case["steps"] > 2500:
        return None
    _, members, fields, _, _ = _ensemble_members(case, seed)
    out = []
    for (_, _, tau), f in zip(members, fields):
        e = _Exact(f, tau, EDGES["nsbc"], 9)
        e.step(case["steps"])
        out.append(torch.stack(e.out()).reshape(3, -1))
    return torch.cat(out, 1)


def _exact_lattice3d(case, seed):
    e = _Exact(_fields3(case, seed), case["tau"], FACES[case["edges"]], case["q"])
    e.step(case["steps"])
    return torch.stack(e.out())


def _net64(params):
    p = closure.unpack_params(params)
    return [torch.tensor(p[k], dtype=torch.float64, device=DEV, requires_grad=True)
            for k in ("W1", "b1", "W2", "b2", "W3", "b3")]


def _forward64(p, x):
    h = torch.tanh(x @ p[0].T + p[1])
    h = torch.tanh(h @ p[2].T + p[3])
    return h @ p[4].T + p[5]


def _loss64(p, x, t):
    loss = ((_forward64(p, x) - t) ** 2).mean()
    return loss, torch.cat([g.reshape(-1) for g in torch.autograd.grad(loss, p)])


def _exact_train(case, seed):
    x, t, rows = _train_inputs(case, seed)
    p = _net64(_net_params(seed))
    loss, g = _loss64(p, x[rows.long()].double(), t[rows.long()].double())
    flat = torch.cat([v.detach().reshape(-1) for v in p])
    # the first Adam step: both moments' bias corrections cancel
    return {"loss": loss.detach().reshape(1), "params": flat - LR * g / (g.abs() + 1e-8)}


def _exact_dataset(case, seed):
    feat, resid = (v.double() for v in _mlp_samples(case, seed))
    mean, sd = feat.mean(0), feat.std(0, unbiased=False)
    used = (torch.arange(96, device=DEV) < 87) & (sd > 1e-30) & (sd > 1e-7 * mean.abs())
    top = sd[:81].reshape(9, 9).amax(0).repeat(9)
    used[:81] &= sd[:81] > 1e-3 * top
    mean, inv = torch.where(used, mean, 0.0), torch.where(used, 1.0 / sd, 0.0)
    scale = resid.square().mean(0).sqrt()
    x, t = (feat - mean) * inv, resid / scale
    p = _net64(_net_params(seed))
    b = case["batch"]
    loss, grads = _loss64(p, x[:b], t[:b])
    with torch.no_grad():
        y = _forward64(p, x)
    return {"x": x, "t": t, "y": y, "grads": grads, "loss": loss.item(), "mean": mean, "inv_std": inv, "scale": scale}


_EXACT = {"lattice": _exact_lattice, "reflection": _exact_reflection, "ensemble": _exact_ensemble,
          "lattice3d": _exact_lattice3d, "train": _exact_train, "dataset": _exact_dataset}


def exact(case, seed):
    return _EXACT[case["kind"]](case, seed)
