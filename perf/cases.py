"""Timing cases of the NEP molecular-dynamics framework: what a user's program does with it,
over the sizes, species, precisions and options it is used at.

A case is one of six kinds of work, each through the package's public entry points:

  serve   one configuration through the allocation-free call (a serving loop)
  frame   one configuration labelled: state in, lists built, energy, virial, forces and
          per-atom energies out (what frame generation and relabelling do)
  md      a segment of dynamics from a given state: NVE, NVT (Nose-Hoover chain) or r-RESPA
          with a surrogate, in default or deterministic accumulation, FP32 or BF16 network
  fit_surrogate   one Adam step of surrogate training (all parameters) over a batch of frames
  fit_network     forward and backward of the energy + force loss through the autograd Function
  check64 FP64 evaluation and FP64 parameter gradient

Boxes are FCC copper-like (a = 3.615 A), of nx x ny x nz cells, thermally displaced, with one
species or a random two-species alloy with 5% vacancies; models are random-weight with the
hyperparameters of ``inputs.FULL_HPARAMS`` and of the 4 / 3 A surrogate.

``exact`` is the plain FP64 definition in torch: descriptors by direct sums over neighbours,
derivatives by automatic differentiation.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2604_24816_amd import autograd as AG
from paper_2604_24816_amd import inputs as I
from paper_2604_24816_amd import nep

DEV = "cuda:0"
LATTICE = 3.615          # A
MASS = 63.546            # amu
XI = 103.642697          # eV fs^2 / (amu A^2)
KB = 8.617333262e-5      # eV / K
VACANCIES = 0.05


def _case(name, kind, nx, ny=None, nz=None, **kw):
    c = {"name": name, "kind": kind, "nx": nx, "ny": ny or nx, "nz": nz or nx, "species": 1, "zbl": 0.0,
         "precision": "fp32", "sigma": 0.08}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest box the 6 A cutoff and 1 A skin admit, evaluated alone in a serving loop:
        # launches and latency are all of it
        _case("serve_256", "serve", 4),
        # one training frame of 4,000 atoms labelled by the full model
        _case("frame_4000", "frame", 10),
        # a trajectory of the size that frame generation runs: 100 steps, thermo every 10
        _case("md_nve_4000", "md", 10, ensemble="nve", steps=100, deterministic=False, sigma=0.05),
        # one optimiser step of surrogate training: 8 frames of 4,000 atoms, every parameter
        _case("fit_surrogate_8x4000", "fit_surrogate", 10, frames=8, sigma=0.12),
        # the loss of two hot 32,000-atom frames, gradients of the full model's network
        _case("fit_network_2x32000", "fit_network", 20, frames=2, sigma=0.17),
        # the FP64 check form on a box used for finite-difference checks
        _case("check64_2048", "check64", 8, sigma=0.08),
        # NVT with the bfloat16 network on an odd-sided box (33,660 atoms)
        _case("md_nvt_bf16_33660", "md", 17, 15, 33, ensemble="nvt", steps=20, deterministic=False,
              precision="bf16"),
        # a reproducible run of an alloy with close-range repulsion (52,531 atoms)
        _case("md_det_alloy_zbl_52531", "md", 24, ensemble="nve", steps=10, deterministic=True, species=2,
              zbl=2.0),
        # multiple time stepping with the 4 / 3 A surrogate, 256,000 atoms, k = 4
        _case("md_mts_256000", "md", 40, ensemble="mts", steps=20, deterministic=False),
        # the 60^3-cell alloy with vacancies (820,800 atoms), labelled once
        _case("frame_alloy_820800", "frame", 60, species=2, sigma=0.05),
        # NVE of an alloy of ordinary production size (95,760 atoms)
        _case("md_alloy_95760", "md", 30, 30, 28, ensemble="nve", steps=20, deterministic=False, species=2),
        # the large box: 4,000,000 atoms, 50 steps
        _case("md_nve_4000000", "md", 100, ensemble="nve", steps=50, deterministic=False),
    ]


def _sides(rng, lo, hi):
    """Three side lengths in cells for a number of sites between lo and hi (log-uniform)."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    e = (n / 4.0) ** (1.0 / 3.0)
    nx = max(4, round(e * rng.uniform(0.8, 1.25)))
    ny = max(4, round(e * rng.uniform(0.8, 1.25)))
    nz = max(4, round(n / 4.0 / (nx * ny)))
    while 4 * nx * ny * nz > hi and nz > 4:
        nz -= 1
    return nx, ny, nz


def draw(rng):
    kind = rng.choice(["serve", "frame", "frame", "md", "md", "md", "md", "fit_surrogate", "fit_network", "check64"])
    kw = {"sigma": round(rng.uniform(0.03, 0.14), 3)}
    if kind == "serve":
        sides = _sides(rng, 256, 16000)
        kw.update(species=rng.choice([1, 1, 2]), precision=rng.choice(["fp32", "bf16"]))
    elif kind == "frame":
        sides = _sides(rng, 256, 900000)
        kw.update(species=rng.choice([1, 2]), zbl=rng.choice([0.0, 0.0, 2.0, 2.5]), precision=rng.choice(["fp32", "fp32", "bf16"]))
    elif kind == "md":
        sides = _sides(rng, 256, 1000000)
        kw.update(ensemble=rng.choice(["nve", "nve", "nvt", "mts"]), steps=4 * rng.randint(2, 10),
                  deterministic=rng.random() < 0.25, species=rng.choice([1, 1, 2]), zbl=rng.choice([0.0, 0.0, 0.0, 2.0, 2.5]),
                  precision=rng.choice(["fp32", "fp32", "bf16"]))
    elif kind == "fit_surrogate":
        sides = _sides(rng, 500, 16000)
        kw.update(frames=rng.randint(1, 8))
    elif kind == "fit_network":
        sides = _sides(rng, 500, 32000)
        kw.update(frames=rng.randint(1, 2), species=rng.choice([1, 1, 2]))
    else:
        sides = _sides(rng, 256, 6000)
        kw.update(species=rng.choice([1, 2]), zbl=rng.choice([0.0, 0.0, 2.0, 2.5]))
    c = _case("", kind, *sides, **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs (made from the seed alone)

def _atoms(case, seed, temperature=600.0):
    """Positions, velocities (FP64), types (int32) on the GPU, the box and the masses."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + 17)
    n3 = (case["nx"], case["ny"], case["nz"])
    ax = [torch.arange(k, device=DEV, dtype=torch.float64) for k in n3]
    cells = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 1, 3)
    basis = torch.tensor([[0.0, 0.0, 0.0], [0.5, 0.5, 0.0], [0.5, 0.0, 0.5], [0.0, 0.5, 0.5]], device=DEV,
                         dtype=torch.float64)
    x = ((cells + basis) * LATTICE).reshape(-1, 3)
    box = np.array(n3, np.float64) * LATTICE
    sites = x.shape[0]
    if case["species"] == 2:
        types = torch.zeros(sites, dtype=torch.int32, device=DEV)
        types[torch.randperm(sites, generator=g, device=DEV)[sites // 2:]] = 1
        keep = torch.ones(sites, dtype=torch.bool, device=DEV)
        keep[torch.randperm(sites, generator=g, device=DEV)[: round(VACANCIES * sites)]] = False
        x, types = x[keep], types[keep].contiguous()
        masses = np.array([MASS, 1.7 * MASS])
    else:
        types = torch.zeros(sites, dtype=torch.int32, device=DEV)
        masses = np.array([MASS])
    n = x.shape[0]
    x = x + case["sigma"] * torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
    L = torch.tensor(box, device=DEV)
    x = torch.remainder(x, L)
    x = torch.where(x >= L, x - L, x).contiguous()
    m = torch.tensor(masses, device=DEV)[types.long()][:, None]
    v = torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64) * torch.sqrt(KB * temperature / (m * XI))
    v = v - (m * v).sum(0) / m.sum()
    ke = 0.5 * XI * float((m * v * v).sum())
    v = v * math.sqrt(temperature * (3 * n - 3) * KB / (2.0 * ke))
    return x, v.contiguous(), types, box, masses


def _hparams(case):
    hp = I.FULL_HPARAMS
    if case["species"] == 2:
        hp = dataclasses.replace(hp, n_types=2, zbl_z=(29.0, 29.0))
    if case["zbl"] > 0:
        hp = dataclasses.replace(hp, zbl_outer=case["zbl"])
    return hp


def _models(case, seed):
    """(full hyperparameters, parameters, surrogate hyperparameters, parameters)"""
    hp = _hparams(case)
    params = I.random_model(hp, seed % 100003)
    shp = dataclasses.replace(I.SURROGATE_SHORTER_HPARAMS, n_types=hp.n_types, zbl_outer=hp.zbl_outer, zbl_z=hp.zbl_z)
    return hp, params, shp, I.surrogate_from_teacher(hp, params, shp, seed % 100003 + 7)


def _student(hp, params, seed):
    """The network weights of a model part-way through training, float32 on the GPU."""
    rng = np.random.default_rng(seed + 5)
    theta = nep.network_params(hp, params)
    return torch.tensor(theta + 0.01 * rng.normal(size=theta.size), dtype=torch.float32, device=DEV)


CAPS = {"cap_radial": 192, "cap_angular": 112}


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "serve":
        hp, params, _, _ = _models(case, seed)
        x, _, types, box, _ = _atoms(case, seed)
        st.update(model=nep.NEPModel(hp, params), x=x, types=types, box=box,
                  F=torch.empty_like(x), U=torch.empty(x.shape[0], dtype=torch.float64, device=DEV))
    elif kind == "frame":
        hp, params, _, _ = _models(case, seed)
        x, _, types, box, masses = _atoms(case, seed)
        st.update(system=nep.NEPSystem(nep.NEPModel(hp, params), x.shape[0], box, **CAPS), x=x, types=types,
                  masses=masses)
    elif kind == "md":
        hp, params, shp, sparams = _models(case, seed)
        x, v, types, box, masses = _atoms(case, seed)
        sur = nep.NEPModel(shp, sparams) if case["ensemble"] == "mts" else None
        s = nep.NEPSystem(nep.NEPModel(hp, params), x.shape[0], box, surrogate=sur, **CAPS)
        s.set_deterministic(case["deterministic"])
        st.update(system=s, x=x, v=v, types=types, masses=masses)
    elif kind == "fit_surrogate":
        hp, params, shp, sparams = _models(case, seed)
        frames = [_atoms(case, 64 * seed + f) for f in range(case["frames"])]
        labels = [_evaluate(hp, params, f[0], f[2], f[3])[:2] for f in frames]
        theta = torch.tensor(sparams, dtype=torch.float32, device=DEV)
        st.update(system=nep.NEPSystem(nep.NEPModel(shp, sparams), frames[0][0].shape[0], frames[0][3],
                                       cap_radial=256, cap_angular=160),
                  frames=frames, E=[e for e, _ in labels], F=[f.to(torch.float32) for _, f in labels], theta=theta,
                  grad=torch.zeros_like(theta), frozen=slice(*shp.offsets()["sigma"]), t=100)
        st["m1"], st["m2"] = _moments(theta, seed)
    elif kind == "fit_network":
        hp, params, _, _ = _models(case, seed)
        st["theta"] = _student(hp, params, seed).requires_grad_(True)
        st["systems"], st["labels"] = [], []
        for f in range(case["frames"]):
            x, _, types, box, masses = _atoms(case, 64 * seed + f)
            s = nep.NEPSystem(nep.NEPModel(hp, params), x.shape[0], box, **CAPS)
            s.set_state(x, types, masses)
            s.build_neighbors(1.0)
            e, F = _evaluate(hp, params, x, types, box)[:2]
            st["systems"].append((s, None))
            st["labels"].append((e, F.to(torch.float32)))
    else:
        hp, params, _, _ = _models(case, seed)
        x, _, types, box, masses = _atoms(case, seed)
        s = nep.NEPSystem(nep.NEPModel(hp, params), x.shape[0], box, **CAPS)
        s.set_state(x, types, masses)
        s.build_neighbors(1.0)
        st.update(system=s, gF=_force_weights(x.shape[0], seed))
    return st


def _moments(theta, seed):
    """Adam moments of a run in progress (gradients of order 0.1)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed + 3)
    m1 = 0.02 * torch.randn(theta.numel(), generator=g, device=DEV)
    m2 = 0.01 * (0.5 + torch.rand(theta.numel(), generator=g, device=DEV))
    return m1, m2


def _force_weights(n, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed + 11)
    return torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)


GE = 0.7   # energy weight of the FP64 gradient check


# ---------------------------------------------------------------- the work

def _single(E, W, F, U):
    """An evaluation's results as a program keeps them: single precision, what they were computed in."""
    return {"E": E, "W": W.astype(np.float32), "F": F.to(torch.float32), "U": U.to(torch.float32)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "serve":
        E, W = nep.compute_energy_forces_virial_noalloc(
            state["model"], state["x"], state["types"], state["box"], precision=case["precision"],
            forces=state["F"], per_atom_energy=state["U"])
        return _single(E, W, state["F"], state["U"])
    if kind == "frame":
        s = state["system"]
        s.set_state(state["x"], state["types"], state["masses"])
        s.build_neighbors(1.0)
        return _single(*s.compute(precision=case["precision"], per_atom=True, on_device=True))
    if kind == "md":
        s = state["system"]
        s.set_state(state["x"], state["types"], state["masses"], state["v"])
        kw = {}
        if case["ensemble"] == "nvt":
            s.set_thermostat(300.0, tau=50.0, chain=3)
        elif case["ensemble"] == "mts":
            kw = {"mts_k": 4, "fallback_rms": 1e9, "fallback_max": 1e9}
        rows = s.step(case["steps"], dt=1.0, rebuild_every=10, skin=1.0, precision=case["precision"],
                      thermo_every=_thermo_every(case), **kw)
        x, v, _ = s.get_state()
        # positions whole, as a restart needs them; velocities and the log in single precision
        return {"x": x, "v": v.astype(np.float32), "thermo": rows.astype(np.float32)}
    if kind == "fit_surrogate":
        s, theta, grad = state["system"], state["theta"], state["grad"]
        n, batch = s.n, case["frames"]
        grad.zero_()
        energies = []
        for (x, _, types, _, masses), e_ref, f_ref in zip(state["frames"], state["E"], state["F"]):
            s.set_state(x, types, masses)
            s.build_neighbors(1.0)
            E, F = s.train_forward_params(0, theta)
            de = (E - e_ref) / n
            s.train_backward_params(0, theta, 2.0 * de / n / batch, (2.0 / (3 * n * batch)) * (F - f_ref), out=grad)
            energies.append(E)
        grad[state["frozen"]] = 0.0
        state["t"] += 1
        s.adam(theta, grad, state["m1"], state["m2"], state["t"], lr=1e-4)
        return {"E": energies, "grad": grad, "theta": theta, "m1": state["m1"], "m2": state["m2"]}
    if kind == "fit_network":
        theta = state["theta"]
        theta.grad = None
        loss = AG.energy_force_loss(state["systems"], theta, state["labels"])
        loss.backward()
        return {"loss": loss.detach().to(torch.float32), "grad": theta.grad}
    s = state["system"]
    E, W, F, U = s.compute(precision="fp64", per_atom=True, on_device=True)
    return {"E": E, "W": W, "F": F, "U": U, "grad": s.train_backward64(GE, state["gF"])}


def _thermo_every(case):
    return 4 if case["ensemble"] == "mts" else 10


# ---------------------------------------------------------------- what a pass cannot do without

# flops per pair inside the cutoffs and per atom, counted from the definition (FMA = 2): basis and
# channel contractions, harmonics, their gradients, the network
FULL = {"rad": 160 + 346, "ang": 460 + 1222, "atom": 5000}
SUR = {"rad": 160 + 346, "ang": 270 + 615, "atom": 1000}


def _sites(case):
    n = 4 * case["nx"] * case["ny"] * case["nz"]
    return n - round(VACANCIES * n) if case["species"] == 2 else n


def _pairs(case, rc):
    occupied = 1.0 - (VACANCIES if case["species"] == 2 else 0.0)
    return 4.0 / 3.0 * math.pi * rc ** 3 * 4.0 / LATTICE ** 3 * occupied


def _eval_flops(case, f, rcR, rcA):
    return _sites(case) * (f["rad"] * _pairs(case, rcR) + f["ang"] * _pairs(case, rcA) + f["atom"])


def work(case):
    n, kind = _sites(case), case["kind"]
    full = _eval_flops(case, FULL, 6.0, 5.0)
    sur = _eval_flops(case, SUR, 4.0, 3.0)
    if kind in ("serve", "frame"):
        return {"bytes": n * (24 + 4 + 24 + 8), "flops": full}       # x, type; F, U
    if kind == "md":
        steps = case["steps"]
        if case["ensemble"] == "mts":
            flops = sur * (steps + 1) + full * (steps // 4 + 1)
        else:
            flops = full * (steps + 1)
        # state in and out; every step reads and writes x, v and reads F twice
        return {"bytes": n * (100 + steps * (96 + 24 + 4)), "flops": flops}
    if kind == "fit_surrogate":
        # forward, the gradient's JVP and the coefficient pass: about twice the evaluation again
        return {"bytes": case["frames"] * n * (28 + 24), "flops": 3.0 * sur * case["frames"]}
    if kind == "fit_network":
        return {"bytes": case["frames"] * n * (28 + 24), "flops": 2.0 * full * case["frames"]}
    return {"bytes": n * (28 + 24 + 8 + 24), "flops": 4.0 * full}


# ---------------------------------------------------------------- exact: the definition in FP64

def _neighbour_table(x, box, rc):
    """Padded neighbour table [N][M] of the atoms within rc (self as padding) from a cell grid."""
    n = x.shape[0]
    L = torch.tensor(box, device=DEV)
    nc = [max(1, int(b // rc)) for b in box]
    ncd = torch.tensor(nc, device=DEV)
    c3 = torch.minimum((x / L * ncd).long(), ncd - 1)
    cell = (c3[:, 0] * nc[1] + c3[:, 1]) * nc[2] + c3[:, 2]
    order = torch.argsort(cell)
    count = torch.bincount(cell, minlength=nc[0] * nc[1] * nc[2])
    start = torch.cumsum(count, 0) - count
    occ = int(count.max())
    offs = sorted({((a % nc[0]), (b % nc[1]), (c % nc[2])) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)})
    offs = torch.tensor(offs, device=DEV)
    slot = torch.arange(occ, device=DEV)
    rows = []
    for a in range(0, n, 16384):
        ids = torch.arange(a, min(n, a + 16384), device=DEV)
        cc = (c3[ids][:, None, :] + offs[None]) % ncd
        cl = (cc[..., 0] * nc[1] + cc[..., 1]) * nc[2] + cc[..., 2]
        cand = start[cl][..., None] + slot
        ok = (slot < count[cl][..., None]).reshape(ids.numel(), -1)
        cand = order[cand.clamp(max=n - 1)].reshape(ids.numel(), -1)
        d = x[cand] - x[ids][:, None]
        d = d - L * torch.round(d / L)
        ok &= ((d * d).sum(-1) < rc * rc) & (cand != ids[:, None])
        m = int(ok.sum(1).max())
        keep = torch.argsort((~ok).to(torch.int8), dim=1, stable=True)[:, :m]
        rows.append(torch.where(ok.gather(1, keep), cand.gather(1, keep), ids[:, None]))
    width = max(r.shape[1] for r in rows)
    out = torch.arange(n, device=DEV)[:, None].repeat(1, width)
    a = 0
    for r in rows:
        out[a:a + r.shape[0], : r.shape[1]] = r
        a += r.shape[0]
    return out


def _basis(r, rc, K):
    """f_k(r) = (T_k(x) + 1) f_c / 2, x = 2 (r/rc - 1)^2 - 1, f_c = (1 + cos(pi r/rc)) / 2; zero from rc on."""
    fc = torch.where(r < rc, 0.5 * (1.0 + torch.cos(math.pi * r / rc)), torch.zeros_like(r))
    y = 2.0 * (r / rc - 1.0) ** 2 - 1.0
    T = [torch.ones_like(y), y]
    for _ in range(2, K):
        T.append(2.0 * y * T[-1] - T[-2])
    return torch.stack([0.5 * (t + 1.0) * fc for t in T], -1)


def _harmonics(u, lmax):
    """q_nl weights folded in: components Y with sum_m Y_lm(a) Y_lm(b) = P_l(a.b)."""
    x, y, z = u.unbind(-1)
    s = math.sqrt
    out = [[y, z, x]]
    out.append([s(3) * x * y, s(3) * y * z, 0.5 * (3 * z * z - 1), s(3) * x * z, 0.5 * s(3) * (x * x - y * y)])
    if lmax > 2:
        out.append([s(5 / 8) * y * (3 * x * x - y * y), s(15) * x * y * z, s(3 / 8) * y * (5 * z * z - 1),
                    0.5 * z * (5 * z * z - 3), s(3 / 8) * x * (5 * z * z - 1), 0.5 * s(15) * z * (x * x - y * y),
                    s(5 / 8) * x * (x * x - 3 * y * y)])
        x2, y2, z2 = x * x, y * y, z * z
        out.append([0.5 * s(35) * x * y * (x2 - y2), 0.25 * s(70) * y * z * (3 * x2 - y2),
                    0.5 * s(5) * x * y * (7 * z2 - 1), 0.25 * s(10) * y * z * (7 * z2 - 3),
                    (35 * z2 * z2 - 30 * z2 + 3) / 8, 0.25 * s(10) * x * z * (7 * z2 - 3),
                    0.25 * s(5) * (x2 - y2) * (7 * z2 - 1), 0.25 * s(70) * x * z * (x2 - 3 * y2),
                    s(35) / 8 * (x2 * x2 - 6 * x2 * y2 + y2 * y2)])
    return [torch.stack(c, -1) for c in out[:lmax]]


def _blocks(hp, p):
    T, nR, nA = hp.n_types, hp.n_max_radial + 1, hp.n_max_angular + 1
    kR, kA, H, D = hp.basis_radial + 1, hp.basis_angular + 1, hp.n_hidden, hp.n_desc
    shapes = [(T, T, nR, kR), (T, T, nA, kA), (D,), (H, D), (H,), (H,), (1,)]
    out, a = [], 0
    for s in shapes:
        k = math.prod(s)
        out.append(p[a:a + k].reshape(s))
        a += k
    return out


def _zbl(hp, r, zi, zj):
    a = 0.8854 * 0.529177210903 / (zi ** 0.23 + zj ** 0.23)
    phi = sum(c * torch.exp(-d * r / a) for c, d in
              ((0.18175, 3.19980), (0.50986, 0.94229), (0.28022, 0.40290), (0.02817, 0.20162)))
    ri, ro = hp.zbl_inner, hp.zbl_outer
    sw = 0.5 * (1.0 + torch.cos(math.pi * (r.clamp(ri, ro) - ri) / (ro - ri)))
    return 14.399645478 * zi * zj / r * phi * sw


def _site_energies(hp, p, d, real, ti, tj):
    """U_i [C] of C centers from pair vectors d [C][M][3] (real: not padding) and species."""
    cR, cA, sigma, W0, b0, w1, b1 = _blocks(hp, p)
    safe = torch.where(real[..., None], d, torch.tensor([1e3, 0.0, 0.0], device=DEV, dtype=torch.float64))
    r = torch.sqrt((safe * safe).sum(-1))
    kR, kA, L3 = hp.basis_radial + 1, hp.basis_angular + 1, hp.l_max_3b

    def channels(f, c):
        """sum_k c^{ti tj}_nk f_k: [C][M][n]"""
        if hp.n_types == 1:
            return f @ c[0, 0].T
        out = 0.0
        for a in range(hp.n_types):
            for b in range(hp.n_types):
                on = ((ti[:, None] == a) & (tj == b)).to(torch.float64)[..., None]
                out = out + on * (f @ c[a, b].T)
        return out

    q = [channels(_basis(r, hp.rc_radial, kR), cR).sum(1)]
    g = channels(_basis(r, hp.rc_angular, kA), cA)
    u = safe / r[..., None]
    ys = _harmonics(u, L3)
    for y in ys:
        s = (g[..., :, None] * y[..., None, :]).sum(1)
        q.append((s * s).sum(-1))
    if hp.l_max_4b == 2:
        eye = torch.eye(3, device=DEV, dtype=torch.float64) / 3.0
        S = (g[..., :, None, None] * (u[..., :, None] * u[..., None, :] - eye)[:, :, None]).sum(1)
        S2 = (S[..., :, :, None] * S[..., None, :, :]).sum(-2)
        q.append((S2 * S.transpose(-1, -2)).sum((-1, -2)))
    q = torch.cat(q, -1) * sigma
    U = torch.tanh(q @ W0.T - b0) @ w1 - b1
    if hp.zbl_outer > 0:
        z = torch.tensor(hp.zbl_z, device=DEV, dtype=torch.float64)
        e = _zbl(hp, torch.where(r < hp.zbl_outer, r, hp.zbl_outer * torch.ones_like(r)), z[ti.long()][:, None],
                 z[tj.long()])
        U = U + 0.5 * torch.where(r < hp.zbl_outer, e, torch.zeros_like(e)).sum(1)
    return U


def _chunks(x, types, box, table, rows):
    L = torch.tensor(box, device=DEV)
    for a in range(0, x.shape[0], rows):
        ids = torch.arange(a, min(x.shape[0], a + rows), device=DEV)
        j = table[ids]
        real = j != ids[:, None]
        d = x[j] - x[ids][:, None]
        d = d - L * torch.round(d / L)
        yield ids, j, real, d, types[ids], types[j]


def _evaluate(hp, params, x, types, box, table=None):
    """E (float), F [N][3], W [3][3], U [N] of the definition, FP64."""
    p = torch.as_tensor(params, dtype=torch.float64, device=DEV)
    table = _neighbour_table(x, box, hp.rc_radial) if table is None else table
    F = torch.zeros_like(x)
    U = torch.empty(x.shape[0], dtype=torch.float64, device=DEV)
    W = torch.zeros(3, 3, dtype=torch.float64, device=DEV)
    for ids, j, real, d, ti, tj in _chunks(x, types, box, table, 16384):
        d.requires_grad_(True)
        u = _site_energies(hp, p, d, real, ti, tj)
        g, = torch.autograd.grad(u.sum(), d)
        U[ids] = u.detach()
        F[ids] += g.sum(1)
        F.index_add_(0, j.reshape(-1), -g.reshape(-1, 3))
        W -= (d.detach()[..., :, None] * g[..., None, :]).sum((0, 1))
    return float(U.sum()), F, W, U


def _param_grad(hp, p, x, types, box, gE, gF):
    """d(gE E + sum gF . F)/dp, FP64."""
    p = torch.as_tensor(p, dtype=torch.float64, device=DEV).detach().clone().requires_grad_(True)
    table = _neighbour_table(x, box, hp.rc_radial)
    out = torch.zeros_like(p)
    for ids, j, real, d, ti, tj in _chunks(x, types, box, table, 4096):
        d.requires_grad_(True)
        u = _site_energies(hp, p, d, real, ti, tj)
        g, = torch.autograd.grad(u.sum(), d, create_graph=True)
        loss = gE * u.sum() + (g * (gF[ids][:, None] - gF[j])).sum()
        out += torch.autograd.grad(loss, p)[0]
    return out


def _trajectory(case, seed):
    hp, params, shp, sparams = _models(case, seed)
    x, v, types, box, masses = _atoms(case, seed)
    n, dt = x.shape[0], 1.0
    L = torch.tensor(box, device=DEV)
    m = torch.tensor(masses, device=DEV)[types.long()][:, None]
    inv = 1.0 / (m * XI)
    vol, rows = float(np.prod(box)), []

    def force(which):
        return _evaluate(*which, x, types, box)[:3]

    def kinetic():
        return 0.5 * XI * float((m * v * v).sum())

    def row(step, E, W, err=(0.0, 0.0)):
        ke = kinetic()
        rows.append([step, E, ke, 2.0 * ke / ((3.0 * n - 3.0) * KB), (2.0 * ke + float(W.trace())) / (3.0 * vol),
                     err[0], err[1], 0.0])

    full, sur, every, steps = (hp, params), (shp, sparams), _thermo_every(case), case["steps"]
    eta, ve = [0.0] * 3, [0.0] * 3

    def chain_half():
        """Half a step of a Nose-Hoover chain of three (explicit reversible Trotter form); scales v."""
        nonlocal v
        kT, tau2, nf, h, ke = KB * 300.0, 50.0 ** 2, 3.0 * n - 3.0, 0.5 * dt, kinetic()
        Q = [nf * kT * tau2, kT * tau2, kT * tau2]

        def pull(k):
            return ((2.0 * ke - nf * kT) if k == 0 else (Q[k - 1] * ve[k - 1] ** 2 - kT)) / Q[k]

        def damped(k):
            d = math.exp(-0.25 * h * ve[k + 1])
            ve[k] = (ve[k] * d + 0.5 * h * pull(k)) * d

        ve[2] += 0.5 * h * pull(2)
        damped(1)
        damped(0)
        scale = math.exp(-h * ve[0])
        ke *= scale * scale
        for k in range(3):
            eta[k] += h * ve[k]
        damped(0)
        damped(1)
        ve[2] += 0.5 * h * pull(2)
        v = v * scale

    if case["ensemble"] == "mts":
        (_, Ff, _), (_, Fs, _) = force(full), force(sur)
        for s in range(0, steps, 4):
            v = v + 0.5 * 4 * dt * (Ff - Fs) * inv
            for _ in range(4):
                v = v + 0.5 * dt * Fs * inv
                x = torch.remainder(x + dt * v, L)
                _, Fs, _ = force(sur)
                v = v + 0.5 * dt * Fs * inv
            E, Ff, W = force(full)
            d2 = ((Ff - Fs) ** 2).sum(1)
            v = v + 0.5 * 4 * dt * (Ff - Fs) * inv
            row(s + 4, E, W, (math.sqrt(float(d2.sum()) / (3 * n)), math.sqrt(float(d2.max()))))
    else:
        _, F, _ = force(full)
        for s in range(1, steps + 1):
            if case["ensemble"] == "nvt":
                chain_half()
            v = v + 0.5 * dt * F * inv
            x = torch.remainder(x + dt * v, L)
            E, F, W = force(full)
            v = v + 0.5 * dt * F * inv
            if case["ensemble"] == "nvt":
                chain_half()
            if s % every == 0 or s == steps:
                row(s, E, W)
    return {"x": x, "v": v, "thermo": np.array(rows)}


def exact(case, seed):
    """What ``run`` returns for these inputs, in FP64; None where it would take too long."""
    kind, n = case["kind"], _sites(case)
    hp, params, shp, sparams = _models(case, seed)
    if kind in ("serve", "frame"):
        x, _, types, box, _ = _atoms(case, seed)
        E, F, W, U = _evaluate(hp, params, x, types, box)
        return {"E": E, "W": W, "F": F, "U": U}
    if kind == "md":
        return None if n * (case["steps"] + 1) > 1200000 else _trajectory(case, seed)
    if kind == "fit_surrogate":
        theta = torch.tensor(sparams, dtype=torch.float32, device=DEV)
        m1, m2 = (m.double() for m in _moments(theta, seed))
        p, grad, energies, batch = theta.double(), 0.0, [], case["frames"]
        for f in range(batch):
            x, _, types, box, _ = _atoms(case, 64 * seed + f)
            e_ref, f_ref = _evaluate(hp, params, x, types, box)[:2]
            E, F = _evaluate(shp, p, x, types, box)[:2]
            grad = grad + _param_grad(shp, p, x, types, box, 2.0 * (E - e_ref) / n / n / batch,
                                      (2.0 / (3 * n * batch)) * (F - f_ref.to(torch.float32).double()))
            energies.append(E)
        grad[slice(*shp.offsets()["sigma"])] = 0.0
        t, b1, b2 = 101, 0.9, 0.999
        m1 = b1 * m1 + (1 - b1) * grad
        m2 = b2 * m2 + (1 - b2) * grad * grad
        p = p - 1e-4 * (m1 / (1 - b1 ** t)) / (torch.sqrt(m2 / (1 - b2 ** t)) + 1e-8)
        return {"E": energies, "grad": grad, "theta": p, "m1": m1, "m2": m2}
    if kind == "fit_network":
        theta = _student(hp, params, seed).double()
        p = torch.cat([torch.tensor(params[: hp.offsets()["W0"][0]], device=DEV), theta])
        loss, grad = 0.0, 0.0
        for f in range(case["frames"]):
            x, _, types, box, _ = _atoms(case, 64 * seed + f)
            e_ref, f_ref = _evaluate(hp, params, x, types, box)[:2]
            E, F = _evaluate(hp, p, x, types, box)[:2]
            de, dF = (E - e_ref) / n, F - f_ref.to(torch.float32).double()
            loss += (de * de + float((dF * dF).sum()) / (3 * n)) / case["frames"]
            grad = grad + _param_grad(hp, p, x, types, box, 2.0 * de / n / case["frames"],
                                      (2.0 / (3 * n * case["frames"])) * dF)
        return {"loss": loss, "grad": grad[hp.offsets()["W0"][0]:]}
    x, _, types, box, _ = _atoms(case, seed)
    E, F, W, U = _evaluate(hp, params, x, types, box)
    return {"E": E, "W": W, "F": F, "U": U,
            "grad": _param_grad(hp, params, x, types, box, GE, _force_weights(n, seed))}
