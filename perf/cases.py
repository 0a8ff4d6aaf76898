"""The work that programs built on this library have it do, one case per use, over the range of each use.

``listed`` gives fixed cases and ``draw`` others of the same ranges.  ``prepare`` makes what a program
holds before the call (inputs and a handle), ``run`` is one pass through the public entry points, ``exact``
computes the same outputs in float64 with plain torch, and ``work`` counts what a pass cannot do without.

Models, lattices, masses, parameter vectors and training-cell ranges are those of
``paper_2205_10046_amd/synth.py`` and ``bench.py``.

Types of the outputs: the library computes energies, forces, virials, descriptors and the sums made of them
in float32 and widens them at its interface, and the order of its float32 sums depends on the kernel shape
that a handle fixes by timing on its first evaluation, so two handles may differ in the last float32 bits.
A program that stores such results (trajectory frames, labelled structures) stores float32, and so do these
cases.  What is float64 by nature (the trainer's mean and scales) comes back as float64.
"""
import itertools
import math

import numpy as np
import torch

from paper_2205_10046_amd import nep, synth

CRYSTAL = {"diamond216": ("diamond", 5.43, 8), "fcc131k": ("fcc", 4.05, 4), "bcc2m": ("bcc", 3.16, 2),
           "serve2": ("fcc", 4.05, 4)}
SKIN = 0.8            # Angstrom, the benchmark's
TEMPERATURE = 300.0   # K
LOSS_WEIGHTS = (1.0, 1.0, 0.1, 1e-4, 1e-4)


def listed():
    return [
        # a single point of a small cell on host arrays: labelling, active learning, a script's first call
        dict(name="evaluate_diamond_216", path="evaluate", model="diamond216", nx=3, ny=3, nz=3, vacancies=0,
             shear=0.0, bf16=False),
        # one step of a relaxation of a mid-sized defective, sheared cell whose arrays stay on the GPU
        dict(name="evaluate_alloy_3995", path="evaluate_dev", model="fcc131k", nx=10, ny=10, nz=10, vacancies=5,
             shear=0.05, bf16=False),
        # a large cell with the bf16 network (the option that the benchmark reports beside float32)
        dict(name="evaluate_alloy_131072_bf16", path="evaluate_dev", model="fcc131k", nx=32, ny=32, nz=32,
             vacancies=0, shear=0.0, bf16=True),
        # one sample of a Green-Kubo run: per-atom heat currents and their total
        dict(name="heat_alloy_32000", path="heat_dev", model="fcc131k", nx=20, ny=20, nz=20, vacancies=0, shear=0.0,
             bf16=False),
        # descriptors of a snapshot for analysis (similarity, farthest-point sampling), on host arrays
        dict(name="descriptors_alloy_6912", path="descriptors", model="fcc131k", nx=12, ny=12, nz=12, vacancies=0,
             shear=0.0, bf16=False),
        # molecular dynamics between two frames: a small cell (launches count), the benchmark's alloy, and the
        # largest system with l_max = 6, 4-body and 5-body terms
        dict(name="md_alloy_2048", path="md_dev", model="fcc131k", nx=8, ny=8, nz=8, vacancies=0, steps=100),
        dict(name="md_alloy_131072", path="md_dev", model="fcc131k", nx=32, ny=32, nz=32, vacancies=0, steps=20),
        dict(name="md_bcc_2000000", path="md_dev", model="bcc2m", nx=100, ny=100, nz=100, vacancies=0, steps=10),
        # thermostatted equilibration on host arrays
        dict(name="nvt_alloy_5323", path="md_ensemble", model="fcc131k", nx=11, ny=11, nz=11, vacancies=1, steps=50,
             ensemble="nvt_berendsen"),
        # scoring a data set of small periodic cells with the current model
        dict(name="score_cells_1000", path="score", structures=1000),
        # one generation of the trainer: sample, evaluate the population, loss, update
        dict(name="generation_200x20", path="generation", structures=200, population=20),
        # a burst of requests to the server: single evaluations and short runs of mixed sizes
        dict(name="serve_10", path="serve", requests=10, largest=4000, steps=20),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def cells(lo, hi, per):  # a box that is not a cube, of about a drawn number of atoms
        side = (log_int(lo, hi) / per) ** (1 / 3)
        nx, ny = (max(3, round(side * rng.uniform(0.75, 1.3))) for _ in "xy")
        return dict(nx=nx, ny=ny, nz=max(3, round(side ** 3 / (nx * ny))))

    path = rng.choice(["evaluate", "evaluate_dev", "evaluate_dev", "heat_dev", "descriptors", "md_dev", "md_dev",
                       "md_ensemble", "score", "generation", "serve"])
    if path in ("evaluate", "evaluate_dev", "heat_dev", "descriptors"):
        model = rng.choice(["diamond216", "fcc131k", "fcc131k", "bcc2m"])
        # bf16 turns a last-bit change of a descriptor into one of 2^-8 here and there: it is drawn at sizes
        # where every handle fixes the same kernel shape
        bf16 = path == "evaluate_dev" and rng.random() < 0.2
        if bf16:
            model = "fcc131k"
        lo, hi = (110000, 160000) if bf16 else (110, 200000) if path.endswith("_dev") else (110, 20000)
        return dict(path=path, model=model, **cells(lo, hi, CRYSTAL[model][2]), vacancies=rng.randint(0, 9),
                    shear=rng.choice([0.0, 0.0, 0.03, 0.08]), bf16=bf16)
    if path == "md_dev":
        model = rng.choice(["fcc131k", "fcc131k", "bcc2m"])
        c = cells(600, 300000, CRYSTAL[model][2])
        n = c["nx"] * c["ny"] * c["nz"] * CRYSTAL[model][2]
        return dict(path=path, model=model, **c, vacancies=rng.randint(0, 9),
                    steps=10 * max(1, min(10, int(400000 / n))) + rng.choice([0, 0, 3]))
    if path == "md_ensemble":
        return dict(path=path, model="fcc131k", **cells(600, 30000, 4), vacancies=rng.randint(0, 9),
                    steps=rng.choice([20, 50]), ensemble=rng.choice(["nvt_berendsen", "nvt_nhc"]))
    if path == "score":
        return dict(path=path, structures=log_int(20, 2000))
    if path == "generation":
        return dict(path=path, structures=log_int(10, 300), population=rng.randint(8, 30))
    return dict(path=path, requests=rng.randint(4, 12), largest=log_int(500, 10000), steps=rng.choice([10, 20]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------


def _hyper(case):
    return synth.WORKLOADS[{"score": "train3", "generation": "train3", "serve": "serve2"}.get(case["path"]) or
                           case["model"]]


def _masses(case):
    return np.array(synth.MASSES[case["model"]])


def _atoms(case):
    return case["nx"] * case["ny"] * case["nz"] * CRYSTAL[case["model"]][2] - case["vacancies"]


def _crystal(case, seed, sigma):
    """Positions, species and box: a replicated crystal with thermal noise, vacancies and a shear."""
    kind, a, _ = CRYSTAL[case["model"]]
    pos, types, box = synth.lattice(kind, (case["nx"], case["ny"], case["nz"]), a, sigma, _hyper(case)["n_types"],
                                    seed)
    gone = np.random.default_rng(seed + 1).permutation(pos.shape[1])[:case["vacancies"]]
    pos, types = np.delete(pos, gone, axis=1), np.delete(types, gone)
    shear = case.get("shear", 0.0)
    pos[0] += shear * pos[1]
    box[3] = shear * box[4]
    return np.ascontiguousarray(pos), types, box


def _moving(case, seed):
    """A crystal at rest positions with velocities at 300 K and parameters that keep it solid."""
    h = _hyper(case)
    pos, types, box = _crystal(case, seed, 0.08 if case["model"] == "bcc2m" else 0.0)
    vel = synth.maxwell_velocities(_masses(case)[types], TEMPERATURE, seed + 2)
    params = synth.solid_params(h, nep.nep_num_descriptors(h), nep.nep_num_params(h), seed=seed + 3)
    return pos, vel, types, box, params


def _training_cells(count, seed):
    """Triclinic periodic cells of 8-256 atoms at 0.05-0.09 atoms per cubic Angstrom, 3 species at random."""
    rng = np.random.default_rng(seed)
    cells = []
    for n in np.random.default_rng(count).integers(8, 257, size=count):  # the sizes are the case's
        m = math.ceil(n ** (1 / 3))
        tilt = rng.uniform(-0.2, 0.2, size=(3, 3))
        np.fill_diagonal(tilt, 1.0)
        box = (n / rng.uniform(0.05, 0.09)) ** (1 / 3) * tilt
        site = np.stack(np.unravel_index(rng.permutation(m ** 3)[:n], (m, m, m)), 1)
        pos = ((site + 0.5 + rng.uniform(-0.2, 0.2, size=(n, 3))) / m) @ box
        cells.append((np.ascontiguousarray(pos.T), rng.integers(0, 3, size=n).astype(np.int32), box.reshape(9)))
    return cells


def _requests(case, seed):
    """Requests of log-uniform sizes from 64 atoms up, every other one a short run."""
    rng = np.random.default_rng(case["largest"])  # the sizes are the case's
    got = []
    for k in range(case["requests"]):
        kind, a, per = (("fcc", 4.05, 4), ("bcc", 3.16, 2))[k % 4 // 2]
        n = case["largest"] if k == 0 else math.exp(rng.uniform(math.log(64), math.log(case["largest"])))
        pos, types, box = synth.lattice(kind, max(2, round((n / per) ** (1 / 3))), a, 0.05, 2, seed + 10 * k)
        r = dict(pos=pos, types=types, box=box, kind=nep.NEP_REQ_EVAL)
        if k % 2:
            masses = np.array(synth.MASSES["serve2"])
            r.update(kind=nep.NEP_REQ_MD, masses=masses, n_steps=case["steps"],
                     vel=synth.maxwell_velocities(masses[types], TEMPERATURE, seed + 10 * k + 1))
        got.append(r)
    return got


def _targets(S, n, seed):
    """Reference energies per atom, forces and virials of a data set."""
    rng = np.random.default_rng(seed)
    return rng.normal(0, 0.3, size=S), rng.normal(0, 1.0, size=(3, n)), rng.normal(0, 0.3, size=(S, 6))


def _rates(n_params):
    return 1.0, (3.0 + math.log(n_params)) / (5.0 * math.sqrt(n_params))


def _random_params(h, seed):
    return synth.random_params(nep.nep_num_params(h), seed=seed)


def _gpu(a, dtype=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _empty(*shape):
    return torch.empty(*shape, dtype=torch.float64, device="cuda")


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------


def prepare(case, seed):
    s = dict(case=case)
    path, h = case["path"], _hyper(case)
    if path in ("evaluate", "evaluate_dev", "heat_dev", "descriptors"):
        pos, types, box = _crystal(case, seed, 0.05)
        n = pos.shape[1]
        s.update(pos=pos, types=types, box=box, handle=nep.Handle(
            h, _random_params(h, seed + 3), nep.NEP_MLP_BF16 if case["bf16"] else nep.NEP_MLP_FP32))
        if path.endswith("_dev"):
            s.update(pos=_gpu(pos), types=_gpu(types, torch.int32))
        if path == "evaluate_dev":
            s.update(energy=_empty(n), force=_empty(3, n), virial=_empty(9, n), totals=_empty(10))
        if path == "heat_dev":
            vel = synth.maxwell_velocities(_masses(case)[types], TEMPERATURE, seed + 2)
            s.update(vel=_gpu(vel), heat=_empty(3, n), total=_empty(3))
    elif path in ("md_dev", "md_ensemble"):
        pos, vel, types, box, params = _moving(case, seed)
        s.update(pos=pos, vel=vel, types=types, box=box, handle=nep.Handle(h, params, skin=SKIN))
        if path == "md_dev":
            s.update(pos=_gpu(pos), vel=_gpu(vel), types=_gpu(types, torch.int32),
                     thermo=_empty(case["steps"] // 10, 13))
        s.update(memory=None)  # the thermostat's, from the run before
    elif path in ("score", "generation"):
        pos, types, boxes, offsets = synth.concat_structures(_training_cells(case["structures"], seed))
        n, S, P = pos.shape[1], boxes.shape[0], case.get("population", 1)
        params = _random_params(h, seed + 3)
        s.update(pos=_gpu(pos), types=_gpu(types, torch.int32), boxes=boxes, offsets=offsets,
                 handle=nep.Handle(h, params), force=_empty(P, 3, n), totals=_empty(P, S, 10))
        if path == "score":
            s.update(energy=_empty(P, n), virial=_empty(P, 9, n))
        else:
            d = params.shape[0]
            e, f, w = _targets(S, n, seed + 4)
            s.update(generator=torch.Generator("cuda").manual_seed(seed), noise=_empty(P, d), population=_empty(P, d),
                     mean=_gpu(params), sigma=torch.full((d,), 0.02, dtype=torch.float64, device="cuda"),
                     loss=_empty(P, 6), targets=(_gpu(e), _gpu(f), _gpu(w)), done=0)
    else:
        handle = nep.Handle(h, _random_params(h, seed + 3))
        s.update(requests=_requests(case, seed), server=nep.Server(handle, 2 << 30, max_slots=64))
    return s


def _single(r, keys):
    return {k: r[k].astype(np.float32) for k in keys}


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "evaluate":
        return _single(s["handle"].compute(s["pos"], s["types"], s["box"]), ("U", "F", "W", "totals"))
    if path == "evaluate_dev":
        s["handle"].compute_dev(s["pos"], s["types"], s["box"], None, s["energy"], s["force"], s["virial"],
                                s["totals"])
        return dict(U=s["energy"].float(), F=s["force"].float(), W=s["virial"].float(), totals=s["totals"].float())
    if path == "heat_dev":
        s["handle"].heat_current_dev(s["pos"], s["vel"], s["types"], s["box"], None, s["heat"], s["total"])
        return dict(J=s["heat"].float(), total=s["total"].float())
    if path == "descriptors":
        return s["handle"].descriptors(s["pos"], s["types"], s["box"]).astype(np.float32)
    if path == "md_dev":
        s["handle"].md_run_dev(s["pos"], s["vel"], s["types"], _masses(case), s["box"], 1.0, case["steps"], 10,
                               s["thermo"])
        return dict(pos=s["pos"].float(), vel=s["vel"].float(), thermo=s["thermo"].float())
    if path == "md_ensemble":
        ens = dict(kind=case["ensemble"], temperature=TEMPERATURE, tau_t=100.0)
        r = s["handle"].md_run_ensemble(s["pos"], s["vel"], s["types"], _masses(case), s["box"], 1.0, case["steps"],
                                        10, ens, s["memory"])
        s["pos"], s["vel"], _, thermo, s["memory"] = r
        return _single(dict(pos=s["pos"], vel=s["vel"], thermo=thermo), ("pos", "vel", "thermo"))
    if path == "score":
        s["handle"].compute_batch(s["offsets"], s["pos"], s["types"], s["boxes"], None, s["energy"], s["force"],
                                  s["virial"], s["totals"])
        return dict(U=s["energy"].float(), F=s["force"].float(), W=s["virial"].float(), totals=s["totals"].float())
    if path == "generation":
        h, e_f_w = s["handle"], s["targets"]
        s["noise"].normal_(generator=s["generator"])
        h.snes_sample(s["mean"], s["sigma"], s["noise"], s["population"])
        h.compute_batch_dev(s["offsets"], s["pos"], s["types"], s["boxes"], s["population"], None, s["force"], None,
                            s["totals"], reuse_rows=s["done"] > 0)
        h.batch_loss(s["offsets"], s["force"], s["totals"], e_f_w[0], e_f_w[1], LOSS_WEIGHTS, s["loss"],
                     virial_target=e_f_w[2], params=s["population"])
        h.snes_step(s["mean"], s["sigma"], s["noise"], s["loss"], *_rates(s["mean"].shape[0]), loss_stride=6)
        s["done"] += 1
        return dict(loss=s["loss"].float(), force=s["force"].float(), totals=s["totals"].float(), mean=s["mean"],
                    sigma=s["sigma"])
    tickets = [s["server"].submit(**r) for r in s["requests"]]
    results = [s["server"].poll(t, wait_ms=-1) for t in tickets]
    return [_single(r, [k for k in ("U", "F", "W", "pos", "vel") if k in r]) for r in results]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------


def _flops(h, density, forces=True):
    """Operations of one atom's evaluation (a multiply-add is two): basis functions and contractions over the
    bonds of a shell of this density, the network, and the chain back to the partial forces."""
    p_r, p_a = (4 / 3 * math.pi * h[k] ** 3 * density for k in ("rc_radial", "rc_angular"))
    n_r, k_r, n_a, k_a = (h[k] + 1 for k in ("n_max_radial", "basis_radial", "n_max_angular", "basis_angular"))
    many = h["l_max_3b"] + (h["l_max_4b"] > 0) + (h["l_max_5b"] > 0)
    b = (h["l_max_3b"] + 1) ** 2 - 1
    nd = n_r + n_a * many
    f = p_r * (10 + 5 * k_r) + 2 * n_r * k_r * h["n_types"]
    f += p_a * (10 + 5 * k_a + 2 * n_a * k_a + 2 * b + 2 * n_a * b) + 3 * n_a * b
    if forces:
        f += 4 * nd * h["n_neurons"] + p_r * (9 + 12 * k_r) + 2 * n_r * k_r * h["n_types"]
        f += p_a * (30 + 12 * k_a + 4 * n_a * k_a + b * (4 * n_a + 10)) + 8 * n_a * b + 6 * p_r
    return f


def work(case):
    path, h = case["path"], _hyper(case)
    if path == "serve":
        total, flops = 0, 0.0
        for r in _requests(case, 0):
            n, steps = r["types"].shape[0], r.get("n_steps", 0)
            total += n * (28 + 104 + (72 if steps else 0))
            flops += n * (steps + 1) * _flops(h, n / np.linalg.det(r["box"].reshape(3, 3)))
        return dict(bytes=total, flops=float(flops))
    if path in ("score", "generation"):
        n, P = 132 * case["structures"], case.get("population", 1)
        per_set = 104 if path == "score" else 48  # outputs, or forces written and read against their targets
        return dict(bytes=n * 28 + P * (n * per_set + 80 * case["structures"]) +
                    (16 * P * nep.nep_num_params(h) if path == "generation" else 0),
                    flops=P * n * _flops(h, 0.07))
    kind, a, per = CRYSTAL[case["model"]]
    n = _atoms(case)
    per_atom = {"evaluate": 28 + 104, "evaluate_dev": 28 + 104, "heat_dev": 52 + 24, "md_dev": 100,
                "md_ensemble": 100, "descriptors": 28 + 8 * nep.nep_num_descriptors(h)}[path]
    return dict(bytes=n * per_atom,
                flops=n * case.get("steps", 1) * _flops(h, per / a ** 3, forces=path != "descriptors"))


# ---------------------------------------------------------------------------
# the same in float64, from the published definitions, with plain torch
# ---------------------------------------------------------------------------

KB = 8.617333262e-5                                              # eV/K
AMU_A2_FS2 = 1.66053906660e-27 * 1e10 / 1.602176634e-19          # 1 amu (Angstrom/fs)^2 in eV


def _there(a):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda" if torch.cuda.is_available() else "cpu")


def _pairs(pos, box, rc):
    """Every (i, j, displacement) with a length below rc, all periodic images, sorted by i."""
    H = box.reshape(3, 3)
    s, n = pos.T @ torch.linalg.inv(H), pos.shape[1]
    s = s - s.floor()
    width = torch.linalg.det(H) / torch.stack([torch.linalg.cross(H[(k + 1) % 3], H[(k + 2) % 3]).norm()
                                               for k in range(3)])
    nearest = bool((width > 2 * rc * (1 + 1e-9)).all())
    reach = [0, 0, 0] if nearest else [int(rc / float(w)) + 1 for w in width]
    images = list(itertools.product(*(range(-r, r + 1) for r in reach)))
    shift = torch.tensor(images, dtype=pos.dtype, device=pos.device)
    found = []
    step = max(1, (1 << 25) // (n * len(images)))
    for a in range(0, n, step):
        ds = s[None] - s[a:a + step, None]
        ds = (ds - ds.round())[:, :, None] if nearest else ds[:, :, None] + shift
        d = ds @ H
        near = (d * d).sum(-1) < rc * rc
        k = torch.arange(a, min(n, a + step), device=pos.device)
        near[k - a, k, images.index((0, 0, 0))] = False
        i, j, _ = near.nonzero(as_tuple=True)
        found.append((i + a, j, d[near]))
    return tuple(torch.cat(x) for x in zip(*found))


def _basis(r, rc, size):
    fc, x = 0.5 + 0.5 * torch.cos(math.pi * r / rc), 2 * (r / rc - 1) ** 2 - 1
    t = [torch.ones_like(x), x]
    while len(t) < size:
        t.append(2 * x * t[-1] - t[-2])
    return torch.stack([fc] + [0.5 * (t[k] + 1) * fc for k in range(1, size)], 1)


def _harmonics(u, L):
    """The real solid harmonics P_l^(m)(z) {Re, Im}(x + iy)^m at unit vectors, and for each the constant of the
    addition theorem; for each l: m = 0, then (Re, Im) of m = 1..l."""
    x, y, z = u.T
    re, im = [torch.ones_like(x)], [torch.zeros_like(x)]
    for _ in range(L):
        re, im = re + [x * re[-1] - y * im[-1]], im + [x * im[-1] + y * re[-1]]
    b, c = [], []
    for l in range(1, L + 1):
        p = np.polynomial.legendre.leg2poly([0] * l + [1])
        for m in range(l + 1):
            v = sum(float(p[k] * math.factorial(k) / math.factorial(k - m)) * z ** (k - m) for k in range(m, l + 1))
            norm = (2 * l + 1) / (4 * math.pi) * (2 if m else 1) * math.factorial(l - m) / math.factorial(l + m)
            b += [v * re[m]] + ([v * im[m]] if m else [])
            c += [norm] * (2 if m else 1)
    return torch.stack(b, 1), torch.tensor(c, dtype=u.dtype, device=u.device)


def _descriptors(h, c_r, c_a, ti, i, tj, d):
    """Descriptors of the atoms 0..n-1 from their entries (i, species of the neighbour, displacement)."""
    n, T = ti.shape[0], h["n_types"]
    r = d.norm(dim=1)
    f = _basis(r, h["rc_radial"], c_r.shape[3])
    sums = torch.zeros(n * T, f.shape[1], dtype=d.dtype, device=d.device).index_add(0, i * T + tj, f)
    q = [(c_r[ti] * sums.reshape(n, T, 1, -1)).sum((1, 3))]
    k = (r < h["rc_angular"]).nonzero(as_tuple=True)[0]
    i, tj, r, d = i[k], tj[k], r[k], d[k]
    g = (c_a[ti[i], tj] * _basis(r, h["rc_angular"], c_a.shape[3])[:, None]).sum(2)
    b, c = _harmonics(d / r[:, None], h["l_max_3b"])
    S = torch.zeros(n, g.shape[1], b.shape[1], dtype=d.dtype, device=d.device)
    S = S.index_add(0, i, g[:, :, None] * b[:, None])
    for l in range(1, h["l_max_3b"] + 1):
        m = slice(l * l - 1, (l + 1) ** 2 - 1)
        q.append((c[m] * S[..., m] ** 2).sum(-1))
    if h["l_max_4b"]:  # the cubic invariant of the traceless tensor sum g (u u - 1/3)
        zz, xz, yz, xy, diff = S[..., 3] * 2 / 3, S[..., 4] / 3, S[..., 5] / 3, S[..., 7] / 6, S[..., 6] / 3
        xx, yy = (diff - zz) / 2, (-diff - zz) / 2
        det = xx * (yy * zz - yz ** 2) - xy * (xy * zz - yz * xz) + xz * (xy * yz - yy * xz)
        q.append(-108 * math.sqrt(2 / 35) * (0.25 * math.sqrt(5 / math.pi)) ** 3 * det)
    if h["l_max_5b"]:
        q.append(7 / 15 * q[1] ** 2)
    return torch.cat(q, 1)


class _Model:
    def __init__(self, h, params):
        p, T = _there(params), h["n_types"]
        n_r, k_r, n_a, k_a = (h[k] + 1 for k in ("n_max_radial", "basis_radial", "n_max_angular", "basis_angular"))
        nn, nd, nets = h["n_neurons"], nep.nep_num_descriptors(h), T if h["nn_per_type"] else 1
        self.h = h
        w = p[:nets * nn * (nd + 2)].reshape(nets, -1)
        self.w0, self.b0, self.w1 = w[:, :nn * nd].reshape(nets, nn, nd), w[:, nn * nd:-nn], w[:, -nn:]
        self.b1 = p[nets * nn * (nd + 2)]
        at = nets * nn * (nd + 2) + 1
        self.c_r = p[at:at + T * T * n_r * k_r].reshape(T, T, n_r, k_r)
        self.c_a = p[at + T * T * n_r * k_r:].reshape(T, T, n_a, k_a)

    def chunks(self, types, entries, at_once=4096):
        i, j, d = entries
        for a in range(0, types.shape[0], at_once):
            b = min(types.shape[0], a + at_once)
            lo, hi = (int(torch.searchsorted(i, k)) for k in (a, b))
            yield a, b, i[lo:hi], j[lo:hi], d[lo:hi]

    def descriptors(self, types, entries):
        return torch.cat([_descriptors(self.h, self.c_r, self.c_a, types[a:b], i - a, types[j], d)
                          for a, b, i, j, d in self.chunks(types, entries)])

    def evaluate(self, types, entries):
        """Site energies, forces (3, n) and per-atom virials (9, n)."""
        n = types.shape[0]
        U, F, W = (entries[2].new_zeros(n, *k) for k in ((), (3,), (9,)))
        for a, b, i, j, d in self.chunks(types, entries):
            d = d.clone().requires_grad_()
            q = _descriptors(self.h, self.c_r, self.c_a, types[a:b], i - a, types[j], d)
            u = torch.zeros_like(q[:, 0])
            for t in range(self.w0.shape[0]):
                k = (types[a:b] == t).nonzero(as_tuple=True)[0] if self.w0.shape[0] > 1 else slice(None)
                site = torch.tanh(q[k] @ self.w0[t].T.contiguous() - self.b0[t]) @ self.w1[t] - self.b1
                u = u.index_put((k,), site) if self.w0.shape[0] > 1 else site
            p, = torch.autograd.grad(u.sum(), d)
            U[a:b] = u.detach()
            F.index_add_(0, i, p).index_add_(0, j, -p)
            W.index_add_(0, j, -(d.detach()[:, :, None] * p[:, None]).reshape(-1, 9))
        return U, F.T, W.T

    def crystal(self, pos, types, box):
        return self.evaluate(types, _pairs(pos, box, self.h["rc_radial"]))


def _totals(U, W):
    return torch.cat([U.sum()[None], W.sum(1)])


def _dynamics(model, pos, vel, types, masses, box, steps, every, berendsen=None):
    """Velocity Verlet at 1 fs; thermo rows [step, E_pot, E_kin, T, virial]; Berendsen's scaling after a step."""
    m = masses[types.long()] * AMU_A2_FS2
    U, F, W = model.crystal(pos, types, box)
    rows = []
    for k in range(1, steps + 1):
        vel = vel + 0.5 * F / m
        pos = pos + vel
        U, F, W = model.crystal(pos, types, box)
        vel = vel + 0.5 * F / m
        kinetic = 0.5 * (m * vel * vel).sum()
        temperature = 2 * kinetic / ((3 * m.shape[0] - 3) * KB)
        if berendsen:
            vel = vel * torch.sqrt(1 + (TEMPERATURE / temperature - 1) / berendsen)
        if every and k % every == 0:
            rows.append(torch.cat([torch.stack([torch.full_like(kinetic, k), U.sum(), kinetic, temperature]),
                                   W.sum(1)]))
    return pos, vel, rows, (U, F, W)


def exact(case, seed):
    path, h = case["path"], _hyper(case)
    if path in ("md_dev", "md_ensemble"):
        if _atoms(case) * case["steps"] > 500000 or case.get("ensemble", "nvt_berendsen") != "nvt_berendsen":
            return None
        pos, vel, types, box, params = _moving(case, seed)
        pos, vel, rows, _ = _dynamics(_Model(h, params), _there(pos), _there(vel), _there(types),
                                      _there(_masses(case)), _there(box), case["steps"], 10,
                                      100.0 if path == "md_ensemble" else None)
        return dict(pos=pos, vel=vel, thermo=torch.stack(rows) if path == "md_dev" else None)
    if path == "serve":
        model, got = _Model(h, _random_params(h, seed + 3)), []
        for r in _requests(case, seed):
            pos, types, box = _there(r["pos"]), _there(r["types"]), _there(r["box"])
            if r["kind"] == nep.NEP_REQ_EVAL:
                got.append(dict(zip("UFW", model.crystal(pos, types, box))))
            else:
                pos, vel, _, last = _dynamics(model, pos, _there(r["vel"]), types, _there(r["masses"]), box,
                                              r["n_steps"], 0)
                got.append(dict(zip("UFW", last), pos=pos, vel=vel))
        return got
    if path in ("score", "generation"):
        return _exact_cells(case, seed, h)
    pos, types, box = (_there(a) for a in _crystal(case, seed, 0.05))
    model = _Model(h, _random_params(h, seed + 3))
    if path == "descriptors":
        return model.descriptors(types, _pairs(pos, box, h["rc_radial"]))
    U, F, W = model.crystal(pos, types, box)
    if path == "heat_dev":
        vel = _there(synth.maxwell_velocities(_masses(case)[types.cpu().numpy()], TEMPERATURE, seed + 2))
        # (the total is a sum that cancels: what is left of the float32 errors in it is a matter of luck)
        return dict(J=(W.reshape(3, 3, -1) * vel).sum(1), total=None)
    return dict(U=U, F=F, W=W, totals=_totals(U, W))


def _exact_cells(case, seed, h):
    cells = _training_cells(case["structures"], seed)
    pos, types, _, offsets = synth.concat_structures(cells)
    n, S = pos.shape[1], len(cells)
    entries = [_pairs(_there(p), _there(b), h["rc_radial"]) for p, _, b in cells]
    entries = (torch.cat([e[0] + int(o) for e, o in zip(entries, offsets)]),
               torch.cat([e[1] + int(o) for e, o in zip(entries, offsets)]), torch.cat([e[2] for e in entries]))
    types, sizes = _there(types), _there(np.diff(offsets))
    which = torch.repeat_interleave(torch.arange(S, device=types.device), sizes)
    params = _random_params(h, seed + 3)

    def one(vector):
        U, F, W = _Model(h, vector).evaluate(types, entries)
        return U, F, W, torch.zeros(S, 10, dtype=U.dtype, device=U.device).index_add(
            0, which, torch.cat([U[None], W]).T.contiguous())

    if case["path"] == "score":
        return dict(zip(("U", "F", "W", "totals"), (x[None] for x in one(params))))
    if case["population"] * n > 1200000 or not torch.cuda.is_available():  # the draws are the GPU's
        return None
    P, d = case["population"], params.shape[0]
    mean, sigma = _there(params), torch.full((d,), 0.02, dtype=torch.float64, device="cuda")
    noise = _empty(P, d).normal_(generator=torch.Generator("cuda").manual_seed(seed))
    population = mean + sigma * noise
    e, f, w = (_there(t) for t in _targets(S, n, seed + 4))
    losses, forces, totals = [], [], []
    for z in population:
        _, F, _, t = one(z.cpu().numpy())
        mine = t / sizes[:, None]
        parts = [((mine[:, 0] - e) ** 2).mean().sqrt(), ((F - f) ** 2).mean().sqrt(),
                 ((mine[:, [1, 5, 9, 2, 6, 7]] - w) ** 2).mean().sqrt(), z.abs().mean(), (z * z).mean().sqrt()]
        losses.append(torch.stack([sum(a * b for a, b in zip(LOSS_WEIGHTS, parts))] + parts))
        forces.append(F)
        totals.append(t)
    losses = torch.stack(losses)
    raw = torch.clamp(math.log(P / 2 + 1) - torch.log(torch.arange(1, P + 1, dtype=torch.float64, device="cuda")), 0)
    use = (raw / raw.sum() - 1 / P)[losses[:, 0].argsort().argsort()]
    step_mean, step_sigma = _rates(d)
    return dict(loss=losses, force=torch.stack(forces), totals=torch.stack(totals),
                mean=mean + step_mean * sigma * (use @ noise),
                sigma=sigma * torch.exp(0.5 * step_sigma * (use @ (noise * noise - 1))))
