"""What the library is timed on: energy-and-force calls as programs make them.

A program keeps one model (weights uploaded, workspace reserved, topology
known from its first call) and calls it once per step with positions that lie
on the GPU.  The engine around it stores forces and energies in its own
mixed-precision arrays (FP32, the ``real`` of a mixed-precision MD engine), so
every pass ends with one conversion of the library's FP64 results.

Kinds of work (``case["kind"]``):

* ``md``      an MD step of a periodic water box, whole system in the index
              group (the water-box scaling benchmark): 64 to 87,000 molecules,
              FP32 and BF16 forms, one network or an ensemble;
* ``relax``   energy and gradient through autograd (geometry optimisation, a
              loss on the energy);
* ``ligand``  a group of molecules inside a larger box, neighbours from the
              MD engine's pair list;
* ``batch``   many separate H/C/N/O molecules in one call (conformers);
* ``replica`` many small periodic water boxes in one call (lambda windows);
* ``embed``   an H/C/N/O solute in fixed-charge MM water through the MM
              potential channel, with or without charges predicted by the
              network, forces on ML and MM atoms;
* ``couple``  the mechanical-embedding Coulomb and Lennard-Jones term.

``tune`` runs the library's tuner once, as the benchmark and a long run of one
large box do.  ``network`` pins a network kernel (-1: the library's choice), as
a program does that keeps the tuner's earlier answer for its box.
"""
import math

import numpy as np
import torch

import paper_2604_21441_amd as nnp

KE = 14.3996454784
VOLUME = 12.42 ** 3 / 64          # A^3 per water molecule at 1.0 g/cm^3
OH, HOH = 0.9572, math.radians(104.52)


# ------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest box of the water-box benchmark: launches and latency
        {"name": "water192", "kind": "md", "n_mol": 64, "prec": "fp32", "members": 1, "tune": False, "network": -1},
        # a ligand-sized ML region in 30,000 MM charges, electrostatic embedding
        {"name": "solute60_mm30000", "kind": "embed", "n_solute": 60, "n_water": 10000, "charges": False,
         "prec": "fp32"},
        # the MM-level coupling of the same system
        {"name": "couple60_30000", "kind": "couple", "n_solute": 60, "n_water": 10000, "cutoff": 12.0},
        # one step of a geometry optimisation through autograd, 700 waters
        {"name": "relax2100", "kind": "relax", "n_mol": 700, "prec": "fp32"},
        # 300 ML waters in a box of 4,096, the engine's pair list
        {"name": "ligand900", "kind": "ligand", "n_mol": 4096, "n_group": 300, "prec": "fp32"},
        # the NVE benchmark box in both forms, and with the eight networks of an ANI ensemble
        {"name": "water12288", "kind": "md", "n_mol": 4096, "prec": "fp32", "members": 1, "tune": False, "network": -1},
        {"name": "water12288_bf16", "kind": "md", "n_mol": 4096, "prec": "bf16", "members": 1, "tune": False,
         "network": -1},
        {"name": "water12288_ens8", "kind": "md", "n_mol": 4096, "prec": "fp32", "members": 8, "tune": False,
         "network": -1},
        # large boxes, tuned once as the benchmark does
        {"name": "water98304", "kind": "md", "n_mol": 32768, "prec": "fp32", "members": 1, "tune": True, "network": -1},
        {"name": "water261000", "kind": "md", "n_mol": 87000, "prec": "fp32", "members": 1, "tune": True,
         "network": -1},
        # the largest box in the BF16 form with the network kernel the tuner picks for it
        {"name": "water261000_bf16", "kind": "md", "n_mol": 87000, "prec": "bf16", "members": 1, "tune": False,
         "network": 9},
        # conformers: 256 molecules of 24 to 300 atoms
        {"name": "batch256", "kind": "batch", "n_sys": 256, "prec": "fp32"},
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))) if hi > lo else lo


def draw(rng):
    """One more case: sizes log-uniform over the listed range, odd ones among them."""
    kind = rng.choice(["md", "md", "md", "md", "relax", "ligand", "batch", "replica", "embed", "couple"])
    prec = "bf16" if rng.random() < 0.25 else "fp32"
    if kind == "md":
        if rng.random() < 0.2:
            return {"kind": "md", "n_mol": _log_int(rng, 64, 4096), "prec": "fp32", "members": rng.randint(2, 8),
                    "tune": False, "network": -1}
        n = _log_int(rng, 64, 86999)
        big = n >= 20000
        return {"kind": "md", "n_mol": n, "prec": prec, "members": 1, "tune": big and prec == "fp32",
                "network": 9 if big and prec == "bf16" else -1}
    if kind == "relax":
        return {"kind": "relax", "n_mol": _log_int(rng, 64, 4096), "prec": "fp32"}
    if kind == "ligand":
        n = _log_int(rng, 512, 16384)
        return {"kind": "ligand", "n_mol": n, "n_group": _log_int(rng, 5, n // 4), "prec": "fp32"}
    if kind == "batch":
        return {"kind": "batch", "n_sys": _log_int(rng, 1, 255), "prec": prec}
    if kind == "replica":
        return {"kind": "replica", "n_sys": _log_int(rng, 2, 64), "n_mol": _log_int(rng, 64, 128), "prec": "fp32"}
    if kind == "embed":
        return {"kind": "embed", "n_solute": _log_int(rng, 14, 107), "n_water": _log_int(rng, 1000, 9999),
                "charges": rng.random() < 0.5, "prec": "fp32"}
    return {"kind": "couple", "n_solute": _log_int(rng, 14, 107), "n_water": _log_int(rng, 1000, 9999),
            "cutoff": rng.choice([9.0, 10.0, 12.0])}


# ------------------------------------------------------------------ inputs
def _config(kind):
    """Hyper-parameters of the two descriptor networks (values as FP32)."""
    f = np.float32
    species = (1, 8) if kind == "water" else (1, 6, 7, 8)
    s = len(species)
    d = 16 * s + 16 * s * (s + 1)
    extra = 1 if kind in ("mm", "ee") else 0
    hidden = (160, 128, 96) if kind == "water" else (256, 192, 160)
    return {"species": species, "rc_rad": f(5.2), "rc_ang": f(3.5), "eta_rad": f(19.7), "eta_ang": f(12.5),
            "zeta": f(14.1), "rad_shift": np.linspace(0.9, 5.2, 16).astype(f),
            "ang_shift": np.linspace(0.9, 3.5, 8).astype(f),
            "ang_sect": ((2 * np.arange(4) + 1) * math.pi / 8).astype(f),
            "widths": (d + extra,) + hidden + (2 if kind == "ee" else 1,), "celu_alpha": f(0.1),
            "extra_inputs": extra, "mm_cutoff": f(12.0), "ke_coulomb": KE}


def _weights(cfg, seed, members=1):
    """Xavier-normal weights per (member, species, layer), flat FP32 in the library's order; the
    output bias is a binding energy of a few eV per atom, as a fitted model has."""
    rng = np.random.Generator(np.random.PCG64(seed + 17))
    w, out = cfg["widths"], []
    for _ in range(members * len(cfg["species"])):
        for fi, fo in zip(w[:-1], w[1:]):
            out.append(rng.standard_normal(fi * fo, dtype=np.float32) * np.float32(math.sqrt(2.0 / (fi + fo))))
            out.append(rng.standard_normal(fo, dtype=np.float32) * np.float32(0.1))
        out[-1][0] -= np.float32(3.0)
    return np.concatenate(out)


def _water(n_mol, seed, edge=None):
    """Rigid waters on a jittered lattice with random orientations: pos [3 n, 3] FP32, Z, L."""
    rng = np.random.Generator(np.random.PCG64(seed + 5))
    L = float(np.float32(edge if edge else (n_mol * VOLUME) ** (1 / 3)))
    side = math.ceil(n_mol ** (1 / 3) - 1e-9)
    site = np.arange(side ** 3) if side ** 3 == n_mol else np.sort(rng.permutation(side ** 3)[:n_mol])
    o = (np.stack(np.unravel_index(site, (side,) * 3), 1) + 0.5) * (L / side) + rng.uniform(-0.3, 0.3, (n_mol, 3))
    q = rng.standard_normal((n_mol, 4))
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    w, x, y, z = q.T
    ex = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y + z * w), 2 * (x * z - y * w)], 1)
    ez = np.stack([2 * (x * z + y * w), 2 * (y * z - x * w), 1 - 2 * (x * x + y * y)], 1)
    p = np.empty((n_mol, 3, 3))
    p[:, 0] = o
    p[:, 1] = o + OH * (math.sin(HOH / 2) * ex + math.cos(HOH / 2) * ez)
    p[:, 2] = o + OH * (-math.sin(HOH / 2) * ex + math.cos(HOH / 2) * ez)
    return p.reshape(-1, 3).astype(np.float32), np.tile(np.array([8, 1, 1], np.int32), n_mol), L


def _molecules(sizes, seed):
    """Self-avoiding walks (bonds 1.0 to 1.5 A, no pair below 0.9 A, H/C/N/O 5:3:1:1), all grown together."""
    dev, m, K = "cuda", len(sizes), 12
    g = torch.Generator(device=dev).manual_seed(seed + 29)
    n = torch.tensor(sizes, device=dev)
    top = int(max(sizes))
    at = torch.full((m, top, 3), 1e4, device=dev, dtype=torch.float64)
    at[:, 0] = 20.0
    have = torch.ones(m, dtype=torch.long, device=dev)
    rows = torch.arange(m, device=dev)
    step = 0
    while step % 50 or bool((have < n).any()):
        step += 1
        v = torch.randn((m, K, 3), generator=g, device=dev, dtype=torch.float64)
        u = torch.rand((m, K, 2), generator=g, device=dev, dtype=torch.float64)
        anchor = have[:, None].expand(m, K) - 1
        late = torch.arange(K, device=dev) >= K - 4      # the last proposals start from earlier atoms
        anchor = torch.where(late, (u[..., 1] * have[:, None]).long().clamp(max=top - 1), anchor)
        p = at[rows[:, None], anchor] + v / v.norm(dim=-1, keepdim=True) * (1.0 + 0.5 * u[..., :1])
        ok = (torch.cdist(p, at) >= 0.9).all(-1) & (p >= 0).all(-1) & (p < 40).all(-1)
        pick = torch.argmax(ok.to(torch.int8), 1)
        grow = ok.any(1) & (have < n)
        slot = torch.where(grow, have, torch.zeros_like(have))
        at[rows, slot] = torch.where(grow[:, None], p[rows, pick], at[rows, slot])
        have += grow
    keep = torch.arange(top, device=dev)[None] < n[:, None]
    z = torch.tensor([1, 1, 1, 1, 1, 6, 6, 6, 7, 8], device=dev)
    z = z[torch.randint(0, 10, (int(n.sum()),), generator=g, device=dev)]
    return at[keep].float().cpu().numpy(), z.cpu().numpy().astype(np.int32)


def _solute_box(case, seed):
    """A walk solute at the centre of a box of MM water: ML and MM positions, Z, L."""
    sites = math.ceil((1.065 * case["n_water"]) ** (1 / 3) - 1e-9) ** 3
    L = max((sites * VOLUME) ** (1 / 3), 2 * 12.0 + 1.0)
    sp, sz = _molecules([case["n_solute"]], seed)
    sp = (sp.astype(np.float64) - 20.0 + L / 2).astype(np.float32)
    wp, _, L = _water(sites, seed, L)
    far = np.ones(sites, bool)
    for a in sp.astype(np.float64):      # waters within 2 A of the solute are left out
        d = wp.astype(np.float64) - a
        d -= L * np.rint(d / L)
        far &= ((d * d).sum(1) > 4.0).reshape(-1, 3).all(1)
    keep = np.nonzero(far)[0][:case["n_water"]]
    return sp, sz, np.ascontiguousarray(wp.reshape(-1, 3, 3)[keep].reshape(-1, 3)), L


def _inputs(case, seed):
    """Host arrays of one case from the seed alone."""
    kind, d = case["kind"], {}
    if kind in ("md", "relax", "ligand"):
        d["pos"], d["Z"], L = _water(case["n_mol"], seed)
        d["box"] = np.full(3, L, np.float32)
        d["cfg"] = _config("water")
        if kind == "ligand":             # the molecules nearest to the box centre, in the engine's atom order
            r = ((d["pos"].reshape(-1, 3, 3)[:, 0].astype(np.float64) - L / 2) ** 2).sum(1)
            mol = np.sort(np.argsort(r)[:case["n_group"]])
            d["group"] = (3 * mol[:, None] + np.arange(3)).reshape(-1).astype(np.int32)
    elif kind == "batch":
        rng = np.random.Generator(np.random.PCG64(case["n_sys"]))   # the sizes belong to the case
        sizes = np.exp(rng.uniform(math.log(24), math.log(301), case["n_sys"])).astype(np.int64).clip(24, 300)
        d["pos"], d["Z"] = _molecules([int(v) for v in sizes], seed)
        d["offsets"] = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        d["cfg"] = _config("hcno")
    elif kind == "replica":
        each = [_water(case["n_mol"], seed + 1000 * k) for k in range(case["n_sys"])]
        d["pos"] = np.concatenate([e[0] for e in each])
        d["Z"] = np.concatenate([e[1] for e in each])
        d["offsets"] = (3 * case["n_mol"] * np.arange(case["n_sys"] + 1)).astype(np.int32)
        d["boxes"] = np.array([[e[2]] * 3 for e in each], np.float32)
        d["cfg"] = _config("water")
    else:
        d["pos"], d["Z"], d["mm_pos"], L = _solute_box(case, seed)
        d["box"] = np.full(3, L, np.float32)
        n_w = len(d["mm_pos"]) // 3
        d["mm_q"] = np.tile(np.array([-0.834, 0.417, 0.417], np.float32), n_w)
        if kind == "embed":
            d["cfg"] = _config("ee" if case["charges"] else "mm")
        else:
            rng = np.random.Generator(np.random.PCG64(seed + 4))
            q = rng.uniform(-0.6, 0.6, len(d["Z"]))
            lj = {1: (2.5, 0.0013), 6: (3.4, 0.0037), 7: (3.25, 0.0073), 8: (3.0, 0.0091)}
            d["ml_par"] = np.array([[c - q.mean(), *lj[int(z)]] for c, z in zip(q, d["Z"])], np.float32)
            d["mm_par"] = np.tile(np.array([[-0.834, 3.1507, 0.0065955], [0.417, 0, 0], [0.417, 0, 0]], np.float32),
                                  (n_w, 1))
    if "cfg" in d:
        d["members"] = case.get("members", 1)
        d["weights"] = _weights(d["cfg"], seed, d["members"])
    return d


def _engine_pairs(pos, group, L, reach):
    """Half pair list of the group's atoms within `reach`, int32 [n, 2] on the GPU."""
    g = torch.from_numpy(group).cuda().long()
    p = pos[g]
    out = []
    for a in range(0, len(g), 2048):
        x = p[a:a + 2048, None] - p[None]
        x = x - L * torch.round(x / L)
        i, j = torch.nonzero((x * x).sum(-1) < reach * reach, as_tuple=True)
        i = i + a
        out.append(torch.stack([g[i[i < j]], g[j[i < j]]], 1))
    return torch.cat(out).to(torch.int32).contiguous()


def prepare(case, seed):
    d = _inputs(case, seed)
    s = {"kind": case["kind"], "case": case}
    pos = torch.from_numpy(d["pos"]).cuda()
    n = len(pos)
    n_mm = len(d["mm_pos"]) if "mm_pos" in d else 0
    n_e = len(d["offsets"]) - 1 if "offsets" in d else 1
    # the library's FP64 results in one buffer, the engine's FP32 copy in another
    buf = torch.zeros(3 * (n + n_mm) + n_e, dtype=torch.float64, device="cuda")
    own = torch.empty_like(buf, dtype=torch.float32)

    def views(b):
        return b[:3 * n].view(n, 3), b[3 * n:3 * (n + n_mm)].view(n_mm, 3), b[3 * (n + n_mm):]

    F, Fmm, E = views(buf)
    s |= {"pos": pos, "box": d.get("box"), "buf": buf, "own": own, "E": E, "F": F, "Fmm": Fmm}
    f, fmm, e = views(own)
    s["result"] = {"energy": e, "forces": f} | ({"mm_forces": fmm} if n_mm else {})
    if n_mm:
        s["mm_pos"] = torch.from_numpy(d["mm_pos"]).cuda()
        s["mm_q"] = torch.from_numpy(d["mm_q"]).cuda()
    if case["kind"] == "couple":
        s["ml_par"] = torch.from_numpy(d["ml_par"]).cuda()
        s["mm_par"] = torch.from_numpy(d["mm_par"]).cuda()
        return s
    m = nnp.NNPModel(d["cfg"], weights=d["weights"], precision=case["prec"], n_members=d["members"])
    s["model"] = m
    if case.get("network", -1) >= 0:
        m.set_variant("network", case["network"])
    # the first evaluation of a run: topology, workspace, graph
    if case["kind"] == "relax":
        s["x"] = pos.requires_grad_(True)
        m.energy(s["x"], d["Z"], s["box"])
    elif case["kind"] == "ligand":
        s["group"] = d["group"]
        s["pairs"] = _engine_pairs(pos, d["group"], float(d["box"][0]), 5.2 + 0.5)
        m.compute_pairs(pos, s["pairs"], d["Z"], s["box"], d["group"], out=(E, F, None))
    elif "offsets" in d:
        s["offsets"], s["boxes"] = d["offsets"], d.get("boxes")
        m.compute_batch(pos, d["Z"], s["offsets"], s["boxes"], out=(E, F))
    elif n_mm:
        m.compute(pos, d["Z"], s["box"], None, s["mm_pos"], s["mm_q"], out=(E, F, Fmm))
    else:
        m.compute(pos, d["Z"], s["box"], out=(E, F, None))
    if case.get("tune"):
        m.autotune()
    return s


def run(s):
    kind = s["kind"]
    if kind == "relax":
        e = s["model"].energy(s["x"], None, s["box"]).float()
        g, = torch.autograd.grad(e, s["x"])
        return {"energy": e.detach(), "gradient": g}
    if kind == "couple":
        nnp.nnp_me_coupling(s["pos"], s["ml_par"], s["mm_pos"], s["mm_par"], s["box"], s["case"]["cutoff"],
                            out=(s["E"], s["F"], s["Fmm"]))
    elif kind == "ligand":
        s["model"].compute_pairs(s["pos"], s["pairs"], None, s["box"], s["group"], out=(s["E"], s["F"], None))
    elif kind in ("batch", "replica"):
        s["model"].compute_batch(s["pos"], None, s["offsets"], s["boxes"], out=(s["E"], s["F"]))
    elif kind == "embed":
        s["model"].compute(s["pos"], None, s["box"], None, s["mm_pos"], s["mm_q"], out=(s["E"], s["F"], s["Fmm"]))
    else:
        s["model"].compute(s["pos"], None, s["box"], out=(s["E"], s["F"], None))
    s["own"].copy_(s["buf"])
    return s["result"]


# -------------------------------------------------------------------- work
def work(case):
    """Positions and charges in, forces and energies out, each weight once; arithmetic of the
    descriptors (155 + 200 operations per radial pair, 150 + 300 per triplet, forward and adjoint)
    and of the networks (two per multiply-add), at 59 pairs and 153 triplets per atom."""
    kind = case["kind"]
    if kind == "couple":
        n, q = case["n_solute"], 3 * case["n_water"]
        return {"bytes": (n + q) * (24 + 24), "flops": 30.0 * n * q}
    n = {"md": 3 * case.get("n_mol", 0), "relax": 3 * case.get("n_mol", 0), "ligand": 3 * case.get("n_group", 0),
         "batch": 121 * case.get("n_sys", 0), "replica": 3 * case.get("n_mol", 0) * case.get("n_sys", 0),
         "embed": case.get("n_solute", 0)}[kind]
    k = case.get("members", 1)
    water = kind in ("md", "relax", "ligand", "replica")
    net = 213184 if water else 713024
    wts = (106784 if water else 4 * 178336) * k * (2 if case.get("prec") == "bf16" else 4)
    flops = n * (59 * 355 + 153 * 450 + net * k)
    if kind == "embed":
        flops += 40.0 * n * 3 * case["n_water"]
    rows = 3 * case["n_mol"] if kind == "ligand" else n + (3 * case["n_water"] if kind == "embed" else 0)
    return {"bytes": float(rows * (12 + 24) + wts), "flops": float(flops)}


# ------------------------------------------------------------------- exact
def _pairs64(x32, L, sys, reach):
    """All ordered pairs (i, j) within `reach`, sorted by i, by direct search in blocks of rows."""
    n, out = len(x32), []
    step = max(256, min(n, (1 << 29) // n))
    for a in range(0, n, step):
        r2 = torch.zeros((min(step, n - a), n), device="cuda")
        for k in range(3):
            t = x32[a:a + step, k, None] - x32[None, :, k]
            if L is not None:
                w = L[k] if not torch.is_tensor(L) else L[sys[a:a + step], k, None]
                t -= torch.round(t / w) * w
            r2.addcmul_(t, t)
        near = r2 < (reach + 1e-3) ** 2
        if sys is not None:
            near &= sys[a:a + step, None] == sys[None]
        near[torch.arange(len(near)), torch.arange(a, a + len(near))] = False
        i, j = torch.nonzero(near, as_tuple=True)
        out.append((i + a, j))
        del r2, t, near
    return torch.cat([o[0] for o in out]), torch.cat([o[1] for o in out])


def _exact_model(d, phi=None):
    """Atomic energies and -dE/dx in float64 (torch autograd), in blocks of centre atoms.
    phi: function of positions giving the MM potential of a block of atoms."""
    cfg = d["cfg"]
    f8 = dict(dtype=torch.float64, device="cuda")
    S, alpha = len(cfg["species"]), float(cfg["celu_alpha"])
    P = S * (S + 1) // 2
    rc, rca, er, ea, zeta = (float(cfg[k]) for k in ("rc_rad", "rc_ang", "eta_rad", "eta_ang", "zeta"))
    rs, ra, th = (torch.tensor(cfg[k].astype(np.float64), **f8) for k in ("rad_shift", "ang_shift", "ang_sect"))
    x = torch.from_numpy(d["pos"]).cuda().double()
    sp = torch.from_numpy(np.searchsorted(np.array(cfg["species"]), d["Z"])).cuda()
    n = len(x)
    sys, L = None, None
    if "offsets" in d:
        sys = torch.repeat_interleave(torch.arange(len(d["offsets"]) - 1), torch.from_numpy(np.diff(d["offsets"])).long()).cuda()
        if d.get("boxes") is not None:
            L = torch.from_numpy(d["boxes"]).cuda().double()
    elif d.get("box") is not None:
        L = [float(v) for v in d["box"]]
    i, j = _pairs64(x.float(), L.float() if torch.is_tensor(L) else L, sys, rc)
    Lrow = None if L is None else (L[sys] if torch.is_tensor(L) else torch.tensor(L, **f8).expand(n, 3))
    # networks
    w = torch.from_numpy(d["weights"]).cuda().double()
    nets, at = [], 0
    for _ in range(d["members"] * S):
        net = []
        for fi, fo in zip(cfg["widths"][:-1], cfg["widths"][1:]):
            net.append((w[at:at + fi * fo].view(fo, fi), w[at + fi * fo:at + fi * fo + fo]))
            at += fi * fo + fo
        nets.append(net)
    cls = torch.zeros((S, S), dtype=torch.long, device="cuda")
    q = 0
    for a in range(S):
        for b in range(a, S):
            cls[a, b] = cls[b, a] = q
            q += 1

    def fc(r, R):
        return 0.5 * torch.cos(math.pi * r / R) + 0.5

    energy, grad = torch.zeros(n, **f8), torch.zeros((n, 3), **f8)
    step = 16384
    first = torch.searchsorted(i, torch.arange(0, n + step, step, device="cuda").clamp(max=n)).tolist()
    for b, a0 in enumerate(range(0, n, step)):
        a1 = min(n, a0 + step)
        m = a1 - a0
        pi, pj = i[first[b]:first[b + 1]], j[first[b]:first[b + 1]]
        xx = x.clone().requires_grad_(True)
        v = xx[pj] - xx[pi]
        if Lrow is not None:
            v = v - (Lrow[pi] * torch.round(v / Lrow[pi])).detach()
        r = v.norm(dim=1)
        keep = torch.nonzero(r.detach() < rc)[:, 0]
        pi, pj, v, r = pi[keep] - a0, pj[keep], v[keep], r[keep]
        rad = torch.zeros((m * S, 16), **f8).index_add(
            0, pi * S + sp[pj], torch.exp(-er * (r[:, None] - rs) ** 2) * fc(r, rc)[:, None])
        # angular neighbours in a padded table, all pairs j < k of each row
        ang = torch.nonzero(r.detach() < rca)[:, 0]
        ai, count = pi[ang], torch.bincount(pi[ang], minlength=m)
        K = max(int(count.max()), 2) if len(ang) else 2
        start = torch.cumsum(count, 0) - count
        slot = torch.arange(len(ang), device="cuda") - start[ai]
        table = torch.full((m, K), -1, dtype=torch.long, device="cuda")
        table[ai, slot] = ang
        tj, tk = torch.triu_indices(K, K, 1, device="cuda")
        row, col = torch.nonzero(table[:, tk] >= 0, as_tuple=True)
        ej, ek = table[row, tj[col]], table[row, tk[col]]
        c = 0.95 * (v[ej] * v[ek]).sum(1) / (r[ej] * r[ek])
        sn = torch.sqrt(1 - c * c)
        A = (1 + c[:, None] * torch.cos(th) + sn[:, None] * torch.sin(th)) ** zeta
        A = A * (2.0 ** (1 - zeta) * fc(r[ej], rca) * fc(r[ek], rca))[:, None]
        B = torch.exp(-ea * ((r[ej] + r[ek])[:, None] / 2 - ra) ** 2)
        angular = torch.zeros((m * P, 32), **f8).index_add(
            0, row * P + cls[sp[pj[ej]], sp[pj[ek]]], (B[:, :, None] * A[:, None, :]).reshape(-1, 32))
        desc = torch.cat([rad.view(m, -1), angular.view(m, -1)], 1)
        ph = None
        if phi is not None:
            ph = phi(xx[a0:a1])
            desc = torch.cat([desc, ph[:, None]], 1)
        e = torch.zeros(m, **f8)
        for s in range(S):
            rows = torch.nonzero(sp[a0:a1] == s)[:, 0]
            if not len(rows):
                continue
            total = 0.0
            for k in range(d["members"]):
                h = desc[rows]
                net = nets[k * S + s]
                for l, (W, bias) in enumerate(net):
                    h = torch.nn.functional.linear(h, W, bias)
                    if l < len(net) - 1:
                        h = torch.nn.functional.celu(h, alpha)
                total = total + (h[:, 0] if h.shape[1] == 1 else h[:, 0] + h[:, 1] * ph[rows])
            e = e.index_add(0, rows, total / d["members"])
        inputs = [xx] + ([d["mm64"]] if phi is not None else [])
        got = torch.autograd.grad(e.sum(), inputs)
        grad += got[0]
        if phi is not None:
            d["mm_grad"] = d.get("mm_grad", 0) + got[1]
        energy[a0:a1] = e.detach()
    return energy, -grad, sys


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    f8 = dict(dtype=torch.float64, device="cuda")
    if kind == "couple":
        a = torch.from_numpy(d["pos"]).cuda().double().requires_grad_(True)
        b = torch.from_numpy(d["mm_pos"]).cuda().double().requires_grad_(True)
        pa, pb = torch.from_numpy(d["ml_par"]).cuda().double(), torch.from_numpy(d["mm_par"]).cuda().double()
        L = float(d["box"][0])
        v = b[None] - a[:, None]
        v = v - (L * torch.round(v / L)).detach()
        r2 = (v * v).sum(-1)
        s6 = ((0.5 * (pa[:, None, 1] + pb[None, :, 1])) ** 2 / r2) ** 3
        eps = torch.sqrt(pa[:, None, 2] * pb[None, :, 2])
        e = KE * pa[:, None, 0] * pb[None, :, 0] / torch.sqrt(r2) + 4 * eps * (s6 * s6 - s6)
        e = torch.where(r2 < case["cutoff"] ** 2, e, torch.zeros((), **f8)).sum()
        ga, gb = torch.autograd.grad(e, [a, b])
        return {"energy": e.detach().reshape(1), "forces": -ga, "mm_forces": -gb}
    if kind == "embed":
        d["mm64"] = torch.from_numpy(d["mm_pos"]).cuda().double().requires_grad_(True)
        q, L, R = torch.from_numpy(d["mm_q"]).cuda().double(), float(d["box"][0]), float(d["cfg"]["mm_cutoff"])

        def phi(x):
            v = d["mm64"][None] - x[:, None]
            v = v - (L * torch.round(v / L)).detach()
            r = torch.sqrt((v * v).sum(-1))
            return (KE * q * torch.where(r < R, (0.5 * torch.cos(math.pi * r / R) + 0.5) / r,
                                         torch.zeros((), **f8))).sum(1)

        e, F, _ = _exact_model(d, phi)
        return {"energy": e.sum().reshape(1), "forces": F, "mm_forces": -d["mm_grad"]}
    if kind == "ligand":
        g = torch.from_numpy(d["group"]).cuda().long()
        sub = dict(d, pos=np.ascontiguousarray(d["pos"][d["group"]]), Z=d["Z"][d["group"]])
        e, Fg, _ = _exact_model(sub)
        F = torch.zeros((len(d["pos"]), 3), **f8)
        F[g] = Fg
        return {"energy": e.sum().reshape(1), "forces": F}
    e, F, sys = _exact_model(d)
    if sys is not None:
        return {"energy": torch.zeros(len(d["offsets"]) - 1, **f8).index_add(0, sys, e), "forces": F}
    if kind == "relax":
        return {"energy": e.sum(), "gradient": -F}
    return {"energy": e.sum().reshape(1), "forces": F}
