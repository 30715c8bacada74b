"""Timed cases: the calls that programs make of the engine, from one small
molecule to a 77,000-atom batch and a 23,001-atom water box.

A case is a dict:
  kind       "forces"  energies and forces of one call (a step of MD)
             "energy"  energies only (scoring conformations)
             "subset"  a molecule inside a larger, otherwise classical system
             "graph"   a captured evaluation, replayed
             "train"   one energy-fitting step: loss, weight gradients and,
                       with pos_grad, position gradients
  system     "conformers"  `mols` jittered copies of one molecule of `atoms`
             "ragged"      `mols` molecules of 10 to 150 atoms (log-uniform)
             "water"       a periodic box of `mols` waters at liquid density
  elements   4 or 7 (networks 384-160-128-96-1 or 1008-256-192-160-1)
  precision  "bf16" or "fp32" networks
  members    networks in the ensemble
  capacity   neighbor list capacity per atom (the default is 128; the
             benchmark gives molecules 64)

The molecules, the boxes and the random weights follow the recipes of the
benchmark: uniform positions at 24 atoms per (10 A)^3 at least 0.9 A apart,
rigid waters at O-O >= 2.6 A, weights N(0, 1/fan_in).
"""
import math

import numpy as np
import torch

from paper_2310_03121_amd import Graph, NNPFunction, Potential

ELEMENT_SHARE = np.array([0.45, 0.3, 0.1, 0.1, 0.02, 0.02, 0.01])
WIDTHS = {4: (384, 160, 128, 96, 1), 7: (1008, 256, 192, 160, 1)}
OUT_SCALE = {4: 5.0, 7: 6.0}   # RMS force near 1 eV/A on the water boxes
ALPHA = 0.1                    # CELU
RC_R, ETA_R, RC_A, ETA_A, ZETA = 5.1, 19.7, 3.5, 12.5, 14.1
SHF_R = np.linspace(0.8, 4.8875, 16).astype(np.float32)
SHF_A = np.linspace(0.8, 2.6, 4).astype(np.float32)
SHF_Z = ((2 * np.arange(8) + 1) * np.pi / 16).astype(np.float32)
RADIAL_SCALE, COS_SCALE = 0.25, 0.95
WATER_VOLUME = 61.2 ** 3 / 7667
SUBSET_TOTAL = 6000            # atoms of the system around a subset

#: neighbors, neighbors in the angular cutoff and pairs of these, of an atom
#: of a molecule and of liquid water: what `work` counts.
NEIGHBORS = {"molecule": (7.8, 5.0), "water": (54.8, 144.0)}
#: features of an atom that are not zero by construction (same for both)
TOUCHED = 130


def _case(name, kind, system, mols, atoms=0, elements=7, precision="bf16", members=1,
          capacity=128, pos_grad=False):
    c = dict(kind=kind, system=system, mols=mols, atoms=atoms, elements=elements,
             precision=precision, members=members, capacity=capacity, pos_grad=pos_grad)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # gas-phase MD of one small molecule: launches and latency
        _case("mol24_fp32", "forces", "conformers", 1, 24, 4, "fp32"),
        # ML/MM: a 53-atom ligand, eight-network ensemble, in a classical system
        _case("ligand53_ens8_bf16", "subset", "conformers", 1, 53, members=8),
        # a captured step of a small packed batch, as a serving loop replays it
        _case("graph_ragged32_bf16", "graph", "ragged", 32, capacity=64),
        # ranking conformations by energy
        _case("screen2048x24_bf16", "energy", "conformers", 2048, 24, 4, capacity=64),
        # the benchmark's batch, both precisions
        _case("conf512x64_bf16", "forces", "conformers", 512, 64, capacity=64),
        _case("conf512x64_fp32", "forces", "conformers", 512, 64, precision="fp32", capacity=64),
        # a full server (about 1 GiB of device memory): mixed sizes, 77,163 atoms
        _case("ragged1500_bf16", "forces", "ragged", 1500, capacity=64),
        # condensed-phase MD, small and large box
        _case("water1500_fp32", "forces", "water", 1500, elements=4, precision="fp32"),
        _case("water7667_bf16", "forces", "water", 7667),
        # committee of eight over a batch of conformations
        _case("ens8_conf512x64_bf16", "forces", "conformers", 512, 64, members=8, capacity=64),
        # training: a minibatch in FP32, and the benchmark's batch with dL/dpos
        _case("train128x64_fp32", "train", "conformers", 128, 64, precision="fp32"),
        _case("train512x64_bf16", "train", "conformers", 512, 64, capacity=64, pos_grad=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forces", "forces", "forces", "energy", "subset", "graph", "train"])
    precision = rng.choice(["bf16", "fp32"])
    elements = rng.choice([4, 7])
    capacity = rng.choice([64, 128])
    if kind == "subset":
        return _case(None, kind, "conformers", 1, _log_int(rng, 10, 150), elements, precision,
                     rng.choice([1, 8]), capacity)
    if kind == "forces" and rng.random() < 0.4:
        # a box of 180 waters is a little over two cutoffs wide
        return _case(None, kind, "water", _log_int(rng, 180, 7667), 0, elements, precision)
    members = rng.choice([1, 1, 8]) if kind == "forces" else 1
    bf16 = precision == "bf16"
    most = {"train": 32768 if bf16 else 8192, "graph": 8192}.get(kind, 80000 if bf16 else 32768)
    if members > 1:
        most = 32768 if bf16 else 4096
    if rng.random() < 0.5:
        mols = _log_int(rng, 1, most // 54)
        return _case(None, kind, "ragged", mols, 0, elements, precision, members, capacity,
                     kind == "train" and rng.random() < 0.5)
    atoms = _log_int(rng, 10, 150)
    mols = _log_int(rng, 1, max(1, most // atoms))
    return _case(None, kind, "conformers", mols, atoms, elements, precision, members, capacity,
                 kind == "train" and rng.random() < 0.5)


# ------------------------------------------------------------------ inputs

def _sizes(case):
    """Atoms per molecule, in a fixed order."""
    if case["system"] == "conformers":
        return np.full(case["mols"], case["atoms"], np.int64)
    if case["system"] == "ragged":
        n = case["mols"]
        q = (np.random.default_rng(n).permutation(n) + 0.5) / n
        return np.floor(np.exp(np.log(10) + q * (np.log(151) - np.log(10)))).astype(np.int64)
    return np.array([3 * case["mols"]], np.int64)


def _molecules(sizes, rng):
    """Positions [M, max size, 3] of molecules placed atom by atom, all
    molecules at once; every accepted atom is 0.9 A from the earlier ones."""
    side = 10.0 * (sizes / 24.0) ** (1.0 / 3.0)
    x = np.full((len(sizes), int(sizes.max()), 3), 1e6)
    for k in range(x.shape[1]):
        todo = np.nonzero(sizes > k)[0]
        while todo.size:
            p = rng.uniform(0.0, 1.0, (todo.size, 3)) * side[todo, None]
            d2 = ((x[todo, :max(k, 1)] - p[:, None]) ** 2).sum(-1).min(1)
            ok = d2 >= 0.81 if k else np.ones(todo.size, bool)
            x[todo[ok], k] = p[ok]
            todo = todo[~ok]
    return x


def _waters(n, L, rng):
    """Rigid waters [3n, 3]: oxygens by random addition, many candidates at a
    time, with random orientations; wrapped into the box."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    O = torch.zeros((0, 3), dtype=torch.float64, device=dev)

    def near(a, b):
        d2 = 0
        for c in range(3):
            d = a[:, None, c] - b[None, :, c]
            d2 = d2 + (d - L * torch.round(d / L)) ** 2
        return d2 < 2.6 * 2.6

    while O.shape[0] < n:
        p = torch.from_numpy(rng.uniform(0.0, L, (4096, 3))).to(dev)
        if O.shape[0]:
            p = p[~near(p, O).any(1)]
        p = p[~torch.tril(near(p, p), -1).any(1)]
        O = torch.cat([O, p])[:n]
    O = O.cpu().numpy()
    q = rng.standard_normal((n, 4))
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    R = np.stack([np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)], -1),
                  np.stack([2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)], -1),
                  np.stack([2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], -1)], 1)
    half = np.deg2rad(104.52) / 2
    h = [0.9572 * np.array([s * np.sin(half), 0.0, np.cos(half)]) for s in (1, -1)]
    pos = np.mod(np.stack([O, O + R @ h[0], O + R @ h[1]], 1).reshape(-1, 3), L).astype(np.float32)
    pos[pos >= np.float32(L)] = 0.0
    return pos


def _inputs(case, seed):
    """Host arrays: pos, species, mol_offsets, box, params (one per member),
    and for a subset idx, pos_all and F_all, for training E_ref."""
    rng = np.random.default_rng(seed)
    S, sizes = case["elements"], _sizes(case)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(off[-1])
    s = dict(off=off, box=None)

    def species(k):
        if S == 4:
            return rng.integers(0, 4, k).astype(np.int32)
        return rng.choice(7, size=k, p=ELEMENT_SHARE / ELEMENT_SHARE.sum()).astype(np.int32)

    if case["system"] == "water":
        L = (case["mols"] * WATER_VOLUME) ** (1.0 / 3.0)
        s["pos"] = _waters(case["mols"], L, rng)
        s["species"] = np.tile(np.array([3, 0, 0], np.int32), case["mols"])
        s["box"] = np.full(3, L, np.float32)
    elif case["system"] == "conformers":
        base = _molecules(sizes[:1], rng)[0]
        pos = base[None] + rng.normal(0.0, 0.05, (case["mols"],) + base.shape)
        s["pos"] = pos.reshape(-1, 3).astype(np.float32)
        s["species"] = np.tile(species(case["atoms"]), case["mols"])
    else:
        x = _molecules(sizes, rng)
        s["pos"] = x[np.arange(x.shape[1])[None] < sizes[:, None]].astype(np.float32)
        s["species"] = species(n)
    s["params"] = []
    w = WIDTHS[S]
    for _ in range(case["members"]):
        parts = []
        for _s in range(S):
            for l in range(4):
                scale = OUT_SCALE[S] if l == 3 else 1.0
                parts += [rng.standard_normal(w[l + 1] * w[l], np.float32) * np.float32(scale / math.sqrt(w[l])),
                          rng.standard_normal(w[l + 1], np.float32) * np.float32(0.1 * scale)]
        s["params"].append(np.concatenate(parts))
    if case["kind"] == "subset":
        s["idx"] = rng.permutation(SUBSET_TOTAL)[:n].astype(np.int32)
        s["pos_all"] = rng.uniform(0.0, 40.0, (SUBSET_TOTAL, 3)).astype(np.float32)
        s["pos_all"][s["idx"]] = s["pos"]
        s["F_all"] = rng.standard_normal((SUBSET_TOTAL, 3)).astype(np.float32)
    if case["kind"] == "train":
        s["E_ref"] = rng.normal(0.0, 20.0, case["mols"])
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    pot = Potential(n_species=case["elements"], rc_rad=RC_R, eta_r=ETA_R, shf_r=SHF_R, rc_ang=RC_A,
                    eta_a=ETA_A, zeta=ZETA, shf_a=SHF_A, shf_z=SHF_Z, radial_prefactor=RADIAL_SCALE,
                    angle_cos_scale=COS_SCALE, widths=WIDTHS[case["elements"]], params=s["params"],
                    celu_alpha=ALPHA, precision=case["precision"], max_neighbors=case["capacity"])
    st = {k: torch.from_numpy(v).cuda() for k, v in s.items()
          if k in ("pos", "species", "off", "idx", "pos_all", "F_all", "E_ref")}
    st.update(kind=case["kind"], pot=pot, box=s["box"])
    if case["kind"] == "graph":
        st["graph"] = Graph(pot, st["pos"], st["species"], st["off"], st["box"])
    if case["kind"] == "train":
        st["params"] = torch.from_numpy(s["params"][0]).cuda().requires_grad_()
        st["pos"].requires_grad_(case["pos_grad"])
    return st


def run(st):
    pot, kind = st["pot"], st["kind"]
    if kind == "forces" or kind == "energy":
        E, F = pot.energy_forces(st["pos"], st["species"], st["off"], st["box"],
                                 forces=kind == "forces")
        return {"E": E, "F": F}
    if kind == "subset":
        F = st["F_all"].clone()   # this step's classical forces
        E = pot.energy_forces_subset(st["idx"], st["pos_all"], st["species"], st["off"], F)
        return {"E": E, "F": F}
    if kind == "graph":
        g, here = st["graph"], torch.cuda.current_stream()
        g.stream.wait_stream(here)
        g.launch()
        here.wait_stream(g.stream)
        return {"E": g.E, "F": g.F}
    pos, params = st["pos"], st["params"]
    E = NNPFunction.apply(pos, params, pot, st["species"], st["off"], st["box"])
    loss = ((E - st["E_ref"]) ** 2).mean()
    if pos.requires_grad:
        gw, gp = torch.autograd.grad(loss, [params, pos])
        return {"E": E.detach(), "gw": gw, "gp": gp}
    return {"E": E.detach(), "gw": torch.autograd.grad(loss, [params])[0]}


def work(case):
    """The inputs and the networks' weights read once (2 or 4 bytes each), the
    outputs written once; the networks over the features that are not zero by
    construction, and the operations of the symmetry functions per neighbor
    (107 forward, 199 adjoint) and per pair of angular neighbors (151, 280)."""
    n, mols = int(_sizes(case).sum()), len(_sizes(case))
    w, S, M = WIDTHS[case["elements"]], case["elements"], case["members"]
    used = 2 if case["system"] == "water" else S
    per = [a * b + b for a, b in zip(w, w[1:])]
    touched = min(TOUCHED, w[0])
    mid = sum(a * b for a, b in zip(w[1:], w[2:])) + touched * w[1]
    rad, ang = NEIGHBORS["water" if case["system"] == "water" else "molecule"]
    train = case["kind"] == "train"
    adjoint = case["kind"] != "energy" and (not train or case["pos_grad"])
    size = 2 if case["precision"] == "bf16" else 4
    flops = 2.0 * n * M * mid * (1 + adjoint + 2 * train - (adjoint and train))
    flops += n * (rad * (107 + 199 * adjoint) + ang * (151 + 280 * adjoint))
    size_w = sum(per) * M * (size * min(used, n) if not train else 4 * S)
    nbytes = n * 16.0 + mols * 8 + size_w + (12.0 * n if adjoint else 0)
    if train:
        nbytes += 4.0 * sum(per) * S + mols * 8
    if case["kind"] == "subset":
        nbytes += 16.0 * n
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------- the same in float64

def _pairs(pos, off, box, a, b):
    """Neighbor pairs (i, j) within the radial cutoff for atoms a..b."""
    if box is not None:
        d = pos[None, :, :] - pos[a:b, None, :]
        d = d - box * torch.round(d / box)
        m = (d * d).sum(-1) < RC_R * RC_R
        m[torch.arange(b - a, device=m.device), torch.arange(a, b, device=m.device)] = False
        i, j = torch.nonzero(m, as_tuple=True)
        return i + a, j
    size = off[1:] - off[:-1]
    mol = torch.repeat_interleave(torch.arange(len(size), device=off.device), size)[a:b]
    j = off[mol][:, None] + torch.arange(int(size.max()), device=off.device)[None]
    ok = (j < off[mol + 1][:, None]) & (j != torch.arange(a, b, device=off.device)[:, None])
    j = torch.where(ok, j, 0)
    d = pos[j] - pos[a:b, None]
    i, k = torch.nonzero(ok & ((d * d).sum(-1) < RC_R * RC_R), as_tuple=True)
    return i + a, j[i, k]


def _features(pos, sp, box, I, J, a, b, S):
    dev, n = pos.device, b - a

    def table(v):
        return torch.from_numpy(v.astype(np.float64)).to(dev)

    def f64(v):
        return float(np.float32(v))

    def fc(d, R):
        return 0.5 * torch.cos(math.pi * d / R) + 0.5

    v = pos[J] - pos[I]
    if box is not None:
        v = v - box * torch.round(v / box)
    d = v.norm(dim=1)
    rcr, rca, zeta, kappa = f64(RC_R), f64(RC_A), f64(ZETA), f64(COS_SCALE)
    rad = RADIAL_SCALE * torch.exp(-f64(ETA_R) * (d[:, None] - table(SHF_R)) ** 2) * fc(d, rcr)[:, None]
    F = WIDTHS[S][0]
    at = ((I - a) * F + 16 * sp[J])[:, None] + torch.arange(16, device=dev)
    G = torch.zeros(n * F, dtype=torch.float64, device=dev).index_add(0, at.reshape(-1), rad.reshape(-1))
    near = torch.nonzero(d.detach() < rca).reshape(-1)   # pairs come sorted by i
    count = torch.bincount(I[near] - a, minlength=n)
    if near.numel() and int(count.max()) > 1:
        first = torch.cumsum(count, 0) - count
        p, q = torch.triu_indices(int(count.max()), int(count.max()), 1, device=dev)
        t, k = torch.nonzero(q[None] < count[:, None], as_tuple=True)
        j, k = near[first[t] + p[k]], near[first[t] + q[k]]
        cosine = (v[j] * v[k]).sum(1) / (d[j] * d[k])
        theta = torch.acos(kappa * cosine)
        f1 = 2.0 ** (1 - zeta) * (1 + torch.cos(theta[:, None] - table(SHF_Z))) ** zeta
        f2 = torch.exp(-f64(ETA_A) * ((d[j] + d[k])[:, None] / 2 - table(SHF_A)) ** 2)
        terms = f2[:, :, None] * f1[:, None, :] * (fc(d[j], rca) * fc(d[k], rca))[:, None, None]
        lo, hi = torch.minimum(sp[J[j]], sp[J[k]]), torch.maximum(sp[J[j]], sp[J[k]])
        block = lo * S - (lo * (lo - 1)) // 2 + hi - lo
        at = (t * F + 16 * S + 32 * block)[:, None] + torch.arange(32, device=dev)
        G = G.index_add(0, at.reshape(-1), terms.reshape(-1))
    return G.reshape(n, F)


def _networks(G, sp, params, S):
    """Atomic energies of one member; params: its flat vector."""
    w, o = WIDTHS[S], 0
    E = torch.zeros(G.shape[0], dtype=torch.float64, device=G.device)
    for s in range(S):
        rows, h = torch.nonzero(sp == s).reshape(-1), None
        for l in range(4):
            W = params[o:o + w[l] * w[l + 1]].reshape(w[l + 1], w[l])
            o += W.numel()
            bias = params[o:o + w[l + 1]]
            o += w[l + 1]
            if rows.numel():
                h = (G[rows] if l == 0 else h) @ W.T + bias
                h = torch.nn.functional.celu(h, float(np.float32(ALPHA))) if l < 3 else h
        if rows.numel():
            E = E.index_add(0, rows, h[:, 0])
    return E


def _energies(s, S, up=None, want_params=False):
    """E [M], dL/dpos and dL/dparams (or None) for L = sum up * E."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    pos = torch.from_numpy(s["pos"].astype(np.float64)).to(dev).requires_grad_(up is not None)
    sp = torch.from_numpy(s["species"].astype(np.int64)).to(dev)
    off = torch.from_numpy(s["off"].astype(np.int64)).to(dev)
    box = None if s["box"] is None else torch.from_numpy(s["box"].astype(np.float64)).to(dev)
    params = [torch.from_numpy(p.astype(np.float64)).to(dev).requires_grad_(want_params) for p in s["params"]]
    n, mols = pos.shape[0], len(off) - 1
    mol = torch.repeat_interleave(torch.arange(mols, device=dev), off[1:] - off[:-1])
    E = torch.zeros(mols, dtype=torch.float64, device=dev)
    gp, gw = torch.zeros_like(pos), [torch.zeros_like(p) for p in params]
    step = 1000 if box is not None else 8192
    for a in range(0, n, step):
        b = min(n, a + step)
        I, J = _pairs(pos.detach(), off, box, a, b)
        with torch.set_grad_enabled(up is not None):
            G = _features(pos, sp, box, I, J, a, b, S)
            e = sum(_networks(G, sp[a:b], p, S) for p in params) / len(params)
            E = E.index_add(0, mol[a:b], e.detach())
            if up is not None:
                to = [pos] + (params if want_params else [])
                g = torch.autograd.grad((up[mol[a:b]] * e).sum(), to)
                gp += g[0]
                for k in range(len(to) - 1):
                    gw[k] += g[k + 1]
    return E, gp.detach(), gw[0] if want_params else None


def exact(case, seed):
    s, S = _inputs(case, seed), case["elements"]
    if case["kind"] == "train":
        E = _energies(s, S)[0]
        up = 2.0 * (E - torch.from_numpy(s["E_ref"]).to(E.device)) / E.numel()
        _, gp, gw = _energies(s, S, up, True)
        return {"E": E, "gw": gw, "gp": gp} if case["pos_grad"] else {"E": E, "gw": gw}
    if case["kind"] == "energy":
        return {"E": _energies(s, S)[0], "F": None}
    E, g, _ = _energies(s, S, torch.ones(case["mols"] if s["box"] is None else 1, dtype=torch.float64,
                                         device="cuda" if torch.cuda.is_available() else "cpu"))
    F = -g
    if case["kind"] == "subset":
        F = torch.from_numpy(s["F_all"].astype(np.float64)).to(g.device)
        F[torch.from_numpy(s["idx"].astype(np.int64)).to(g.device)] -= g
    return {"E": E, "F": F}
