"""The work that a program using this library has it do, as cases that can be timed and checked.

A case is one pass through a public entry point on a synthetic system: a jittered periodic
water box or a jittered FCC (Cu-like) crystal, with a seeded random model of one of the
repository's model shapes.  The weights of a model are fixed (a program keeps its model); the
positions come from the seed.  Entry points:

    plan      energy, atomic energies, forces and virial through a device plan (the inner call
              of an MD engine that keeps its positions on the GPU)
    autograd  energy and its gradient through the torch wrapper
    energy    energy and atomic energies only (Monte Carlo moves, scoring a configuration)
    frames    two unrelated frames of the same composition in turn through one plan (scoring
              a data set): every evaluation has to build its neighbour list
    host      the host-pointer call, positions in and forces out (coupling to a CPU MD engine)
    serve     one velocity-Verlet step of every system of a resident batch through the server

Results are handed on in the type the path computes in: float64 and float32 as such, float32
work with BF16 products as bfloat16.  BF16 plans give no virial: the pressure of these systems is
a small remainder of cancelling terms, which BF16 products do not resolve.
"""
from __future__ import annotations

import math

import numpy as np
import torch

SPACING = 12.42 / 4            # water: one molecule per site of this grid (64 in a 12.42 A cube)
FCC_A = 3.61                   # lattice constant of the crystal
MASS = (1.008, 15.999, 63.546)  # amu, of H, O, Cu
ACCEL = 9.648533212e-3         # (eV/A) / amu in A/fs^2
KB = 8.617333262e-5            # eV / K
DT_FS = 1.0                    # time step of the served velocity-Verlet steps

# The model shapes of the repository: n_species, L, K, r_c, hidden layers x width, first-layer
# weight scale, bias scale, angular scale, form.  Species: water (H, O), crystal (Cu), serving
# (H, O, Cu).
MODELS = {
    "water": dict(ns=2, L=2, K=8, r_c=5.0, nh=2, H=64, w1=2.0, bias=1.0, ang=1.0 / 5.0, form="reann"),
    "water-plain": dict(ns=2, L=2, K=8, r_c=5.0, nh=2, H=64, w1=1.0, bias=0.0, ang=1.0, form="reann"),
    "cu": dict(ns=1, L=2, K=12, r_c=6.0, nh=3, H=128, w1=1.0, bias=1.0, ang=1.0 / 6.0, form="reann"),
    "serving": dict(ns=3, L=2, K=12, r_c=5.0, nh=3, H=128, w1=2.0, bias=1.0, ang=1.0 / 5.0, form="reann"),
    "cu-radial": dict(ns=1, L=0, K=12, r_c=6.0, nh=3, H=128, w1=1.0, bias=1.0, ang=1.0, form="radial"),
    "water-radial": dict(ns=2, L=0, K=8, r_c=5.0, nh=2, H=64, w1=1.0, bias=1.0, ang=1.0, form="radial"),
}
DTYPE = {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.bfloat16}


def _case(name, entry, system, nx, ny, nz, model, T, precision="fp32", skin=1.0, split=1):
    return dict(name=name, entry=entry, system=system, nx=nx, ny=ny, nz=nz, model=model, T=T,
                precision=precision, skin=skin, split=split)


def listed():
    return [
        # the 64-molecule reference box: the smallest call, where launches and latency count
        _case("water-192", "plan", "water", 4, 4, 4, "water-plain", 2),
        # a small training-sized box through torch autograd
        _case("water-1512-autograd", "autograd", "water", 9, 8, 7, "water", 3),
        # an ordinary MD cell
        _case("fcc-4000", "plan", "fcc", 10, 10, 10, "cu", 3),
        # the throughput workload, in both precisions that MD is run in
        _case("fcc-100800", "plan", "fcc", 30, 30, 28, "cu", 3),
        _case("fcc-100800-bf16", "plan", "fcc", 30, 30, 28, "cu", 3, "bf16"),
        # the largest: 402,432 molecules in 2x2x2 subdomains with the per-layer ghost exchange
        _case("water-1207296-split", "plan", "water", 48, 64, 131, "water", 3, split=2),
        # a middle-sized box split in subdomains, BF16 products
        _case("water-65772-bf16-split", "plan", "water", 28, 27, 29, "water", 3, "bf16", split=2),
        # reference precision: validation runs, phonons, energy-conserving dynamics
        _case("fcc-6864-fp64", "plan", "fcc", 11, 12, 13, "cu", 3, "fp64"),
        # energies without forces, a ragged size
        _case("water-20520-energy", "energy", "water", 19, 18, 20, "water", 3),
        # the second message form
        _case("fcc-31920-radial", "plan", "fcc", 20, 21, 19, "cu-radial", 3),
        # unrelated frames of one composition: a neighbour list for each
        _case("water-3000-frames", "frames", "water", 10, 10, 10, "water", 2),
        # a batch of resident systems, 64 to 20,000 atoms, one MD step of each
        dict(name="mix-16-serve", entry="serve", count=16, n_min=64, n_max=20000, model="serving", T=3,
             precision="bf16", skin=1.0),
    ]


def _dims(rng, system, lo, hi):
    """Cells (or molecule sites) along x, y, z for about a log-uniform number of atoms, ragged."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    side = (n / (3 if system == "water" else 4)) ** (1.0 / 3.0)
    return tuple(max(2, int(round(side * rng.uniform(0.8, 1.25)))) for _ in range(3))


def draw(rng):
    entry = rng.choice(["plan", "plan", "plan", "autograd", "energy", "frames", "host", "serve"])
    if entry == "serve":
        return dict(entry="serve", count=rng.randint(3, 16), n_min=rng.randint(48, 400),
                    n_max=rng.randint(2000, 20000), model="serving", T=rng.randint(2, 3),
                    precision=rng.choice(["bf16", "fp32"]), skin=1.0)
    # two random frames of a crystal can lie within half a skin of each other: frames are water
    system = "water" if entry == "frames" else rng.choice(["water", "fcc"])
    precision = rng.choice(["fp32", "fp32", "fp32", "bf16", "bf16", "fp64"])
    hi = {"fp64": 8000}.get(precision, 100000)
    if entry in ("frames", "host", "autograd"):
        hi = min(hi, 20000)
    nx, ny, nz = _dims(rng, system, 64, hi)
    model = "water" if system == "water" else "cu"
    if rng.random() < 0.2:
        model += "-radial"
    c = _case("", entry, system, nx, ny, nz, model, rng.randint(1, 4), precision,
              skin=rng.choice([0.5, 1.0]), split=rng.choice([1, 1, 2]))
    del c["name"]
    return c


# ------------------------------------------------------------------------- inputs --

class _Params:
    """Model parameters in the layout the library's Model takes."""


def _model_params(name, T):
    """Weights N(0, 1/fan_in) (the first layer scaled), biases N(0, bias^2), c0 ~ N(0, 1)."""
    m = MODELS[name]
    rng = np.random.default_rng(0)
    p = _Params()
    p.elements = ["H", "O", "Cu"][:m["ns"]] if m["ns"] > 1 else ["Cu"]
    p.n_species, p.L, p.K, p.r_c, p.T_max = m["ns"], m["L"], m["K"], m["r_c"], max(T, 2)
    p.n_hidden, p.hidden, p.ang_scale, p.energy_scale, p.form = m["nh"], m["H"], m["ang"], 1.0, m["form"]
    p.F = p.K if p.form == "radial" else (p.L + 1) * p.K * (p.K + 1) // 2
    p.centres = np.linspace(0.0, p.r_c, p.K)
    p.alphas = np.full(p.K, 2.0)   # width 0.5 A
    p.c0 = rng.normal(size=(p.n_species, p.K))

    def nn(out):
        dims, parts = [p.F] + [p.hidden] * p.n_hidden + [out], []
        for k in range(1, len(dims)):
            sd = (m["w1"] if k == 1 else 1.0) / math.sqrt(dims[k - 1])
            parts += [rng.normal(scale=sd, size=dims[k] * dims[k - 1]),
                      rng.normal(size=dims[k]) * m["bias"]]
        return np.concatenate(parts)

    # a message NN per layer (the first T_max - 1) and species, an energy NN per species
    p.msg_blob = np.concatenate([nn(p.K) for _ in range((p.T_max - 1) * p.n_species)])
    p.energy_blob = np.concatenate([nn(1) for _ in range(p.n_species)])
    return p


def _water(nx, ny, nz, rng):
    """One molecule per grid site (O jittered by 0.2 A), uniformly random orientations."""
    g = np.stack(np.meshgrid(np.arange(nx), np.arange(ny), np.arange(nz), indexing="ij"), -1).reshape(-1, 3)
    o = (g + 0.5) * SPACING + rng.normal(scale=0.2, size=g.shape)
    q = rng.normal(size=(len(g), 4))
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    w, x, y, z = q.T
    half = math.radians(104.5) / 2.0
    # columns 0 and 2 of the rotation matrix: the molecule lies in the body's x-z plane
    ex = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y + z * w), 2 * (x * z - y * w)], 1) * (0.96 * math.sin(half))
    ez = np.stack([2 * (x * z + y * w), 2 * (y * z - x * w), 1 - 2 * (x * x + y * y)], 1) * (0.96 * math.cos(half))
    pos = np.stack([o, o + ez + ex, o + ez - ex], 1).reshape(-1, 3)
    return pos, np.tile(np.array([1, 0, 0], np.int32), len(g)), np.array([nx, ny, nz]) * SPACING


def _fcc(nx, ny, nz, rng):
    """Conventional cells of 4 atoms, displaced by 0.1 A."""
    basis = np.array([[0, 0, 0], [0, 0.5, 0.5], [0.5, 0, 0.5], [0.5, 0.5, 0]])
    g = np.stack(np.meshgrid(np.arange(nx), np.arange(ny), np.arange(nz), indexing="ij"), -1).reshape(-1, 1, 3)
    pos = ((g + basis) * FCC_A).reshape(-1, 3)
    pos = pos + rng.normal(scale=0.1, size=pos.shape)
    return pos, np.zeros(len(pos), np.int32), np.array([nx, ny, nz]) * FCC_A


def _system(pos, species, box):
    return dict(pos=np.ascontiguousarray(pos), species=species, cell=np.diag(box).astype(np.float64),
                pbc=np.ones(3, np.int32))


def _frames(case, seed):
    """The case's systems (frames: two of the same composition, serve: the batch, else one)."""
    rng = np.random.default_rng([int(seed), 7])
    if case["entry"] == "serve":
        out = []
        for k in range(case["count"]):
            f = k / max(1, case["count"] - 1)
            n = case["n_min"] ** (1 - f) * case["n_max"] ** f
            water = k % 2 == 0
            side = (n / (3 if water else 4)) ** (1.0 / 3.0)
            nx, ny = max(2, int(round(side))), max(2, int(round(side)))
            nz = max(2, int(round(side ** 3 / (nx * ny))))
            pos, sp, box = (_water if water else _fcc)(nx, ny, nz, rng)
            s = _system(pos, sp if water else sp + 2, box)   # species over (H, O, Cu)
            sd = np.sqrt(KB * 300.0 / np.asarray(MASS)[s["species"]] * ACCEL)
            s["vel"] = rng.normal(size=pos.shape) * sd[:, None]   # 300 K
            out.append(s)
        return out
    make = _water if case["system"] == "water" else _fcc
    return [_system(*make(case["nx"], case["ny"], case["nz"], rng)) for _ in range(2 if case["entry"] == "frames" else 1)]


def prepare(case, seed):
    import paper_2505_06711_amd as rn
    systems = _frames(case, seed)
    entry, T, precision = case["entry"], case["T"], case["precision"]
    dt = DTYPE[precision]
    st = dict(entry=entry, T=T, precision=precision, dtype=dt, skin=case["skin"], systems=systems)
    st["model"] = model = rn.Model(_model_params(case["model"], T))
    if entry == "serve":
        st["server"] = srv = rn.Server(model, T=T, precision=precision, skin=case["skin"])
        srv.set_masses(MASS)
        st["ids"] = [srv.add_system(s, s["vel"]) for s in systems]
        return st
    st["ctx"] = ctx = rn.Context(0)
    st["decomp"] = (case["split"],) * 3
    if entry == "host":
        return st
    s = systems[0]
    n = s["pos"].shape[0]
    st["plan"] = plan = rn.Plan(ctx, model, s, T=T, precision=precision, decomp=st["decomp"], skin=case["skin"])
    st["pos"] = [torch.tensor(f["pos"], dtype=torch.float64, device="cuda") for f in systems]
    # one block of results: forces, atomic energies, virial, energy
    st["out"] = out = torch.zeros(4 * n + 10, dtype=torch.float64, device="cuda")
    st["n"] = n
    st["views"] = _views(out, n)
    if entry == "autograd":
        st["pos"][0].requires_grad_(True)
    if entry != "frames":
        plan.update_list(st["pos"][0].detach())   # the list an MD run arrives with
    return st


def _views(out, n):
    return out[:3 * n].view(n, 3), out[3 * n:4 * n], out[4 * n:4 * n + 9].view(3, 3), out[4 * n + 9]


def run(state):
    entry, dt = state["entry"], state["dtype"]
    if entry == "serve":
        srv, ids = state["server"], state["ids"]
        waiting = {sid: srv.submit_vv(sid, DT_FS, skip=("positions", "velocities")) for sid in ids}
        got = {}
        while waiting:
            for sid, ticket in list(waiting.items()):
                r = srv.poll(ticket, sid)
                if r is not None:
                    del waiting[sid]
                    got[sid] = r
        return [[torch.tensor(got[sid]["energy"], dtype=dt), torch.from_numpy(got[sid]["forces"]).to(dt)]
                for sid in ids]
    if entry == "host":
        import paper_2505_06711_amd as rn
        E, F, W = rn.energy_forces(state["ctx"], state["model"], state["systems"][0], T=state["T"],
                                   precision=state["precision"], decomp=state["decomp"], skin=state["skin"])
        virial = [] if dt == torch.bfloat16 else [torch.from_numpy(W).to(dt)]
        return [torch.from_numpy(F).to(dt)] + virial + [torch.tensor(E, dtype=dt)]
    plan = state["plan"]
    if entry == "autograd":
        from paper_2505_06711_amd.autograd import reann_energy
        e = reann_energy(state["pos"][0], plan)
        (g,) = torch.autograd.grad(e, state["pos"][0])
        return [g.to(dt), e.detach().to(dt)]
    n = state["n"]
    F, Eat, W, E = state["views"]
    if entry == "energy":
        plan.forward(state["pos"][0], E, atom_energy=Eat)
        _, Eat, _, E = _views(state["out"].to(dt), n)
        return [Eat, E]
    if entry == "frames":
        res = []
        for pos in state["pos"]:
            plan.forward(pos, E)
            plan.backward(F)
            f, _, _, e = _views(state["out"].to(dt, copy=True), n)
            res.append([f, e])
        return res
    plan.forward(state["pos"][0], E, atom_energy=Eat)
    bf16 = dt == torch.bfloat16
    plan.backward(F, virial=None if bf16 else W)
    F, Eat, W, E = _views(state["out"].to(dt), n)
    return [F, Eat, E] if bf16 else [F, Eat, W, E]


# --------------------------------------------------------------------------- work --

def work(case):
    """Bytes: positions in, results out, weights once.  Operations: the edge sums, their adjoint and
    the atomic NNs in both directions, at the mean number of neighbours within the cutoff."""
    m = MODELS[case["model"]]
    K, L, H, nh, T = m["K"], m["L"], m["H"], m["nh"], case["T"]
    NL = (L + 1) * (L + 2) * (L + 3) // 6
    F = K if m["form"] == "radial" else (L + 1) * K * (K + 1) // 2
    sphere = 4.0 / 3.0 * math.pi * m["r_c"] ** 3
    edges = atoms = 0
    if case["entry"] == "serve":
        systems = [(len(s["pos"]), abs(np.linalg.det(s["cell"]))) for s in _frames(case, 0)]
    elif case["system"] == "water":
        g = case["nx"] * case["ny"] * case["nz"]
        systems = [(3 * g, g * SPACING ** 3)]
    else:
        g = case["nx"] * case["ny"] * case["nz"]
        systems = [(4 * g, g * FCC_A ** 3)]
    if case["entry"] == "frames":
        systems *= 2
    for n, vol in systems:
        atoms += n
        edges += n * n / vol * sphere
    back = case["entry"] != "energy"
    nn = 2.0 * (F * H + (nh - 1) * H * H)   # per atom and layer, without the output layer
    dens = 0.0 if m["form"] == "radial" else 3.0 * K * (K + 1) / 2 * NL
    flops = 0.0
    for t in range(T):
        out = 2.0 * H * (K if t < T - 1 else 1)
        fwd = edges * (2 * NL * K + 7 * K + 40) + atoms * (nn + out + dens)
        bwd = edges * (4 * NL * K + 12 * K + 80 + (2 * NL * K if t > 0 else 0)) + atoms * (nn + out + 2 * dens)
        flops += fwd + (bwd if back else 0.0)
    weights = m["ns"] * T * (nn / 2 + H * K) * 4
    return {"bytes": float(24 * atoms + (24 * atoms if back else 8 * atoms) + weights), "flops": float(flops)}


# -------------------------------------------------------------------------- exact --

def exact(case, seed):
    systems = _frames(case, seed)
    p = _model_params(case["model"], case["T"])
    if case["entry"] == "serve":
        res = []
        for s in systems:
            # the server evaluates the first forces at the given positions, then steps
            r = _evaluate(p, s, case["T"], True)
            a = r["forces"] * (ACCEL / np.asarray(MASS)[s["species"]])[:, None]
            moved = dict(s, pos=s["pos"] + s["vel"] * DT_FS + 0.5 * a * DT_FS ** 2)
            r = _evaluate(p, moved, case["T"], True)
            res.append([r["energy"], r["forces"]])
        return res
    if case["entry"] == "frames":
        res = [_evaluate(p, s, case["T"], True) for s in systems]
        return [[r["forces"], r["energy"]] for r in res]
    r = _evaluate(p, systems[0], case["T"], case["entry"] != "energy")
    bf16 = case["precision"] == "bf16"
    return {"plan": lambda: [r["forces"], r["atoms"]] + ([] if bf16 else [r["virial"]]) + [r["energy"]],
            "host": lambda: [r["forces"]] + ([] if bf16 else [r["virial"]]) + [r["energy"]],
            "autograd": lambda: [-r["forces"], r["energy"]],
            "energy": lambda: [r["atoms"], r["energy"]]}[case["entry"]]()


def _neighbours(pos, box, r_c):
    """Padded neighbour arrays of a periodic orthorhombic box, in chunks of rows: a list of
    (first row, neighbour atom [m, D], displacement [m, D, 3], live [m, D])."""
    dev = pos.device
    n = pos.shape[0]
    w = pos - torch.floor(pos / box) * box
    reach = [int(math.floor(r_c / float(b))) + 1 for b in box]
    ys, owners = [w], [torch.arange(n, device=dev)]
    for sx in range(-reach[0], reach[0] + 1):
        for sy in range(-reach[1], reach[1] + 1):
            for sz in range(-reach[2], reach[2] + 1):
                if sx == sy == sz == 0:
                    continue
                y = w + torch.tensor([sx, sy, sz], dtype=pos.dtype, device=dev) * box
                near = ((y > -r_c) & (y < box + r_c)).all(1).nonzero().squeeze(1)
                ys.append(y[near])
                owners.append(near)
    y, owner = torch.cat(ys), torch.cat(owners)
    nb = torch.clamp(torch.floor((box + 2 * r_c) / r_c), min=1).to(torch.int64)
    size = (box + 2 * r_c) / nb
    cell3 = torch.minimum(torch.clamp(((y + r_c) / size).to(torch.int64), min=0), nb - 1)
    stride = torch.stack([nb[1] * nb[2], nb[2], torch.ones_like(nb[0])])
    cell = (cell3 * stride).sum(1)
    order = torch.argsort(cell, stable=True)
    count = torch.bincount(cell, minlength=int(nb.prod()))
    start = torch.cumsum(count, 0) - count
    cap = int(count.max())
    offs = torch.stack(torch.meshgrid(*[torch.arange(-1, 2, device=dev)] * 3, indexing="ij"), -1).reshape(27, 3)
    rows = max(1, min(n, 40_000_000 // (27 * cap)))
    res = []
    for a in range(0, n, rows):
        b = min(n, a + rows)
        c3 = cell3[a:b, None, :] + offs
        ok = ((c3 >= 0) & (c3 < nb)).all(2)
        c = torch.where(ok, (c3 * stride).sum(2), torch.zeros_like(c3[..., 0]))
        k = torch.arange(cap, device=dev)
        cand = (start[c][..., None] + k).reshape(b - a, -1)
        ok = (ok[..., None] & (k < count[c][..., None])).reshape(b - a, -1)
        e = order[torch.where(ok, cand, torch.zeros_like(cand))]
        d = y[e] - w[a:b, None, :]
        hit = ok & ((d * d).sum(2) < r_c * r_c) & (e != torch.arange(a, b, device=dev)[:, None])
        D = max(1, int(hit.sum(1).max()))
        pick = torch.topk(hit.to(torch.int8), D, dim=1).indices
        live = torch.gather(hit, 1, pick)
        res.append((a, owner[torch.gather(e, 1, pick)],
                    torch.gather(d, 1, pick[..., None].expand(-1, -1, 3)).contiguous(), live))
    return res


def _mlp(blob, dims, index):
    size = sum(dims[k] * dims[k - 1] + dims[k] for k in range(1, len(dims)))
    o, out = index * size, []
    for k in range(1, len(dims)):
        W = blob[o:o + dims[k] * dims[k - 1]].view(dims[k], dims[k - 1])
        o += W.numel()
        out.append((W, blob[o:o + dims[k]]))
        o += dims[k]
    return out


def _evaluate(p, system, T, with_forces):
    """Energy, atomic energies, forces and virial in 64 bits with torch: the orbital sums
    S[l,m] = sum_j c_j[m] A_l(d) exp(-a_m (r - r_m)^2) f_c(r), f_c = (cos(pi r / r_c) / 2 + 1/2)^2,
    their weighted pair products of each angular order as features (the radial form: the sums
    themselves, with a residual on c), SiLU networks for the messages and the energy, and
    torch's autograd with respect to the displacements."""
    from torch.utils.checkpoint import checkpoint
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    t64 = lambda a: torch.tensor(np.asarray(a, np.float64), device=dev)  # noqa: E731
    pos, box = t64(system["pos"]), t64(np.diag(system["cell"]))
    spec = torch.as_tensor(system["species"].astype(np.int64), device=dev)
    n, K, radial = pos.shape[0], p.K, p.form == "radial"
    cen, alp, c0 = t64(p.centres), t64(p.alphas), t64(p.c0)
    msg, en = t64(p.msg_blob), t64(p.energy_blob)
    lams = [(l, (a, b, l - a - b)) for l in range(p.L + 1) for a in range(l, -1, -1) for b in range(l - a, -1, -1)]
    fact = math.factorial
    wl = t64([fact(l) / (fact(x) * fact(y) * fact(z)) for l, (x, y, z) in lams])
    iu = torch.triu_indices(K, K, device=dev)

    def sums(d, live, j, c):
        r = torch.sqrt(torch.where(live, (d * d).sum(2), torch.ones_like(d[..., 0])))
        fc = torch.where(live, (0.5 * torch.cos(math.pi * r / p.r_c) + 0.5) ** 2, torch.zeros_like(r))
        w = c[j] * torch.exp(-alp * (r[..., None] - cen) ** 2) * fc[..., None]
        u = d * p.ang_scale
        one = torch.ones_like(r)
        pw = [[one, u[..., a], u[..., a] * u[..., a]] for a in range(3)]
        A = torch.stack([pw[0][x] * pw[1][y] * pw[2][z] for _, (x, y, z) in lams], 1)
        return torch.bmm(A, w)

    def features(S):
        if radial:
            return S[:, 0]
        parts = []
        for l in range(p.L + 1):
            q = [k for k, (ll, _) in enumerate(lams) if ll == l]
            Sl = S[:, q[0]:q[-1] + 1]
            G = torch.bmm((Sl * wl[q[0]:q[-1] + 1, None]).transpose(1, 2).contiguous(), Sl)
            parts.append(G[:, iu[0], iu[1]])
        return torch.cat(parts, 1)

    def network(x, blob, dims, first):
        out = torch.zeros(n, dims[-1], dtype=torch.float64, device=dev)
        for s in range(p.n_species):
            at = (spec == s).nonzero().squeeze(1)
            h = x[at]
            layers = _mlp(blob, dims, first + s)
            for k, (W, b) in enumerate(layers):
                h = h @ W.T + b
                if k + 1 < len(layers):
                    h = torch.nn.functional.silu(h)
            out = out.index_copy(0, at, h)
        return out

    edges = [(a, j, d.requires_grad_(with_forces), live) for a, j, d, live in _neighbours(pos, box, p.r_c)]
    # rows of a chunk split further, so that a chunk's [rows, D, K] intermediates stay small
    dims = [p.F] + [p.hidden] * p.n_hidden
    with torch.set_grad_enabled(with_forces):
        c = c0[spec]
        for t in range(T):
            S = []
            for a, j, d, live in edges:
                step = max(1, 4_000_000 // j.shape[1])
                for b in range(0, j.shape[0], step):
                    part = (d[b:b + step], live[b:b + step], j[b:b + step], c)
                    S.append(checkpoint(sums, *part, use_reentrant=False) if with_forces else sums(*part))
            x = features(torch.cat(S))
            if t < T - 1:
                c = network(x, msg, dims + [K], t * p.n_species) + (c if radial else 0.0)
            else:
                e = network(x, en, dims + [1], 0)[:, 0]
        energy = e.sum()
    out = dict(energy=np.float64(energy.detach().item()), atoms=e.detach().cpu().numpy())
    if with_forces:
        g = torch.autograd.grad(energy, [d for _, _, d, _ in edges])
        F, W = torch.zeros_like(pos), torch.zeros(3, 3, dtype=torch.float64, device=dev)
        for (a, j, d, live), gd in zip(edges, g):
            gd = torch.where(live[..., None], gd, torch.zeros_like(gd))
            F[a:a + j.shape[0]] += gd.sum(1)
            F.index_add_(0, j.reshape(-1), -gd.reshape(-1, 3))
            W -= d.detach().reshape(-1, 3).T.contiguous() @ gd.reshape(-1, 3)
        out["forces"], out["virial"] = F.cpu().numpy(), W.cpu().numpy()
    return out
