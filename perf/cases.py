"""Timed workloads of the library: what a program that uses it has it do.

The path is the translational scan (spread, transform, correlate, mask, average) and what goes
before and after it: the receptor's grids and spectra, the energies of one configuration, poses drawn
from a finished scan, and the proposal network that chooses configurations.  Sizes are those of the
repository's own workloads (a 16 A-class site grid at 0.25 A in a 128-point transform, its coarse form
at 0.5 A in 64, a 62 A whole-surface grid in 256, a 32-point grid in double precision) and odd ones
around them.  Inputs are synthetic and made from the seed: receptor atoms in a shell around a cavity (or
a ball), compact self-avoiding trees as ligands, uniform rotations, jittered snapshots.

exact() evaluates the same quantities in 64 bits with plain torch: the grids of pairwise terms, the
trilinear and ball rasters, the correlations by torch's own transforms, the averages.  A record's energies
are kept in the context's precision by the library (the record itself is double), so run() hands them on
in that precision.  The index of the lowest energy is not handed on: which of two energies that agree to
rounding is the lower one is decided by the order of the transforms' rounding.
"""
import math

import numpy as np
import torch

import paper_1708_07045_amd as fd

T_KELVIN = 300.0
KT = 1.987204259e-3 * T_KELVIN
C_STANDARD = 6.02214076e-4
COULOMB = 332.05
OCC_F = 0.5
LJR_CAP = 10.0
N_IN = 21      # inputs of the proposal network: 18 configuration features and 3 of a coarse scan
WIDTH = 256


def scan_case(name=None, **kw):
    c = dict(kind="scan", n_rec=96, n_fft=128, h=0.25, precision="f32", mode="occ", rec_atoms=2600, snaps=1,
             ligands=1, atoms_lo=25, atoms_hi=25, conformers=8, cfgs=1000, select=1.0, graph=False)
    c.update(kw)
    return dict({"name": name} if name else {}, **c)


SURFACE = dict(n_rec=248, n_fft=256)
COARSE = dict(n_rec=48, n_fft=64, h=0.5)
TINY = dict(n_rec=32, n_fft=32, h=0.5, precision="f64", mode="cap", rec_atoms=300, atoms_lo=12, atoms_hi=12,
            conformers=1, cfgs=100)


def listed():
    return [
        # the tiny plain case in double precision: a check of settings, the smallest scan there is
        scan_case("scan 32 f64 cap", **TINY),
        # a few configurations of one ligand scored again, for instance after a visual check
        scan_case("scan 128 few", cfgs=24, conformers=3),
        # one ligand against one receptor structure, exhaustively: the repository's headline workload
        scan_case("scan 128 site", cfgs=8000),
        # uneven ligands against an ensemble of snapshots in one batch
        scan_case("scan 128 batch", ligands=9, atoms_lo=8, atoms_hi=40, conformers=4, cfgs=1800, snaps=10),
        # an importance-sampled scan: one configuration in ten, the others only counted, weights in the average
        scan_case("scan 128 selected", ligands=6, atoms_lo=8, atoms_hi=40, cfgs=6000, snaps=3, select=0.1),
        # the coarse pre-scan that ranks configurations before the fine one
        scan_case("scan 64 coarse", ligands=12, atoms_lo=8, atoms_hi=40, conformers=4, cfgs=6000, snaps=5, **COARSE),
        # the whole receptor surface
        scan_case("scan 256 surface", cfgs=64, **SURFACE),
        # the energies of one configuration at every translation, out of a ligand's thousand
        scan_case("energies 128", kind="energies", cfgs=1000),
        # poses drawn from a finished scan for the solvation leg
        scan_case("poses 128", kind="poses", cfgs=1000, draws=100),
        # a new receptor structure: its grids and spectra, and the first configurations on it
        scan_case("receptor 128", kind="receptor", cfgs=8),
        # the proposal's prediction for a pool of configurations, in the blocks the proposal driver uses
        dict(name="network forward", kind="forward", rows=20000, block=512),
        # its training: a few batches of 512 rows
        dict(name="network train", kind="train", rows=20000, block=512, batch=512, steps=20),
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["site"] * 6 + ["coarse"] * 3 + ["double"] * 2 + ["surface", "energies", "poses", "receptor",
                                                                        "forward", "train"])
    if kind == "forward":
        return dict(kind="forward", rows=log_int(rng, 1, 20000), block=rng.choice([512, 512, 1000, 4096]))
    if kind == "train":
        return dict(kind="train", rows=log_int(rng, 600, 20000), block=512, batch=rng.choice([512, 512, 256, 500, 77]),
                    steps=rng.randint(1, 20))
    lo = rng.randint(6, 30)
    many = rng.random() < 0.5
    c = scan_case(ligands=rng.randint(2, 8) if many else 1, atoms_lo=lo, atoms_hi=min(44, lo + rng.randint(0, 20)),
                  conformers=rng.randint(1, 4), rec_atoms=rng.randint(2000, 2800), n_rec=rng.randint(80, 112))
    if kind == "site":
        c.update(snaps=rng.choice([1, 1, 2, 3, 5, 10]), graph=rng.random() < 0.2)
        c["cfgs"] = log_int(rng, c["ligands"], 7000 // c["snaps"])
        if rng.random() < 0.2:
            c["select"] = rng.choice([0.05, 0.1, 0.3])
    elif kind == "coarse":
        c.update(n_rec=rng.randint(40, 56), n_fft=64, h=0.5, snaps=rng.choice([1, 2, 5, 10]))
        c["cfgs"] = log_int(rng, c["ligands"], 24000 // c["snaps"])
    elif kind == "double":
        n = rng.choice([32, 64])
        c.update(n_fft=n, n_rec=rng.randint(26, 32) if n == 32 else rng.randint(40, 56), h=0.5, precision="f64",
                 mode=rng.choice(["occ", "cap"]), rec_atoms=300, atoms_hi=min(c["atoms_hi"], lo + 4), ligands=1)
        if n == 32:
            c.update(atoms_lo=rng.randint(6, 12), atoms_hi=12)
        c["cfgs"] = log_int(rng, 1, 1000)
    elif kind == "surface":
        c.update(n_rec=rng.randint(180, 248), n_fft=256, ligands=1, cfgs=log_int(rng, 1, 48))
    elif kind == "energies":
        c.update(kind="energies", ligands=1, cfgs=log_int(rng, 1, 2000))
    elif kind == "poses":
        c.update(kind="poses", ligands=1, cfgs=log_int(rng, 10, 1000), draws=rng.choice([10, 50, 100]))
    else:
        c.update(kind="receptor", ligands=1, cfgs=8)
    return c


# ------------------------------------------------------------------ inputs
class Ligand:
    def __init__(self, q, sigma, eps, conformers, cfg_conf, cfg_quat):
        self.q, self.sigma, self.eps, self.conformers = q, sigma, eps, conformers
        self.cfg_conf, self.cfg_quat = cfg_conf, cfg_quat
        self.n_atoms, self.n_cfg = q.shape[0], cfg_conf.shape[0]


def atom_parameters(g, n, tiny):
    q = g.normal(0.0, 0.4 if tiny else 0.1, n)
    eps = g.uniform(0.05, 0.2, n) if tiny else g.uniform(0.025, 0.1, n)
    return q, g.uniform(3.0, 4.0, n), eps


def directions(g, n):
    v = g.normal(size=(n, 3))
    return v / np.linalg.norm(v, axis=1, keepdims=True)


def receptor_atoms(g, c):
    """Atoms of every snapshot [snaps][n][3] and their parameters; charges neutral in groups of about four."""
    tiny, n = c["rec_atoms"] <= 300, c["rec_atoms"]
    r_in, r_out = (0.0, 8.0) if tiny else (10.0, 19.3)
    r = (r_in ** 3 + (r_out ** 3 - r_in ** 3) * g.random(n)) ** (1.0 / 3.0)
    xyz = directions(g, n) * r[:, None]
    q, sigma, eps = atom_parameters(g, n, tiny)
    centre = xyz[g.choice(n, max(1, n // 4), replace=False)]
    lab = np.argmin(((xyz ** 2).sum(1)[:, None] - 2.0 * xyz @ centre.T + (centre ** 2).sum(1)[None]), axis=1)
    mean = np.bincount(lab, q, len(centre)) / np.maximum(1, np.bincount(lab, minlength=len(centre)))
    snaps = np.stack([xyz + (g.normal(0.0, 0.3, xyz.shape) if s else 0.0) for s in range(c["snaps"])])
    return snaps, q - mean[lab], sigma, eps


def compact_tree(g, n):
    """A self-avoiding tree: each atom 1.5 A from an earlier one (near the centroid by preference, at most three
    bonds each), 2.5 A from all others."""
    while True:
        x, bonds, i, tries = np.zeros((n, 3)), np.zeros(n, int), 1, 0
        while i < n and tries < 20 * n:
            free = np.flatnonzero(bonds[:i] < 3)
            d = np.linalg.norm(x[free] - x[:i].mean(0), axis=1)
            p = np.exp(-(d - d.min()) / 1.5)
            to = free[g.choice(len(free), 64, p=p / p.sum())]
            new = x[to] + 1.5 * directions(g, 64)
            far = np.linalg.norm(new[:, None] - x[None, :i], axis=2)
            far[np.arange(64), to] = 9.0
            ok = np.flatnonzero(far.min(1) >= 2.5)
            tries += 1
            if not len(ok):
                continue
            x[i] = new[ok[0]]
            bonds[to[ok[0]]] += 1
            bonds[i] += 1
            i += 1
        if i == n:
            return x


def rotations(g, n):
    u1, u2, u3 = g.random(n), 2 * np.pi * g.random(n), 2 * np.pi * g.random(n)
    a, b = np.sqrt(1.0 - u1), np.sqrt(u1)
    return np.stack([a * np.sin(u2), a * np.cos(u2), b * np.sin(u3), b * np.cos(u3)], axis=1)


def inputs(c, seed):
    """(receptor atoms, ligands, select mask or None, weights or None): host arrays, from the seed alone."""
    g = np.random.Generator(np.random.PCG64([seed, 5]))
    rec = receptor_atoms(g, c)
    nl = c["ligands"]
    share = g.uniform(0.2, 2.0, nl)
    cuts = np.floor(np.cumsum(share) / share.sum() * (c["cfgs"] - nl) + 0.5).astype(int)
    counts = np.diff(np.concatenate([[0], cuts])) + 1
    ligs = []
    # one configuration's energies: a given ligand (its extents are the result's shape) on a new receptor
    gl = np.random.Generator(np.random.PCG64(17)) if c["kind"] == "energies" else g
    for k in range(nl):
        n = int(gl.integers(c["atoms_lo"], c["atoms_hi"] + 1))
        q, sigma, eps = atom_parameters(g, n, c["rec_atoms"] <= 300)
        conf = np.stack([compact_tree(gl, n) for _ in range(c["conformers"])])
        m = int(counts[k])
        ligs.append(Ligand(q - q.mean(), sigma, eps, conf, (np.arange(m) * c["conformers"] // m).astype(np.int32),
                           rotations(gl, m)))
    if c["select"] >= 1.0:
        return rec, ligs, None, None
    sel = (g.random(c["cfgs"]) < c["select"]).astype(np.uint8)
    sel[0] = 1
    return rec, ligs, sel, np.where(sel > 0, 1.0 / c["select"], 0.0)


def grid_origin(c):
    return np.full(3, -0.5 * (c["n_rec"] - 1) * c["h"])


def network_data(c, seed):
    g = np.random.Generator(np.random.PCG64([seed, 7]))
    n = c["rows"]
    x = np.zeros((n, N_IN), np.float32)
    x[:, :4] = rotations(g, n)
    x[np.arange(n), 4 + g.integers(0, 8, n)] = 1.0
    x[:, 12:18] = g.uniform(0.2, 1.1, (n, 6))
    x[:, 18], x[:, 19], x[:, 20] = -5.0 * g.random(n) ** 2, 5.0 * g.random(n), 0.1 * g.random(n)
    layers = []
    for r, k in ((WIDTH, N_IN), (WIDTH, WIDTH), (WIDTH, WIDTH), (1, WIDTH)):
        a = 1.0 / math.sqrt(k)
        layers += [g.uniform(-a, a, r * k), g.uniform(-a, a, r)]
    p = np.concatenate(layers).astype(np.float32)
    t = np.clip(x[:, 18] + 0.3 * g.normal(size=n), -5.0, 0.0).astype(np.float32)
    w = np.where(t > -1.0, 10.0, 1.0).astype(np.float32)
    idx = g.integers(0, n, c.get("steps", 1) * c.get("batch", 1)).astype(np.int32)
    return x, p, t, w, idx


# ------------------------------------------------------------------ the calls
def context(c):
    ctx = fd.FFTDG(c["n_rec"], c["n_fft"], c["h"], grid_origin(c), c["precision"], c["mode"], LJR_CAP, OCC_F)
    if c["n_fft"] > 128:
        ctx.set_tuning(energy_xy_direct=2)  # what the autotuner keeps at this size
    if c["graph"]:
        ctx.set_tuning(use_graph=1)
    return ctx


def receptors(ctx, rec):
    xyz, q, sigma, eps = rec
    both = [ctx.receptor_grids(x, q, sigma, eps) for x in xyz]
    grids = torch.stack([b[0] for b in both])
    occ = torch.stack([b[1] for b in both]) if both[0][1] is not None else None
    ctx.set_receptors(grids, occ)
    return grids, occ


def prepare(case, seed):
    c = case
    if c["kind"] in ("forward", "train"):
        x, p, t, w, idx = network_data(c, seed)
        net = fd.Network(N_IN, WIDTH, c["block"])
        net.set_skip(18, 1.0)
        net.set_params(p)
        to = lambda a: torch.as_tensor(a, device="cuda")  # noqa: E731
        return dict(c=c, net=net, x=to(x), t=to(t), w=to(w), idx=to(idx).view(-1, c.get("batch", 1)))
    rec, ligs, sel, weight = inputs(c, seed)
    ctx = context(c)
    batch = fd.Batch(ligs, sel)
    s = dict(c=c, ctx=ctx, batch=batch, rec=rec)
    if c["kind"] == "receptor":
        return s
    receptors(ctx, rec)
    s["weight"] = None if weight is None else torch.as_tensor(weight, device="cuda")
    s["out"] = ctx.alloc_partials(batch)
    if c["kind"] == "poses":
        ctx.scan(batch, T_KELVIN, s["out"])
        s["u"] = np.random.Generator(np.random.PCG64([seed, 9])).random(2 * c["draws"])
    return s


def scan_outputs(s, out):
    c, ctx, batch = s["c"], s["ctx"], s["batch"]
    B, res = ctx.reduce(batch, out, T_KELVIN, s.get("weight"))
    kind, host = (torch.float32, np.float32) if c["precision"] == "f32" else (torch.float64, np.float64)
    v = out.view(torch.float64).view(ctx.n_snap, batch.n_cfg, 5)[..., :3].to(kind)
    k = out.view(torch.int32).view(ctx.n_snap, batch.n_cfg, 10)
    return {"m": v[..., 0], "s": v[..., 1], "psi_min": v[..., 2], "n_valid": k[..., 6], "n_finite": k[..., 7],
            "scanned": k[..., 9], "B": B.astype(host), "dG": res["dG"].astype(host), "v_site": res["v_site"],
            "psi_best": res["psi_min"].astype(host), "finite": res["n_finite"], "samples": res["n_samples"]}


def run(s):
    c = s["c"]
    if c["kind"] == "forward":
        return s["net"].forward(s["x"])
    if c["kind"] == "train":
        for k in range(c["steps"]):
            s["net"].train_step(s["x"], s["t"], s["w"], s["idx"][k], 1e-3)
        return s["net"].get_params()
    ctx, batch = s["ctx"], s["batch"]
    if c["kind"] == "energies":
        return ctx.energy_grid(0, batch, c["cfgs"] // 3, T_KELVIN)
    if c["kind"] == "poses":
        cfg, t, psi = ctx.sample_poses(batch, s["out"], 0, 0, T_KELVIN, s["u"])
        return {"cfg": cfg, "t": t, "psi": psi.astype(np.float32)}
    if c["kind"] == "receptor":
        grids, occ = receptors(ctx, s["rec"])
        return dict(scan_outputs(s, ctx.scan(batch, T_KELVIN)), grids=grids, occ=occ)
    return scan_outputs(s, ctx.scan(batch, T_KELVIN, s["out"]))


# ------------------------------------------------------------------ what cannot be done without
def work(case):
    c = case
    if c["kind"] in ("forward", "train"):
        per = 2.0 * (WIDTH * N_IN + 2 * WIDTH * WIDTH + WIDTH)
        n_par = per / 2 + 3 * WIDTH + 1
        if c["kind"] == "forward":
            return {"bytes": 4.0 * (c["rows"] * (N_IN + 1) + n_par), "flops": per * c["rows"]}
        rows = c["steps"] * c["batch"]
        return {"bytes": 4.0 * (rows * (N_IN + 3) + 6 * n_par * c["steps"]), "flops": 3.0 * per * rows}
    n, n3, e = c["n_rec"], float(c["n_rec"]) ** 3, 4 if c["precision"] == "f32" else 8
    occ = c["mode"] == "occ"
    atoms = 0.5 * (c["atoms_lo"] + c["atoms_hi"])
    edge = max(4.0, n - 4.0 - 2.8 * atoms ** (1.0 / 3.0) / c["h"])   # box-valid translations along an axis
    # energies: at every translation that may be free of clashes, by the 8-point sum or by transforms
    share = (0.7 if n * c["h"] > 40 else 0.032) if occ and c["kind"] != "energies" else 1.0
    fft = 10.0 * c["n_fft"] ** 3 * 3 * math.log2(c["n_fft"])
    per = min(fft, edge ** 3 * (share * atoms * 48.0 + 1.0))
    scans = c["cfgs"] * c["select"] * c["snaps"]
    grid_bytes = c["snaps"] * n3 * (3 * e + (1 if occ else 0))
    if c["kind"] == "energies":
        return {"bytes": grid_bytes + edge ** 3 * (e + 1), "flops": per}
    if c["kind"] == "poses":
        return {"bytes": grid_bytes + 40.0 * c["cfgs"], "flops": per * c["draws"]}
    make = n3 * c["rec_atoms"] * 25.0 * c["snaps"] if c["kind"] == "receptor" else 0.0
    return {"bytes": grid_bytes + c["cfgs"] * (40.0 * c["snaps"] + 12.0 * atoms), "flops": make + per * scans}


# ------------------------------------------------------------------ 64 bits
def exact_grids(c, xyz, q, sigma, eps, dev):
    n, h, o = c["n_rec"], c["h"], grid_origin(c)[0]
    ax = o + h * torch.arange(n, dtype=torch.float64, device=dev)
    out = torch.zeros((3, n, n, n), dtype=torch.float64, device=dev)
    hit = torch.zeros((n, n, n), dtype=torch.bool, device=dev)
    rex = 2.0 ** (-1.0 / 6.0) * sigma
    se, s3 = np.sqrt(eps), sigma ** 3
    step = max(1, (1 << 26) // (n * n * n))
    for a in range(0, len(q), step):
        col = lambda v: torch.as_tensor(v[a:a + step], device=dev)[:, None, None, None]  # noqa: E731
        dx, dy, dz = (col(xyz[:, d].copy()) for d in range(3))
        d2 = (dx - ax[None, None, None, :]) ** 2 + (dy - ax[None, None, :, None]) ** 2 + (dz - ax[None, :, None, None]) ** 2
        near = d2 < col(rex * rex)
        hit |= (d2 < col((OCC_F * rex) ** 2)).any(0)
        r6 = 1.0 / (d2 * d2 * d2)
        keep = ~near
        out[0] += (col(COULOMB * q) * torch.rsqrt(d2) * keep).sum(0)
        out[2] += (col(se * s3) * r6 * keep).sum(0)
        rep = col(se * s3 * s3) * r6 * r6
        out[1] += (rep if c["mode"] == "cap" else torch.where(keep, rep, torch.zeros_like(rep))).sum(0)
    if c["mode"] == "cap":
        out[1].clamp_(max=LJR_CAP)
    return out, hit


def exact_place(c, L):
    """Lattice coordinates (2^-16 grid units) [cfg][atom][3] and valid translations [cfg][3] (x, y, z)."""
    X = L.conformers - L.conformers.mean(1, keepdims=True)
    w, x, y, z = (L.cfg_quat / np.linalg.norm(L.cfg_quat, axis=1, keepdims=True)).T
    R = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                  2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                  2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], axis=1).reshape(-1, 3, 3)
    Y = np.einsum("cde,cne->cnd", R, X[L.cfg_conf])
    U = np.floor(((Y - Y.min(1, keepdims=True)) / c["h"] + 2.0) * 65536.0 + 0.5).astype(np.int64)
    box = -(-U.max(1) // 65536) + 2
    return U, np.maximum(c["n_rec"] - box, 0)


def exact_energies(c, spec, L, U, dev):
    """Psi and the clash mask on the whole periodic grid for the configurations U, one snapshot's spectra."""
    N, nb, na = c["n_fft"], U.shape[0], U.shape[1]
    u = torch.as_tensor(U, device=dev)
    i, f = u >> 16, (u & 65535).double() / 65536.0
    s3, se = L.sigma ** 3, np.sqrt(L.eps)
    gam = torch.as_tensor(np.stack([L.q, se * s3 * s3, -2.0 * se * s3]), device=dev)
    occ = len(spec) == 4
    G = torch.zeros((nb, len(spec), N * N * N), dtype=torch.float64, device=dev)
    for k in range(8):
        d = [(k >> b) & 1 for b in range(3)]
        wgt = torch.stack([f[..., b] if d[b] else 1.0 - f[..., b] for b in range(3)]).prod(0)
        p = (((i[..., 2] + d[2]) % N) * N + (i[..., 1] + d[1]) % N) * N + (i[..., 0] + d[0]) % N
        for ch in range(3):
            G[:, ch].scatter_add_(1, p, wgt * gam[ch])
    if occ:
        thr = np.ceil((OCC_F * 2.0 ** (-1.0 / 6.0) * L.sigma / c["h"]) ** 2 * 4294967296.0)
        r = int(math.sqrt(thr.max()) / 65536.0) + 1
        o = torch.arange(-r, r + 2, device=dev)
        at = [i[..., b, None] + o for b in range(3)]
        sq = [(at[b] * 65536 - u[..., b, None]) ** 2 for b in range(3)]
        D = sq[2][..., :, None, None] + sq[1][..., None, :, None] + sq[0][..., None, None, :]
        p = ((at[2][..., :, None, None] % N) * N + at[1][..., None, :, None] % N) * N + at[0][..., None, None, :] % N
        ins = D < torch.as_tensor(thr, device=dev)[None, :, None, None, None]
        row = torch.arange(nb, device=dev)[:, None, None, None, None].expand_as(p)
        G[row[ins], 3, p[ins]] = 1.0
    F = torch.fft.rfftn(G.view(nb, len(spec), N, N, N), dim=(2, 3, 4)).conj()
    back = lambda P: torch.fft.irfftn(P, s=(N, N, N), dim=(1, 2, 3))  # noqa: E731
    for s in spec[0]:
        psi = back(sum(spec[ch][s] * F[:, ch] for ch in range(3)))
        yield psi, (back(spec[3][s] * F[:, 3]) > 0.5 if occ else None)


def exact_spectra(c, rec, dev, grids=None):
    N, n = c["n_fft"], c["n_rec"]
    spec = [{} for _ in range(4 if c["mode"] == "occ" else 3)]
    for s, x in enumerate(rec[0]):
        g, hit = exact_grids(c, x, *rec[1:], dev)
        if grids is not None:
            grids.append(g.clone())
        if c["precision"] == "f32":
            g = g.float().double()
        for ch in range(len(spec)):
            pad = torch.zeros((N, N, N), dtype=torch.float64, device=dev)
            pad[:n, :n, :n] = g[ch] if ch < 3 else hit.double()
            spec[ch][s] = torch.fft.rfftn(pad)
    return spec


def exact_scan(c, spec, ligs, sel, weight, dev):
    S, C, nb = c["snaps"], c["cfgs"], max(1, (1 << 25) // c["n_fft"] ** 3)
    m = torch.full((S, C), -math.inf, dtype=torch.float64, device=dev)
    s, low = torch.zeros_like(m), torch.full_like(m, math.inf)
    n_valid, base = np.zeros(C), 0
    t = torch.arange(c["n_fft"], device=dev)
    for L in ligs:
        U, V = exact_place(c, L)
        n_valid[base:base + L.n_cfg] = V.prod(1)
        todo = np.flatnonzero((V.min(1) > 0) & (sel[base:base + L.n_cfg] > 0 if sel is not None else True))
        for a in range(0, len(todo), nb):
            k = todo[a:a + nb]
            v = torch.as_tensor(V[k], device=dev)
            box = ((t < v[:, 2, None])[:, :, None, None] & (t < v[:, 1, None])[:, None, :, None]
                   & (t < v[:, 0, None])[:, None, None, :])
            at = torch.as_tensor(base + k, device=dev)
            for sn, (psi, clash) in enumerate(exact_energies(c, spec, L, U[k], dev)):
                x = torch.where(box if clash is None else box & ~clash, psi, torch.full_like(psi, math.inf)).flatten(1)
                lo = x.min(1).values
                low[sn, at], m[sn, at] = lo, -lo / KT
                fin = torch.isfinite(lo)
                s[sn, at] = torch.where(fin, torch.exp((torch.where(fin, lo, torch.zeros_like(lo))[:, None] - x) / KT).sum(1),
                                        torch.zeros_like(lo))
        base += L.n_cfg
    m, s, low = m.cpu().numpy(), s.cpu().numpy(), low.cpu().numpy()
    B, dG, vs, best, base = [], [], [], [], 0
    wt = np.ones(C) if weight is None else weight
    with np.errstate(divide="ignore", invalid="ignore"):
        lz = m + np.log(s) + np.log(wt)[None, :]
        lz[~np.isfinite(m) | (wt <= 0)[None, :]] = -math.inf
    for L in ligs:
        z, n = lz[:, base:base + L.n_cfg], n_valid[base:base + L.n_cfg]
        top = z.max(1, keepdims=True)
        top[~np.isfinite(top)] = 0.0
        with np.errstate(divide="ignore"):
            b = -KT * (top[:, 0] + np.log(np.exp(z - top).sum(1)) - math.log(n.sum()))
        v = c["h"] ** 3 * n.mean()
        lead = b.min()
        B.append(b)
        vs.append(v)
        dG.append(math.inf if not math.isfinite(lead) else
                  lead - KT * math.log(np.exp(-(b - lead) / KT).mean()) - KT * math.log(v * C_STANDARD))
        best.append(low[:, base:base + L.n_cfg].min())
        base += L.n_cfg
    return {"m": m, "s": s, "psi_min": low, "n_valid": None, "n_finite": None, "scanned": None, "B": np.stack(B),
            "dG": np.array(dG), "v_site": np.array(vs), "psi_best": np.array(best), "finite": None, "samples": None}


def exact_network(c, seed, dev):
    x, p, t, w, idx = (torch.as_tensor(a, device=dev) for a in network_data(c, seed))
    p = p.double().requires_grad_(c["kind"] == "train")

    def forward(rows):
        a, at = rows.double(), 0
        for k, (r, n) in enumerate(((WIDTH, N_IN), (WIDTH, WIDTH), (WIDTH, WIDTH), (1, WIDTH))):
            a = a @ p[at:at + r * n].view(r, n).T + p[at + r * n:at + r * n + r]
            at += r * n + r
            a = torch.nn.functional.silu(a) if k < 3 else a
        return a[:, 0] + rows[:, 18].double()

    if c["kind"] == "forward":
        return forward(x)
    opt = torch.optim.Adam([p], lr=1e-3)
    for k in idx.view(c["steps"], c["batch"]).long():
        opt.zero_grad()
        wk = w[k].double()
        ((wk * (forward(x[k]) - t[k].double()) ** 2).sum() / wk.sum()).backward()
        opt.step()
    return p.detach()


def exact(case, seed):
    c = case
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if c["kind"] in ("forward", "train"):
        return exact_network(c, seed, dev)
    rec, ligs, sel, weight = inputs(c, seed)
    if c["cfgs"] * c["select"] * (4 + 2 * c["snaps"]) * c["n_fft"] ** 3 > 2.5e11:
        return None  # minutes of double-precision transforms
    grids = []
    spec = exact_spectra(c, rec, dev, grids)
    if c["kind"] == "receptor":
        return dict(exact_scan(c, spec, ligs, sel, weight, dev), grids=torch.stack(grids), occ=None)
    if c["kind"] == "scan":
        return exact_scan(c, spec, ligs, sel, weight, dev)
    L = ligs[0]
    U, V = exact_place(c, L)

    def energies(k):
        psi, clash = next(exact_energies(c, spec, L, U[k:k + 1], dev))
        x, y, z = V[k]
        return psi[0, :z, :y, :x], clash[0, :z, :y, :x]

    if c["kind"] == "energies":
        return energies(c["cfgs"] // 3)[0], None
    u = np.random.Generator(np.random.PCG64([seed, 9])).random(2 * c["draws"])
    part = exact_scan(c, spec, ligs, None, None, dev)
    z = np.where(np.isfinite(part["m"][0]), np.exp(part["m"][0] - part["m"][0].max()) * part["s"][0], 0.0)
    cdf = np.cumsum(z)
    psi = np.zeros(c["draws"])
    pick = np.minimum(np.searchsorted(cdf, u[0::2] * cdf[-1], side="right"), len(z) - 1)
    for k in np.unique(pick):
        e, clash = energies(int(k))
        e = e.flatten()
        x = torch.where(clash.flatten(), torch.zeros_like(e), torch.exp((e[~clash.flatten()].min() - e) / KT))
        run_sum = x.cumsum(0)
        mine = np.flatnonzero(pick == k)
        at = torch.searchsorted(run_sum, torch.as_tensor(u[1::2][mine], device=dev) * run_sum[-1], right=True)
        psi[mine] = e[at.clamp(max=len(e) - 1)].cpu().numpy()
    return {"cfg": None, "t": None, "psi": psi}
