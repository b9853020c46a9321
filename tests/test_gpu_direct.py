"""Energies of the fused path at the edges of its two ways of forming them:
summed at the clash-free translations where these are few, by the transforms
where they are many.  One batch holds both, the choice differing between
snapshots (the second has its receptor far outside the box: everything is
free), over chunks of two configurations, eager and replayed from a graph.

Tolerances: raw FP32 energies agree with the oracle to 1e-5 of the largest
|Psi| (1e-10 in FP64), so a minimum does too and a log-sum-exp to beta times
that; counts are integers."""
import numpy as np
import pytest

import oracle
from workload import synth

pytestmark = pytest.mark.gpu


def _workload(n_fft, n_rec, h, precision, sizes, seed):
    w = synth.tiny(seed=seed, n_rec=n_rec, n_fft=n_fft, h=h, n_rec_atoms=60, n_lig_atoms=2, n_cfg=1, n_snap=2,
                   precision=precision)
    w.receptor.xyz[1] += 60.0 + n_rec * h
    rs = synth.streams(seed + 1)
    w.ligands = [synth.make_ligand(rs[1], rs[2], na, 1, nc) for na, nc in sizes]
    return w


# (n_fft, n_rec, h, precision, (atoms, configurations) per ligand): pairs of
# free translations and atoms from a few hundred to 2 million, planes of one
# to over 256 free translations, rows of one to four words
CASES = [(32, 30, 0.5, "f32", [(1, 2), (6, 3)]), (64, 48, 0.5, "f32", [(1, 3), (3, 2), (10, 2)]),
         (64, 48, 0.5, "f64", [(3, 1), (8, 2)]), (128, 100, 0.25, "f32", [(1, 1), (3, 2), (14, 2)])]
# enough configurations for the choice to be offered on the small grids; one
# atom or eight and more (at most 32 or at least 97 runs: the clash test's known
# defect, held by its own test, is between)
CASES += [(32, 30, 0.5, "f32", [(1, 140), (8, 60)]), (32, 30, 0.5, "f64", [(1, 10), (8, 6)]),
          (64, 48, 0.5, "f32", [(1, 14), (10, 10)]), (64, 48, 0.5, "f64", [(1, 1), (8, 3)])]


@pytest.mark.parametrize("n_fft,n_rec,h,precision,sizes", CASES)
def test_partials(n_fft, n_rec, h, precision, sizes):
    import torch
    import paper_1708_07045_amd as fd
    w = _workload(n_fft, n_rec, h, precision, sizes, 11)
    r = w.receptor
    rel = 1e-5 if precision == "f32" else 1e-10
    beta = 1.0 / oracle.kT(w.T)
    want = []
    for s in range(2):
        g, o = oracle.receptor_grids(w, s)
        for l, L in enumerate(w.ligands):
            for c in range(L.n_cfg):
                e = oracle.config_eval(w, g, o, l, c)
                top = np.abs(e["psi"]).max() if e["psi"].size else 0.0
                want.append(np.concatenate([e["partial"], [top]]))
    want = np.array(want).reshape(2, -1, 7)
    free = want[..., 3] * np.concatenate([np.full(L.n_cfg, L.n_atoms) for L in w.ligands])[None]
    assert free.min() < free.max() / 8  # the batch spans both sides
    for fused in (1, 2):
        for graph in (0, 1):
            ctx = fd.FFTDG.from_workload(w)
            ctx.set_tuning(fused=fused, use_graph=graph, configs_per_chunk=2)
            both = [ctx.receptor_grids(r.xyz[s], r.q, r.sigma, r.eps) for s in range(2)]
            ctx.set_receptors(torch.stack([b[0] for b in both]), torch.stack([b[1] for b in both]), r.weights)
            b = fd.Batch(w.ligands)
            out = ctx.alloc_partials(b)
            for _ in range(3):
                out.fill_(255)
                P = ctx.partials_numpy(ctx.scan(b, w.T, out), 2, b.n_cfg)
                assert np.array_equal(P["n_valid"], want[..., 2]) and np.array_equal(P["n_finite"], want[..., 3])
                ok = want[..., 3] > 0
                tol = rel * want[..., 6][ok] + 1e-30
                assert np.all(np.abs(P["psi_min"][ok] - want[..., 4][ok]) <= tol)
                dz = (P["m"][ok] + np.log(P["s"][ok])) - (want[..., 0][ok] + np.log(want[..., 1][ok]))
                assert np.all(np.abs(dz) <= beta * tol + rel)
                assert np.all(np.isposinf(P["psi_min"][~ok])) and np.all(P["argmin"][~ok] == -1)
