"""Clash test on bits (fused path) where its tables and loops have edges: one
to four output words per row, receptor grids that fill the transform (rows
continued past both ends, balls that wrap), ligands of a few runs up to runs
cut into pieces.  The mask and the counts are integers: equal to the oracle's."""
import numpy as np
import pytest

import oracle
from workload import synth

pytestmark = pytest.mark.gpu


# rows of a ligand with at most 96 runs count as decided after phase 1, whose
# strided walk misses runs where the stride shares a factor with their number
MISSED = pytest.mark.xfail(strict=True, reason="phase 1's stride misses runs of this ligand (at most 96 of them)")

# (n_fft, n_rec, h, ligand atoms, occ_f): words per row 1, 1, 2, 2, 3, 4; the
# last two have balls wide enough for long unions and for the table's margin
CASES = [(32, 32, 1.0, 2, 0.5), (64, 31, 0.5, 3, 0.5), pytest.param(64, 64, 0.5, 5, 0.5, marks=MISSED),
         (128, 70, 0.25, 4, 0.5), (128, 112, 0.25, 1, 0.5), pytest.param(128, 128, 0.5, 2, 0.5, marks=MISSED),
         (64, 64, 0.5, 12, 0.5), (128, 128, 0.25, 3, 0.5), (128, 100, 0.25, 12, 0.55), (64, 60, 0.25, 9, 0.5)]


@pytest.mark.parametrize("n_fft,n_rec,h,n_at,occ_f", CASES)
def test_mask_and_counts(n_fft, n_rec, h, n_at, occ_f):
    import paper_1708_07045_amd as fd
    w = synth.tiny(seed=7 + n_rec, n_rec=n_rec, n_fft=n_fft, h=h, n_rec_atoms=40, n_lig_atoms=n_at, n_cfg=3,
                   occ_f=occ_f, precision="f32")
    ctx = fd.FFTDG.from_workload(w)
    r = w.receptor
    g, o = ctx.receptor_grids(r.xyz[0], r.q, r.sigma, r.eps)
    ctx.set_receptors(g[None], o[None], r.weights)
    b = fd.Batch(w.ligands)
    P = ctx.partials_numpy(ctx.scan(b, w.T), 1, b.n_cfg)[0]
    go, oo = oracle.receptor_grids(w)
    for c in range(b.n_cfg):
        e = oracle.config_eval(w, go, oo, 0, c)
        if e["psi"].size == 0:
            assert P["n_valid"][c] == 0
            continue
        assert P["n_valid"][c] == e["psi"].size
        assert P["n_finite"][c] == int((e["clash"] == 0).sum())
        _, mask = ctx.energy_grid(0, b, c)
        assert np.array_equal(mask.cpu().numpy(), e["clash"])


@pytest.mark.parametrize("n_at,n_rec", [(12, 110), (9, 100)])
def test_long_runs(n_at, n_rec):
    """A straight chain along x, y or z: along x its rows are unions of
    overlapping balls longer than one piece of a run (63 points), across bit
    64 of the row."""
    import paper_1708_07045_amd as fd
    w = synth.tiny(seed=3, n_rec=n_rec, n_fft=128, h=0.25, n_rec_atoms=50, n_lig_atoms=n_at, n_cfg=1, precision="f32")
    L = w.ligands[0]
    x = np.zeros((1, n_at, 3))
    x[0, :, 0] = 1.5 * np.arange(n_at)
    r = np.sqrt(0.5)
    quat = np.array([[1.0, 0, 0, 0], [r, 0, 0, r], [r, 0, r, 0], [0.98, 0.02, 0.05, 0.1]])
    w.ligands = [synth.Ligand(L.q, L.sigma, L.eps, x, np.zeros(4, np.int32), quat)]
    ctx = fd.FFTDG.from_workload(w)
    rc = w.receptor
    g, o = ctx.receptor_grids(rc.xyz[0], rc.q, rc.sigma, rc.eps)
    ctx.set_receptors(g[None], o[None], rc.weights)
    b = fd.Batch(w.ligands)
    go, oo = oracle.receptor_grids(w)
    for c in range(4):
        e = oracle.config_eval(w, go, oo, 0, c)
        _, mask = ctx.energy_grid(0, b, c)
        assert np.array_equal(mask.cpu().numpy(), e["clash"])
