"""A configuration's record is its own: equal, bit for bit, whether the call scans it alone, among a few or
with all others of the batch (a selected or sharded scan is then a part of the whole one)."""
import numpy as np
import pytest

from workload import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_fft,n_rec,h,precision,n_cfg", [(32, 30, 0.5, "f32", 420), (32, 30, 0.5, "f64", 60),
                                                           (64, 48, 0.5, "f32", 60), (64, 48, 0.5, "f64", 20),
                                                           (128, 96, 0.25, "f32", 20)])
def test_record_does_not_depend_on_the_others(n_fft, n_rec, h, precision, n_cfg):
    import paper_1708_07045_amd as fd
    w = synth.tiny(seed=4, n_rec=n_rec, n_fft=n_fft, h=h, n_rec_atoms=60, n_lig_atoms=6, n_cfg=n_cfg, precision=precision)
    r = w.receptor
    ctx = fd.FFTDG.from_workload(w)
    g, o = ctx.receptor_grids(r.xyz[0], r.q, r.sigma, r.eps)
    ctx.set_receptors(g[None], o[None], r.weights)
    b = fd.Batch(w.ligands)
    whole = ctx.partials_numpy(ctx.scan(b, w.T), 1, n_cfg)[0].copy()
    assert (whole["n_finite"] > 0).any()
    for pick in ([0], [n_cfg - 1], [3, 4, 11]):
        sel = np.zeros(n_cfg, np.uint8)
        sel[pick] = 1
        part = ctx.partials_numpy(ctx.scan(b.with_select(sel), w.T), 1, n_cfg)[0]
        assert part[pick].tobytes() == whole[pick].tobytes()
