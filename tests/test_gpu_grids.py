"""Receptor grids (Eqs. 7, 10) where the kernel's tiling has edges: grid rows
that are no multiple of a thread's points, atom counts around a staged block,
atoms exactly on grid points, numerators that are not finite.

Tolerance: FP64 sums of the same terms in the same order; each term's
inverse distance is good to about 2 ulp and enters to the 12th power, so
1e-13 of the largest value of its channel is far above what rounding gives.
Occupancy is a set of decisions: equal."""
import numpy as np
import pytest

import oracle
from workload import synth

pytestmark = pytest.mark.gpu


def _case(n_rec, n_atoms, mode):
    w = synth.tiny(seed=n_rec + n_atoms, n_rec=n_rec, n_fft=n_rec, h=0.5, n_rec_atoms=n_atoms, clash_mode=mode)
    # one atom on a grid point, one on a face
    w.receptor.xyz[0, 0] = np.asarray(w.origin) + 0.5 * np.array([1, n_rec // 2, n_rec - 1])
    if n_atoms > 1:
        w.receptor.xyz[0, 1] = np.asarray(w.origin)
    return w


@pytest.mark.parametrize("mode", ["occ", "cap"])
@pytest.mark.parametrize("n_rec,n_atoms", [(5, 1), (9, 127), (18, 128), (31, 129), (44, 300)])
def test_grids(n_rec, n_atoms, mode):
    import paper_1708_07045_amd as fd
    w = _case(n_rec, n_atoms, mode)
    r = w.receptor
    want, occ = oracle.receptor_grids(w)
    for precision, rel in (("f64", 1e-13), ("f32", 1e-7)):
        t = fd.GridTools(n_rec, w.h, w.origin, precision, mode, w.ljr_cap, w.occ_f)
        g, o = t.build(r.xyz[0], r.q, r.sigma, r.eps)
        g = g.double().cpu().numpy()
        for ch in range(3):
            assert np.all(np.abs(g[ch] - want[ch]) <= rel * np.abs(want[ch]).max())
        if mode == "occ":
            assert np.array_equal(o.cpu().numpy(), occ)


def test_numerator_that_is_not_finite():
    """Only the points an atom acts on see its charge."""
    import paper_1708_07045_amd as fd
    w = _case(24, 40, "occ")
    r = w.receptor
    q = r.q.copy()
    q[7] = np.inf
    t = fd.GridTools(24, w.h, w.origin, "f64", "occ", w.ljr_cap, w.occ_f)
    g, _ = t.build(r.xyz[0], q, r.sigma, r.eps)
    g = g.cpu().numpy()
    want, _ = oracle.receptor_grids(w)
    ax = [w.origin[d] + w.h * np.arange(24) for d in range(3)]
    d = np.sqrt((ax[0][None, None, :] - r.xyz[0, 7, 0]) ** 2 + (ax[1][None, :, None] - r.xyz[0, 7, 1]) ** 2
                + (ax[2][:, None, None] - r.xyz[0, 7, 2]) ** 2)
    inside = d < 2.0 ** (-1.0 / 6.0) * r.sigma[7]
    assert inside.any() and np.all(np.isfinite(g[0][inside])) and np.all(np.isinf(g[0][~inside]))
    assert np.all(np.abs(g[1] - want[1]) <= 1e-13 * np.abs(want[1]).max())
