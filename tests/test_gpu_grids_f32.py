"""FP32 receptor grids (Eqs. 7, 10) at the edges of their kernel: atom counts around its staged blocks (512 atoms
for n_rec below 40, 256 from there on), both tilings, numerators that are not finite, and atoms at no finite
distance.

Tolerance: the sums are FP64, their terms good to a few ulp, and rounded once to FP32: half an ulp, 6e-8, of a
value; 1e-7 of the largest value of the channel holds both."""
import numpy as np
import pytest

import oracle
from workload import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["occ", "cap"])
@pytest.mark.parametrize("n_rec", [24, 44])
def test_atoms_at_no_finite_distance(n_rec, mode):
    """At infinity, or so far off that a squared distance overflows, an atom adds nothing (its terms are a numerator
    over infinity): the grids equal, bit for bit, those without it."""
    import paper_1708_07045_amd as fd
    w = synth.tiny(seed=n_rec, n_rec=n_rec, n_fft=64, h=0.5, n_rec_atoms=40, clash_mode=mode)
    r = w.receptor
    far = np.array([[np.inf, 0, 0], [0, -np.inf, 0], [1e155, 0, 0], [-3e200, 2e200, 1.0], [0, 0, 9e160]])
    more = lambda a, v: np.concatenate([a, np.full(len(far), v)])  # noqa: E731
    t = fd.GridTools(n_rec, w.h, w.origin, "f32", mode, w.ljr_cap, w.occ_f)
    want, occ = t.build(r.xyz[0], r.q, r.sigma, r.eps)
    g, o = t.build(np.concatenate([r.xyz[0], far]), more(r.q, 0.5), more(r.sigma, 3.0), more(r.eps, 0.1))
    assert np.all(np.isfinite(want.cpu().numpy()))
    assert np.array_equal(g.cpu().numpy(), want.cpu().numpy())
    if mode == "occ":
        assert np.array_equal(o.cpu().numpy(), occ.cpu().numpy())


@pytest.mark.parametrize("mode", ["occ", "cap"])
@pytest.mark.parametrize("n_rec,n_atoms", [(24, 511), (24, 512), (24, 513), (15, 1100), (39, 300), (40, 255), (41, 256),
                                           (44, 257), (42, 600)])
def test_staged_blocks(n_rec, n_atoms, mode):
    import paper_1708_07045_amd as fd
    w = synth.tiny(seed=n_rec + n_atoms, n_rec=n_rec, n_fft=64, h=0.5, n_rec_atoms=n_atoms, clash_mode=mode)
    r = w.receptor
    r.xyz[0, n_atoms - 1] = np.asarray(w.origin) + 0.5 * np.array([n_rec - 1, 2, 3])  # the last atom on a grid point
    want, occ = oracle.receptor_grids(w)
    t = fd.GridTools(n_rec, w.h, w.origin, "f32", mode, w.ljr_cap, w.occ_f)
    g, o = t.build(r.xyz[0], r.q, r.sigma, r.eps)
    g = g.double().cpu().numpy()
    for ch in range(3):
        assert np.all(np.abs(g[ch] - want[ch]) <= 1e-7 * np.abs(want[ch]).max())
    if mode == "occ":
        assert np.array_equal(o.cpu().numpy(), occ)


@pytest.mark.parametrize("what,value", [("q", np.inf), ("q", np.nan), ("eps", np.inf)])
@pytest.mark.parametrize("n_rec,mode", [(24, "occ"), (24, "cap"), (44, "occ"), (44, "cap")])
def test_numerators_that_are_not_finite(n_rec, mode, what, value):
    """Only the points an atom acts on see its parameters: the FP64 grids, which add plain quotients, rounded."""
    import paper_1708_07045_amd as fd
    w = synth.tiny(seed=n_rec, n_rec=n_rec, n_fft=64, h=0.5, n_rec_atoms=40, clash_mode=mode)
    r = w.receptor
    p = dict(q=r.q.copy(), sigma=r.sigma, eps=r.eps.copy())
    p[what][7] = value
    r.xyz[0, 7] = np.asarray(w.origin) + 0.25 * n_rec  # in the box, its excluded ball too
    both = [fd.GridTools(n_rec, w.h, w.origin, k, mode, w.ljr_cap, w.occ_f).build(r.xyz[0], **p)[0].double().cpu().numpy()
            for k in ("f64", "f32")]
    fine = np.isfinite(both[0])
    assert not fine.all() and fine[0 if what == "q" else 2].any()
    assert np.array_equal(np.isfinite(both[1]), fine)
    assert np.array_equal(both[0][~fine], both[1][~fine], equal_nan=True)
    for ch in range(3):
        v = both[0][ch][fine[ch]]
        assert np.all(np.abs(both[1][ch][fine[ch]] - v) <= 1e-7 * np.abs(v).max())
