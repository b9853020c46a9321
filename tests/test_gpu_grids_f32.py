"""FP32 receptor grids (Eqs. 7, 10) with atoms at no finite distance: at infinity, or so far off that a
squared distance overflows.  Such an atom adds nothing (its terms are a numerator over infinity), in both
tilings of the kernel (n_rec below and from 40): the grids equal, bit for bit, those without it."""
import numpy as np
import pytest

from workload import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["occ", "cap"])
@pytest.mark.parametrize("n_rec", [24, 44])
def test_atoms_at_no_finite_distance(n_rec, mode):
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
