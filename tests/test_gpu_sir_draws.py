"""Translation draws against running sums over the exported grid itself:
fewer translations than one segment of the kernel, segments and threads'
shares with no clash-free translation, uniforms at both ends.

Sums of up to 3e5 positive FP64 terms in two orders differ by less than
1e-10 of the total, so a draw may differ only where its uniform lies that
close to a boundary of the running sums."""
import numpy as np
import pytest

import oracle
from workload import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rec,n_fft,atoms,mode,precision,r_ball", [
    (16, 32, 1, "occ", "f64", 0.5), (24, 32, 6, "occ", "f64", 1.5), (18, 32, 12, "cap", "f64", 4.0),
    (60, 64, 600, "occ", "f32", 9.0), (72, 128, 300, "occ", "f32", 7.0)])
def test_draws(n_rec, n_fft, atoms, mode, precision, r_ball):
    import paper_1708_07045_amd as fd
    w = synth.tiny(seed=n_rec, n_rec=n_rec, n_fft=n_fft, h=0.5, n_rec_atoms=atoms, n_lig_atoms=3, n_cfg=1,
                   clash_mode=mode, precision=precision, r_ball=r_ball)
    r = w.receptor
    ctx = fd.FFTDG.from_workload(w)
    g, o = ctx.receptor_grids(r.xyz[0], r.q, r.sigma, r.eps)
    ctx.set_receptors(g[None].contiguous(), o[None].contiguous() if o is not None else None, r.weights)
    b = fd.Batch(w.ligands)
    T = 30000.0  # weights over many translations
    part = ctx.scan(b, T)
    psi, clash = (x.cpu().numpy() for x in ctx.energy_grid(0, b, 0, T))
    f, ok = psi.astype(np.float64).ravel(), clash.ravel() == 0
    assert ok.any()
    K = 150
    u = synth.uniforms(n_rec, 2 * K)
    u[1], u[3] = 0.0, 1.0 - 2.0 ** -53
    cfg, t, e = ctx.sample_poses(b, part, 0, 0, T, u)
    kT = oracle.kT(T)
    cw = np.cumsum(np.where(ok, np.exp(-(f - f[ok].min()) / kT), 0.0))
    lin = (t[:, 2] * psi.shape[1] + t[:, 1]) * psi.shape[2] + t[:, 0]
    assert np.all(ok[lin]) and np.array_equal(e, f[lin])
    for k in range(K):
        x = u[2 * k + 1] * cw[-1]
        want = min(int(np.searchsorted(cw, x, side="right")), int(np.flatnonzero(ok)[-1]))
        assert lin[k] == want or np.min(np.abs(cw - x)) <= 1e-10 * cw[-1], (k, lin[k], want)


def test_one_configuration_of_a_batch():
    """The grid of one configuration does not depend on the others of its
    batch, and a batch with one that cannot be placed is refused whole."""
    import copy
    import paper_1708_07045_amd as fd
    w = synth.tiny(seed=5, n_rec=24, n_fft=32, h=0.5, n_rec_atoms=6, n_lig_atoms=4, n_cfg=5, r_ball=1.5)
    r = w.receptor
    ctx = fd.FFTDG.from_workload(w)
    g, o = ctx.receptor_grids(r.xyz[0], r.q, r.sigma, r.eps)
    ctx.set_receptors(g[None].contiguous(), o[None].contiguous(), r.weights)
    for c in (0, 3, 4):
        alone = copy.deepcopy(w.ligands)
        alone[0].cfg_conf, alone[0].cfg_quat = alone[0].cfg_conf[c:c + 1], alone[0].cfg_quat[c:c + 1]
        a = ctx.energy_grid(0, fd.Batch(w.ligands), c, w.T)
        b = ctx.energy_grid(0, fd.Batch(alone), 0, w.T)
        assert a[0].numel() > 0 and all(bool((x == y).all()) for x, y in zip(a, b))
    for k in range(3):
        ligands = copy.deepcopy(w.ligands)
        if k == 0:
            ligands[0].cfg_quat[2] = 0.0
        elif k == 1:
            ligands[0].cfg_quat[2] = 1e-170
        else:
            ligands[0].conformers[ligands[0].cfg_conf[2]][0] += 1e5
        with pytest.raises(fd.FFTDGError):
            ctx.energy_grid(0, fd.Batch(ligands), 0, w.T)
