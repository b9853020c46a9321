"""Scans whose chunk takes its snapshots in several groups, and whose listed configurations are more than the
blocks of a launch over a list: what a group leaves to the next (forward planes made, lists, both buffer sets)
and the loops over a second item of a block.  Each record equals, bit for bit, that of its snapshot alone in chunks
of two configurations, where there is one group and no block has a second item."""
import numpy as np
import pytest

from workload import synth

pytestmark = pytest.mark.gpu


# as many snapshots a group as keep a set of its buffers under half a GiB: three groups, two
@pytest.mark.parametrize("n_fft,n_rec,h,precision,n_cfg,snaps,groups", [(128, 110, 0.25, "f32", 700, 9, 3),
                                                                        (64, 64, 0.5, "f32", 1700, 16, 2),
                                                                        (64, 64, 0.5, "f64", 1700, 16, 2)])
def test_groups_of_snapshots_and_long_lists(n_fft, n_rec, h, precision, n_cfg, snaps, groups):
    import torch
    import paper_1708_07045_amd as fd
    w = synth.tiny(seed=8, n_rec=n_rec, n_fft=n_fft, h=h, n_rec_atoms=60, n_lig_atoms=2, n_cfg=1, n_snap=snaps,
                   precision=precision)
    # snapshots 2, 6 and the last: the receptor far outside, everything free, all configurations take the transforms
    for s in (2, 6, snaps - 1):
        w.receptor.xyz[s] += 60.0 + n_rec * h
    rs = synth.streams(21)
    w.ligands = [synth.make_ligand(rs[1], rs[2], na, 1, n_cfg // 2) for na in (9, 12)]
    r = w.receptor
    ctx = fd.FFTDG.from_workload(w)
    both = [ctx.receptor_grids(r.xyz[s], r.q, r.sigma, r.eps) for s in range(snaps)]
    grids, occ = torch.stack([b[0] for b in both]), torch.stack([b[1] for b in both])
    b = fd.Batch(w.ligands)
    sel = np.zeros(n_cfg, np.uint8)
    sel[::23] = 1
    pick = np.flatnonzero(sel)
    want = []
    one = fd.FFTDG.from_workload(w)
    one.set_tuning(configs_per_chunk=2)
    for s in range(snaps):
        one.set_receptors(grids[s:s + 1], occ[s:s + 1])
        want.append(one.partials_numpy(one.scan(b.with_select(sel), w.T), 1, n_cfg)[0][pick].tobytes())
    ctx.set_receptors(grids, occ)
    for fused in (1, 2):
        for graph in (0, 1):
            ctx.set_tuning(fused=fused, use_graph=graph, configs_per_chunk=n_cfg)
            for turn in range(3):
                got = ctx.partials_numpy(ctx.scan(b, w.T), snaps, n_cfg)
                if fused == 1:
                    assert [got[s][pick].tobytes() for s in range(snaps)] == want
                else:
                    first = got if graph == 0 and turn == 0 else first
                    assert got.tobytes() == first.tobytes()
    # the clash test and the choice are counted as one launch each a group
    ctx.set_tuning(fused=1, use_graph=0)
    ctx.profile(True)
    ctx.scan(b, w.T)
    assert ctx.profile_read()["clash"][1] == 2 * groups
