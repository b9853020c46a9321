"""What the host runtime allocates and launches, without a GPU: libfftdg.so over a stand-in of the HIP calls
(hip_host.cpp), which notes the kernels' names and gives device memory of a set size.  Each test is a
process of its own, so nothing else sees the stand-in."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

DRIVER = '''
import ctypes, re, sys
import numpy as np
host = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
host.host_capacity.argtypes = [ctypes.c_size_t]
host.host_in_use.restype = ctypes.c_size_t
host.host_launches.restype = ctypes.c_char_p
import paper_1708_07045_amd as fd
from paper_1708_07045_amd import _lib as lib
from workload import synth
L = fd.load()
NO_LIMIT = 2 ** 64 - 1
OUT = ctypes.c_void_p(4096)  # never read: kernels do nothing


def create(n_fft, n_rec, precision="f32", mode="occ", h=0.5):
    g = lib.GridDesc(n_rec, n_fft, h, (ctypes.c_double * 3)(0, 0, 0), lib.F64 if precision == "f64" else lib.F32,
                     lib.OCC if mode == "occ" else lib.CAP, 10.0, 0.5)
    c = ctypes.c_void_p()
    assert L.fftdg_create(ctypes.byref(c), ctypes.byref(g), 0, None) == lib.OK
    return c


def receptors(c, n):
    return L.fftdg_set_receptors(c, n, OUT, OUT, None)


def ligand(n_cfg, n_at=6):
    rs = synth.streams(5)
    return synth.make_ligand(rs[1], rs[2], n_at, 1, n_cfg)


def kernels():
    """(name, integer and bool template arguments) of the launches since the last call"""
    t = host.host_launches().decode().split()
    host.host_clear()
    parts = [re.match(r"_ZN5fftdg(\\d+)(.*)", n) for n in t]
    return [(m[2][:int(m[1])], re.findall(r"L[ib](\\d+)E", m[2])) for m in parts]


def scan(c, b):
    """(status, kernels launched)"""
    kernels()
    return L.fftdg_scan(c, ctypes.byref(b.c), 300.0, OUT), kernels()

'''


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("hip") / "hip_host.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-o", so, os.path.join(HERE, "hip_host.cpp"), "-ldl"])
    return so


def drive(stand_in, body):
    r = subprocess.run([sys.executable, "-c", DRIVER + body, stand_in], cwd=os.path.dirname(HERE), capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


@pytest.mark.parametrize("precision,n_fft,n_rec", [("f32", 32, 30), ("f64", 32, 30), ("f32", 64, 48), ("f32", 128, 96)])
def test_only_live_planes_are_transformed(stand_in, precision, n_fft, n_rec):
    """A scan in occupancy mode runs the form of the z pass that skips z-translations without a clash-free one
    (last template argument), however few configurations it has; an export runs the other form."""
    drive(stand_in, f'''
c = create({n_fft}, {n_rec}, "{precision}")
assert receptors(c, 2) == lib.OK
shape = np.zeros(3, np.int32)
for fused in (1, 2):
    t = lib.Tuning(256, 0, 1, 0, fused, 1)
    assert L.fftdg_set_tuning(c, ctypes.byref(t)) == lib.OK
    for n in (1, 700):
        b = fd.Batch([ligand(n)])
        rc, ks = scan(c, b)
        z = [a for k, a in ks if k in ("k_zplanes", "k_zfused")]
        assert rc == lib.OK and z and all(a[-1] == "1" for a in z), (n, z)
    assert L.fftdg_energy_grid(c, 0, ctypes.byref(b.c), 0, 300.0, OUT, OUT, shape.ctypes.data) == lib.OK
    z = [a for k, a in kernels() if k in ("k_zplanes", "k_zfused")]
    assert z and all(a[-1] == "0" for a in z), z
''')


@pytest.mark.parametrize("precision,n_fft,n_rec", [("f32", 32, 30), ("f64", 32, 30), ("f32", 64, 48), ("f64", 64, 48),
                                                   ("f32", 128, 96)])
def test_way_of_the_energies_goes_by_the_grid(stand_in, precision, n_fft, n_rec):
    """Which kernels form the energies does not depend on how many configurations a scan has."""
    drive(stand_in, f'''
c = create({n_fft}, {n_rec}, "{precision}")
for snaps in (1, 3):
    assert receptors(c, snaps) == lib.OK
    used = []
    for n in (1, 700):
        rc, ks = scan(c, fd.Batch([ligand(n)]))
        assert rc == lib.OK
        used.append({{k for k, _ in ks}})
    assert used[0] == used[1], used[0] ^ used[1]
    assert ("k_direct" in used[0]) == ({n_fft} >= 64)
''')


@pytest.mark.parametrize("mode,n_fft,n_rec", [("occ", 32, 30), ("occ", 64, 48), ("cap", 64, 48), ("occ", 256, 200)])
def test_receptors_that_do_not_fit_leave_none(stand_in, mode, n_fft, n_rec):
    """Whichever allocation of set_receptors fails, the context then has no receptors: nothing is launched over the
    buffers that the call gave up, and the next set is taken as the first was."""
    drive(stand_in, f'''
b = fd.Batch([ligand(3)])
c = create({n_fft}, {n_rec}, mode="{mode}")
failed = set()
for part in np.linspace(0, 1, 60):
    host.host_capacity(NO_LIMIT)
    assert receptors(c, 2) == lib.OK
    assert scan(c, b)[0] == lib.OK
    base = host.host_in_use()
    if not failed:
        assert receptors(c, 40) == lib.OK
        full = host.host_in_use()
        L.fftdg_destroy(c)
        c = create({n_fft}, {n_rec}, mode="{mode}")
        assert receptors(c, 2) == lib.OK and scan(c, b)[0] == lib.OK
    host.host_capacity(int(base + part * (full - base) * 0.98))
    rc = receptors(c, 40)
    failed.add(rc)
    host.host_capacity(NO_LIMIT)
    if rc != lib.OK:
        assert rc == lib.E_NOMEM
        assert scan(c, b) == (lib.E_STATE, [])
        res, B = np.zeros(1, lib.RESULT_DTYPE), np.zeros((1, 2))
        assert L.fftdg_reduce(c, ctypes.byref(b.c), OUT, None, 300.0, B.ctypes.data, res.ctypes.data) == lib.OK
        shape = np.zeros(3, np.int32)
        assert L.fftdg_energy_grid(c, 0, ctypes.byref(b.c), 0, 300.0, OUT, OUT, shape.ctypes.data) == lib.E_STATE
    L.fftdg_destroy(c)
    c = create({n_fft}, {n_rec}, mode="{mode}")
assert lib.E_NOMEM in failed
''')


@pytest.mark.parametrize("n_fft,n_rec,snaps", [(64, 48, 6), (128, 96, 3)])
def test_scan_on_a_full_device_goes_on_with_less(stand_in, n_fft, n_rec, snaps):
    """As the memory shrinks a scan gives up the launches over several snapshots, then the copy of the grids (and
    takes the transforms, over live planes), and only then says that it does not fit: at what it needed without
    either.  Draws from it fit where it does."""
    drive(stand_in, f'''
b = fd.Batch([ligand(40)])
grids = {snaps} * 3 * {n_rec} ** 3 * 4


def attempt(capacity):
    """(statuses of set_receptors, scan and an export, kernels of the scan, bytes in use)"""
    host.host_capacity(NO_LIMIT)
    c = create({n_fft}, {n_rec})
    base = host.host_in_use()
    host.host_capacity(capacity + base if capacity < NO_LIMIT else capacity)
    rc = [receptors(c, {snaps})]
    s, ks = scan(c, b)
    shape = np.zeros(3, np.int32)
    rc += [s, L.fftdg_energy_grid(c, 0, ctypes.byref(b.c), 0, 300.0, OUT, OUT, shape.ctypes.data)]
    used = host.host_in_use() - base
    L.fftdg_destroy(c)
    return rc, [k for k, _ in ks], [a for k, a in ks if k in ("k_zplanes", "k_zfused")], used


rc, ks, _, full = attempt(NO_LIMIT)
assert rc == [lib.OK] * 3 and ks.count("k_direct") == 1
seen, least = set(), full
for capacity in np.linspace(full, 0.3 * full, 400).astype(int).tolist():
    rc, ks, z, used = attempt(capacity)
    assert used <= capacity
    if rc != [lib.OK] * 3:
        assert set(rc) <= {{lib.OK, lib.E_NOMEM, lib.E_STATE}}
        break
    least = capacity
    assert ks.count("k_direct") in (0, 1, {snaps}) and all(a[-1] == "1" for a in z)
    seen.add(ks.count("k_direct"))
assert seen == {{0, 1, {snaps}}}, seen
assert least < full - 1.1 * grids
''')


def test_counters_beyond_two_to_the_31(stand_in):
    """One configuration in 600 000 scanned against 2000 snapshots: the clash test's counters number 2.4e9."""
    drive(stand_in, '''
n = 600_000
sel = np.zeros(n, np.uint8)
sel[7] = 1
b = fd.Batch([ligand(n, 1)]).with_select(sel)
c = create(32, 20)
assert receptors(c, 2000) == lib.OK
rc, ks = scan(c, b)
assert rc == lib.OK, L.fftdg_last_error(c)
assert [k for k, _ in ks].count("k_zero32") == 3
''')
