"""Edges of the kernels' work splits on the GPU, against the CPU FP64 oracle:
block sizes around a tile, strip or group boundary, at the tolerances of the
parity tests (FP64 1e-10, FP32 1e-5, relative Frobenius and per row)."""
import numpy as np
import pytest

import synth
from oracle import exx
from tests.helpers import dev, host, max_row_rel, rel_fro, report

pytestmark = pytest.mark.gpu

TOL = {"c128": 1e-10, "c64": 1e-5}


def _dtype(prec):
    import torch
    return torch.complex128 if prec == "c128" else torch.complex64


# strips of the pair pass: 4 or 8 occupied orbitals (one over, one under, a
# remainder behind full strips)
@pytest.mark.parametrize("n,prec,nocc,ntgt", [
    ((48, 48, 48), "c64", 5, 3), ((96, 96, 96), "c64", 9, 2), ((96, 96, 96), "c64", 7, 1),
    ((96, 96, 96), "c128", 5, 2), ((96, 96, 128), "c128", 3, 2), ((96, 96, 128), "c64", 10, 1),
])
def test_pair_pass_strips(n, prec, nocc, ntgt):
    from paper_1305_7313_amd import fock as F
    s = synth.make_system(synth.ortho_cell(*(x / 4.0 for x in n)), n)
    occ, tgt = synth.random_orbitals(s.a, s.miller, nocc, 1), synth.random_orbitals(s.a, s.miller, ntgt, 2)
    f = np.linspace(0.5, 1.0, nocc)
    print(f"[case] strips {n} {prec} {nocc} x {ntgt}", flush=True)
    v = host(F.fock_apply(F.Cell(s.a, s.n, s.miller), (0.0, 0.0, 0.0), dev(occ, _dtype(prec)), dev(f),
                          dev(tgt, _dtype(prec))))
    ref = exx.fock_apply(s.a, s.n, s.miller, np.zeros(3), occ, f, tgt)
    e, er = rel_fro(v, ref), max_row_rel(v, ref)
    report(f"strips {n} {prec} {nocc}x{ntgt}", rel=e, maxband=er)
    assert e < TOL[prec] and er < TOL[prec]


def _sphere(n, kind):
    """A system on grid n whose plane-wave list is the full sphere in random
    order, a ragged part of it (not symmetric, columns missing), or G = 0 alone."""
    s = synth.make_system(synth.ortho_cell(*(x / 4.0 for x in n)), n)
    rng = np.random.default_rng(5)
    m = s.miller[rng.permutation(s.npw)]
    if kind == "ragged":
        m = m[(m[:, 1] > -3) & (m[:, 2] % 3 != 1)]
    elif kind == "one":
        m = np.zeros((1, 3), dtype=np.int32)
    s.miller = np.ascontiguousarray(m)
    return s


SPHERES = [((24, 24, 24), "full"), ((48, 48, 64), "full"), ((64, 64, 64), "ragged"), ((72, 72, 72), "full"),
           ((96, 96, 96), "ragged"), ((128, 96, 128), "full"), ((72, 48, 48), "ragged"), ((24, 72, 72), "one")]


# sphere passes and the band loops' one-dimensional passes on every line length,
# with plane waves in any order
@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n,kind", SPHERES)
def test_sphere_passes(n, kind, prec):
    import torch
    from oracle import bands
    from paper_1305_7313_amd import fock as F
    s = _sphere(n, kind)
    rng = np.random.default_rng(6)
    nb = 3
    c = rng.standard_normal((nb, s.npw)) + 1j * rng.standard_normal((nb, s.npw))
    c /= np.linalg.norm(c, axis=1)[:, None]
    w = np.array([2.0, 0.5, 1.25])
    v, k = rng.standard_normal(n), np.array([0.07, -0.02, 0.05])
    cell = F.Cell(s.a, s.n, s.miller)
    cd, wd = dev(c, _dtype(prec)), dev(w)
    print(f"[case] sphere {n} {kind} {prec}: {s.npw} plane waves", flush=True)
    rho = host(F.fock_band_density(cell, cd, wd))
    e1 = rel_fro(rho, bands.band_density(s.a, s.n, s.miller, c, w))
    vd = dev(v, torch.float64 if prec == "c128" else torch.float32)
    e2 = rel_fro(host(F.fock_band_force(cell, k, cd, wd, vd)), bands.band_force(s.a, s.n, s.miller, k, c, w, v))
    q = np.array([0.03, 0.01, -0.02])
    ref = exx.fock_apply(s.a, s.n, s.miller, q, c[:2], w[:2], c[2:])
    e3 = rel_fro(host(F.fock_apply(cell, q, cd[:2], wd[:2], cd[2:])), ref)
    report(f"sphere {n} {kind} {prec}", density=e1, force=e2, apply=e3)
    assert max(e1, e2, e3) < TOL[prec]


# bands around the chunk and group boundaries of the band loops
@pytest.mark.parametrize("prec,nb", [("c128", 1), ("c128", 65), ("c64", 9), ("c64", 70)])
def test_band_chunks(prec, nb):
    import torch
    from oracle import bands
    from paper_1305_7313_amd import fock as F
    s = synth.make_system(synth.cubic_cell(12.0), (48, 48, 48))
    c = synth.random_orbitals(s.a, s.miller, nb, 3)
    w = np.linspace(0.5, 2.0, nb)
    v = np.random.default_rng(7).standard_normal(s.n)
    cell = F.Cell(s.a, s.n, s.miller)
    cd, wd = dev(c, _dtype(prec)), dev(w)
    print(f"[case] band chunks {prec} {nb}", flush=True)
    e1 = rel_fro(host(F.fock_band_density(cell, cd, wd)), bands.band_density(s.a, s.n, s.miller, c, w))
    vd = dev(v, torch.float64 if prec == "c128" else torch.float32)
    k = np.zeros(3)
    e2 = rel_fro(host(F.fock_band_force(cell, k, cd, wd, vd)), bands.band_force(s.a, s.n, s.miller, k, c, w, v))
    report(f"band chunks {prec} {nb}", density=e1, force=e2)
    assert max(e1, e2) < TOL[prec]


# few targets: the occupied loop of the fused pass in parts, and tiles wider
# than the square edge (one target; parts with a remainder; several tiles; the
# part count at its limit; the streaming schedule of the 96 x 128 FP64 plane)
@pytest.mark.parametrize("n,prec,nocc,ntgt", [
    ((24, 24, 24), "c64", 35, 1), ((24, 24, 24), "c128", 70, 3), ((24, 24, 24), "c128", 4, 17),
    ((48, 48, 48), "c128", 40, 5), ((48, 48, 64), "c64", 70, 17), ((48, 48, 48), "c128", 290, 1),
    ((96, 96, 128), "c128", 9, 2),
])
def test_few_targets(n, prec, nocc, ntgt):
    from paper_1305_7313_amd import fock as F
    s = synth.make_system(synth.ortho_cell(*(x / 2.5 for x in n)), n)
    rng = np.random.default_rng(8)
    occ = rng.standard_normal((nocc, s.npw)) + 1j * rng.standard_normal((nocc, s.npw))
    tgt = rng.standard_normal((ntgt, s.npw)) + 1j * rng.standard_normal((ntgt, s.npw))
    f, g = np.linspace(0.2, 1.0, nocc), np.linspace(1.0, 0.5, ntgt)
    q = np.array([0.04, -0.01, 0.02])
    cell = F.Cell(s.a, s.n, s.miller)
    od, td, fd, gd = dev(occ, _dtype(prec)), dev(tgt, _dtype(prec)), dev(f), dev(g)
    print(f"[case] few targets {n} {prec} {nocc} x {ntgt}", flush=True)
    v = host(F.fock_apply(cell, q, od, fd, td))
    # the oracle on a sample of the targets
    js = sorted({0, ntgt // 2, ntgt - 1})
    ref = exx.fock_apply(s.a, s.n, s.miller, q, occ, f, tgt[js])
    e, er = rel_fro(v[js], ref), max_row_rel(v[js], ref)
    # E = 1/2 sum_j g_j Re <psi_j | V_x psi_j>, all targets, from a second path
    ex = float(host(F.fock_energy(cell, q, od, fd, td, gd)))
    e_v = 0.5 * float(np.sum(g * np.sum(np.conj(tgt) * v.astype(np.complex128), axis=1).real))
    report(f"few targets {n} {prec} {nocc}x{ntgt}", rel=e, maxband=er, energy=abs(ex - e_v) / abs(ex))
    assert e < TOL[prec] and er < TOL[prec] and abs(ex - e_v) < TOL[prec] * abs(ex)


# a workspace full of NaN: no pass reads a line that this call has not written
# (dead columns cleared once for several tiles; sphere lines; first tiles that
# overwrite their accumulators)
@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n,nb", [((24, 24, 24), 70), ((48, 48, 48), 35), ((64, 64, 64), 34), ((72, 72, 72), 18)])
def test_stale_workspace(n, nb, prec):
    import torch
    from paper_1305_7313_amd import fock as F
    s = synth.make_system(synth.ortho_cell(*(x / 3.0 for x in n)), n)
    c = synth.random_orbitals(s.a, s.miller, nb, 9)
    f = np.linspace(0.3, 1.0, nb)
    cell = F.Cell(s.a, s.n, s.miller)
    cd, fd = dev(c, _dtype(prec)), dev(f)
    q0, q1 = np.zeros(3), np.array([0.03, -0.02, 0.05])
    code = F.dtype_code(cd)

    def nan(nbytes):
        return torch.full((nbytes // 8,), float("nan"), dtype=torch.float64, device="cuda").view(torch.uint8)

    print(f"[case] stale workspace {n} {prec} {nb}", flush=True)
    js = [0, nb // 2, nb - 1]
    size = F.fock_workspace_size(cell, code, nb, nb)
    own = host(F.fock_apply(cell, q0, cd, fd, cd, ws=nan(size)))[js]
    e1 = rel_fro(own, exx.fock_apply(s.a, s.n, s.miller, q0, c, f, c[js]))
    k = nb // 2
    other = host(F.fock_apply(cell, q1, cd, fd, cd[:k].clone(), ws=nan(size)))[[0, k - 1]]
    e2 = rel_fro(other, exx.fock_apply(s.a, s.n, s.miller, q1, c, f, c[[0, k - 1]]))
    ex = float(host(F.fock_energy(cell, q0, cd, fd, cd, fd, ws=nan(size))))
    vx = host(F.fock_apply(cell, q0, cd, fd, cd, ws=nan(size)))
    e3 = abs(ex - 0.5 * float(np.sum(f * np.sum(np.conj(c) * vx, axis=1).real))) / abs(ex)
    g = synth.gamma_orbitals(s.a, s.miller, 19, 4)
    gd, hd = dev(g, _dtype(prec)), dev(f[:19] if nb >= 19 else np.ones(19))
    lib = F.lib()
    import ctypes
    gsize = int(lib.fock_workspace_size_gamma(ctypes.byref(cell.c), code, 19))
    gv = host(F.fock_apply_gamma(cell, gd, hd, ws=nan(gsize)))[[0, 18]]
    e4 = rel_fro(gv, exx.fock_apply(s.a, s.n, s.miller, q0, g, host(hd), g[[0, 18]]))
    bsize = int(lib.fock_band_workspace_size(ctypes.byref(cell.c), code, nb))
    rho = host(F.fock_band_density(cell, cd, fd, ws=nan(bsize)))
    e5 = abs(rho.sum() * s.volume / np.prod(n) - f.sum()) / f.sum()
    report(f"stale {n} {prec} {nb}", self=e1, other=e2, energy=e3, gamma=e4, charge=e5)
    assert max(e1, e2, e3, e4, e5) < TOL[prec]
