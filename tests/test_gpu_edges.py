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
