"""Pair-buffer accesses, plain and marked non-temporal: the same plan with a
buffer on either side of the line (within the 32 MB of L2, within the 256 MB
last-level cache, above it), one size per form of the passes.  The two runs
differ in the accesses and in the order of the sums over partners; tolerances
are those of the parity tests (1e-12 FP64 and mixed energies of equal spectra;
V_x 1e-12 FP64 sums, 1e-5 FP32 sums; E_x 1e-9 of FP32 spectra, whose roundings
do not change)."""
import sys

import numpy as np
import pytest

from paper_1111_0716_amd import inputs

pytestmark = pytest.mark.gpu

MIB = 1 << 20
CASES = [  # precision, grid, bands, default buffer in MiB (at least, below), small buffer (MiB)
    ("c128", (30, 30, 30), 24, 32, 256, 8), ("c64", (30, 30, 30), 30, 32, 256, 8),  # line path: plain, marked
    ("c128", (36, 36, 36), 27, 256, 512, 64),                                       # line path: marked, plain
    ("c64", (32, 32, 32), 46, 256, 512, 128), ("c64", (64, 64, 64), 16, 256, 512, 128),  # slab: marked, plain
    ("c64", (60, 40, 40), 27, 256, 512, 128), ("c64", (40, 72, 72), 18, 256, 512, 128),  # plane-wise
    ("mixed", (32, 32, 32), 28, 256, 512, 64), ("mixed", (40, 40, 40), 20, 256, 512, 64),
    ("mixed_inv", (32, 32, 32), 28, 256, 512, 64), ("mixed_inv", (40, 40, 40), 20, 256, 512, 64)]


@pytest.mark.parametrize("prec,grid,nb,least,below,small", CASES)
def test_plain_and_marked_accesses_agree(prec, grid, nb, least, below, small, device):
    import torch

    from paper_1111_0716_amd import fock

    print(f"pair stream {prec} {grid} {nb}", file=sys.stderr, flush=True)
    inst = dict(lattice=inputs.cubic_lattice(10.0), grid=grid, kfrac=np.zeros((1, 3)), nbands=nb, mu=0.106)
    n = int(np.prod(grid))
    point = {"c64": 8, "c128": 16}.get(prec, 24)
    pairs = nb * (nb + 1) // 2
    assert least * MIB < pairs * n * point < below * MIB
    gen = torch.Generator(device=device)
    gen.manual_seed(970 + nb)
    res = []
    for tuning in (None, {"tbuf_mb": small}):
        plan = fock.Plan([inst], precision=prec, device=device, tuning=tuning)
        if not res:
            psi = torch.randn((1, nb, n), dtype=plan.cdtype, device=device, generator=gen) / n ** 0.5
            occ = torch.rand((1, nb), dtype=torch.float64, device=device, generator=gen)
        (v,), _, ex = plan.fock_apply_energy([psi], [occ])
        e2 = plan.fock_energy([psi], [occ])
        (g,) = plan.fock_energy_backward([psi], [occ], torch.ones(1, dtype=torch.float64, device=device), 1.0)
        torch.cuda.synchronize()
        res.append((v, g, ex, e2))
        plan.close()
    sums32 = prec in ("c64", "mixed_inv")
    for a, b in zip(res[0][:2], res[1][:2]):
        d = torch.linalg.vector_norm(a - b, dim=2) / torch.linalg.vector_norm(b, dim=2)
        assert float(d.max()) <= (1e-5 if sums32 else 1e-12)
    es = [float(x.item()) for r in res for x in r[2:]]
    for a, b in ((es[0], es[2]), (es[1], es[3])):
        assert abs(a - b) <= (1e-9 if prec == "c64" else 1e-12) * abs(b)
