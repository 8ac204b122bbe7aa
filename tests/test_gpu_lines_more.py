"""Line path where the small grids of the length sweep do not go: the one-lane
accumulate of long FP32 lines, ragged tiles of planes, large grids N1 x L x L in
FP64 and both schedules of them, against the FP64 oracle (tolerances of the
parity tests: 1e-12 FP64; V_x 1e-5, E_x 1e-6 FP32)."""
import sys

import numpy as np
import pytest

from oracle.fock_oracle import Oracle
from paper_1111_0716_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"c128": dict(e=1e-12, v=1e-12), "c64": dict(e=1e-6, v=1e-5)}


def _run(inst, prec, device, tuning=None):
    import torch

    from paper_1111_0716_amd import fock

    u = np.ascontiguousarray(inst.psi.astype(np.complex64 if prec == "c64" else np.complex128))
    plan = fock.Plan([inst], precision=prec, device=device, tuning=tuning)
    psi, occ = torch.from_numpy(u).to(device), torch.from_numpy(np.ascontiguousarray(inst.occ)).to(device)
    (v,), _, ex2 = plan.fock_apply_energy([psi], [occ])
    ex = plan.fock_energy([psi], [occ])
    (g,) = plan.fock_energy_backward([psi], [occ], torch.ones(1, dtype=torch.float64, device=device), 1.0)
    torch.cuda.synchronize()
    res = dict(u=u.astype(np.complex128), v=v.cpu().numpy(), g=g.cpu().numpy(), e=[float(ex.item()), float(ex2.item())],
               stats=plan.stats())
    plan.close()
    return res


def _band_err(got, ref):
    return max(np.linalg.norm(got[k, n].reshape(-1) - ref[k, n].reshape(-1)) / np.linalg.norm(ref[k, n])
               for k in range(ref.shape[0]) for n in range(ref.shape[1]) if np.any(ref[k, n]))


@pytest.mark.parametrize("tbuf", [None, 600])  # one triangular batch; blocks, with rows of both sides of a batch
@pytest.mark.parametrize("grid", [(72, 64, 72), (54, 64, 72)])
def test_one_lane_accumulate_of_long_fp32_lines(grid, tbuf, device):
    """More than 2048 waves of whole lines (72 line blocks x 30 rows): FP32 lines
    of 54 and 72 points stay in one lane.  Three outputs against the oracle."""
    nb = 30
    assert (grid[1] * grid[2] + 63) // 64 * nb > 2048
    print(f"one lane {grid} {tbuf}", file=sys.stderr, flush=True)
    inst = inputs.small_instance(grid=grid, kmesh=(1, 1, 1), nbands=nb, seed=(1000, grid[0]))
    r = _run(inst, "c64", device, {"tbuf_mb": tbuf} if tbuf else None)
    assert r["stats"]["apply_fft_pairs"] == nb * (nb + 1) // 2
    outputs = [(0, 0), (0, 14), (0, 29)]
    vref, _ = Oracle.from_instance(inst).apply(r["u"], inst.occ, outputs=outputs)
    for k, n in outputs:
        ref = vref[k, n].reshape(-1)
        assert np.linalg.norm(r["v"][k, n].reshape(-1) - ref) <= 1e-5 * np.linalg.norm(ref)


def _tile(grid, pairs, prec):
    """Planes of a tile of the plane passes."""
    n1, plane = grid[0], grid[1] * grid[2]
    g = max(1, min(n1, (1440 if prec == "c128" else 2880) // plane))
    while g > 1 and pairs * -(-n1 // g) < 1024:
        g = (g + 1) // 2
    return g


@pytest.mark.parametrize("prec,grid,kmesh,nb", [
    ("c128", (16, 16, 16), (1, 1, 1), 40),                                        # 5, 5, 5 and 1 planes
    ("c64", (25, 5, 9), (1, 1, 1), 25), ("c128", (25, 5, 9), (1, 1, 1), 25),      # 7, 7, 7 and 4
    ("c64", (32, 10, 12), (2, 1, 1), 24), ("c128", (20, 12, 20), (1, 1, 1), 46),  # 24 and 8; 6, 6, 6 and 2
    ("c64", (72, 4, 6), (1, 1, 1), 46), ("c128", (50, 8, 10), (1, 1, 1), 46)])    # one tile; 18, 18 and 14
def test_ragged_tiles_match_oracle(prec, grid, kmesh, nb, device):
    orb = nb * kmesh[0]
    g = _tile(grid, orb * (orb + 1) // 2, prec)
    print(f"ragged {prec} {grid} {nb}: {g} planes a tile", file=sys.stderr, flush=True)
    assert g > 1 and (grid[0] % g != 0 or g == grid[0])
    inst = inputs.small_instance(grid=grid, kmesh=kmesh, nbands=nb, seed=(1001, nb), full_grid=True)
    r = _run(inst, prec, device)
    assert r["stats"]["apply_fft_pairs"] == orb * (orb + 1) // 2
    vref, eref = Oracle.from_instance(inst).apply(r["u"], inst.occ)
    assert _band_err(r["v"], vref) <= TOL[prec]["v"]
    for e in r["e"]:
        assert abs(e - eref) <= TOL[prec]["e"] * abs(eref)


@pytest.mark.parametrize("grid", [(32, 32, 32), (24, 24, 24), (40, 40, 40), (64, 64, 64), (64, 40, 40), (36, 36, 36),
                                  (54, 50, 50)])
@pytest.mark.parametrize("tuning", [None, {"tbuf_mb": 6}, {"no_pair_symmetry": 1, "tbuf_mb": 24}])
def test_fp64_n1_l_l_grids_match_oracle(grid, tuning, device):
    """FP64 on grids that once had register-line kernels: unordered pairs, the
    same in blocks of one or two orbitals, ordered pairs in small batches."""
    print(f"fp64 {grid} {tuning}", file=sys.stderr, flush=True)
    inst = inputs.small_instance(grid=grid, kmesh=(2, 1, 1), nbands=2, seed=(1002, grid[0]))
    r = _run(inst, "c128", device, tuning)
    assert r["stats"]["apply_fft_pairs"] == (16 if tuning and "no_pair_symmetry" in tuning else 10)
    o = Oracle.from_instance(inst)
    vref, eref = o.apply(r["u"], inst.occ)
    assert _band_err(r["v"], vref) <= 1e-12
    for e in r["e"]:
        assert abs(e - eref) <= 1e-12 * abs(eref)
    gref = o.gradient(r["u"], inst.occ, vref) / (2.0 * o.dv)
    assert _band_err(r["g"], gref.reshape(r["g"].shape)) <= 1e-12
