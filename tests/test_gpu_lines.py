"""General grids (line path): every axis length in every position.

For each {2,3,5}-smooth length the grids (L, 5, 9), (6, L, 10) and (4, 3, L)
run through fock_apply, fock_apply_energy, fock_energy, fock_energy_backward
and dft3 against the FP64 oracle: the axis-1 transforms of one lane and of
lane pairs, every radix pair of the plane passes, tiles of several planes with
a remainder, lines that do not fill a wave.  A pair buffer of 1 MB forces
blocks of orbitals with a ragged last one on the larger grids; an explicit
k-pair list runs the ordered schedule.  Tolerances are those of the parity
tests (1e-12 FP64; 1e-5, energies 1e-6, FP32)."""
import ctypes
import sys

import numpy as np
import pytest

from oracle.fock_oracle import Oracle
from paper_1111_0716_amd import fock, inputs

LENGTHS = [2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64, 72]
TOL = {"c128": dict(e=1e-12, v=1e-12), "c64": dict(e=1e-6, v=1e-5)}


def _band_err(got, ref):
    got = got.reshape(ref.shape)
    return max(np.linalg.norm(got[k, n] - ref[k, n]) / np.linalg.norm(ref[k, n])
               for k in range(ref.shape[0]) for n in range(ref.shape[1]))


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("L", LENGTHS)
def test_every_axis_length_matches_oracle(L, prec, device):
    import torch

    dt = np.complex64 if prec == "c64" else np.complex128
    tol = TOL[prec]
    for j, grid in enumerate([(L, 5, 9), (6, L, 10), (4, 3, L)]):
        print(f"lines {grid} {prec}", file=sys.stderr, flush=True)
        inst = inputs.small_instance(grid=grid, kmesh=(2, 1, 1), nbands=4, seed=(960, L, j), full_grid=True)
        inst.occ[1, 3] = 0.25
        kpairs = [[[0, 0], [0, 1], [1, 0]]] if L % 3 == 0 and j == 1 else None
        n = inst.npoints
        bs = n + 3
        plan = fock.Plan([inst], precision=prec, device=device, band_stride=[bs], tuning={"tbuf_mb": 1},
                         kpairs=[np.array(kpairs[0], dtype=np.int32)] if kpairs else None)
        u = inst.psi.astype(dt)
        psi = torch.zeros((inst.nk, inst.nbands, bs), dtype=plan.cdtype, device=device)
        psi[:, :, :n] = torch.from_numpy(np.ascontiguousarray(u)).to(device)
        occ = torch.from_numpy(np.ascontiguousarray(inst.occ)).to(device)
        out = torch.full_like(psi, 7.0)
        plan.fock_apply([psi], [occ], out=[out])
        (v2,), _, ex2 = plan.fock_apply_energy([psi], [occ])
        ex = plan.fock_energy([psi], [occ])
        gex = torch.full((1,), 0.75, dtype=torch.float64, device=device)
        o = Oracle.from_instance(inst, kpairs=[tuple(x) for x in kpairs[0]] if kpairs else None)
        (g,) = plan.fock_energy_backward([psi], [occ], gex, 2.0 * o.dv)
        torch.cuda.synchronize()
        assert torch.equal(out[:, :, :n], v2[:, :, :n])
        assert torch.all(out[:, :, n:] == 7.0)  # the padding is never written
        vref, eref = o.apply(u.astype(np.complex128), inst.occ)
        gref = 0.75 * o.gradient(u.astype(np.complex128), inst.occ, vref)
        assert _band_err(out[:, :, :n].cpu().numpy(), vref) <= tol["v"]
        assert _band_err(g[:, :, :n].cpu().numpy(), gref) <= tol["v"]
        for e in (ex, ex2):
            assert abs(float(e.item()) - eref) <= tol["e"] * abs(eref)
        rng = np.random.default_rng([960, L, j])
        x = (rng.standard_normal((3, n)) + 1j * rng.standard_normal((3, n))).astype(dt)
        for sign in (-1, 1):
            d = torch.from_numpy(x).to(device)
            plan.dft3(d, sign)
            x3 = x.astype(np.complex128).reshape((3,) + grid)
            ref = np.fft.fftn(x3, axes=(1, 2, 3)) if sign < 0 else np.fft.ifftn(x3, axes=(1, 2, 3)) * n
            err = np.linalg.norm(d.cpu().numpy().reshape(ref.shape) - ref) / np.linalg.norm(ref)
            assert err <= (1e-5 if prec == "c64" else 1e-12), (sign, err)
        plan.close()


def _fft_pairs(grid, kmesh, nb, kpairs=None, tuning=None):
    keep = []
    d = fock.make_desc(inputs.cubic_lattice(10.0), grid, inputs.gamma_mesh(*kmesh), None, nb, None, 0.106, kpairs, keep)
    h, fft = ctypes.c_void_p(), ctypes.c_int64()
    tn = fock.FockTuning(**tuning) if tuning else None
    assert fock.lib().fock_plan_tuned((fock.FockDesc * 1)(d), 1, fock.FOCK_C64, None, ctypes.byref(tn) if tn else None,
                                      ctypes.byref(h)) == fock.FOCK_OK
    fock.lib().fock_plan_stats(h, None, ctypes.byref(fft), None, None)
    fock.lib().fock_destroy(h)
    return fft.value


def _plan_stats(grid, nb, prec):
    keep = []
    d = fock.make_desc(inputs.cubic_lattice(10.0), grid, inputs.gamma_mesh(1, 1, 1), None, nb, None, 0.106, None, keep)
    h, fft, size = ctypes.c_void_p(), ctypes.c_int64(), ctypes.c_size_t()
    assert fock.lib().fock_plan((fock.FockDesc * 1)(d), 1, prec, None, ctypes.byref(h)) == fock.FOCK_OK
    fock.lib().fock_plan_stats(h, None, ctypes.byref(fft), None, None)
    fock.lib().fock_workspace_size(h, ctypes.byref(size))
    fock.lib().fock_destroy(h)
    return fft.value, size.value


@pytest.mark.parametrize("L,prec,nb", [(16, fock.FOCK_C128, 9), (16, fock.FOCK_C128, 40), (16, fock.FOCK_C128, 56)])
def test_small_cubes_stay_within_the_static_workspace(L, prec, nb):
    """The whole-pair kernel (one transform per ordered pair, no pair buffer)
    fits all of these; where the three-pass path would not, it is kept."""
    fft, size = _plan_stats((L, L, L), nb, prec)
    assert size <= fock.STATIC_WORKSPACE_BYTES
    pair_bytes = L ** 3 * (8 if prec == fock.FOCK_C64 else 16)
    if nb * (nb + 1) // 2 * pair_bytes < fock.STATIC_WORKSPACE_BYTES // 2:
        assert fft == nb * (nb + 1) // 2


def test_general_grids_transform_unordered_pairs():
    assert _fft_pairs((24, 30, 45), (2, 1, 1), 5) == 55
    assert _fft_pairs((24, 30, 45), (2, 1, 1), 5, tuning={"tbuf_mb": 1}) == 55  # blocks
    assert _fft_pairs((24, 30, 45), (2, 1, 1), 5, tuning={"no_pair_symmetry": 1}) == 100
    assert _fft_pairs((24, 30, 45), (2, 1, 1), 5, kpairs=[[0, 0], [0, 1], [1, 1]]) == 75  # not closed under swapping
