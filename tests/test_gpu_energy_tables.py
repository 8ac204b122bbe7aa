"""Energies whose passes read their own kernel table, in plans with and without
room for it in the static workspace: fock_energy, and E_x after an apply,
against the oracle (1e-6 FP32, 1e-12 FP64, as the parity tests)."""
import sys

import numpy as np
import pytest

from oracle.fock_oracle import Oracle
from paper_1111_0716_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,grid,kmesh,nb,own", [
    # FP32 general grid: the grid-order table takes 559872 bytes
    ("c64", (12, 16, 27), (2, 2, 2), 7, False), ("c64", (12, 16, 27), (2, 2, 2), 6, True),
    # FP64 16^3 on the three-pass path: the whole-pair kernel's table
    ("c128", (16, 16, 16), (1, 1, 1), 9, True), ("c128", (16, 16, 16), (2, 1, 1), 20, True)])
def test_energy_tables(prec, grid, kmesh, nb, own, device):
    import torch

    from paper_1111_0716_amd import fock

    print(f"energy table {prec} {grid} {kmesh} {nb}", file=sys.stderr, flush=True)
    inst = inputs.small_instance(grid=grid, kmesh=kmesh, nbands=nb, seed=(990, nb), full_grid=True)
    plan = fock.Plan([inst], precision=prec, device=device)
    size = plan.workspace_bytes
    assert size <= fock.STATIC_WORKSPACE_BYTES
    if prec == "c64":  # (2, 2, 2): 27 distinct transfers
        assert (size + 27 * inst.npoints * 4 > fock.STATIC_WORKSPACE_BYTES) == (not own)
    u = inst.psi.astype(np.complex64 if prec == "c64" else np.complex128)
    psi, occ = torch.from_numpy(np.ascontiguousarray(u)).to(device), torch.from_numpy(inst.occ).to(device)
    _, _, ex2 = plan.fock_apply_energy([psi], [occ])
    ex = plan.fock_energy([psi], [occ])
    plan.profile(True)
    plan.fock_energy([psi], [occ])
    kinds = {k for k, v in plan.profile_read().items() if v[1]}
    plan.close()
    assert ("energy_fused" in kinds) == (prec == "c128")
    _, eref = Oracle.from_instance(inst).apply(u.astype(np.complex128), inst.occ)
    for e in (ex, ex2):
        assert abs(float(e.item()) - eref) <= (1e-6 if prec == "c64" else 1e-12) * abs(eref)


@pytest.mark.parametrize("nb", [1, 6, 7, 23])
def test_energy_finished_by_its_last_workgroup(nb, device):
    """FP32 general grid, ordered pairs x 8 slabs on either side of the 288
    partials up to which the pencil pass sums them: E_x after an apply against the
    oracle, the same bits from call to call, and from a graph replayed between
    eager calls."""
    import torch

    from paper_1111_0716_amd import fock

    print(f"energy last workgroup {nb}", file=sys.stderr, flush=True)
    inst = inputs.small_instance(grid=(5, 8, 6), kmesh=(1, 1, 1), nbands=nb, seed=(991, nb), full_grid=True)
    assert (nb * nb * 8 <= 288) == (nb <= 6)
    u = inst.psi.astype(np.complex64)
    psi, occ = torch.from_numpy(np.ascontiguousarray(u)).to(device), torch.from_numpy(inst.occ).to(device)
    _, eref = Oracle.from_instance(inst).apply(u.astype(np.complex128), inst.occ)
    plan = fock.Plan([inst], precision="c64", device=device)
    eager = [float(plan.fock_apply_energy([psi], [occ])[2].item()) for _ in range(3)]
    assert abs(eager[0] - eref) <= 1e-6 * abs(eref)
    assert len(set(eager)) == 1
    plan.close()
    stream = torch.cuda.Stream(device=device)
    with torch.cuda.stream(stream):
        graph = fock.Plan([inst], precision="c64", device=device, stream=stream)
        graph.set_graph(True)
        out, ex = torch.empty_like(psi), torch.empty(1, dtype=torch.float64, device=device)
        for _ in range(4):
            ex.zero_()
            graph.fock_apply_energy([psi], [occ], out=[out], ex=ex)
            graph.fock_energy([psi], [occ])
            stream.synchronize()
            assert float(ex.item()) == eager[0]
        graph.close()


def _klist(nk, kind):
    if kind == "diagonal":
        return [[k, k] for k in range(nk)]
    if kind == "upper":
        return [[k, kp] for k in range(nk) for kp in range(k, nk)]
    return [[0, kp] for kp in range(nk)] + [[k, k] for k in range(1, nk - 1)]  # the last k has no partner


@pytest.mark.parametrize("kind", ["diagonal", "upper", "uneven"])
@pytest.mark.parametrize("grid,nb", [((5, 8, 6), 1), ((5, 8, 6), 3), ((12, 10, 9), 4)])
def test_energy_of_several_groups_in_one_launch(grid, nb, kind, device):
    """FP32 general grid, k-points with partner lists of their own: the ordered
    pairs of all of them go through one pass each, with and without the finishing
    workgroup; E_x against the oracle, eagerly and from a replayed graph."""
    import torch

    from paper_1111_0716_amd import fock

    print(f"energy groups {grid} {nb} {kind}", file=sys.stderr, flush=True)
    inst = inputs.small_instance(grid=grid, kmesh=(4, 1, 1), nbands=nb, seed=(992, nb), full_grid=True)
    kpairs = np.array(_klist(inst.nk, kind), dtype=np.int32)
    u = inst.psi.astype(np.complex64)
    psi, occ = torch.from_numpy(np.ascontiguousarray(u)).to(device), torch.from_numpy(inst.occ).to(device)
    vref, eref = Oracle.from_instance(inst, kpairs=kpairs).apply(u.astype(np.complex128), inst.occ)
    stream = torch.cuda.Stream(device=device)
    with torch.cuda.stream(stream):
        plan = fock.Plan([inst], precision="c64", device=device, stream=stream, kpairs=[kpairs])
        plan.profile(True)
        (v,), _, ex = plan.fock_apply_energy([psi], [occ])
        first = float(ex.item())
        launches = plan.profile_read()
        plan.profile(False)
        assert launches["energy_plane"][1] == launches["energy_pencil"][1] == 1
        assert abs(first - eref) <= 1e-6 * abs(eref)
        vh = v.cpu().numpy()
        assert np.linalg.norm(vh - vref) <= 1e-6 * np.linalg.norm(vref)
        plan.set_graph(True)
        for _ in range(3):
            ex.zero_()
            plan.fock_apply_energy([psi], [occ], out=[v], ex=ex)
            e2 = plan.fock_energy([psi], [occ])
            stream.synchronize()
            assert float(ex.item()) == first
            assert abs(float(e2.item()) - eref) <= 1e-6 * abs(eref)
        plan.close()


@pytest.mark.parametrize("cells,reduces", [
    # (grid, k-points, bands): batches of 32 to 288 partials and up to 19200 points,
    # one of more partials, one of more points
    ([((5, 8, 6), 1, 6), ((4, 3, 9), 2, 4), ((12, 10, 9), 2, 2), ((16, 3, 16), 1, 5)], 0),
    ([((5, 8, 6), 1, 2), ((16, 3, 16), 1, 6)], 2),
    ([((5, 8, 6), 1, 2), ((12, 10, 9), 2, 2), ((5, 8, 6), 1, 24)], 2),
    # the middle one on the whole-pair kernel
    ([((5, 8, 6), 1, 2), ((16, 16, 16), 1, 2), ((4, 3, 9), 2, 4)], 1)])
def test_energies_of_small_instances(cells, reduces, device):
    """FP32 instances whose energy batches sum themselves, alone and beside others:
    E_x of each against the oracle, the same bits from call to call, and no
    launches but those of the sums that are left."""
    import torch

    from paper_1111_0716_amd import fock

    print(f"energy small instances {cells}", file=sys.stderr, flush=True)
    insts = [inputs.small_instance(grid=g, kmesh=(nk, 1, 1), nbands=nb, seed=(993, i), full_grid=True)
             for i, (g, nk, nb) in enumerate(cells)]
    us = [i.psi.astype(np.complex64) for i in insts]
    psi = [torch.from_numpy(np.ascontiguousarray(u)).to(device) for u in us]
    occ = [torch.from_numpy(i.occ).to(device) for i in insts]
    plan = fock.Plan(insts, precision="c64", device=device)
    plan.profile(True)
    ex = [plan.fock_apply_energy(psi, occ)[2].cpu().numpy()]
    assert plan.profile_read()["energy_reduce"][1] == reduces
    plan.profile(False)
    ex += [plan.fock_apply_energy(psi, occ)[2].cpu().numpy() for _ in range(2)]
    plan.close()
    assert all(np.array_equal(e, ex[0]) for e in ex)
    for inst, u, e in zip(insts, us, ex[0]):
        _, eref = Oracle.from_instance(inst).apply(u.astype(np.complex128), inst.occ)
        assert abs(e - eref) <= 1e-6 * abs(eref)
