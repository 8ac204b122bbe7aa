"""fock_dft3 on either side of the sizes where FP32 batches change kernels:
20 MB and 256 MB of data, with the axis lengths that do so, in both
directions; every grid of the batch against numpy in FP64."""
import sys

import numpy as np
import pytest

from paper_1111_0716_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,counts", [((36, 36, 36), (56, 57, 719, 720)), ((40, 40, 40), (41,)), ((48, 48, 48), (24,)),
                                         ((48, 36, 36), (43,)), ((36, 24, 24), (130,)), ((16, 40, 40), (110,)),
                                         ((24, 48, 48), (48,))])
def test_dft3_around_the_cached_sizes(grid, counts, device):
    """Bound per grid: eps log2 N (16 to 17 butterfly levels, each within eps of the
    data in the root mean square) of FP32, 1e-6."""
    import torch

    from paper_1111_0716_amd import fock

    n = int(np.prod(grid))
    inst = dict(lattice=inputs.cubic_lattice(10.0), grid=grid, kfrac=np.zeros((1, 3)), nbands=1, mu=0.106)
    plan = fock.Plan([inst], precision="c64", device=device)
    rng = np.random.default_rng([980, n])
    for count in counts:
        some = min(count, 8)  # distinct grids, repeated through the batch
        x = (rng.standard_normal((some, n)) + 1j * rng.standard_normal((some, n))).astype(np.complex64)
        src = torch.from_numpy(x).to(device)
        for sign in (-1, 1):
            print(f"dft {grid} {count} {sign}", file=sys.stderr, flush=True)
            d = src.repeat((count + some - 1) // some, 1)[:count].contiguous()
            plan.dft3(d, sign)
            x3 = x.astype(np.complex128).reshape((some,) + grid)
            ref = np.fft.fftn(x3, axes=(1, 2, 3)) if sign < 0 else np.fft.ifftn(x3, axes=(1, 2, 3)) * n
            got = d[:some].cpu().numpy().reshape(ref.shape)
            for g, r in zip(got, ref):
                assert np.linalg.norm(g - r) <= 1e-6 * np.linalg.norm(r)
            for i in range(some, count):  # the rest of the batch, bit for bit
                assert torch.equal(d[i], d[i % some])
    plan.close()
