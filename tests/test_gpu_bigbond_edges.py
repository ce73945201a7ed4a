"""The two-site update above D = 32 where its blocks of columns change: one column over the 64 that the
exchange buffer holds, one block of rounds more or fewer, odd sizes, the full 128 columns; sites with
one, two and three legs, so that Theta' comes taller, wider and square.

Every <Z> of every step against the oracle: complex64 within 1e-5, its parity; complex128 within 1e-10 at
a cutoff of 1e-4 (one vector set is recovered through 1/sigma, good to 2^-52 sigma_0 / sigma).
"""

import math

import numpy as np
import pytest

import oracle.su as su
from heavyhex import heavy_hex

pytestmark = pytest.mark.gpu
TJ = -math.pi / 2


@pytest.mark.parametrize("d,precision,cutoff,tol", [(33, "c64", 1e-6, 1e-5), (33, "c128", 1e-4, 1e-10), (40, "c64", 1e-6, 1e-5),
                                                    (49, "c128", 1e-4, 1e-10), (63, "c64", 1e-6, 1e-5), (64, "c128", 1e-4, 1e-10)])
def test_bigbond_edges(d, precision, cutoff, tol):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(2, 5, False)
    print(f"[gpu case] heavy_hex 2x5 D={d} {precision}, cutoff {cutoff}, 8 steps", flush=True)
    s = Simulator([g], [0], [0.8], [TJ], d_max=d, precision=precision, trunc_rel=cutoff, max_steps=8)
    s.step(8)
    (h,) = s.z_history()
    s.close()
    assert np.max(np.abs(h - su.evolve_graph(g, 0.8, TJ, d, 8, cutoff).z)) < tol
