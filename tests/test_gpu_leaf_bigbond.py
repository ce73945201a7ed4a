"""The two-site update above D = 32 on a graph whose sites have one, two and three legs: Theta' comes square,
taller and wider, the complex64 absorb splits the rows of three-leg ends over workgroups (33 and 63
columns leave remainders in its tiles), and the largest case runs all 128 columns.

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


@pytest.mark.parametrize("d,precision,cutoff,tol,steps", [(33, "c64", 1e-6, 1e-5, 8), (40, "c64", 1e-6, 1e-5, 8), (63, "c64", 1e-6, 1e-5, 8),
                                                          (64, "c64", 1e-6, 1e-5, 8), (33, "c128", 1e-4, 1e-10, 8),
                                                          (49, "c128", 1e-4, 1e-10, 8), (64, "c128", 1e-4, 1e-10, 9)])
def test_bigbond_on_a_graph_with_leaves(d, precision, cutoff, tol, steps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(3, 7, False)
    assert set(g.degrees()) == {1, 2, 3}
    print(f"[gpu case] 25 qubits with leaves D={d} {precision}, cutoff {cutoff}, {steps} steps", flush=True)
    s = Simulator([g], [0], [0.8], [TJ], d_max=d, precision=precision, trunc_rel=cutoff, max_steps=steps)
    s.step(steps)
    (h,) = s.z_history()
    assert max(np.max(x) for x in s.bond_dims()) == d
    s.close()
    assert np.max(np.abs(h - su.evolve_graph(g, 0.8, TJ, d, steps, cutoff).z)) < tol
