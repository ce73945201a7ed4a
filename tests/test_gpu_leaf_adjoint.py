"""Adjoint with every bond at d_max, odd ones among them, on a graph whose sites have one, two and three legs:
the second 16-wide tile of its kernels, the clamped columns past an odd bond and the elimination of more than
16 rows.

The QR backward regularises with 1e-13 of the largest diagonal entry of R^H R: directions under its root,
3.2e-7 of the largest, are damped, and a gradient through some thirty gates in sequence agrees with the
oracle to 1e-5.  complex128 only: on these states a complex64 gradient is 5e-5 to 6e-4 off, in the forms of
the kernels before these as well, from the rounding of the stored tensors in such directions.
"""

import numpy as np
import pytest

import oracle.grad as G
from heavyhex import heavy_hex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [9, 15, 17, 23, 31])
def test_adjoint_at_saturated_bonds(d):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(3, 7, False)
    steps = 6
    got = []
    for mode in (1, 2):
        print(f"[gpu case] adjoint {mode}: 25 qubits with leaves D={d} c128, {steps} steps", flush=True)
        s = Simulator([g], [0], [0.5], [-1.2], d_max=d, precision="c128", trunc_rel=1e-12, max_steps=steps, adjoint=mode)
        s.step(steps)
        assert max(np.max(x) for x in s.bond_dims()) == d
        (dh,), (dj,) = s.backward([np.full(g.n_nodes, 1.0 / g.n_nodes)])
        s.close()
        got.append((float(dh), float(dj)))
    r = G.loss_and_grad_graph(g, 0.5, -1.2, d, steps, 1e-12)
    assert got[0] == got[1]
    assert abs(got[0][0] - r.dtheta_h) < 1e-5 and abs(got[0][1] - r.dtheta_j) < 1e-5
