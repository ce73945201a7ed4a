"""Adjoint at the bond dimensions where its small-matrix kernel changes size (16 | 17) and where its
16 x 16 tiles end, on vertices with one, two and three edges.

After four steps no bond exceeds 16, so nothing is cut from d_max = 16 on: the two sizes of the kernel
work on the same state.  complex128 against the gradient oracle within 1e-8, the bound of the other
complex128 gradients.
"""

import numpy as np
import pytest

import oracle.grad as G
from heavyhex import heavy_hex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 5, 16, 17, 32])
def test_adjoint_edges(d):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(2, 9, False)
    steps = 4
    print(f"[gpu case] adjoint heavy_hex 2x9 D={d} c128 {steps} steps", flush=True)
    s = Simulator([g], [0], [0.5], [-1.2], d_max=d, precision="c128", trunc_rel=1e-12, max_steps=steps, adjoint=True)
    s.step(steps)
    (dh,), (dj,) = s.backward([np.full(g.n_nodes, 1.0 / g.n_nodes)])
    s.close()
    r = G.loss_and_grad_graph(g, 0.5, -1.2, d, steps, 1e-12)
    assert np.isfinite([dh, dj]).all()
    assert abs(dh - r.dtheta_h) < 1e-8 and abs(dj - r.dtheta_j) < 1e-8
