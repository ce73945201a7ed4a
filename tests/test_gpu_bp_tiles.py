"""Belief propagation at the bond dimensions where its 16 x 16 tiles end: half a tile, one tile, one
more column, two tiles, the smallest bonds; saturated bonds, senders with one, two and three legs.

complex128 states against the BP oracle within 1e-10 (the parity of the complex128 path; the message
products are float64 in both).
"""

import math

import numpy as np
import pytest

import oracle.bp as bp
import oracle.su as su
from heavyhex import heavy_hex

pytestmark = pytest.mark.gpu
TJ = -math.pi / 2


@pytest.mark.parametrize("d", [1, 2, 5, 8, 9, 15, 16, 17, 20, 31, 32])
def test_bp_tile_edges(d):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(2, 9, False)
    steps = max(2, math.ceil(math.log2(d)) + 1)
    print(f"[gpu case] heavy_hex 2x9 D={d} c128 {steps} steps, BP 3 iterations", flush=True)
    s = Simulator([g], [0], [0.8], [TJ], d_max=d, precision="c128", trunc_rel=1e-12, max_steps=steps)
    s.step(steps)
    (z,), res = s.bp_expect_z(3)
    s.close()
    ref = bp.run(su.evolve_graph(g, 0.8, TJ, d, steps, 1e-12, keep_state=True).peps, 3)
    assert np.max(np.abs(z - ref.z)) < 1e-10
    assert abs(res - ref.residual) < 1e-10
