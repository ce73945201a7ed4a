"""Belief propagation with senders of one, two and three legs at the bond dimensions where its 16 x 16 tiles
end, every bond saturated.

complex128 states against the BP oracle within 1e-10, the parity of the complex128 path.
"""

import math

import numpy as np
import pytest

import oracle.bp as bp
import oracle.su as su
from heavyhex import heavy_hex

pytestmark = pytest.mark.gpu
TJ = -math.pi / 2


@pytest.mark.parametrize("d", [1, 2, 5, 8, 9, 15, 16, 17, 23, 31, 32])
def test_bp_with_leaves(d):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(3, 7, False)
    assert set(g.degrees()) == {1, 2, 3}
    steps = max(2, math.ceil(math.log2(d)) + 1)
    print(f"[gpu case] 25 qubits with leaves D={d} c128 {steps} steps, BP 3 iterations", flush=True)
    s = Simulator([g], [0], [0.8], [TJ], d_max=d, precision="c128", trunc_rel=1e-12, max_steps=steps)
    s.step(steps)
    assert max(np.max(x) for x in s.bond_dims()) == d
    (z,), res = s.bp_expect_z(3)
    s.close()
    ref = bp.run(su.evolve_graph(g, 0.8, TJ, d, steps, 1e-12, keep_state=True).peps, 3)
    assert np.max(np.abs(z - ref.z)) < 1e-10
    assert abs(res - ref.residual) < 1e-10
