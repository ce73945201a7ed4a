"""The complex128 two-site SVD on few columns: the forms that leave row blocks and waves out, up to 8, 16
and 32 columns and at odd numbers between, on a graph with ends of one, two and three legs, so that
Theta' comes square, taller and wider at every size.

Every <Z> of every step within 1e-10 of the oracle, the parity of the complex128 path.
"""

import math

import numpy as np
import pytest

import oracle.su as su
from heavyhex import heavy_hex

pytestmark = pytest.mark.gpu
TJ = -math.pi / 2


def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


@pytest.mark.parametrize("d,threads", [(2, 256), (3, 256), (3, 64), (4, 256), (5, 256), (6, 64), (9, 256), (10, 64), (11, 256),
                                       (13, 256), (17, 256), (20, 256), (23, 256)])
def test_few_columns(d, threads):
    _need_gpu()
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(3, 7, False)
    assert set(g.degrees()) == {1, 2, 3}
    steps = max(3, math.ceil(math.log2(d)) + 2)
    print(f"[gpu case] 25 qubits with leaves D={d} c128 {threads} threads, {steps} steps", flush=True)
    s = Simulator([g], [0], [0.8], [TJ], d_max=d, precision="c128", trunc_rel=1e-12, max_steps=steps)
    s.set_tiles(16, 2, threads)
    s.step(steps)
    (h,) = s.z_history()
    assert max(np.max(x) for x in s.bond_dims()) == d
    s.close()
    assert np.max(np.abs(h - su.evolve_graph(g, 0.8, TJ, d, steps, 1e-12).z)) < 1e-10


@pytest.mark.parametrize("d,instances", [(5, 40), (5, 100), (9, 70)])
def test_workgroups_that_share_a_cu_give_the_same_bits(d, instances):
    """More workgroups a launch than CUs: from the 257th on a workgroup numbers its waves differently."""
    _need_gpu()
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(3, 7, False)
    steps = 6
    print(f"[gpu case] 25 qubits x {instances} D={d} c128, {steps} steps", flush=True)
    s = Simulator([g], [0] * instances, [0.8] * instances, [TJ] * instances, d_max=d, precision="c128", trunc_rel=1e-12,
                  max_steps=steps)
    s.step(steps)
    h = s.z_history()
    s.close()
    assert np.max(np.abs(h[0] - su.evolve_graph(g, 0.8, TJ, d, steps, 1e-12).z)) < 1e-10
    assert all(np.array_equal(x, h[0]) for x in h[1:])
