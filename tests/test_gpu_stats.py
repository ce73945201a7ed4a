"""The SVD statistics are counted on several lines of memory and added up when asked for."""

import math

import pytest

from heavyhex import heavy_hex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,precision,instances", [(3, "c128", 1), (8, "c64", 30), (20, "c128", 2), (40, "c64", 1)])
def test_statistics_add_up(d, precision, instances):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(3, 7, False)
    print(f"[gpu case] statistics: 25 qubits x {instances} D={d} {precision}, 4 steps", flush=True)
    s = Simulator([g], [0] * instances, [0.8] * instances, [-math.pi / 2] * instances, d_max=d, precision=precision, trunc_rel=1e-6,
                  max_steps=4)
    for steps in (4, 1):  # a reset starts them again
        s.reset()
        s.step(steps)
        st = s.stats()
        assert st["svds"] == steps * instances * len(g.edges) and st["not_converged"] == 0
        assert 0 < st["max_sweeps"] <= st["jacobi_sweeps"] <= st["max_sweeps"] * st["svds"]
    s.close()
