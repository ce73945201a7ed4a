"""The complex128 two-site SVD (sorted Householder QR, register Jacobi with accumulated rotations) at
the bond dimensions where its lane groups, column padding and tiles change, with ends of one, two and
three legs, so that Theta' comes taller, wider and square.

Every <Z> of every step within 1e-10 of the oracle: the parity of the complex128 path, at a cutoff of
1e-12 that keeps singular values twelve orders under the largest.
"""

import math

import numpy as np
import pytest

import oracle.su as su
from heavyhex import heavy_hex

pytestmark = pytest.mark.gpu
TJ = -math.pi / 2


@pytest.mark.parametrize("d,threads", [(1, 256), (2, 256), (3, 64), (7, 256), (8, 64), (9, 256), (15, 64), (16, 256),
                                       (16, 64), (17, 256), (24, 256), (31, 256), (32, 256)])
def test_c128_svd_bond_edges(d, threads):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(2, 9, False)
    steps = max(3, math.ceil(math.log2(d)) + 2)
    print(f"[gpu case] heavy_hex 2x9 D={d} c128 {threads} threads, {steps} steps", flush=True)
    s = Simulator([g], [0], [0.8], [TJ], d_max=d, precision="c128", trunc_rel=1e-12, max_steps=steps)
    s.set_tiles(16, 2, threads)
    s.step(steps)
    (h,) = s.z_history()
    s.close()
    assert np.max(np.abs(h - su.evolve_graph(g, 0.8, TJ, d, steps, 1e-12).z)) < 1e-10
