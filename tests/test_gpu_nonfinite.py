"""A state that has gone non-finite ends in the numeric status at the next synchronising call, in each form
of the two-site SVD and in the reverse sweep, and a reset makes the context whole again."""

import math

import numpy as np
import pytest

import oracle.su as su
from heavyhex import heavy_hex

pytestmark = pytest.mark.gpu
TJ = -math.pi / 2


def _spoil(sim):
    """NaN into the first element of the first site tensor, where the workspace begins."""
    import torch
    sim.sync()
    t = torch.float64 if sim.cfg.precision == 1 else torch.float32
    sim.workspace[:16].view(t)[:2].fill_(float("nan"))
    torch.cuda.synchronize()


@pytest.mark.parametrize("d,precision,threads", [(8, "c128", 256), (8, "c128", 64), (16, "c128", 256), (20, "c128", 256), (40, "c128", 256),
                                                 (8, "c64", 256), (16, "c64", 64), (20, "c64", 256), (40, "c64", 256)])
def test_nan_ends_in_the_status(d, precision, threads):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(3, 7, False)
    steps = 4
    print(f"[gpu case] 25 qubits D={d} {precision} {threads} threads, NaN after two of {steps} steps", flush=True)
    cut = 1e-4 if d > 32 else 1e-12 if precision == "c128" else 1e-6
    s = Simulator([g], [0], [0.8], [TJ], d_max=d, precision=precision, trunc_rel=cut, max_steps=steps)
    s.set_tiles(16, 1, threads)
    s.step(2)
    _spoil(s)
    s.step(2)
    with pytest.raises(Exception, match="non-finite"):
        s.sync()
    s.reset()
    s.step(steps)
    (h,) = s.z_history()
    s.close()
    tol = 1e-10 if precision == "c128" else 1e-5
    assert np.max(np.abs(h - su.evolve_graph(g, 0.8, TJ, d, steps, cut).z)) < tol


@pytest.mark.parametrize("d,precision,threads", [(8, "c128", 64), (16, "c128", 256), (20, "c128", 256), (16, "c64", 256), (20, "c64", 256)])
def test_nan_before_a_reverse_sweep(d, precision, threads):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2309_15642_amd.simulator import Simulator
    g = heavy_hex(3, 7, False)
    for mode in (1, 2):
        print(f"[gpu case] 25 qubits D={d} {precision} {threads} threads, adjoint {mode}, NaN after two of four steps", flush=True)
        s = Simulator([g], [0], [0.8], [TJ], d_max=d, precision=precision, trunc_rel=1e-12 if precision == "c128" else 1e-6,
                      max_steps=4, adjoint=mode)
        s.set_tiles(16, 1, threads)
        s.step(2)
        _spoil(s)
        s.step(2)
        with pytest.raises(Exception, match="non-finite"):
            s.backward([np.full(g.n_nodes, 1.0 / g.n_nodes)])
        s.close()


@pytest.mark.parametrize("d,precision", [(2, "c128"), (8, "c64"), (20, "c128")])
def test_infinite_element_under_a_vanishing_weight(d, precision):
    """An infinite element where lambda^2 is zero in float64 is no zero term: the readout reports it."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from heavyhex import ring
    from paper_2309_15642_amd.simulator import Simulator
    g = ring(12)
    print(f"[gpu case] ring of 12 D={d} {precision}, infinity under lambda 1e-170", flush=True)
    s = Simulator([g], [0], [0.8], [TJ], d_max=d, precision=precision, trunc_rel=0.0, max_steps=2)
    s.step(2)
    s.sync()
    esize = 16 if precision == "c128" else 8
    n_gamma = sum(2 * d ** int(k) for k in g.degrees())
    off_lam = -(-n_gamma * esize // 256) * 256  # the weights [edge][d] follow the site tensors
    lam = s.workspace[off_lam : off_lam + 8 * d * len(g.edges)].view(torch.float64).view(-1, d)
    inner = max(e for e, (u, v) in enumerate(g.edges) if 0 in (u, v))  # the last leg of qubit 0
    assert lam[inner, 1] > 0  # that leg has a second index
    lam[inner, 1] = 1e-170
    s.workspace[: 2 * esize].view(torch.float64 if precision == "c128" else torch.float32)[2] = float("inf")  # its element [0][0][1]
    torch.cuda.synchronize()
    with pytest.raises(Exception, match="non-finite"):
        s.expect_z()
    s.close()
