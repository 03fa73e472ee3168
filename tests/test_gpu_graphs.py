"""Captured graphs outlive changes of the phase and of the weights (they read both from
device memory): after any sequence of changes a context gives, bit for bit, what a fresh
context with the same phase and weights gives, in the cycle, the recorded cycles and their
reverse.  (The same kernels run on the same values, so equality is exact.)
"""
import numpy as np
import pytest
import torch

import helm_inputs as hi

pytestmark = pytest.mark.gpu


def _context(c, prec):
    from paper_2404_02493_amd import Helmholtz

    return Helmholtz(c.velocity, c.k, levels=c.levels, precision=prec, damping_cells=c.damping_cells)


def _results(H, g, K=2):
    u = torch.zeros_like(g)
    H.cycle(g, u)
    uk = H.cycle_record(K, g, torch.empty_like(g))
    gphi, gw = H.cycle_reverse(K, g, uk)
    torch.cuda.synchronize()
    return [t.clone() for t in (u, uk, gphi, gw)]


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_graphs_follow_phase_and_weights(prec):
    c = hi.make_problem(128, 60.0, 4, seed=2, medium="grf", phase="fmm", damping_cells=8)
    H = _context(c, prec)
    g = torch.as_tensor(c.g).to(H.cdtype).to("cuda:0")
    w = H.weights
    phases = [np.asarray(c.phi), 0.9 * np.asarray(c.phi), np.asarray(c.phi)[::-1, ::-1].copy()]
    weights = [w, np.concatenate([[0.9 * w[0]], 1.1 * w[1:]]), w]
    # the buffers stay the same, so every round after the first replays the first one's graphs
    for rnd, (phi, wt) in enumerate(zip(phases, weights)):
        if rnd == 2:  # other phase arrays in between
            H.set_rays(3)
            H.cycle(g, torch.zeros_like(g))
        H.set_phase(phi)
        H.set_weights(wt)
        got = _results(H, g)
        F = _context(c, prec)
        F.set_phase(phi)
        F.set_weights(wt)
        for name, a, b in zip(("cycle", "record", "grad_phi", "grad_w"), got, _results(F, g)):
            assert torch.equal(a, b), f"round {rnd}: {name}"
        F.close()
    H.close()
