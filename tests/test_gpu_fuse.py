"""GPU parity of the ADR levels joined across their Gram passes (the default form of
levels that do not march) against the FP64 oracle: one ADR step and whole cycles.

Grids: level 2 smaller than one 32 x 32 tile, of exactly one, of several in either
direction, two ADR levels, all of them, and more tiles than the consumers sum themselves
(512 and 257..: the one-block solve between the passes).  Tolerances as in the other
parity tests: 1e-12 (FP64 cycles) and 1e-5 (FP32 cycles), relative 2-norm and element by
element.
"""
import numpy as np
import pytest
import torch

import helm_inputs as hi
from gpu_util import TOL, assert_close, make_pair, rand_grid, rounded, to_dev
from oracle.adr import adr_step
from oracle.cycle import cycle

pytestmark = pytest.mark.gpu

# (rows, columns, levels, adr_levels)
GRIDS = [(16, 16, 3, 3), (32, 64, 4, 3), (64, 64, 3, 3), (64, 64, 4, 2), (128, 128, 4, 3), (32, 512, 4, 3),
         (512, 32, 4, 3), (256, 256, 6, 0), (256, 512, 5, 3), (512, 4096, 5, 3)]


@pytest.mark.parametrize("ny,nx,levels,adr_levels", GRIDS)
@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_joined_adr_levels(ny, nx, levels, adr_levels, prec):
    c = hi.make_problem(nx, 0.5 * max(nx, ny), levels, seed=7 + nx + ny, medium="grf", phase="fmm",
                        damping_cells=8 if min(nx, ny) > 16 else 2, ny=ny)
    P, H = make_pair(c, prec, adr_levels=adr_levels) if adr_levels else make_pair(c, prec, adr_levels=levels - 1)
    rng = np.random.default_rng(nx + 3 * ny)
    cd = H.cdtype
    u2, g2 = (rounded(rand_grid(rng, (ny // 2, nx // 2)), cd) for _ in range(2))
    out = H.debug_op(9, 2, to_dev(u2, cd), to_dev(g2, cd))
    assert_close(out, adr_step(P, g2, u2), TOL[prec], "ADR step")
    u, g = rounded(rand_grid(rng, (ny, nx)), cd), rounded(torch.as_tensor(c.g), cd)
    ref = cycle(P, g, u)
    gd = to_dev(g, cd)
    for rep in range(2):  # the second cycle replays the captured graph on the same buffers
        ud = to_dev(u, cd) if rep == 0 else ud.copy_(u.to(cd))
        H.cycle(gd, ud)
        assert_close(ud, ref, TOL[prec], f"cycle {rep}")
    H.close()


def test_separate_passes_of_a_large_class():
    """40 problems of 256^2 (64 tiles each, more than five blocks per CU together) take separate
    passes: solves equal those on the same contexts, and a context's cycle the oracle's."""
    from oracle.cycle import Problem
    from paper_2404_02493_amd import HelmholtzBatch

    cases = [hi.make_problem(256, 0.5 * 256, 5, seed=31 + p, medium="grf", phase="fmm", damping_cells=8)
             for p in range(2)]
    B = HelmholtzBatch([dict(velocity=c.velocity, k=c.k, levels=c.levels, damping_cells=c.damping_cells, phi=c.phi)
                        for c in cases * 20], precision="c64", lanes=1)
    gs = [torch.as_tensor(c.g).to("cuda:0") for c in cases * 20]
    us, its, rr, st = B.solve(gs, tol=1e-6, maxit=400, mode=1)
    torch.cuda.synchronize()
    assert np.all(st == 0) and np.all(rr < 1e-6) and np.all(B.classes() == B.classes()[0])
    for p in (0, 39):
        u, it, r, _ = B.problem(p).solve(gs[p], tol=1e-6, maxit=400, mode=1)
        assert it == its[p] and r == rr[p] and torch.equal(u, us[p])
    c = cases[0]
    H = B.problem(0)
    P = Problem(c.velocity, c.k, c.levels, damping_cells=c.damping_cells, phi=c.phi)
    H.set_weights(P.weights.numpy())
    u = rounded(rand_grid(np.random.default_rng(3), (256, 256)), H.cdtype)
    g = rounded(torch.as_tensor(c.g), H.cdtype)
    ud = to_dev(u, H.cdtype)
    H.cycle(to_dev(g, H.cdtype), ud)
    assert_close(ud, cycle(P, g, u), TOL["c64"], "cycle")
    B.close()
