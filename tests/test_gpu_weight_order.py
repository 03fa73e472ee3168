"""helm_set_weights right behind queued work, on a non-blocking stream and on the null one:
cycles, recordings and reverses queued before it still take the weights before it (the tables
that they read are rewritten only once they are done), bit for bit as when the host waits in
between.  A spinning kernel ahead of them keeps the queued work from starting before the call.
"""
import numpy as np
import pytest
import torch

import helm_inputs as hi

pytestmark = pytest.mark.gpu

K = 3


def _calls(H, g, what):
    if what == "cycle":
        u = torch.zeros_like(g)
        H.cycle(g, u)
        return [u]
    if what == "backward":
        return list(H.cycle_backward(K, g, g))
    u = torch.empty_like(g)
    H.cycle_record(K, g, u)
    return [u] if what == "record" else [u, *H.cycle_reverse(K, g, g)]


@pytest.mark.parametrize("what", ["cycle", "record", "reverse", "backward"])
@pytest.mark.parametrize("graphs,own_stream", [(1, True), (0, True), (1, False)])
def test_set_weights_behind_queued_work(what, graphs, own_stream):
    from paper_2404_02493_amd import Helmholtz

    c = hi.make_problem(128, 60.0, 4, seed=5, medium="grf", phase="fmm", damping_cells=8)
    H = Helmholtz(c.velocity, c.k, levels=c.levels, precision="c64", damping_cells=c.damping_cells, use_graphs=graphs)
    H.set_phase(c.phi)
    g = torch.as_tensor(c.g).to(H.cdtype).to("cuda:0")
    w = H.weights
    other = np.concatenate([[0.5 * w[0]], 2.0 * w[1:]])
    H.set_weights(other)
    changed = [t.clone() for t in _calls(H, g, what)]
    torch.cuda.synchronize()
    H.set_weights(w)
    expect = [t.clone() for t in _calls(H, g, what)]
    torch.cuda.synchronize()
    assert not any(torch.equal(a, b) for a, b in zip(changed, expect))
    side = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(50_000_000)
        got = _calls(H, g, what)
    H.set_weights(other)
    side.synchronize()
    for a, b in zip(got, expect):
        assert torch.equal(a, b)
    # the new weights are in effect behind it
    again = _calls(H, g, what)
    torch.cuda.synchronize()
    for a, b in zip(again, changed):
        assert torch.equal(a, b)
    H.close()
