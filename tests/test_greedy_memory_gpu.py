"""The greedy's device memory: allocated with the grouping, none by a call,
whatever the batch, the inbox size or the launch shape; batches of several
resident generations against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


@pytest.mark.parametrize("P,M,comm", [(4, 12, 3), (8, 6, 900), (32, 5, 900)])
def test_calls_allocate_nothing(P, M, comm):
    """comm 900: most stages arrive far ahead, so the rings go on into device
    memory and the inboxes grow between calls."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng([P, M])
    prob = W.compile_instance(W.pipeline_instance(P, M, rng.integers(1, 30, (P, M)), comm=comm, act=2))
    g, G, cls = W.priority_groups(prob)
    sizes = (3, 2049, 20000, 64)
    prio = W.rollout_priorities(cls, 64, seed=5)
    want = O.greedy(prob, g, G, prio, stride=prob.stride, threads=16)[1]
    rows = torch.from_numpy(np.ascontiguousarray(prio[np.arange(max(sizes)) % 64])).to(DEV)
    out = None
    for first in (True, False):                            # the first handle loads the kernels
        sim = dip.Sim(prob)
        assert sim.configure_greedy(G, g) == dip.OK
        if out is None:
            out = sim.outputs(max(sizes), DEV)
        sim.greedy(rows[:1], out=tuple(t[:1] for t in out), orders=False)     # brings the costs
        torch.cuda.synchronize()
        free, held = torch.cuda.mem_get_info()[0], sim.info["scratch_bytes"]
        for inbox in (0, 1, 0):
            assert sim.set_greedy_inbox(inbox) == dip.OK
            for n in sizes * 2:
                print(f"P={P} M={M} first {first} inbox {inbox} n={n} held {held}", flush=True)
                part = tuple(t[:n] for t in out)
                for t in part:
                    t.fill_(77)
                sim.greedy(rows[:n], out=part, orders=False)
                torch.cuda.synchronize()
                assert sim.info["scratch_bytes"] == held
                assert first or torch.cuda.mem_get_info()[0] == free
                at = np.arange(n) % 64
                for t, w in zip(part, (want.makespan, want.bubble, want.peak, want.flags)):
                    np.testing.assert_array_equal(t.cpu().numpy(), w[at])
        sim.close()
