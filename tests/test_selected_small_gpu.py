"""The re-timed evaluate of candidates of few ops, where the general kernel takes
over from the simulation kernel as batches grow: both sides of that line and of
the op counts' limits, the automatic choice against both kernels."""
import numpy as np
import pytest

import workloads as W
from workloads.strategies import strategy_table

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


@pytest.mark.parametrize("P,M,n", [(1, 1, 1), (1, 24, 51200), (1, 24, 51201), (1, 25, 53000),
                                   (2, 8, 5200), (2, 8, 5201), (4, 8, 4600), (4, 8, 4601),
                                   (5, 24, 13500), (5, 25, 13500), (8, 16, 7100), (8, 16, 7101),
                                   (8, 22, 9500), (64, 2, 3800), (64, 3, 3800)])
def test_both_kernels(P, M, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng([P, M, n])
    prob = W.compile_instance(W.pipeline_instance(P, M, rng.integers(0, 40, (P, M)), comm=3, act=2,
                                                  mem_cap=M))
    base = W.OrderGenerator(prob, W.MODE_LIST, 2, 0, 3, 0).generate(0, min(n, 96))
    for c in range(2, len(base), 7):
        r = int(rng.integers(P))
        a, b = int(prob.rank_off[r]), int(prob.rank_off[r + 1])
        base[c, a:b] = rng.permutation(b - a)
    if len(base) > 5:
        base[4, 0] = base[4, 1]                            # a repeated id
    orders = torch.from_numpy(np.ascontiguousarray(base[np.arange(n) % len(base)])).to(DEV)
    choice = rng.integers(0, 2, (n, prob.n_slots)).astype(np.uint8)
    if n > 5:
        choice[5, 0] = 9                                   # beyond any pair's candidates
    choice = torch.from_numpy(choice).to(DEV)
    sim = dip.Sim(prob)
    tab = strategy_table(prob)
    assert dip.configure_memopt(sim.h, tab.slot_layers, tab.time, tab.mem, 5) == dip.OK
    sim.evaluate(orders[:1])
    got = []
    for variant in (0, 9, 4):
        assert sim.configure(variant) == dip.OK
        out = sim.outputs(n, DEV)
        for t in out:
            t.fill_(77)
        print(f"P={P} M={M} n={n} variant {variant}", flush=True)
        dip.evaluate_selected(sim.h, orders, choice, n, *out)
        torch.cuda.synchronize()
        got.append(out)
    for other in got[1:]:
        for g, w in zip(got[0], other):
            assert torch.equal(g, w)
    sim.close()
