"""The re-timed evaluate through the simulation kernel against the general
kernel (any dependence graph) on the same schedules and choices: rank counts,
random and invalid choices, deadlocked and invalid orders, caps, batches
within the direct kernel's resident groups; and a sample against the simulator
oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from workloads.strategies import strategy_table

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


def problem(P, M, v, seed):
    rng = np.random.default_rng([P, M, v, seed])
    inst = W.pipeline_instance(P, M, rng.integers(0, 60, (P * v, M)), comm=int(rng.integers(0, 9)),
                               act=int(rng.integers(1, 50)), v=v, mem_cap=int(20 * M))
    return W.compile_instance(inst), rng


def run(sim, orders, choice, n):
    out = sim.outputs(n, DEV)
    for t in out:
        t.fill_(77)
    dip.evaluate_selected(sim.h, orders, choice, n, *out)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


@pytest.mark.parametrize("P,M,v", [(1, 6, 1), (2, 70, 1), (3, 5, 2), (4, 33, 1), (8, 20, 1),
                                   (12, 6, 2), (16, 12, 2), (33, 4, 1), (64, 9, 1)])
@pytest.mark.parametrize("n", [1, 67, 3000])
def test_matches_general_kernel(P, M, v, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob, rng = problem(P, M, v, n)
    rows = W.OrderGenerator(prob, W.MODE_LIST, 2, 0, 5, 0).generate(0, n)
    for c in range(2, n, 5):                               # mostly deadlocks
        for r in range(P):
            a, b = int(prob.rank_off[r]), int(prob.rank_off[r + 1])
            rows[c, a:b] = rng.permutation(b - a)
    if n > 10:
        rows[7, 0] = rows[7, 1]                            # a repeated id
        rows[8, prob.n_total - 1] = 30000                  # out of range
        rows[9, 0] = -1
    tab = strategy_table(prob)
    sim = dip.Sim(prob)
    assert dip.configure_memopt(sim.h, tab.slot_layers, tab.time, tab.mem, 5) == dip.OK
    orders = torch.from_numpy(rows).to(DEV)
    sim.evaluate(orders[:1])
    choice = rng.integers(0, 2, (n, prob.n_slots)).astype(np.uint8)
    if n > 10:
        choice[3, 0] = 200                                 # beyond any pair's candidates
        choice[4, -1] = 7
    choice = torch.from_numpy(choice).to(DEV)
    print(f"P={P} M={M} v={v} n={n} variant {sim.info['variant']}", flush=True)
    got = run(sim, orders, choice, n)
    again = run(sim, orders, choice, n)
    assert sim.configure(4) == dip.OK
    want = run(sim, orders, choice, n)
    for g, g2, w in zip(got, again, want):
        np.testing.assert_array_equal(g, w)
        np.testing.assert_array_equal(g2, w)
    sim.close()


def test_fastest_choices_are_the_plain_evaluate():
    """Every pair on its fastest candidate: the oracle's plain simulation."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for cid, n in ((2, 300), (3, 40), (4, 20)):
        prob = W.make_problem(cid)
        rows = W.generator_for(prob, cid).generate(0, n)
        want = O.evaluate(prob, rows, threads=16)
        tab = strategy_table(prob)
        sim = dip.Sim(prob)
        assert dip.configure_memopt(sim.h, tab.slot_layers, tab.time, tab.mem, 4) == dip.OK
        orders = torch.from_numpy(rows).to(DEV)
        sim.evaluate(orders)
        choice = torch.zeros((n, prob.n_slots), dtype=torch.uint8, device=DEV)
        got = run(sim, orders, choice, n)
        print(f"config {cid}", flush=True)
        for g, w in zip(got, (want.makespan, want.bubble, want.peak, want.flags)):
            np.testing.assert_array_equal(g, w)
        sim.close()
