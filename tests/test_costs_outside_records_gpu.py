"""Costs outside the simulation kernel's records (an op cost of 2**20, a
latency of 2**11) run variant 8 whatever is configured after they came, as a
handle's first costs and after others; evaluate against the oracle, the
re-timed evaluate against the general kernel."""
import copy

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


def selected(sim, orders, choice):
    out = sim.outputs(len(orders), DEV)
    for t in out:
        t.fill_(77)
    dip.evaluate_selected(sim.h, orders, choice, len(orders), *out)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


@pytest.mark.parametrize("P", [4, 6])
@pytest.mark.parametrize("field", ["cost", "comm"])
@pytest.mark.parametrize("first", [True, False])
def test_configure_after_costs_outside_the_records(P, field, first):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng([P, 3])
    inside = W.compile_instance(W.pipeline_instance(P, 7, rng.integers(1, 90, (P, 7)), comm=5, act=2,
                                                    mem_cap=9))
    outside = copy.deepcopy(inside)
    if field == "cost":
        outside.op_cost[3] = 1 << 20
    else:
        outside.edge_comm[3] = 1 << 11
    rows = W.OrderGenerator(inside, W.MODE_LIST, 2, 0, 7, 0).generate(0, 70)
    orders = torch.from_numpy(rows).to(DEV)
    sim = dip.Sim(inside)
    tab = strategy_table(inside)
    assert dip.configure_memopt(sim.h, tab.slot_layers, tab.time, tab.mem, 4) == dip.OK
    choice = torch.from_numpy(rng.integers(0, 2, (70, inside.n_slots)).astype(np.uint8)).to(DEV)

    def compare(prob, variant):
        print(f"P={P} {field} first={first} variant {sim.info['variant']}", flush=True)
        assert sim.info["variant"] == variant
        want = O.evaluate(prob, rows)
        out = sim.evaluate(orders)
        torch.cuda.synchronize()
        for g, w in zip(out, (want.makespan, want.bubble, want.peak, want.flags)):
            np.testing.assert_array_equal(g.cpu().numpy(), w)

    if not first:
        sim.evaluate(orders)
    sim.costs = dip.HostCosts.of(outside)
    sim.evaluate(orders[:1], resend_costs=True)
    for configure in (lambda: sim.configure(0), lambda: sim.configure_pool(8),
                      lambda: sim.configure_pool(4), lambda: sim.configure_pool(0),
                      lambda: sim.configure(9), lambda: sim.configure(9, 4),
                      lambda: sim.configure(0)):
        assert configure() == dip.OK
        compare(outside, 8)
    got = selected(sim, orders, choice)
    assert sim.configure(4) == dip.OK
    for g, w in zip(got, selected(sim, orders, choice)):
        np.testing.assert_array_equal(g, w)
    # and back within them
    assert sim.configure(0) == dip.OK
    sim.costs = dip.HostCosts.of(inside)
    sim.evaluate(orders[:1], resend_costs=True)
    compare(inside, 9)
    sim.close()
