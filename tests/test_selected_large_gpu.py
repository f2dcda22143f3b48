"""The re-timed evaluate beyond the direct kernel's resident groups: 8-slot
pools and the direct kernel over the list of those that filled, and, where a
schedule's end times do not fit in LDS, 32-slot pools and the general kernel
over its list.  A part of the orders fills any pool, another deadlocks.  Against
the general kernel on every schedule."""
import numpy as np
import pytest

import workloads as W
from workloads.strategies import strategy_table

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


def crowded(prob, base, M, rng):
    """Every other row runs all forwards first and needs the last rank's last
    one at once; every eighth is a random permutation on the last rank."""
    P = prob.n_ranks
    ahead = np.concatenate([np.argsort(prob.op_kind[a:b], kind="stable")
                            for a, b in zip(prob.rank_off[:-1], prob.rank_off[1:])])
    last = ahead[int(prob.rank_off[P - 1]):]
    last[:M] = last[:M][::-1].copy()
    base[1::2, :prob.n_total] = ahead
    a, b = int(prob.rank_off[P - 1]), int(prob.rank_off[P])
    for c in range(4, len(base), 8):
        base[c, a:b] = rng.permutation(b - a)


@pytest.mark.parametrize("P,M,n", [(64, 40, 3000), (8, 60, 12500), (12, 60, 9000), (4, 160, 20000),
                                   (8, 330, 700), (8, 330, 3000), (33, 80, 1500)])
def test_beyond_the_resident_groups(P, M, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng([P, M, n])
    prob = W.compile_instance(W.pipeline_instance(P, M, rng.integers(1, 50, (P, M)), comm=2, act=3,
                                                  mem_cap=2 * M))
    base = W.OrderGenerator(prob, W.MODE_LIST, 2, 0, 3, 0).generate(0, 64)
    crowded(prob, base, M, rng)
    base[6, 0] = base[6, 1]                                # a repeated id
    orders = torch.from_numpy(np.ascontiguousarray(base[np.arange(n) % 64])).to(DEV)
    choice = rng.integers(0, 2, (64, prob.n_slots)).astype(np.uint8)
    choice[10, 0] = 200                                    # beyond any pair's candidates
    choice = torch.from_numpy(np.ascontiguousarray(choice[np.arange(n) % 64])).to(DEV)
    sim = dip.Sim(prob)
    tab = strategy_table(prob)
    assert dip.configure_memopt(sim.h, tab.slot_layers, tab.time, tab.mem, 5) == dip.OK
    sim.evaluate(orders[:1])
    print(f"P={P} M={M} n={n} {sim.info}", flush=True)
    got = []
    for variant in (0, 0, 4):
        assert sim.configure(variant) == dip.OK
        out = sim.outputs(n, DEV)
        for t in out:
            t.fill_(77)
        dip.evaluate_selected(sim.h, orders, choice, n, *out)
        torch.cuda.synchronize()
        got.append(out)
    for other in got[1:]:
        for g, w in zip(got[0], other):
            assert torch.equal(g, w)
    flags = got[0][3].cpu().numpy()
    assert (flags & 1).any() and (flags & 4).any() and ((flags & 5) == 0).any()
    sim.close()
