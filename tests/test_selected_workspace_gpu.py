"""The re-timed evaluate's working rows: kept with the selection's tables,
never allocated, replaced or freed by a call; worked through in steps by a
batch larger than them; shared by calls on several streams; left alone by a
captured call, whose replays are compared after larger eager calls."""
import numpy as np
import pytest

import workloads as W
from workloads.strategies import strategy_table

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


def setup(P, M, n, seed=0):
    """A handle with a selection and costs; n schedules (some deadlocked) and
    choices, and what the general kernel makes of them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng([P, M, n, seed])
    prob = W.compile_instance(W.pipeline_instance(P, M, rng.integers(1, 60, (P, M)), comm=4, act=3,
                                                  mem_cap=2 * M))
    base = W.OrderGenerator(prob, W.MODE_LIST, 2, 0, seed, 0).generate(0, min(n, 64))
    for c in range(3, len(base), 9):
        a, b = int(prob.rank_off[P - 1]), int(prob.rank_off[P])
        base[c, a:b] = rng.permutation(b - a)
    orders = torch.from_numpy(np.ascontiguousarray(base[np.arange(n) % len(base)])).to(DEV)
    choice = torch.from_numpy(rng.integers(0, 2, (n, prob.n_slots)).astype(np.uint8)).to(DEV)
    sim = dip.Sim(prob)
    tab = strategy_table(prob)
    assert dip.configure_memopt(sim.h, tab.slot_layers, tab.time, tab.mem, 5) == dip.OK
    sim.evaluate(orders[:1])
    print(f"P={P} M={M} n={n} scratch {sim.info['scratch_bytes']}", flush=True)
    assert sim.configure(4) == dip.OK
    want = sim.outputs(n, DEV)
    dip.evaluate_selected(sim.h, orders, choice, n, *want)
    torch.cuda.synchronize()
    assert sim.configure(0) == dip.OK
    return sim, orders, choice, want


def same(got, want, n=None):
    for g, w in zip(got, want):
        assert torch.equal(g, w if n is None else w[:n])


@pytest.mark.parametrize("P,M,n", [(2, 2, 65536 + 1), (2, 2, 2 * 65536 + 77), (3, 2, 70001)])
def test_batches_beyond_the_rows(P, M, n):
    sim, orders, choice, want = setup(P, M, n)
    assert sim.configure(9) == dip.OK              # (chosen by itself, the general kernel runs)
    for _ in range(2):
        out = sim.outputs(n, DEV)
        dip.evaluate_selected(sim.h, orders, choice, n, *out)
        torch.cuda.synchronize()
        same(out, want)
    sim.close()


def test_calls_allocate_nothing():
    sim, orders, choice, want = setup(4, 20, 4000)
    out = sim.outputs(4000, DEV)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    scratch = sim.info["scratch_bytes"]
    for n in (1, 4000, 64):
        dip.evaluate_selected(sim.h, orders, choice, n, *out)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free and sim.info["scratch_bytes"] == scratch
    dip.evaluate_selected(sim.h, orders, choice, 4000, *out)
    torch.cuda.synchronize()
    same(out, want)
    sim.close()


def test_captured_call_beside_larger_ones():
    n, small = 4000, 500
    sim, orders, choice, want = setup(4, 20, n)
    out, big = sim.outputs(small, DEV), sim.outputs(n, DEV)
    dip.evaluate_selected(sim.h, orders, choice, small, *out)      # an eager call before it
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dip.evaluate_selected(sim.h, orders, choice, small, *out)
    for k in range(4):
        for t in out + big:
            t.fill_(77)
        dip.evaluate_selected(sim.h, orders, choice, n, *big)
        graph.replay()
        torch.cuda.synchronize()
        print(f"replay {k}", flush=True)
        same(out, want, small)
        same(big, want)
    sim.close()


def test_calls_on_several_streams():
    n = 3000
    sim, orders, choice, want = setup(8, 12, n)
    streams = [torch.cuda.Stream() for _ in range(3)]
    parts = [slice(0, 1000), slice(1000, 1200), slice(1200, n)]
    args = []
    for p in parts:
        m = p.stop - p.start
        args.append((orders[p].contiguous(), choice[p].contiguous(), m, sim.outputs(m, DEV)))
    torch.cuda.synchronize()
    for k in range(6):
        for (o, c, m, out), s in zip(args, streams[k % 3:] + streams[:k % 3]):
            dip.evaluate_selected(sim.h, o, c, m, *out, stream=s)
    torch.cuda.synchronize()
    for p, (_, _, _, out) in zip(parts, args):
        same(out, [w[p] for w in want])
    sim.close()
