"""The simulation kernel's own passes, which the direct kernel would hide on
small batches: publishing counts below, at and above the pools' sizes with
variant 9 fixed, and ranks of many ops of which few are read elsewhere, whose
batches fit the groups resident with 16 slots and not the direct kernel's.
Against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from test_sim_shapes_gpu import compare, instance, rows_of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


def fixed(sim):
    assert sim.configure(9) == dip.OK


@pytest.mark.parametrize("P,M,v", [(4, 4, 1), (4, 5, 1), (4, 8, 1), (4, 9, 1), (4, 16, 1), (4, 17, 1),
                                   (7, 8, 1), (8, 20, 3), (64, 8, 1), (64, 30, 1)])
@pytest.mark.parametrize("n", [1, 65, 257, 2500])
def test_pool_bounds_with_the_variant_fixed(P, M, v, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob, rng = instance(P, M, v, 2)
    rows = rows_of(prob, n, rng)
    print(f"P={P} M={M} v={v} n={n}", flush=True)
    compare(prob, rows, fixed)


@pytest.mark.parametrize("linked", [4, 5, 8, 9])
def test_few_ops_read_elsewhere(linked):
    """4 ranks of 80 ops; only the first microbatches' stages cross ranks: at
    most 8, 10, 16 or 18 end times a rank are published."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P, M, n = 4, 40, 40000
    rng = np.random.default_rng([linked, 7])
    prob = W.compile_instance(W.pipeline_instance(P, M, rng.integers(1, 50, (P, M)), comm=2, act=1,
                                                  mem_cap=M))
    rank = np.repeat(np.arange(P), prob.n_ops)
    ptr, op, comm = [0], [], []
    for g in range(prob.n_total):
        lid = g - int(prob.rank_off[rank[g]])
        for e in range(int(prob.pred_ptr[g]), int(prob.pred_ptr[g + 1])):
            p = int(prob.pred_op[e])
            if rank[p] == rank[g] or lid // 2 < linked:
                op.append(p)
                comm.append(int(prob.edge_comm[e]))
        ptr.append(len(op))
    prob.pred_ptr = np.array(ptr, np.int32)
    prob.pred_op = np.array(op, np.int32)
    prob.edge_comm = np.array(comm, np.int32)
    base = W.OrderGenerator(prob, W.MODE_LIST, 2, 0, 3, 0).generate(0, 64)
    a, b = int(prob.rank_off[P - 1]), int(prob.rank_off[P])
    for c in range(3, 64, 4):                              # most of them deadlock
        base[c, a:b] = rng.permutation(b - a)
    want = O.evaluate(prob, base, threads=16)
    at = np.arange(n) % 64
    orders = torch.from_numpy(np.ascontiguousarray(base[at])).to(DEV)
    for slots in (0, 4, 8, 16):
        sim = dip.Sim(prob)
        if slots:
            assert sim.configure_pool(slots) == dip.OK
        out = sim.evaluate(orders)
        torch.cuda.synchronize()
        print(f"linked {linked} slots {slots} {dip.last_retries(sim.h)}", flush=True)
        for g, w in zip(out, (want.makespan, want.bubble, want.peak, want.flags)):
            np.testing.assert_array_equal(g.cpu().numpy(), w[at])
        sim.close()
