"""Evaluate on rank counts that are no power of two, with batches on both sides
of the lines between the direct, the simulation and the pool kernel; a part of
the orders deadlocks or fills the pools.  Against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


@pytest.mark.parametrize("P,M,sizes", [
    (3, 16, (50000, 120000, 240000)),
    (5, 33, (40000, 60000)),
    (12, 16, (25000, 30001, 120000)),
    (12, 33, (25000, 60000)),                              # 792 ops
    (12, 34, (25000, 60000)),
    (20, 16, (5000, 14001, 60000)),                        # 640 ops
    (20, 17, (14001, 60000)),
    (33, 8, (5000, 9999, 12000)),
    (63, 40, (2000, 4100, 9000)),
    (33, 128, (3000, 5000))])
def test_sizes(P, M, sizes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng([P, M])
    prob = W.compile_instance(W.pipeline_instance(P, M, rng.integers(1, 50, (P, M)), comm=3, act=1,
                                                  mem_cap=M + 1))
    base = W.OrderGenerator(prob, W.MODE_LIST, 2, 0, 3, 0).generate(0, 64)
    ends = list(zip(prob.rank_off[:-1].tolist(), prob.rank_off[1:].tolist()))
    ahead = np.concatenate([np.argsort(prob.op_kind[a:b], kind="stable") for a, b in ends])
    last = ahead[ends[-1][0]:]
    last[:M] = last[:M][::-1].copy()                       # needs the last forward first
    base[1::16, :prob.n_total] = ahead.astype(base.dtype)
    for c in range(5, 64, 16):
        a, b = ends[int(rng.integers(P))]
        base[c, a:b] = rng.permutation(b - a)
    base[7, 0] = base[7, 1]                                # a repeated id
    want = O.evaluate(prob, base, threads=16)
    want = [torch.from_numpy(w).to(DEV) for w in (want.makespan, want.bubble, want.peak, want.flags)]
    pool = torch.from_numpy(base).to(DEV)
    sim = dip.Sim(prob)
    for n in sizes:
        at = torch.arange(n, device=DEV) % 64
        out = sim.outputs(n, DEV)
        for t in out:
            t.fill_(77)
        sim.evaluate(pool[at].contiguous(), out=out)
        torch.cuda.synchronize()
        print(f"P={P} M={M} n={n} {dip.last_retries(sim.h)}", flush=True)
        for t, w in zip(out, want):
            assert torch.equal(t, w[at])
    sim.close()
