"""GPU parity of the rollout priorities where the kernel's rows per block
change (4 rows up to 2,048 rollouts, doubling to 64, fewer for many classes),
with a ragged last block."""
import numpy as np
import pytest

import oracle.mcts as OM
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


@pytest.mark.parametrize("M,R", [(1, 1), (3, 3), (8, 2047), (8, 4097), (3, 40003), (500, 70)])
def test_rows_per_block(M, R):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob = W.compile_instance(W.pipeline_instance(1, M, 3, comm=1))
    g, G, cls = W.priority_groups(prob)
    n = int(cls.max()) + 1
    sim = dip.Sim(prob)
    assert sim.configure_greedy(G, g) == dip.OK
    sim.greedy(torch.zeros((1, G), dtype=torch.int32, device=DEV))
    assert dip.configure_rollouts(sim.h, n, cls) == dip.OK
    prefix = list(range(n - 1, n - 1 - n // 3, -1))
    rest = [c for c in range(n) if c not in set(prefix)]
    prio = torch.empty((R, G), dtype=torch.int32, device=DEV)
    ms = torch.empty(R, dtype=torch.int32, device=DEV)
    fl = torch.empty(R, dtype=torch.uint8, device=DEV)
    key = torch.full((1,), -1, dtype=torch.int64, device=DEV)
    print(f"classes {n} rollouts {R}", flush=True)
    dip.rollouts(sim.h, prefix, R, 31, 2, prio, ms, fl, key)
    rows = sorted(set(range(min(R, 70))) | set(range(max(0, R - 70), R)) |
                  set(range(0, R, max(1, R // 100))))
    want = np.stack([OM.priorities_of(prefix + OM.shuffled(rest, 31, 2, i), cls, n) for i in rows])
    np.testing.assert_array_equal(prio.cpu().numpy()[rows], want)
    sim.close()
