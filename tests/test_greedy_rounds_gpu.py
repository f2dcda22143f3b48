"""GPU parity of the greedy's rounds of several commits: the queue forms a
rank goes through (runs of equal times, later stages in LDS and in device
memory, joins of stages committed together) on both launch shapes (a wave per
candidate, several candidates a wave), against the one-commit-a-step oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


def pipeline(P, M, v, fcost, comm, cap=-1):
    inst = W.pipeline_instance(P, M, fcost, comm=comm, act=3, mem_cap=cap, v=v)
    return W.compile_instance(inst)


def check(prob, prio, inbox=0, tag=""):
    g, G, _ = W.priority_groups(prob)
    print(f"{tag}: P={prob.n_ranks} N={prob.n_total} G={G} n={len(prio)} inbox={inbox}", flush=True)
    want_o, want = O.greedy(prob, g, G, prio, stride=prob.stride, threads=16)
    sim = dip.Sim(prob)
    assert sim.configure_greedy(G, g) == dip.OK
    assert sim.set_greedy_inbox(inbox) == dip.OK
    ords, (ms, bub, pk, fl) = sim.greedy(torch.from_numpy(prio).to(DEV))
    torch.cuda.synchronize()
    N = prob.n_total
    np.testing.assert_array_equal(ords.cpu().numpy()[:, :N], want_o[:, :N])
    np.testing.assert_array_equal(ms.cpu().numpy(), want.makespan)
    np.testing.assert_array_equal(bub.cpu().numpy(), want.bubble)
    np.testing.assert_array_equal(pk.cpu().numpy(), want.peak)
    np.testing.assert_array_equal(fl.cpu().numpy(), want.flags)
    sim.close()


@pytest.mark.parametrize("P,M,v", [(1, 5, 1), (2, 40, 1), (3, 7, 3), (4, 33, 2), (5, 9, 1),
                                   (8, 16, 2), (12, 10, 2), (16, 9, 3), (17, 6, 1), (32, 12, 2),
                                   (33, 5, 1), (64, 8, 1)])
@pytest.mark.parametrize("shape", ["zero", "ties", "spread"])
@pytest.mark.parametrize("inbox", [0, 1])
def test_queue_forms(P, M, v, shape, inbox):
    """zero: most stages cost nothing (floods of equal times); ties: all costs
    equal, no latency; spread: latencies far above the costs pile up later
    stages (inbox 1 sends nearly all of them to device memory)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L = P * v
    rng = np.random.default_rng([P, M, v])
    cost = {"zero": np.where(rng.random((L, M)) < 0.7, 0, rng.integers(1, 9, (L, M))),
            "ties": np.full((L, M), 5), "spread": rng.integers(1, 40, (L, M))}[shape]
    prob = pipeline(P, M, v, cost, comm={"zero": 0, "ties": 0, "spread": 700}[shape],
                    cap=3 * (M + 1) if shape == "spread" else -1)
    _, G, _ = W.priority_groups(prob)
    prio = rng.integers(-2, 3, (37, G)).astype(np.int32)
    prio[0] = np.iinfo(np.int32).min
    prio[1] = np.iinfo(np.int32).max
    prio[2] = np.arange(G)
    prio[3] = np.where(np.arange(G) % 2, np.iinfo(np.int32).min, np.iinfo(np.int32).max)
    check(prob, prio, inbox, shape)


@pytest.mark.parametrize("n", [2100, 8 * 256 + 5])
def test_several_candidates_a_wave(n):
    """Batches too large for a wave per candidate; the last wave ragged."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for P, M, v in ((3, 4, 1), (8, 5, 1), (16, 3, 1), (32, 3, 1)):
        rng = np.random.default_rng([P, n])
        prob = pipeline(P, M, v, rng.integers(0, 6, (P * v, M)), comm=2)
        _, G, _ = W.priority_groups(prob)
        check(prob, rng.integers(0, 4, (n, G)).astype(np.int32), 0, "dense")


def test_joins_outside_lds():
    """More joins than a block's LDS holds beside the bitmaps of 64 ranks:
    their accumulators lie in device memory."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P, M, joins = 64, 512, 17800
    rng = np.random.default_rng(5)
    prob = pipeline(P, M, 1, rng.integers(3, 30, (P, M)), comm=4)
    preds = [list(prob.pred_op[prob.pred_ptr[o]:prob.pred_ptr[o + 1]]) for o in range(prob.n_total)]
    comms = [list(prob.edge_comm[prob.pred_ptr[o]:prob.pred_ptr[o + 1]])
             for o in range(prob.n_total)]
    made = 0
    for r in range(1, P):
        for u in range(1, M):
            if made == joins:
                break
            f = int(prob.rank_off[r]) + 2 * u                  # F(u, r) also waits for F(u-1, r-1)
            preds[f].append(int(prob.rank_off[r - 1]) + 2 * (u - 1))
            comms[f].append(4)
            made += 1
    assert made == joins
    prob.pred_ptr[1:] = np.cumsum([len(p) for p in preds])
    prob.pred_op = np.array([x for p in preds for x in p], np.int32)
    prob.edge_comm = np.array([x for c in comms for x in c], np.int32)
    _, G, cls = W.priority_groups(prob)
    check(prob, W.rollout_priorities(cls, 3, seed=4), 0, "joins")
