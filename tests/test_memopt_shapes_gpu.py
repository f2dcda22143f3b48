"""The memory selection's kernel at the edges of its shapes, against the
selection oracle: pair counts around multiples of a group's lanes, groups of
16 lanes (many problems) and of 64 (few), batches that leave groups of a block
without a problem, orders whose backwards come before their forwards, invalid
orders between valid ones, caps from out of reach to slack, and searches that
stop early, find better leaves or end proven."""
import numpy as np
import pytest

import oracle.memopt as MO
import workloads as W
from workloads.strategies import strategy_table

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


def problem(M, seed):
    rng = np.random.default_rng([M, seed])
    prob = W.compile_instance(W.pipeline_instance(2, M, rng.integers(5, 60, (2, M)), comm=2, act=9))
    rows = W.OrderGenerator(prob, W.MODE_LIST, 2, 0, 7, 0).generate(0, 6)
    a, b = int(prob.rank_off[0]), int(prob.rank_off[1])
    rows[1, a:b] = rng.permutation(b - a)                  # backwards first for some pairs
    fwd_first = np.argsort(prob.op_kind[a:b], kind="stable")
    rows[2, a:b] = fwd_first
    return prob, rows


def select(prob, tab, rows, n, S, nodes):
    sim = dip.Sim(prob)
    assert dip.configure_memopt(sim.h, tab.slot_layers, tab.time, tab.mem, S, nodes) == dip.OK
    idx = np.arange(n) % len(rows)
    t = torch.empty((n, 2), dtype=torch.int64, device=DEV)
    p = torch.empty((n, 2), dtype=torch.int32, device=DEV)
    s = torch.empty((n, 2), dtype=torch.uint8, device=DEV)
    c = torch.full((n, prob.n_slots), 99, dtype=torch.uint8, device=DEV)
    orders = torch.from_numpy(np.ascontiguousarray(rows[idx])).to(DEV)
    assert dip.memopt(sim.h, orders, n, t, p, s, c) in (None, dip.OK)
    torch.cuda.synchronize()
    sim.close()
    return idx, [x.cpu().numpy() for x in (t, p, s, c)]


@pytest.mark.parametrize("M", [1, 2, 15, 16, 17, 33, 64, 65, 96, 97, 129])
@pytest.mark.parametrize("frac,S,nodes", [(0.05, 6, 512), (0.5, 8, 40), (0.6, 6, 3),
                                          (0.85, 4, 512), (0.97, 6, 1), (1.0, 6, 512)])
def test_selection_shapes(M, frac, S, nodes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob, rows = problem(M, S)
    tab = strategy_table(prob)
    cands = MO.pair_candidates(tab, S)
    # the cap: a part of the first schedule's peak under the fastest choices
    peaks = [MO.greedy_select(c, live, -1)[3] for _, c, live in
             (MO.rank_problem(prob, tab, cands, rows[0], r) for r in range(2))]
    prob.mem_cap[:] = [int(x * frac) for x in peaks]
    if M > 1:
        rows[4, 0] = rows[4, 1]                            # a repeated id on rank 0
    rows[5, int(prob.rank_off[1])] = 2 * M                 # out of range on rank 1
    bad = {(4, 0)} if M > 1 else set()
    bad.add((5, 1))
    want = {}
    for i, row in enumerate(rows):
        for r in range(2):
            if (i, r) in bad:
                continue
            slots, cc, live = MO.rank_problem(prob, tab, cands, row, r)
            pf, pb = MO.rank_positions(prob, tab, row, r)
            want[i, r] = slots, MO.select(cc, live, pf, pb, int(prob.mem_cap[r]), nodes)
    order = np.argsort(tab.slot_rank, kind="stable")       # pairs by rank, then slot
    col = np.empty_like(order)
    col[order] = np.arange(len(order))
    for n in (3, 61, 4999):
        print(f"M={M} frac={frac} S={S} nodes={nodes} n={n}", flush=True)
        idx, (t, p, s, c) = select(prob, tab, rows, n, S, nodes)
        for i in range(min(n, len(rows))):
            at = idx == i
            for r in range(2):
                if (i, r) in bad:
                    assert (s[at, r] == 2).all() and (t[at, r] == -1).all()
                    continue
                slots, (cur, total, status, peak) = want[i, r]
                assert (s[at, r] == status).all(), (i, r, status, np.unique(s[at, r]))
                assert (t[at, r] == total).all() and (p[at, r] == peak).all()
                np.testing.assert_array_equal(c[at][:, col[slots]],
                                              np.broadcast_to(cur, (at.sum(), len(cur))))


@pytest.mark.parametrize("M", [250, 257, 512])
def test_selection_largest_ranks(M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob, rows = problem(M, 1)
    rows = rows[[0, 2]]
    tab = strategy_table(prob)
    cands = MO.pair_candidates(tab, 4)
    peaks = [MO.greedy_select(c, live, -1)[3] for _, c, live in
             (MO.rank_problem(prob, tab, cands, rows[0], r) for r in range(2))]
    prob.mem_cap[:] = [int(x * 0.7) for x in peaks]
    want = MO.optimise(prob, tab, cands, rows)
    print(f"M={M}", flush=True)
    idx, (t, p, s, c) = select(prob, tab, rows, 5, 4, 512)
    for k, i in enumerate(idx):
        for r in range(2):
            total, status, peak, _ = want[i][r]
            assert (t[k, r], s[k, r], p[k, r]) == (total, status, peak)
        np.testing.assert_array_equal(c[k], MO.choice_row(tab, want[i]))
