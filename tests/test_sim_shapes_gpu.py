"""GPU parity of the simulation kernel on rank counts that leave lanes of a
candidate's group without a rank, and on batches from one candidate up, with
orders that deadlock, fill pools and exceed caps."""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


def instance(P, M, v, seed):
    rng = np.random.default_rng([P, M, v, seed])
    inst = W.pipeline_instance(P, M, rng.integers(0, 50, (P * v, M)), comm=int(rng.integers(0, 9)),
                               act=2, v=v, mem_cap=M + 2)
    return W.compile_instance(inst), rng


def rows_of(prob, n, rng):
    """List schedules, a third of them with swaps, a third random permutations."""
    gen = W.OrderGenerator(prob, W.MODE_LIST, 3, 0, 11, 0)
    rows = gen.generate(0, n)
    for c in range(0, n, 3):
        for r in range(prob.n_ranks):
            a, b = int(prob.rank_off[r]), int(prob.rank_off[r + 1])
            rows[c, a:b] = rng.permutation(b - a)
    return rows


def compare(prob, rows, configure=None):
    want = O.evaluate(prob, rows, threads=16)
    sim = dip.Sim(prob)
    if configure:
        configure(sim)
    out = sim.evaluate(torch.from_numpy(rows).to(DEV))
    torch.cuda.synchronize()
    assert sim.info["variant"] == 9
    for got, exp in zip(out, (want.makespan, want.bubble, want.peak, want.flags)):
        np.testing.assert_array_equal(got.cpu().numpy(), exp)
    sim.close()


@pytest.mark.parametrize("P", [3, 5, 7, 12, 17, 24, 33, 48, 63])
@pytest.mark.parametrize("M,v", [(1, 1), (9, 1), (6, 3)])
def test_any_rank_count(P, M, v):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob, rng = instance(P, M, v, 1)
    rows = rows_of(prob, 150, rng)
    print(f"P={P} M={M} v={v} N={prob.n_total}", flush=True)
    for slots in (4, 0, 16):
        compare(prob, rows, lambda s: s.configure_pool(slots))


@pytest.mark.parametrize("P,M,v", [(4, 8, 1), (4, 9, 1), (4, 16, 1), (4, 17, 1), (4, 33, 1),
                                   (8, 20, 3), (16, 5, 2), (64, 8, 1), (64, 30, 1)])
@pytest.mark.parametrize("n", [1, 3, 65, 257, 2500])
def test_small_batches_and_pool_bounds(P, M, v, n):
    """Batches within the resident groups (spread over the blocks), and rank
    publishing counts below, at and above the pools' sizes (8, 16 and 32
    slots), where the later passes are left out or run."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob, rng = instance(P, M, v, 2)
    rows = rows_of(prob, n, rng)
    print(f"P={P} M={M} v={v} n={n}", flush=True)
    compare(prob, rows)
    compare(prob, rows, lambda s: s.configure_pool(4))


@pytest.mark.parametrize("P,M,n", [(4, 90, 20000), (8, 70, 9000), (64, 40, 3000)])
def test_pools_that_fill_in_large_batches(P, M, n):
    """Batches beyond the resident groups whose first ranks run far ahead of
    the last one (all forwards first, the last rank's in reverse): every pool
    size fills, and the candidates end in the kernel that keeps all end times,
    started over a list; a part of the batch deadlocks there."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng([P, M, n])
    prob = W.compile_instance(W.pipeline_instance(P, M, rng.integers(1, 50, (P, M)), comm=2, act=1, mem_cap=2 * M))
    base = W.OrderGenerator(prob, W.MODE_LIST, 2, 0, 3, 0).generate(0, 64)
    fwd_first = np.concatenate([np.argsort(prob.op_kind[a:b], kind="stable") for a, b in
                                zip(prob.rank_off[:-1], prob.rank_off[1:])])
    last = fwd_first[int(prob.rank_off[P - 1]):]
    last[:M] = last[:M][::-1].copy()                       # needs the last forward first
    base[1::2] = fwd_first.astype(base.dtype)
    for c in range(5, 64, 8):
        a, b = int(prob.rank_off[P - 1]), int(prob.rank_off[P])
        base[c, a:b] = rng.permutation(b - a)
    rows = np.ascontiguousarray(base[np.arange(n) % 64])
    print(f"P={P} M={M} n={n}", flush=True)
    want = O.evaluate(prob, base, threads=16)
    sim = dip.Sim(prob)
    out = sim.evaluate(torch.from_numpy(rows).to(DEV))
    torch.cuda.synchronize()
    for got, exp in zip(out, (want.makespan, want.bubble, want.peak, want.flags)):
        np.testing.assert_array_equal(got.cpu().numpy(), exp[np.arange(n) % 64])
    sim.close()
