"""GPU parity of the cost tables where the register kernel can go wrong:
every kind count, batch sizes at its lane and block edges, items of no, few
and many rows, entries that leave as vectors or one by one, kind bytes at any
alignment, kinds out of range."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


class Table:
    pass


def reference(t, kinds, coef):
    """Row by row in float64, as the entry point defines it."""
    out = np.zeros((coef.shape[0], len(t.item_ptr) - 1), np.int64)
    for i in range(out.shape[1]):
        s = np.zeros(coef.shape[0])
        bad = False
        for r in range(t.item_ptr[i], t.item_ptr[i + 1]):
            k = int(t.kind[r])
            bad |= k >= kinds
            c = coef[:, min(k, kinds - 1)]
            s = s + np.maximum(np.maximum(c[:, 0] * t.n_fop[r], c[:, 1] * t.n_mem[r]),
                               c[:, 2] * t.n_net[r])
        us = np.ceil(s * 1e6)
        out[:, i] = np.where(bad | ~(us <= 2147483647.0), -1, us)
    return out.astype(np.int32)


@pytest.mark.parametrize("kinds", [1, 2, 3, 4, 5, 6, 7, 8, 9, 17])
@pytest.mark.parametrize("n,items", [(1, 1), (64, 3), (65, 4), (128, 40), (129, 7), (256, 1),
                                     (257, 5), (300, 2050)])
def test_shapes(kinds, n, items):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng([kinds, n, items])
    t = Table()
    rows = rng.integers(0, 40, items) if items < 100 else rng.integers(0, 4, items)
    rows[0] = 9
    t.item_ptr = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    R = int(t.item_ptr[-1])
    t.n_fop, t.n_mem, t.n_net = (rng.random(R) * 10.0 ** rng.integers(0, 6, R) for _ in range(3))
    t.kind = rng.integers(0, kinds, R).astype(np.uint8)
    if items > 3:
        t.kind[int(t.item_ptr[2])] = min(255, kinds + int(rng.integers(0, 3)))
        t.kind[-1] = 255 if kinds < 255 else 0
    coef = rng.random((n, kinds, 3)) * 1e-6
    want = reference(t, kinds, coef)
    print(f"kinds {kinds} n {n} items {items} rows {R}", flush=True)
    dt = dip.DeviceOpTable(t, kinds, DEV)
    c = torch.from_numpy(coef).to(DEV)
    # rows of the output at 16-byte alignment and 4 bytes off it
    for off in (0, 1):
        buf = torch.full((n * items + off + 8,), -7, dtype=torch.int32, device=DEV)
        out = buf[off:off + n * items].view(n, items)
        dip.cost_tables(dt, c, out)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), want)
        assert (buf[:off] == -7).all() and (buf[off + n * items:] == -7).all()
