"""Cost tables of one to three items with long runs of rows, on both sides of
the line between the kernels; every count of configurations a lane at seven and
eight kinds."""
import numpy as np
import pytest

from test_costmodel_shapes_gpu import Table, reference

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


@pytest.mark.parametrize("kinds", [1, 2, 3, 6, 7, 8])
@pytest.mark.parametrize("items", [1, 2, 3])
@pytest.mark.parametrize("n", [1, 65, 256, 257, 530])
def test_few_items(kinds, items, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng([kinds, items, n])
    t = Table()
    t.item_ptr = np.concatenate([[0], np.cumsum(rng.integers(60, 90, items))]).astype(np.int32)
    R = int(t.item_ptr[-1])
    t.n_fop, t.n_mem, t.n_net = (rng.random(R) * 10.0 ** rng.integers(0, 6, R) for _ in range(3))
    t.kind = rng.integers(0, kinds, R).astype(np.uint8)
    if items == 3:
        t.kind[-2] = kinds                                 # out of range: the last item is -1
    coef = rng.random((n, kinds, 3)) * 1e-6
    print(f"kinds {kinds} items {items} n {n}", flush=True)
    out = torch.full((n, items), -7, dtype=torch.int32, device=DEV)
    dip.cost_tables(dip.DeviceOpTable(t, kinds, DEV), torch.from_numpy(coef).to(DEV), out)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy(), reference(t, kinds, coef))
