"""Cost tables of as many items as 32 bits count, where rounding the count up
to whole chunks must not overflow: nearly all items empty (priced 0), one row
in each of the first, a middle and the last item."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_14145_amd as dip

DEV = "cuda:0"


class Table:
    def __init__(self, n_items, n_rows, kinds):
        self.n_items = n_items
        self.ptr = torch.full((n_items + 1,), 1, dtype=torch.int32, device=DEV)
        self.ptr[0] = 0
        self.ptr[n_items // 2 + 1:] = 2
        self.ptr[n_items] = 3
        self.rows = [torch.tensor([2e-6, 5e-6, 9e-6], dtype=torch.float64, device=DEV)
                     for _ in range(3)]
        self.kind = torch.tensor([0, kinds - 1, 0], dtype=torch.uint8, device=DEV)
        self.c = dip.OpTable(n_items, n_rows, kinds, self.ptr.data_ptr(),
                             *(r.data_ptr() for r in self.rows), self.kind.data_ptr())


@pytest.mark.parametrize("kinds", [1, 5])
@pytest.mark.parametrize("n_items", [2**31 - 2, 2**31 - 1])
def test_item_count_near_int32_max(kinds, n_items):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 20 GiB of device memory")
    print(f"{kinds} kinds, {n_items} items", flush=True)
    table = Table(n_items, 3, kinds)
    coef = torch.ones((1, kinds, 3), dtype=torch.float64, device=DEV)
    out = torch.full((1, n_items), -7, dtype=torch.int32, device=DEV)
    dip.cost_tables(table, coef, out)
    torch.cuda.synchronize()
    got = out[0]
    assert [int(got[i]) for i in (0, n_items // 2, n_items - 1)] == [2, 5, 9]
    for i in (0, n_items // 2, n_items - 1):
        got[i] = 0
    for lo in range(0, n_items, 1 << 28):
        assert int(got[lo:lo + (1 << 28)].abs().max()) == 0
