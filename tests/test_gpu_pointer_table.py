"""ss_pointer_table: addresses arrive in order, also where they need more than one launch, and
nothing beyond them is written."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 127, 128, 129, 300])
def test_pointer_table(n):
    from paper_2404_04270_amd import binding as B
    values = [0x7000_0000_0000 + 4096 * i + n for i in range(n)]
    table = torch.full((n + 3,), -1, dtype=torch.int64, device="cuda")
    B.ss_pointer_table(table, values)
    assert table.tolist() == values + [-1] * 3
