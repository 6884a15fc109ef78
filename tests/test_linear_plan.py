"""Which kernel takes a dense product of few rows, seen through the workspace its splits ask for (no GPU needed)."""
import pytest

from paper_2507_00715_amd import binding as B


def splits(rows, k, n):
    return B.earn_linear_workspace_bytes(rows, k, n) // (rows * n * 4)


@pytest.mark.parametrize("rows,k,n,want", [
    # up to 64 rows: 64-column tiles, 256 workgroups at most
    (64, 4096, 6144, 2), (64, 16384, 4096, 4), (1, 4096, 8192, 2),
    # 65 - 96 rows: 128-column tiles where their splits are one round of every XCD
    (65, 4096, 6144, 5), (96, 3072, 5632, 5), (80, 8192, 7680, 4), (96, 11008, 4096, 8),
    # and 64-column tiles where they are not, or the inner dimension is short
    (96, 4096, 6400, 2), (80, 8192, 8192, 2), (65, 3008, 6144, 2), (96, 8192, 4096, 4), (72, 16384, 2560, 6),
    # wide outputs stay whole
    (160, 4096, 11008, 0), (16, 4096, 11008, 0)])
def test_splits_of_products_with_few_rows(rows, k, n, want):
    assert splits(rows, k, n) == want
