"""Which kernel takes a dense product of few rows, seen through the workspace its splits ask for (no GPU needed)."""
import pytest

from paper_2507_00715_amd import binding as B


def splits(rows, k, n):
    return B.earn_linear_workspace_bytes(rows, k, n) // (rows * n * 4)


# the count that a launch with room for it takes (of 65 - 160 rows and wide or short products in 128-column tiles, else in 64-column ones)
@pytest.mark.parametrize("rows,k,n,want", [
    # 64-column tiles, 256 workgroups at most
    (64, 16384, 4096, 4), (1, 4096, 8192, 2), (16, 4096, 11008, 0), (32, 4096, 4096, 4),
    # 128-column tiles, by a count of the time
    (64, 4096, 6144, 5), (65, 4096, 6144, 5), (96, 3072, 5632, 4), (80, 8192, 7680, 4), (96, 11008, 4096, 8), (96, 4096, 6400, 5),
    (72, 16384, 2560, 12), (160, 4096, 4096, 5), (160, 4096, 6144, 4), (160, 4096, 11008, 2), (160, 11008, 4096, 8), (160, 896, 4864, 2),
    # Q/K/V products as wide need two splits for the kernel of few rows
    (160, 8192, 10240, 3), (160, 8192, 28672, 2),
    # more rows: 256-row tiles
    (161, 4096, 6144, 5), (200, 4096, 4096, 8), (16512, 4096, 4096, 0), (161, 4096, 11008, 0)])
def test_splits_of_products_with_few_rows(rows, k, n, want):
    assert splits(rows, k, n) == want


@pytest.mark.parametrize("k,n", [(64, 8), (896, 1152), (4096, 11008), (11008, 4096), (2048, 16384)])
def test_workspace_is_splits_of_whole_outputs(k, n):
    """Whole fp32 copies of the output, rounded up to 256 bytes, no more of them than there are pairs of 64-wide tiles."""
    for rows in (1, 31, 33, 64, 65, 96, 97, 160, 161, 700):
        size = B.earn_linear_workspace_bytes(rows, k, n)
        z = size // (rows * n * 4)
        assert size == (0 if z == 0 else (z * rows * n * 4 + 255) // 256 * 256) and z != 1 and z <= max(16, k // 256)
