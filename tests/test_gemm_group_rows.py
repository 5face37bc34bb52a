"""Tile heights of the launches of several directions together (host arithmetic, no GPU needed)."""
import pytest


@pytest.mark.parametrize("dirs", [2, 3, 4])
@pytest.mark.parametrize("d", [704, 832, 960, 1088, 1344, 1472, 1728, 1984, 2112, 2368, 1024, 1536, 2048, 2560])
def test_no_higher_tile_than_the_rows_fill_and_a_price_for_each_height(d, dirs):
    """A height is not doubled where that leaves the count of tiles as it is; and in launches of several rounds tiles of 256 rows, of which a round takes at least
    1.3 times as long as one of 128-row tiles, save that many rounds."""
    from paper_2503_12668_amd import binding as b
    cu = 256
    seen = set()
    for tokens in list(range(17, 132, 3)) + [150, 185, 192, 200, 255, 256, 257, 300, 384, 512]:
        for N, K, nprob in ((d, d, 6), (d, d, 2), (4 * d, d, 2), (d, 4 * d, 2)):
            rows = b.op_gemm_group_rows(b.BF16, tokens, N, K, nprob, dirs, 64 << 20)
            assert rows in (0, 64, 128, 256)
            seen.add(rows)
            if rows == 0:
                continue
            assert rows == 64 or (tokens + rows - 1) // rows < (tokens + rows // 2 - 1) // (rows // 2), (tokens, N, K, nprob, rows)
            if rows == 256:
                pieces = b.op_gemm_choice(b.BF16, tokens, N, K, nprob, 64 << 20)[1]
                rounds = [-(-pieces * nprob * dirs * ((N + 127) // 128) * -(-tokens // h) // cu) for h in (128, 256)]
                assert rounds[1] == 1 or 1.3 * rounds[1] <= rounds[0], (tokens, N, K, nprob)
    assert 64 in seen and 128 in seen
