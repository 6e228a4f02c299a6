"""GPU: row starts of permuted matrices, a scan of the lengths in tiles of 2048:
one entry short of a tile, a whole tile and one past it, with few tiles (each
adds up the sums before its own) and around 8192 of them (the sums scanned by a
launch of their own)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mx = pytest.importorskip("paper_2308_00106_amd.mxe")

TILE = 2048


@pytest.mark.parametrize("nrows", [8193, 5 * TILE - 2, 5 * TILE - 1, 5 * TILE, 8192 * TILE - 1, 8192 * TILE, 8193 * TILE + 1])
def test_row_starts_at_tile_edges(nrows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lens = np.zeros(nrows, np.int32)
    lens[::7] = 1
    lens[[1, nrows // 2, nrows - 1]] = 1
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = np.arange(rp[-1], dtype=np.int32) % 97
    with mx.Context(0) as ctx:
        a = ctx.register_matrix(nrows, 97, *(torch.from_numpy(v).cuda() for v in (rp, col, col.astype(np.float64))))
        b = ctx.permute(a, 5, mx.ROWS)
        rperm, _ = ctx.get_permutation(b)
        got_rp, got_col, _ = ctx.export_csr(b)
    assert np.array_equal(got_rp, np.concatenate([[0], np.cumsum(lens[rperm])]))
    rows = rperm[lens[rperm] == 1]
    assert np.array_equal(got_col, col[rp[rows]])
