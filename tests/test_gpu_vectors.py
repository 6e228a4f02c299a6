"""GPU: the vector permutes of Eq. 1 (mxe_gather_x, mxe_scatter_y) move rows bit
for bit: widths around the pieces a row is cut into (4, 8 and 16 bytes) and
around a wavefront of them, leading dimensions and first columns that allow only
narrow pieces, sizes around a workgroup, rectangular shapes; the columns beside
a written block stay as they were."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mx = pytest.importorskip("paper_2308_00106_amd.mxe")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = mx.Context(0)
    yield c
    c.close()


# k, leading dimension, first column
SHAPES = [(1, 1, 0), (1, 2, 0), (1, 3, 1), (2, 2, 0), (2, 3, 1), (3, 3, 0), (4, 4, 0), (4, 6, 1), (4, 8, 2),
          (8, 8, 0), (8, 12, 4), (12, 12, 0), (16, 16, 0), (16, 17, 1), (100, 100, 0), (300, 304, 4), (513, 513, 0)]


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nrows,ncols", [(1, 1), (255, 257), (1031, 2500)])
def test_rows_move_bit_for_bit(ctx, nrows, ncols, storage):
    dt = torch.float64 if storage == "f64" else torch.float32
    m = min(nrows, ncols)
    A = ctx.register(synth.from_entries(nrows, ncols, np.arange(m), np.arange(m), np.ones(m)), storage)
    B = ctx.permute(A, 5)
    rperm, cperm = (torch.from_numpy(p).long().cuda() for p in ctx.get_permutation(B))
    for i, (k, ld, c0) in enumerate(SHAPES):
        g = torch.Generator(device="cuda").manual_seed(i)
        for n, move, perm in ((ncols, ctx.gather_x, cperm), (nrows, ctx.scatter_y, rperm)):
            src = torch.rand((n, ld), dtype=dt, device="cuda", generator=g)
            dst = torch.full((n, ld), -1.0, dtype=dt, device="cuda")
            move(B, src[:, c0:c0 + k], dst[:, c0:c0 + k])
            want = torch.full_like(dst, -1.0)
            if move == ctx.gather_x:
                want[:, c0:c0 + k] = src[perm, c0:c0 + k]
            else:
                want[perm, c0:c0 + k] = src[:, c0:c0 + k]
            assert torch.equal(dst, want), (k, ld, c0)
    ctx.release(B)
    ctx.release(A)
