"""GPU: entropies at the edges of their kernels, bit for bit against the oracle:
more regions than the pinned result buffer holds, one workgroup and several per
region, levels finer than the grid, bins with more entries than the counted
range, grids around a workgroup, calls in turn with different sizes."""
import numpy as np
import pytest

import oracle
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


def _dense_corner(n, corner, seed):
    """A full corner x corner block and a diagonal: heavy bins beside light ones."""
    i = np.arange(corner)
    r = np.concatenate([np.repeat(i, corner), np.arange(corner, n)])
    c = np.concatenate([np.tile(i, corner), np.arange(corner, n)])
    return synth.from_entries(n, n, r, c, np.random.default_rng(seed).uniform(-1, 1, len(r)))


CASES = [(lambda: synth.clustered_n4096(1), 128, 128, (64, 3)),          # 4105 regions
         (lambda: synth.clustered_n4096(2), 16, 100, (2, 4, 8, 64)),
         (lambda: synth.clustered_n4096(3), 200, 200, (1, 2)),           # several workgroups per region
         (lambda: _dense_corner(3000, 300, 4), 1, 1, (1,)),
         (lambda: _dense_corner(3000, 300, 5), 5, 7, (2, 3)),            # bins above 4096 entries
         (lambda: _dense_corner(3000, 300, 6), 255, 1, (4,)),
         (lambda: _dense_corner(3000, 300, 7), 16, 16, (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16))]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_entropies_bit_for_bit(ctx, case):
    make, gr, gc, levels = CASES[case]
    A0 = make()
    A = ctx.register(A0)
    ref = oracle.block_hist(A0.nrows, A0.ncols, A0.row_ptr, A0.col, gr, gc)
    bits, nats, hist = ctx.entropy(A, gr, gc, hist=True)
    assert np.array_equal(hist, ref) and (bits, nats) == oracle.entropy(ref)
    for (hb, hn), (wb, wn) in zip(ctx.entropy_levels(A, gr, gc, levels), oracle.entropy_levels(ref, levels)):
        assert np.array_equal(hb, wb) and np.array_equal(hn, wn), hb.shape
    assert ctx.entropy(A, gr, gc) == (bits, nats)
    ctx.release(A)
