"""GPU: random permutations and gradient shuffles where their kernels change
(one workgroup up to 8192 indices, small buckets up to 131072, several
permutations in one launch), against the oracle, with the permuted row starts:
rows and columns on either side of each line, gradient pivots that put a part's
end there, a single row or column."""
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


def _step(nrows, ncols, pivot):
    """One entry in every row up to the pivot (none in the first), three after
    it: the counts rise most at the pivot."""
    lens = np.ones(nrows, np.int64)
    lens[0] = 0 if pivot else 1
    lens[pivot + 1:] = 3
    lens = np.minimum(lens, ncols)
    r = np.repeat(np.arange(nrows), lens)
    within = np.arange(len(r)) - np.repeat(np.cumsum(lens) - lens, lens)
    return synth.from_entries(nrows, ncols, r, (r * 7 + within) % ncols, np.arange(len(r)) + 1.0)


def _check(ctx, A0, mode, seed):
    A = ctx.register(A0)
    B = ctx.permute(A, seed, mode)
    if mode & mx.GRADIENT:
        er, ec, want = oracle.permute_gradient(A0, seed, mode)
    else:
        s_r, s_c = oracle.stream_seeds(seed)
        er = oracle.permutation(A0.nrows, s_r) if mode & mx.ROWS else np.arange(A0.nrows)
        ec = oracle.permutation(A0.ncols, s_c) if mode & mx.COLS else np.arange(A0.ncols)
        want = oracle.permute_csr(A0, er, ec)
    rperm, cperm = ctx.get_permutation(B)
    assert np.array_equal(rperm, er) and np.array_equal(cperm, ec)
    for got, w in zip(ctx.export_csr(B), want):
        assert np.array_equal(got, w)
    ctx.release(B)
    ctx.release(A)


@pytest.mark.parametrize("nrows,ncols", [(1, 1), (1, 9000), (8191, 8193), (8192, 131_072), (8193, 8192),
                                         (131_072, 131_073), (131_073, 5), (300_001, 8000)])
def test_rows_and_columns_together(ctx, nrows, ncols):
    A0 = _step(nrows, ncols, nrows // 2)
    for seed, mode in enumerate((mx.ROWS | mx.COLS, mx.ROWS, mx.COLS, 0, mx.ROWS | mx.COLS | mx.GRADIENT)):
        _check(ctx, A0, mode, seed + 3)


@pytest.mark.parametrize("n,pivot", [(20_000, 0), (20_000, 8191), (20_000, 8192), (20_000, 11_806), (20_000, 19_998),
                                     (150_000, 131_071), (150_000, 131_072), (150_000, 18_926), (262_144, 131_071),
                                     (400_000, 131_071)])
def test_gradient_parts(ctx, n, pivot):
    _check(ctx, _step(n, 9000, pivot), mx.ROWS | mx.COLS | mx.GRADIENT, 5)
    _check(ctx, _step(n, n, pivot), mx.ROWS | mx.COLS | mx.GRADIENT, 6)
