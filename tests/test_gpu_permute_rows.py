"""GPU: permuted CSR and gradient shuffles at the edges of their kernels, bit for
bit against the oracle: rows around the lengths where the ranking of a row's new
columns changes (32 entries, 512, 1024) and groups of rows that fill a
wavefront's stage exactly, overflow it or are empty, few rows and many; column counts of more than
a million entries, with one column per bucket edge, heavy columns and fewer
columns than a bucket."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import expected_export

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


def _rows(ncols, lens, seed, low=0, high=None):
    """CSR with the given row lengths, distinct columns in [low, high) in each row."""
    rng = np.random.default_rng(seed)
    high = ncols if high is None else high
    c = [np.sort(rng.permutation(high - low)[:n]) + low for n in lens]
    r = np.repeat(np.arange(len(lens)), lens)
    return synth.from_entries(len(lens), ncols, r, np.concatenate(c), rng.uniform(-1, 1, len(r)))


ROWS = {
    "around_pairs": lambda: _rows(3000, [30, 31, 32, 33, 34, 0, 1, 2] * 20, 1),
    "stage_exact": lambda: _rows(3000, [32] * 16 + [256, 256] + [0] * 14 + [33] * 15 + [17] + [512] * 16, 2),
    "around_stage": lambda: _rows(3000, [511, 1, 512, 0, 513, 7, 1023, 1024, 1025, 2, 600, 400, 100, 12, 1, 0, 3], 3),
    "heavy_band": lambda: _rows(20_000, [8] * 500 + [256] * 200 + [8] * 300, 4),
    "narrow_columns": lambda: _rows(100_000, [200, 3, 90, 512, 41, 0, 0, 33] * 9, 5, 777, 1400),
    "all_columns": lambda: _rows(64, [64] * 50, 6),
    "two_columns": lambda: _rows(2, [2, 0, 1, 2, 2] * 30, 7),
}


def _many_rows(nrows):
    """Enough rows for groups of long ones to be moved by a launch of their
    own: in the middle, one row past the stage, and the last, partial group."""
    rng = np.random.default_rng(nrows)
    lens = rng.integers(0, 4, nrows)
    lens[160:176] = 40
    lens[176:192] = 32                                     # exactly the stage
    lens[5000:5004] = [600, 1025, 512, 1]
    lens[-3:] = 300
    r = np.repeat(np.arange(nrows), lens)
    c = rng.integers(0, 5000, len(r))
    c = synth._dedupe(r, c, 5000, lambda idx: rng.integers(0, 5000, len(idx)))
    return synth.from_entries(nrows, 5000, r, c, rng.uniform(-1, 1, len(r)))


for _n in (131_071, 131_072, 131_075):
    ROWS[f"many_{_n}"] = lambda n=_n: _many_rows(n)


@pytest.mark.parametrize("mode", [mx.ROWS | mx.COLS, mx.COLS, mx.ROWS, mx.ROWS | mx.COLS | mx.GRADIENT])
@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("name", list(ROWS))
def test_rows_of_every_length(ctx, name, storage, mode):
    A0 = ROWS[name]()
    A = ctx.register(A0, storage)
    B = ctx.permute(A, 11, mode)
    rperm, cperm = ctx.get_permutation(B)
    for got, want in zip(ctx.export_csr(B), expected_export(A0, rperm, cperm, storage)):
        assert np.array_equal(got, want)
    ctx.release(B)
    ctx.release(A)


def _columns(nrows, ncols, counts_of, seed):
    """CSR whose column j holds counts_of[j] entries, in random distinct rows."""
    rng = np.random.default_rng(seed)
    c = np.repeat(np.arange(ncols), counts_of)
    start = np.repeat(rng.integers(0, nrows, ncols), counts_of)
    within = np.arange(len(c)) - np.repeat(np.cumsum(counts_of) - counts_of, counts_of)
    return synth.from_entries(nrows, ncols, (start + within) % nrows, c, np.ones(len(c)))


def _bucket_edges():
    rng = np.random.default_rng(8)
    n = rng.integers(90, 110, 3 * 4096 + 1)
    n[[0, 4095, 4096, 8191, 8192, 12288]] = [3, 9001, 1, 0, 7000, 5]
    return n


def _heavy_columns():
    n = np.full(20_000, 45)
    n[5000:5100] = 9000                                    # several workgroups share this bucket
    return n


COLUMNS = {
    "bucket_edges": lambda: _columns(9100, 3 * 4096 + 1, _bucket_edges(), 1),
    "heavy_columns": lambda: _columns(10_000, 20_000, _heavy_columns(), 2),
    "few_columns": lambda: _columns(30_000, 50, np.random.default_rng(3).integers(20_000, 25_000, 50), 3),
    "just_below": lambda: _columns(9000, 4000, np.full(4000, 262), 4),          # 1,048,000 entries
    "just_above": lambda: _columns(9000, 4000, np.full(4000, 263), 5),          # 1,052,000
    "many_columns": lambda: _columns(400, 5_000_000, (np.arange(5_000_000) % 5 == 0).astype(int) + (np.arange(5_000_000) > 4_900_000), 6),
}


@pytest.mark.parametrize("name", list(COLUMNS))
def test_column_gradient_of_many_entries(ctx, name):
    A0 = COLUMNS[name]()
    A = ctx.register(A0)
    B = ctx.permute(A, 13, mx.COLS | mx.GRADIENT)
    er, ec, want = oracle.permute_gradient(A0, 13, oracle.COLS)
    rperm, cperm = ctx.get_permutation(B)
    assert np.array_equal(rperm, er) and np.array_equal(cperm, ec)
    for got, w in zip(ctx.export_csr(B), want):
        assert np.array_equal(got, w)
    ctx.release(B)
    ctx.release(A)
