"""GPU: the slab product's reads of X rows and its sums by row: every number of
right-hand sides, rows on no 8 or 16 byte boundary, leading dimensions past the
24-bit offsets, chunks whose entries all lie in one row, in rows of two, or in
rows that cross the 16-lane edges; NaN and infinities stay in the rows that hold
their column."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import TOL, spmv_error, torch_vec

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


def _rows(nrows, ncols, lens, seed):
    rng = np.random.default_rng(seed)
    lens = np.resize(np.asarray(lens, np.int64), nrows)
    r = np.repeat(np.arange(nrows), lens)
    c = rng.integers(0, ncols, len(r))
    c = synth._dedupe(r, c, ncols, lambda idx: rng.integers(0, ncols, len(idx)))
    return synth.from_entries(nrows, ncols, r, c, rng.uniform(-1, 1, len(r)))


MATRICES = {
    "single_entries": lambda: _rows(3001, 900, [1], 1),
    "pairs": lambda: _rows(3001, 900, [2], 2),
    "three_and_five": lambda: _rows(3001, 900, [3, 5, 0, 1], 3),
    "across_edges": lambda: _rows(2000, 900, [15, 2, 30, 1, 17], 4),
    "whole_chunks": lambda: _rows(300, 900, [64, 128, 200, 7], 5),
}
VARIANTS = [mx.variant(mx.VAR_SLAB, 1), mx.variant(mx.VAR_SLAB, 16), mx.variant(mx.VAR_WINDOW, 32)]


def _set(ctx, H, k, v):
    try:
        ctx.set_variant(H, k, v)
    except mx.MxeError:
        return False
    return True


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("name", list(MATRICES))
def test_every_number_of_right_hand_sides(ctx, name, storage):
    A0 = MATRICES[name]()
    A = ctx.register(A0, storage)
    dt = torch.float64 if storage == "f64" else torch.float32
    tol = TOL["f64"] if storage == "f64" else TOL["f32"]      # against the stored values
    for k in range(1, 17):
        for ld, c0 in ((k, 0), (k + 1, 1), (k + 3, 2)):
            X = synth.vector(A0.ncols, 20 + k, k=k).reshape(A0.ncols, k)
            Xf = X.astype(np.float32).astype(np.float64) if storage != "f64" else X
            Xs = torch.full((A0.ncols, ld), float("nan"), dtype=dt, device="cuda")
            Xs[:, c0:c0 + k] = torch_vec(Xf, dt)
            for v in VARIANTS:
                if not _set(ctx, A, k, v):
                    continue
                Y = torch.full((A0.nrows, k), float("nan"), dtype=dt, device="cuda")
                ctx.spmv(A, Xs[:, c0:c0 + k], Y)
                err = spmv_error(A0, Xf, Y.cpu().numpy().astype(np.float64), storage, ref_stored=True)
                assert err <= tol, (name, storage, k, ld, hex(v), err)
    ctx.release(A)


@pytest.mark.parametrize("semiring", [mx.SR_MIN_PLUS, mx.SR_OR_AND])
def test_semirings_of_several_right_hand_sides(ctx, semiring):
    for name in MATRICES:
        A0 = MATRICES[name]()
        A = ctx.register(A0)
        for k in (1, 2, 3, 5, 8, 11, 16):
            X = synth.vector(A0.ncols, k, k=k).reshape(A0.ncols, k)
            X[::5] = 0.0
            if not _set(ctx, A, k, mx.variant(mx.VAR_SLAB, 1)):
                continue
            Y = torch.empty((A0.nrows, k), dtype=torch.float64, device="cuda")
            ctx.spmv_semiring(A, semiring, torch_vec(X, torch.float64), Y)
            ref = oracle.spmm_semiring(semiring, A0.nrows, A0.row_ptr, A0.col, A0.val, X)
            assert np.array_equal(Y.cpu().numpy(), np.asarray(ref).reshape(Y.shape)), (name, k)
        ctx.release(A)


@pytest.mark.parametrize("k", [2, 3, 8])
def test_strides_past_24_bits(ctx, k):
    A0 = _rows(200, 40, [6], 9)
    A = ctx.register(A0, "f32")
    X = torch.zeros((40, (1 << 22) + 1), dtype=torch.float32, device="cuda")
    X[:, 5:5 + k] = torch_vec(synth.vector(40, 1, k=k), torch.float32)
    ctx.set_variant(A, k, mx.variant(mx.VAR_SLAB, 16))
    Y = torch.full((200, k), float("nan"), dtype=torch.float32, device="cuda")
    want = torch.full_like(Y, float("nan"))
    ctx.spmv(A, X[:, 5:5 + k], Y)
    ctx.spmv(A, X[:, 5:5 + k].contiguous(), want)
    assert torch.equal(Y, want)
    ctx.release(A)


@pytest.mark.parametrize("k", [1, 2, 4, 7, 8, 16])
def test_not_finite_x_stays_in_its_rows(ctx, k):
    """Chunks that are not full read row 0 of X for their padding."""
    A0 = MATRICES["three_and_five"]()
    X = synth.vector(A0.ncols, 4, k=k).reshape(A0.ncols, k)
    X[0], X[17] = np.nan, np.inf
    touched = np.zeros(A0.nrows, bool)
    rows = np.repeat(np.arange(A0.nrows), A0.row_lengths())
    touched[rows[(A0.col == 0) | (A0.col == 17)]] = True
    for storage, dt in (("f64", torch.float64), ("f32", torch.float32)):
        A = ctx.register(A0, storage)
        for v in VARIANTS:
            if not _set(ctx, A, k, v):
                continue
            Y = torch.empty((A0.nrows, k), dtype=dt, device="cuda")
            ctx.spmv(A, torch_vec(X, dt), Y)
            bad = ~np.isfinite(Y.cpu().numpy())
            assert np.array_equal(bad.any(1), touched) and np.array_equal(bad.all(1), touched), (k, storage, hex(v))
        ctx.release(A)


# rows of the layout's build: batches of 256 entries cut inside and between rows,
# more than 64 rows (or empty rows) starting in one batch, rows of several batches
BUILDS = {
    "empty_runs": [5] + [0] * 200 + [3, 0, 1],
    "all_single": [1],
    "batch_sized": [256, 256, 0, 255, 1, 257],
    "long_and_short": [1500] + [1] * 90 + [0] * 70 + [513, 2],
    "last_rows_empty": [4] * 40 + [0] * 500,
}


@pytest.mark.parametrize("ncols,unit", [(8192, 1), (8193, 1), (40_001, 1), (500_000, 1), (40_001, 16)])   # 1, 2, 5, 62 and 1 slabs
@pytest.mark.parametrize("name", list(BUILDS))
def test_rows_of_the_layout(ctx, name, ncols, unit):
    """Whole numbers, so that every row's sum is exact."""
    for nrows in (1, 17, 4003):
        rng = np.random.default_rng(nrows + ncols)
        lens = np.resize(np.asarray(BUILDS[name], np.int64), nrows)
        r = np.repeat(np.arange(nrows), lens)
        c = rng.integers(0, ncols, len(r))
        c = synth._dedupe(r, c, ncols, lambda idx: rng.integers(0, ncols, len(idx)))
        A0 = synth.from_entries(nrows, ncols, r, c, rng.integers(-9, 10, len(r)).astype(np.float64))
        x = rng.integers(-9, 10, ncols).astype(np.float64)
        A = ctx.register(A0)
        ctx.set_variant(A, 1, mx.variant(mx.VAR_SLAB, unit))
        Y = torch.full((nrows,), float("nan"), dtype=torch.float64, device="cuda")
        ctx.spmv(A, torch_vec(x, torch.float64), Y)
        torch.cuda.synchronize()
        rows = np.repeat(np.arange(nrows), np.diff(A0.row_ptr))
        want = np.bincount(rows, A0.val * x[A0.col], nrows)
        assert np.array_equal(Y.cpu().numpy(), want)
        ctx.release(A)
