"""GPU: the column-panel product (MXE_VAR_PANEL, one right-hand side) against
the CPU oracle at the edges of its layout: matrices one column short of and
past a whole panel, one panel and many, rectangular ones, chunks whose rows are
nearly all empty or that hold more rows than the row starts kept in LDS, long
rows, strided X and Y. Products stay within the normalized
errors of the other variants (1e-13 FP64, 1e-5 FP32, 1e-2 BF16 against the FP64
oracle); (min, +) and (or, and) match bit for bit in FP64."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import TOL, spmv_error, torch_vec

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mx = pytest.importorskip("paper_2308_00106_amd.mxe")

PANEL = mx.variant(mx.VAR_PANEL)


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = mx.Context(0)
    yield c
    c.close()


def _rows(nrows, ncols, lens, seed):
    """CSR with the given row lengths, distinct uniform columns in each row."""
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens, np.int64)
    r = np.repeat(np.arange(nrows), lens)
    c = rng.integers(0, ncols, len(r))
    c = synth._dedupe(r, c, ncols, lambda idx: rng.integers(0, ncols, len(idx)))
    return synth.from_entries(nrows, ncols, r, c, rng.uniform(-1, 1, len(r)))


def _mostly_empty(n, ncols, seed):
    """Long rows at both ends, nothing between: a chunk with thousands of empty rows."""
    lens = np.zeros(n, np.int64)
    lens[7:57] = 400
    lens[-60:-9] = 391
    return _rows(n, ncols, lens, seed)


CASES = {
    "one_panel": lambda: synth.clustered_n4096(1),
    "8191_columns": lambda: _rows(5000, 8191, np.full(5000, 9), 1),
    "8193_columns": lambda: _rows(9001, 8193, np.full(9001, 7), 2),
    "16385_columns": lambda: _rows(6000, 16385, np.full(6000, 12), 3),
    "many_panels": lambda: _rows(60_011, 90_001, np.random.default_rng(4).integers(0, 40, 60_011), 4),
    "skewed": lambda: synth.skewed_clustered(40_000, 2.0, 1.0, 256, 2000.0, 5),
    "mostly_empty": lambda: _mostly_empty(30_000, 3000, 6),
    "all_but_one_empty": lambda: _rows(4000, 5000, [3000] + [0] * 3999, 7),
    "long_rows": lambda: _rows(700, 20_000, [4095] + [60] * 698 + [4095], 8),
    # more chunks than CUs, in FP32 too
    "several_waves": lambda: _rows(800_000, 300_000, np.full(800_000, 11), 9),
    # 318 panels in FP64, 159 in FP32
    "wide": lambda: _rows(60_000, 2_600_000, np.full(60_000, 12), 10),
}


def _spmv(ctx, H, A0, x, dt, semiring=None, flags=mx.SPACE_PERMUTED):
    y = torch.full((A0.nrows,), float("nan"), dtype=dt, device="cuda")
    if semiring is None:
        ctx.spmv(H, torch_vec(x, dt), y, flags=flags)
    else:
        ctx.spmv_semiring(H, semiring, torch_vec(x, dt), y, flags=flags)
    torch.cuda.synchronize()
    return y


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("name", list(CASES))
def test_panel_product(ctx, name, storage):
    A0 = CASES[name]()
    x = synth.vector(A0.ncols, 2)
    dt = torch.float64 if storage == "f64" else torch.float32
    A = ctx.register(A0, storage)
    B = ctx.permute(A, 3)
    for H, flags in ((A, mx.SPACE_PERMUTED), (B, mx.SPACE_ORIGINAL)):
        ctx.set_variant(H, 1, PANEL)
        y = _spmv(ctx, H, A0, x, dt, flags=flags)
        assert torch.equal(y, _spmv(ctx, H, A0, x, dt, flags=flags))       # repeatable
        err = spmv_error(A0, x, y.cpu().numpy().astype(np.float64), storage)
        assert err <= TOL[storage], (name, storage, err)
    # columns of wider X and Y: strides above one, the neighbours untouched
    X = torch.zeros((A0.ncols, 3), dtype=dt, device="cuda")
    X[:, 1] = torch_vec(x, dt)
    Y = torch.full((A0.nrows, 2), 7.0, dtype=dt, device="cuda")
    ctx.spmv(A, X[:, 1:2], Y[:, 0:1])
    torch.cuda.synchronize()
    assert torch.equal(Y[:, 0], _spmv(ctx, A, A0, x, dt)) and bool((Y[:, 1] == 7.0).all())
    ctx.release(B)
    ctx.release(A)


@pytest.mark.parametrize("semiring", [mx.SR_MIN_PLUS, mx.SR_OR_AND])
@pytest.mark.parametrize("name", ["8193_columns", "skewed", "mostly_empty"])
def test_panel_semirings(ctx, name, semiring):
    A0 = CASES[name]()
    x = synth.vector(A0.ncols, 4)
    x[:: 7] = 0.0
    if semiring == mx.SR_MIN_PLUS:
        x[3] = np.inf
    A = ctx.register(A0)
    ctx.set_variant(A, 1, PANEL)
    y = _spmv(ctx, A, A0, x, torch.float64, semiring)
    ref = oracle.spmm_semiring(semiring, A0.nrows, A0.row_ptr, A0.col, A0.val, x)
    assert np.array_equal(y.cpu().numpy(), ref)
    ctx.release(A)


def test_panel_infinite_x_stays_in_its_rows(ctx):
    """Padding entries multiply by the first x of their panel: an infinity or
    a NaN there reaches only the rows that hold its column."""
    A0 = CASES["8193_columns"]()
    x = synth.vector(A0.ncols, 4)
    x[0], x[8192] = np.inf, np.nan
    A = ctx.register(A0)
    ctx.set_variant(A, 1, PANEL)
    y = _spmv(ctx, A, A0, x, torch.float64).cpu().numpy()
    touched = np.zeros(A0.nrows, bool)
    rows = np.repeat(np.arange(A0.nrows), A0.row_lengths())
    touched[rows[(A0.col == 0) | (A0.col == 8192)]] = True
    assert np.array_equal(~np.isfinite(y), touched)
    ctx.release(A)


def test_panel_declines(ctx):
    """A row longer than half a chunk, runs too short to be worth their
    padding, several right-hand sides, lanes."""
    long_row = ctx.register(_rows(50, 20_000, [9000] + [4] * 49, 1))
    sparse = ctx.register(_rows(1000, 2_000_000, np.full(1000, 3), 1))
    small = ctx.register(synth.clustered_n4096(1))
    for h, k, v in ((long_row, 1, PANEL), (sparse, 1, PANEL), (small, 2, PANEL)):
        with pytest.raises(mx.MxeError) as e:
            ctx.set_variant(h, k, v)
        assert e.value.status == mx.ERR_UNSUPPORTED
    with pytest.raises(mx.MxeError) as e:
        ctx.set_variant(small, 1, mx.variant(mx.VAR_PANEL, 1))
    assert e.value.status == mx.ERR_INVALID_ARG
    for h in (long_row, sparse, small):
        ctx.release(h)


def test_panel_tuned_matrix_in_a_batch(ctx):
    """A batch runs a panel item on slab units; the product stays the item's own."""
    A0 = CASES["many_panels"]()
    x = synth.vector(A0.ncols, 2)
    A = ctx.register(A0)
    ctx.set_variant(A, 1, PANEL)
    y = torch.full((A0.nrows,), float("nan"), dtype=torch.float64, device="cuda")
    ctx.spmv_batch([(A, torch_vec(x, torch.float64), y)])
    torch.cuda.synchronize()
    assert spmv_error(A0, x, y.cpu().numpy(), "f64") <= TOL["f64"]
    ctx.release(A)


def test_panel_product_in_a_graph(ctx):
    """The product captured in a graph: every replay equals the eager result,
    with eager work and new inputs in between."""
    A0 = CASES["many_panels"]()
    A = ctx.register(A0)
    ctx.set_variant(A, 1, PANEL)
    x = torch_vec(synth.vector(A0.ncols, 2), torch.float64)
    y = torch.empty(A0.nrows, dtype=torch.float64, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx.spmv(A, x, y)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ctx.spmv(A, x, y)
    for i in range(4):
        x.copy_(torch_vec(synth.vector(A0.ncols, 20 + i), torch.float64))
        want = torch.empty_like(y)
        ctx.spmv(A, x, want)
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want), i
    del g
    ctx.release(A)
