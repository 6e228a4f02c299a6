"""GPU: the longest row, which sizes the column-panel layout, asked for while
the permuted matrix is still being written on another stream, in memory that
held a matrix of shorter rows: matrix_info, set_variant and a panel product
without a synchronization in between, for a permuted matrix and for a
permutation of one."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import TOL, torch_vec

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mx = pytest.importorskip("paper_2308_00106_amd.mxe")

N, LONG = 20_000, 3000


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = mx.Context(0)
    yield c
    c.close()


def _rows(lens, seed):
    rng = np.random.default_rng(seed)
    r = np.repeat(np.arange(N), lens)
    c = rng.integers(0, N, len(r))
    c = synth._dedupe(r, c, N, lambda idx: rng.integers(0, N, len(idx)))
    return synth.from_entries(N, N, r, c, rng.uniform(-1, 1, len(r)))


@pytest.mark.parametrize("times", [1, 2])
def test_longest_row_of_a_matrix_on_its_way(ctx, times):
    short, long = np.full(N, 4), np.full(N, 4)
    long[::400] = LONG
    # the predecessor: as many rows of four entries; its blocks are the next ones taken
    A = ctx.register(_rows(short, 1))
    made = [A]
    for i in range(times):
        made.append(ctx.permute(made[-1], 2 + i))
    assert ctx.matrix_info(made[-1]).max_row == 4
    A0 = _rows(long, 5)
    A = ctx.register(A0)
    torch.cuda.synchronize()
    for h in reversed(made):
        ctx.release(h)
    side = torch.cuda.Stream()
    x = torch_vec(synth.vector(N, 3), torch.float64)
    y = torch.full((N,), float("nan"), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)                  # some milliseconds ahead of the permutation
    made = [A]
    for i in range(times):
        made.append(ctx.permute(made[-1], 7 + i, stream=side))
    B = made[-1]
    assert ctx.matrix_info(B).max_row == LONG
    ctx.set_variant(B, 1, mx.variant(mx.VAR_PANEL))
    ctx.spmv(B, x, y, stream=side)
    side.synchronize()
    rp, col, val = ctx.export_csr(B)
    ref = oracle.spmm(N, rp, col, val, synth.vector(N, 3))
    err = oracle.normalized_error(N, rp, col, val, synth.vector(N, 3), y.cpu().numpy(), ref)
    assert err <= TOL["f64"]
    for h in reversed(made):
        ctx.release(h)


def test_longest_row_first_asked_for_by_set_variant(ctx):
    """set_variant, the first call to need it, on a permutation of a permuted matrix."""
    lens = np.full(N, 4)
    lens[::400] = LONG
    A = ctx.register(_rows(lens, 6))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
    B = ctx.permute(A, 1, stream=side)
    C = ctx.permute(B, 2, stream=side)
    ctx.set_variant(C, 1, mx.variant(mx.VAR_PANEL))
    assert ctx.matrix_info(C).max_row == LONG and ctx.matrix_info(A).max_row == LONG
    side.synchronize()
    for h in (C, B, A):
        ctx.release(h)
