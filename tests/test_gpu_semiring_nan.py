"""GPU: (min, +) where a value and an x add up to NaN (an infinity of each sign,
or a NaN in x): such a term is no path, whatever kernel runs the product, and
takes no other term with it. (or, and): a NaN is not zero. Against a loop over
each row in the accumulation type, bit for bit, for each storage type, k = 1 and
several, both index spaces."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import torch_vec

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mx = pytest.importorskip("paper_2308_00106_amd.mxe")

N = 40_000


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = mx.Context(0)
    yield c
    c.close()


def _matrix():
    A0 = synth.skewed_clustered(N, 2.0, 1.0, 256, 2000.0, 5)
    val = A0.val.copy()
    val[::17] = np.inf
    val[5::23] = -np.inf
    val[3::31] = 0.0
    return synth.CSR(A0.nrows, A0.ncols, A0.row_ptr, A0.col, val)


def _expected(A0, storage, X, semiring):
    acc = np.float64 if storage == "f64" else np.float32
    stored = oracle.stored_values(A0.val, storage).astype(acc)
    rows = np.repeat(np.arange(N), np.diff(A0.row_ptr))
    out = np.full((N, X.shape[1]), np.inf if semiring == mx.SR_MIN_PLUS else 0, acc)
    for q in range(X.shape[1]):
        x = X[:, q].astype(acc)[A0.col]
        if semiring == mx.SR_MIN_PLUS:
            with np.errstate(invalid="ignore"):
                t = stored + x
            np.minimum.at(out[:, q], rows[~np.isnan(t)], t[~np.isnan(t)])
        else:
            out[:, q][rows[(stored != 0) & (x != 0)]] = 1
    return out


VARIANTS = {
    "group": lambda k: mx.variant(mx.VAR_GROUP, 16),
    "slab": lambda k: mx.variant(mx.VAR_SLAB, 1),
    "slab_one_per_cu": lambda k: mx.variant(mx.VAR_SLAB, 4 | mx.SLAB_ONE_PER_CU),
    "panel": lambda k: mx.variant(mx.VAR_PANEL),
}


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("name,k", [("group", 1), ("group", 5), ("slab", 1), ("slab", 2), ("slab", 8),
                                    ("slab_one_per_cu", 1), ("slab_one_per_cu", 3), ("panel", 1)])
def test_terms_that_are_not_numbers(ctx, name, k, storage):
    A0 = _matrix()
    X = synth.vector(N, 4, k=k).reshape(N, k)
    X[::7] = 0.0
    X[3::11] = np.inf
    X[4::13] = -np.inf
    X[5::29] = np.nan
    dt = torch.float64 if storage == "f64" else torch.float32
    A = ctx.register(A0, storage)
    B = ctx.permute(A, 9)
    for semiring in (mx.SR_MIN_PLUS, mx.SR_OR_AND):
        want = _expected(A0, storage, X, semiring)
        for H, flags in ((A, mx.SPACE_PERMUTED), (B, mx.SPACE_ORIGINAL)):
            ctx.set_variant(H, k, VARIANTS[name](k))
            Y = torch.full((N, k), float("nan"), dtype=dt, device="cuda")
            ctx.spmv_semiring(H, semiring, torch_vec(X, dt), Y, flags=flags)
            torch.cuda.synchronize()
            assert np.array_equal(Y.cpu().numpy(), want), (semiring, flags, int((Y.cpu().numpy() != want).sum()))
    ctx.release(B)
    ctx.release(A)
