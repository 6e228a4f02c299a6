"""GPU: eager products on one stream while another stream is captured. Neither
the library's reuse of memory, which asks whether other streams' blocks are still
in use, nor its reuse of events, some of which marked uses of matrices in an
earlier capture, ends the capture."""
import pytest

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


def test_eager_products_beside_a_capture(ctx):
    n = 30_000
    A0 = synth.skewed_clustered(n, 2.0, 1.0, 64, 500.0, 3)
    A = ctx.register(A0)
    x = synth.vector(n, 5)
    X = torch_vec(x, torch.float64)
    captured, eager, third = (torch.cuda.Stream() for _ in range(3))
    group = mx.variant(mx.VAR_GROUP, 8)

    def matrix(seed):
        B = ctx.permute(A, seed)
        ctx.set_variant(B, 1, group)
        return B

    # matrices used in a capture of the stream and released: their events are free
    for seed in range(6):
        B = matrix(seed)
        Y = torch.empty_like(X)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=captured):
            ctx.spmv(B, X, Y)
        g.replay()
        torch.cuda.synchronize()
        assert spmv_error_permuted(ctx, A0, B, x, Y) <= TOL["f64"]
        del g
        ctx.release(B)
    B, C = matrix(10), matrix(11)
    Y, Z = torch.empty_like(X), torch.empty((8, n), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    # blocks of a third stream, still in use, lie where the eager stream looks
    with torch.cuda.stream(third):
        torch.cuda._sleep(20_000_000)
    for i in range(3):
        ctx.spmv(C, X, Z[i], flags=mx.SPACE_ORIGINAL, stream=third)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=captured):
        ctx.spmv(B, X, Y, flags=mx.SPACE_ORIGINAL)
        for i in range(3, 8):
            ctx.spmv(C, X, Z[i], flags=mx.SPACE_ORIGINAL, stream=eager)
        ctx.spmv(B, X, Y, flags=mx.SPACE_ORIGINAL)
    for _ in range(3):
        Y.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for y in (Y, *Z):
            assert spmv_error(A0, x, y.cpu().numpy(), "f64") <= TOL["f64"]
    del g
    for h in (C, B, A):
        ctx.release(h)


def spmv_error_permuted(ctx, A0, B, x, y):
    Bo = synth.CSR(A0.nrows, A0.ncols, *ctx.export_csr(B))
    return spmv_error(Bo, x, y.cpu().numpy(), "f64")
