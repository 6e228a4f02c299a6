"""GPU: calls that take workspaces from the context's device memory leave
independent streams independent. A product queued on one stream behind the same
product and a long wait on another ends before that wait does."""
import pytest

import synth
from gpu_common import TOL, spmv_error, torch_vec

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mx = pytest.importorskip("paper_2308_00106_amd.mxe")

WAIT = 40_000_000                                      # cycles: tenths of a second


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = mx.Context(0)
    yield c
    c.close()


def _independent_streams():
    """Two streams that do not share a hardware queue."""
    a = torch.cuda.Stream()
    t = torch.zeros(1, device="cuda")
    for _ in range(8):
        b = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(a):
            torch.cuda._sleep(WAIT)
            done = torch.cuda.Event()
            done.record()
        with torch.cuda.stream(b):
            t.add_(1)
        b.synchronize()
        apart = not done.query()
        torch.cuda.synchronize()
        if apart:
            return a, b
    pytest.skip("the runtime put every stream on one hardware queue")


@pytest.mark.parametrize("variant", [mx.variant(mx.VAR_GROUP, 8), mx.variant(mx.VAR_PANEL)])
def test_products_of_two_streams_stay_independent(ctx, variant):
    n = 60_000
    A0 = synth.skewed_clustered(n, 2.0, 1.0, 64, 500.0, 3)
    A = ctx.register(A0)
    B = ctx.permute(A, 4)
    ctx.set_variant(B, 1, variant)
    xs = [synth.vector(n, 7 + i) for i in range(2)]
    X = [torch_vec(x, torch.float64) for x in xs]
    Y = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2)]
    ctx.spmv(B, X[0], Y[0], flags=mx.SPACE_ORIGINAL)  # builds the layout
    a, b = _independent_streams()
    for _ in range(3):                                 # workspaces of both streams, in turn
        with torch.cuda.stream(a):
            torch.cuda._sleep(WAIT)
            ctx.spmv(B, X[0], Y[0], flags=mx.SPACE_ORIGINAL, stream=a)
            done = torch.cuda.Event()
            done.record()
        ctx.spmv(B, X[1], Y[1], flags=mx.SPACE_ORIGINAL, stream=b)
        b.synchronize()
        assert not done.query(), "the product waited for the other stream"
        torch.cuda.synchronize()
        for x, y in zip(xs, Y):
            assert spmv_error(A0, x, y.cpu().numpy(), "f64") <= TOL["f64"]
    ctx.release(B)
    ctx.release(A)
