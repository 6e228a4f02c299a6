"""GPU: the context's reused device memory. Products that take workspaces
(original index space, merge path) from several streams and threads at once,
matrices registered, permuted, multiplied and released in turn on different
streams, a captured product replayed between eager ones: every result equals the
one computed alone, bit for bit."""
import threading

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


def _matrix(ctx, n, seed, k):
    A = ctx.register(synth.skewed_clustered(n, 2.0, 1.0, 64, 500.0, seed))
    B = ctx.permute(A, seed)
    ctx.set_variant(B, k, mx.variant(mx.VAR_MERGE if k <= 4 else mx.VAR_GROUP, 0 if k <= 4 else 8))
    return A, B


def test_workspaces_of_streams_and_threads(ctx):
    jobs = []
    for i, (n, k) in enumerate([(30_000, 1), (30_000, 3), (70_001, 2), (5000, 4), (70_001, 8)]):
        A, B = _matrix(ctx, n, 20 + i, k)
        X = torch_vec(synth.vector(n, 3 + i, k=k), torch.float64)
        ref = torch.empty((n, k), dtype=torch.float64, device="cuda")
        ctx.spmv(B, X, ref, flags=mx.SPACE_ORIGINAL)
        jobs.append((A, B, X, ref))
    torch.cuda.synchronize()
    errors = []

    def work(j, stream):
        A, B, X, ref = jobs[j]
        outs = [torch.full_like(ref, float("nan")) for _ in range(20)]
        torch.cuda.synchronize()
        for Y in outs:
            ctx.spmv(B, X, Y, flags=mx.SPACE_ORIGINAL, stream=stream)
        stream.synchronize()
        if not all(torch.equal(Y, ref) for Y in outs):
            errors.append(j)

    threads = [threading.Thread(target=work, args=(j % 5, s))
               for j, s in enumerate([torch.cuda.default_stream()] + [torch.cuda.Stream() for _ in range(9)])]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for A, B, _, _ in jobs:
        ctx.release(B)
        ctx.release(A)


def test_matrices_in_turn_on_different_streams(ctx):
    streams = [torch.cuda.default_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    rng = np.random.default_rng(5)
    kept = []
    for i in range(24):
        n = int(rng.choice([4096, 9000, 20_000, 20_500]))
        s = streams[i % 3]
        A0 = synth.skewed_clustered(n, 2.0, 1.0, 64, 300.0, i)
        A = ctx.register(A0)
        x = synth.vector(n, i)
        X = torch_vec(x, torch.float64)
        Y = torch.empty(n, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        B = ctx.permute(A, i, stream=s)
        ctx.set_variant(B, 1, mx.variant(mx.VAR_SLAB, 4) if i % 2 else mx.variant(mx.VAR_MERGE))
        ctx.spmv(B, X, Y, flags=mx.SPACE_ORIGINAL, stream=s)
        ctx.release(B)
        ctx.release(A)
        kept.append((A0, x, Y))
    torch.cuda.synchronize()
    for A0, x, Y in kept:
        assert spmv_error(A0, x, Y.cpu().numpy(), "f64") <= TOL["f64"]


def test_captured_product_between_eager_ones(ctx):
    A, B = _matrix(ctx, 40_000, 9, 2)
    X = torch_vec(synth.vector(40_000, 1, k=2), torch.float64)
    Y = torch.empty((40_000, 2), dtype=torch.float64, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx.spmv(B, X, Y, flags=mx.SPACE_ORIGINAL)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ctx.spmv(B, X, Y, flags=mx.SPACE_ORIGINAL)
    for i in range(5):
        X.copy_(torch_vec(synth.vector(40_000, 30 + i, k=2), torch.float64))
        Y.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()                                         # on the current stream, eager ones on s and here
        want, here = torch.empty_like(Y), torch.empty_like(Y)
        ctx.spmv(B, X, want, flags=mx.SPACE_ORIGINAL, stream=s)
        ctx.spmv(B, X, here, flags=mx.SPACE_ORIGINAL)
        torch.cuda.synchronize()
        assert torch.equal(Y, want) and torch.equal(here, want), i
    del g
    ctx.release(B)
    ctx.release(A)
