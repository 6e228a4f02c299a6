"""GPU: the allocation-free batch captured in a graph, one of its stated uses.
Its descriptor table is built in host memory that is gone when the call returns,
so the graph has to hold the table itself. Every replay equals the eager batch,
with new X contents, eager batches (which rewrite the shared table) and other
host work in between; one item, and more pieces than one store launch takes."""
import numpy as np
import pytest

import synth
from gpu_common import torch_vec

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


@pytest.mark.parametrize("count", [1, 2, 40])
def test_captured_batch_replays(ctx, count):
    ks = [1 + i % 5 for i in range(count)]
    mats, handles = [], []
    for i in range(count):
        A0 = synth.skewed_clustered(3000 + 97 * i, 2.0, 1.0, 64, 300.0, i)
        A = ctx.register(A0, "f32")
        B = ctx.permute(A, i)
        ctx.release(A)
        for k in set(ks):
            ctx.set_variant(B, k, mx.variant(mx.VAR_SLAB, 4) if i % 2 else mx.variant(mx.VAR_GROUP, 8))
        mats.append(A0)
        handles.append(B)
    X = [torch.zeros((A0.ncols, k), dtype=torch.float32, device="cuda") for A0, k in zip(mats, ks)]
    Y = [torch.zeros((A0.nrows, k), dtype=torch.float32, device="cuda") for A0, k in zip(mats, ks)]
    W = [torch.zeros_like(y) for y in Y]
    ctx.spmv_batch(list(zip(handles, X, W)))           # tunes nothing more, builds the layouts
    ctx.spmv_batch_noalloc(list(zip(handles, X, W)))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    print(f"capture of {count} items", flush=True)
    with torch.cuda.graph(g, stream=s):
        ctx.spmv_batch_noalloc(list(zip(handles, X, Y)), stream=s)
    held = [np.full(1 << 16, 0xA5, np.uint8) for _ in range(64)]      # host memory taken again
    for rep in range(3):
        for i, (x, k) in enumerate(zip(X, ks)):
            x.copy_(torch_vec(synth.vector(x.shape[0], 10 * rep + i, k=k).reshape(x.shape), torch.float32))
        ctx.spmv_batch_noalloc(list(zip(handles, X, W)))
        for y in Y:
            y.fill_(float("nan"))
        torch.cuda.synchronize()
        print(f"replay {rep}", flush=True)
        g.replay()
        torch.cuda.synchronize()
        for i, (y, w) in enumerate(zip(Y, W)):
            assert torch.equal(y, w), (rep, i)
    assert len(held) == 64
    del g
    for h in handles:
        ctx.release(h)
