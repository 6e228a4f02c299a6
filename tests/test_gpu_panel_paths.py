"""GPU: a matrix tuned or set to the column panels on every path a product can
take (single, batch, plan, allocation-free batch, serving), choices made before
the panels kept by its batches, and the slab variants accepted wherever the
tests of the slab product count on them."""
import numpy as np
import pytest

import synth
from gpu_common import TOL, spmv_error, torch_vec
from test_gpu_slab_rows import MATRICES, VARIANTS

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


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
def test_slab_variants_are_accepted(ctx, storage):
    """Only the window may decline, where it finds no LDS."""
    for name, make in MATRICES.items():
        A = ctx.register(make(), storage)
        for k in range(1, 17):
            for v in VARIANTS:
                if v & 0xf00 == mx.VAR_SLAB:
                    ctx.set_variant(A, k, v)
                    continue
                try:
                    ctx.set_variant(A, k, v)
                except mx.MxeError as e:
                    assert e.status == mx.ERR_UNSUPPORTED, (name, k)
        ctx.release(A)


def test_a_forced_panel_product_builds_its_layout(ctx):
    A0 = synth.skewed_clustered(50_000, 2.0, 1.0, 64, 500.0, 2)
    A = ctx.register(A0, "f32")
    ctx.set_variant(A, 1, PANEL)
    held = ctx.matrix_info(A).device_bytes
    y = torch.empty(A0.nrows, dtype=torch.float32, device="cuda")
    ctx.spmv(A, torch_vec(synth.vector(A0.ncols, 1), torch.float32), y)
    assert ctx.matrix_info(A).device_bytes - held >= 8 * A0.nnz
    ctx.release(A)


def test_panel_tuned_matrix_on_every_path(ctx):
    A0 = synth.skewed_clustered(1_200_000, 2.0, 1.0, 256, 2000.0, 5)
    f32, n = torch.float32, A0.nrows
    A = ctx.register(A0, "f32")
    B = ctx.permute(A, 2)
    assert ctx.tune(B, 1) == PANEL
    xs = [synth.vector(n, 3 + i) for i in range(4)]
    X = [torch_vec(x, f32) for x in xs]
    Bo = synth.CSR(A0.nrows, A0.ncols, *ctx.export_csr(B))

    def right(i, y):
        return spmv_error(Bo, xs[i], y.cpu().numpy().astype(np.float64), "f32") <= TOL["f32"]

    alone, batch, noalloc, plan = (torch.full((n,), float("nan"), dtype=f32, device="cuda") for _ in range(4))
    ctx.spmv(B, X[0], alone)
    ctx.spmv_batch([(B, X[0], batch)])
    ctx.spmv_batch_noalloc([(B, X[0], noalloc)])
    p = ctx.batch_create([(B, X[0], plan)])
    ctx.batch_launch(p)
    torch.cuda.synchronize()
    ctx.batch_destroy(p)
    assert torch.equal(batch, noalloc) and torch.equal(batch, plan)
    assert right(0, alone) and right(0, batch)
    for merge, batch_items in ((1, 1), (8, 8)):
        ctx.serve_start(streams=2, max_inflight=16, max_batch=batch_items, max_merge_k=merge)
        Y = [torch.full((n,), float("nan"), dtype=f32, device="cuda") for _ in range(9)]
        torch.cuda.synchronize()
        ctx.wait(ctx.submit(B, X[0], Y[8]))                  # a lone request is the product alone
        for t in [ctx.submit(B, X[i % 4], Y[i]) for i in range(8)]:
            ctx.wait(t)
        ctx.serve_stop()
        torch.cuda.synchronize()
        assert torch.equal(Y[8], alone)
        assert all(right(i % 4, Y[i]) for i in range(8))
        if merge == 1:
            assert torch.equal(Y[0], alone) and torch.equal(Y[4], alone)
    ctx.release(B)
    ctx.release(A)


@pytest.mark.parametrize("before", [mx.variant(mx.VAR_SLAB, 4), mx.variant(mx.VAR_GROUP, 16), None])
def test_batches_keep_the_choice_made_before_the_panels(ctx, before):
    A0 = synth.skewed_clustered(70_000, 2.0, 1.0, 64, 500.0, 6)
    x = synth.vector(A0.ncols, 7)
    X = torch_vec(x, torch.float64)
    A = ctx.register(A0)
    first, second, third = (torch.full((A0.nrows,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3))
    if before is None:
        ctx.tune(A, 1)
    else:
        ctx.set_variant(A, 1, before)
    ctx.spmv_batch([(A, X, first)])
    ctx.set_variant(A, 1, PANEL)
    ctx.spmv_batch([(A, X, second)])
    ctx.spmv(A, X, third)
    torch.cuda.synchronize()
    assert torch.equal(first, second)
    for y in (second, third):
        assert spmv_error(A0, x, y.cpu().numpy(), "f64") <= TOL["f64"]
    ctx.release(A)
