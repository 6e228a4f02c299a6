"""python child.py SHIM NAME: one case of the library without device memory to
give, in a process whose hipMallocAsync goes through the shim. Prints 'ok'."""
import ctypes
import os
import sys

shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)     # before the HIP runtime
shim.shim_fail.argtypes = [ctypes.c_size_t, ctypes.c_int]
sys.path[:0] = [os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__)))),
                os.path.dirname(os.path.dirname(os.path.abspath(__file__)))]

import numpy as np                                           # noqa: E402
import torch                                                 # noqa: E402

import synth                                                 # noqa: E402
from gpu_common import TOL, spmv_error, torch_vec            # noqa: E402
from paper_2308_00106_amd import mxe as mx                   # noqa: E402

mx.load_library()
runtime = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
assert shim.shim_runtime(runtime.encode()), runtime
MiB = 1 << 20


def product(ctx, B, A0, seed, flags=mx.SPACE_ORIGINAL, dt=torch.float64):
    x = synth.vector(A0.ncols, seed)
    y = torch.full((A0.nrows,), float("nan"), dtype=dt, device="cuda")
    ctx.spmv(B, torch_vec(x, dt), y, flags=flags)
    torch.cuda.synchronize()
    return x, y


def room_from_another_context():
    """A failed allocation gets back what another context holds unused, and the
    call goes on as if nothing had happened."""
    A0 = synth.skewed_clustered(300_000, 2.0, 1.0, 64, 500.0, 1)
    with mx.Context(0) as one, mx.Context(0) as two:
        A = one.register(A0)
        B = one.permute(A, 2)
        one.set_variant(B, 1, mx.variant(mx.VAR_GROUP, 8))
        product(one, B, A0, 3)
        one.release(B)                                       # about 60 MB unused
        free0 = torch.cuda.mem_get_info()[0]
        shim.shim_fail(4 * MiB, 1)
        A2 = two.register(A0)
        assert shim.shim_failed() == 1
        assert torch.cuda.mem_get_info()[0] > free0 - 16 * MiB
        B2 = two.permute(A2, 2)
        two.set_variant(B2, 1, mx.variant(mx.VAR_GROUP, 8))
        x, y = product(two, B2, A0, 4)
        assert spmv_error(A0, x, y.cpu().numpy(), "f64") <= TOL["f64"]
        shim.shim_fail(4 * MiB, -1)                          # no memory at all: reported, nothing lost
        try:
            two.permute(A2, 5)
            raise AssertionError("a permutation without memory")
        except mx.MxeError as e:
            assert e.status == mx.ERR_OUT_OF_MEMORY
        shim.shim_fail(0, 0)
        x, y = product(two, B2, A0, 6)
        assert spmv_error(A0, x, y.cpu().numpy(), "f64") <= TOL["f64"]
        two.release(two.permute(A2, 5))


def tuning_without_room_for_the_panels():
    """The tuner tries the column panels last; without room for their layout, or
    for their products alone, it chooses among the others."""
    A0 = synth.skewed_clustered(300_000, 2.0, 1.0, 64, 500.0, 1)
    # budget: exact sizes. FP64: no room for the layout's values; BF16: for the
    # workspace of FP32 products, larger than every other variant's largest block
    for storage, largest in (("f64", 8 * A0.nnz), ("bf16", 4 * A0.nnz)):
        dt = torch.float64 if storage == "f64" else torch.float32
        with mx.Context(0, budget_bytes=1 << 34) as ctx:
            A = ctx.register(A0, storage)
            B = ctx.permute(A, 2)
            shim.shim_fail(largest + 8192, -1)
            x, y = product(ctx, B, A0, 3, dt=dt)
            assert shim.shim_failed() > 0
            assert spmv_error(A0, x, y.cpu().numpy().astype(np.float64), storage) <= TOL[storage]
            assert ctx.tune(B, 1) & 0xf00 != mx.VAR_PANEL
            held = ctx.matrix_info(B).device_bytes
            shim.shim_fail(0, 0)
            ctx.set_variant(B, 1, mx.variant(mx.VAR_PANEL))  # it was the memory alone
            x, y = product(ctx, B, A0, 4, dt=dt)
            assert spmv_error(A0, x, y.cpu().numpy().astype(np.float64), storage) <= TOL[storage]
            assert ctx.matrix_info(B).device_bytes > held
            ctx.release(B)
            ctx.release(A)


def products_without_a_workspace():
    """A panel product without room for its workspace: the same bits, over each
    semiring, with infinities and NaN in x, a strided X and Y, and so on the next
    call with room. A new stream finds no block of the context's to reuse."""
    from test_gpu_panel import CASES
    for name in ("one_panel", "8193_columns", "many_panels", "mostly_empty", "all_but_one_empty", "long_rows",
                 "several_waves", "wide"):
        A0 = CASES[name]()
        for storage in ("f64", "f32", "bf16"):
            dt = torch.float64 if storage == "f64" else torch.float32
            x = synth.vector(A0.ncols, 2)
            x[:: 7] = 0.0
            x[0], x[A0.ncols // 2], x[-1] = np.inf, np.nan, -np.inf
            X = torch.zeros((A0.ncols, 3), dtype=dt, device="cuda")
            X[:, 1] = torch_vec(x, dt)
            with mx.Context(0) as ctx:
                A = ctx.register(A0, storage)
                ctx.set_variant(A, 1, mx.variant(mx.VAR_PANEL))
                for semiring in (mx.SR_PLUS_TIMES, mx.SR_MIN_PLUS, mx.SR_OR_AND):
                    Y = torch.full((3, A0.nrows, 2), 7.0, dtype=dt, device="cuda")
                    side = torch.cuda.Stream()
                    torch.cuda.synchronize()
                    ctx.spmv_semiring(A, semiring, X[:, 1:2], Y[0][:, 0:1])
                    shim.shim_fail(0, -1)
                    ctx.spmv_semiring(A, semiring, X[:, 1:2], Y[1][:, 0:1], stream=side)
                    assert shim.shim_failed() > 0
                    shim.shim_fail(0, 0)
                    ctx.spmv_semiring(A, semiring, X[:, 1:2], Y[2][:, 0:1], stream=side)
                    torch.cuda.synchronize()
                    bits = Y.view(torch.int64 if storage == "f64" else torch.int32)
                    for other in (1, 2):
                        assert torch.equal(bits[0], bits[other]), (name, storage, semiring, other)
                    assert bool((Y[:, :, 1] == 7.0).all())
            print(name, storage, flush=True)


def tuned_panels_without_room_for_the_layout():
    """A matrix made again with the seed it was tuned for, whose panel layout is
    not built yet and finds no room, on the device or in the budget: the product
    runs all the same. A forced choice says what is missing."""
    A0 = synth.skewed_clustered(1_200_000, 2.0, 1.0, 256, 2000.0, 5)
    csr, f32 = 8 * A0.nnz, torch.float32
    budget = 16 * csr                                        # for every layout of the tuning at once
    with mx.Context(0, budget_bytes=budget) as ctx:
        A = ctx.register(A0, "f32")
        B = ctx.permute(A, 2)
        assert ctx.tune(B, 1) == mx.variant(mx.VAR_PANEL)
        x, y = product(ctx, B, A0, 3, dt=f32)
        for semiring in (mx.SR_PLUS_TIMES, mx.SR_MIN_PLUS):
            ctx.release(B)
            B = ctx.permute(A, 2)                            # the same key; its layout is to be built
            held = ctx.matrix_info(B).device_bytes
            shim.shim_fail(1 << 31, 1)                       # empties the pool of the last one's layout
            ctx.probe_gather(1 << 31, 1 << 20)
            assert shim.shim_failed() == 1
            Y = [torch.empty_like(y) for _ in range(2)]
            side = torch.cuda.Stream()
            torch.cuda.synchronize()
            shim.shim_fail(0, -1)
            ctx.spmv_semiring(B, semiring, torch_vec(x, f32), Y[0], stream=side)
            assert shim.shim_failed() > 0 and ctx.matrix_info(B).device_bytes == held
            shim.shim_fail(0, 0)
            ctx.spmv_semiring(B, semiring, torch_vec(x, f32), Y[1], stream=side)
            torch.cuda.synchronize()
            assert ctx.matrix_info(B).device_bytes > held
            if semiring == mx.SR_MIN_PLUS:
                assert torch.equal(Y[0], Y[1])
            else:
                Bo = synth.CSR(A0.nrows, A0.ncols, *ctx.export_csr(B))
                for got in Y:
                    assert spmv_error(Bo, x, got.cpu().numpy().astype(np.float64), "f32") <= TOL["f32"]
        ctx.release(B)                                       # the budget used up but for half a layout
        B = ctx.permute(A, 2)
        n = A0.nrows
        left = budget - sum(ctx.matrix_info(m).device_bytes for m in (A, B)) - csr // 2
        while left > 8 * n:
            nnz = min((left - 4 * (n + 1)) // 12, 20 * n)
            rp = np.minimum(np.arange(n + 1, dtype=np.int64) * 20, nnz).astype(np.int32)
            M = ctx.register_matrix(n, n, rp, np.arange(nnz, dtype=np.int32) % 20, np.ones(nnz))
            left -= ctx.matrix_info(M).device_bytes
        held = ctx.matrix_info(B).device_bytes
        z = torch.empty_like(y)
        ctx.spmv(B, torch_vec(x, f32), z)
        torch.cuda.synchronize()
        assert ctx.matrix_info(B).device_bytes == held
        assert spmv_error(Bo, x, z.cpu().numpy().astype(np.float64), "f32") <= TOL["f32"]
        ctx.set_variant(B, 1, mx.variant(mx.VAR_PANEL))
        try:
            ctx.spmv(B, torch_vec(x, f32), z)
            raise AssertionError("a forced layout without room")
        except mx.MxeError as e:
            assert e.status == mx.ERR_BUDGET


def batches_of_panel_matrices_without_room_for_slabs():
    """A matrix tuned to the column panels, whose slab layouts find no room in the
    budget or on the device any more: batches, the allocation-free ones too, and
    serving rounds run it as row tiles."""
    A0 = synth.skewed_clustered(1_200_000, 2.0, 1.0, 256, 2000.0, 5)
    csr, f32 = 8 * A0.nnz, torch.float32
    budget = 16 * csr
    with mx.Context(0, budget_bytes=budget) as ctx:
        A = ctx.register(A0, "f32")
        B = ctx.permute(A, 2)
        assert ctx.tune(B, 1) == mx.variant(mx.VAR_PANEL)
        x, y = product(ctx, B, A0, 3, dt=f32)
        Bo = synth.CSR(A0.nrows, A0.ncols, *ctx.export_csr(B))
        X = torch_vec(x, f32)

        def batches():
            Y = torch.full((2, A0.nrows), float("nan"), dtype=f32, device="cuda")
            ctx.spmv_batch([(B, X, Y[0])])
            ctx.spmv_batch_noalloc([(B, X, Y[1])])
            torch.cuda.synchronize()
            assert torch.equal(Y[0], Y[1])
            assert spmv_error(Bo, x, Y[0].cpu().numpy().astype(np.float64), "f32") <= TOL["f32"]

        held = ctx.matrix_info(B).device_bytes
        shim.shim_fail(1 << 31, 1)                           # empties the pool
        ctx.probe_gather(1 << 31, 1 << 20)
        shim.shim_fail(csr // 4, -1)
        batches()
        batches()
        assert shim.shim_failed() > 0 and ctx.matrix_info(B).device_bytes == held
        shim.shim_fail(0, 0)
        n = A0.nrows                                         # the budget used up but for half a layout
        left = budget - sum(ctx.matrix_info(m).device_bytes for m in (A, B)) - csr // 2
        while left > 8 * n:
            nnz = min((left - 4 * (n + 1)) // 12, 20 * n)
            rp = np.minimum(np.arange(n + 1, dtype=np.int64) * 20, nnz).astype(np.int32)
            M = ctx.register_matrix(n, n, rp, np.arange(nnz, dtype=np.int32) % 20, np.ones(nnz))
            left -= ctx.matrix_info(M).device_bytes
        held = ctx.matrix_info(B).device_bytes
        batches()
        plan = ctx.batch_create([(B, X, y)])
        ctx.batch_launch(plan)
        torch.cuda.synchronize()
        assert spmv_error(Bo, x, y.cpu().numpy().astype(np.float64), "f32") <= TOL["f32"]
        ctx.batch_destroy(plan)
        assert ctx.matrix_info(B).device_bytes == held


def serving_within_the_budget():
    """A lone request on a panel matrix takes its workspace where the budget has
    room for it beside the vectors, and runs without it, same bits, where not. The
    shim refuses blocks of the workspace's size: it counts who asks for them."""
    A0 = synth.skewed_clustered(200_000, 2.0, 1.0, 64, 500.0, 1)
    n, panel = A0.nrows, mx.variant(mx.VAR_PANEL)
    x = synth.vector(n, 3)
    X = torch_vec(x, torch.float64)
    with mx.Context(0) as ctx:
        A = ctx.register(A0)
        B = ctx.permute(A, 2)
        ctx.set_variant(B, 1, panel)
        want = torch.empty_like(X)
        ctx.spmv(B, X, want, flags=mx.SPACE_ORIGINAL)
        torch.cuda.synchronize()
        resident = sum(ctx.matrix_info(m).device_bytes for m in (A, B))
    vectors, workspace = 16 * n, 8 * A0.nnz                  # and its padding
    for budget, asks in ((0, True), (resident + vectors + 2 * workspace, True), (resident + vectors + 1024, False),
                         (resident + vectors + workspace // 2, False)):
        with mx.Context(0, budget_bytes=budget) as ctx:
            A = ctx.register(A0)
            B = ctx.permute(A, 2)
            ctx.set_variant(B, 1, panel)
            y = torch.empty_like(X)
            ctx.spmv(B, X, y, flags=mx.SPACE_ORIGINAL)       # builds the layout
            torch.cuda.synchronize()
            ctx.serve_start(streams=2, max_inflight=8, max_batch=4, max_merge_k=1)
            shim.shim_fail(workspace, -1)
            Y = torch.full((6, n), float("nan"), dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            for t in [ctx.submit(B, X, Y[i], flags=mx.SPACE_ORIGINAL) for i in range(6)]:
                ctx.wait(t)
            assert (shim.shim_failed() > 0) == asks, (budget, shim.shim_failed())
            shim.shim_fail(0, 0)
            ctx.serve_stop()
            torch.cuda.synchronize()
            assert all(torch.equal(row, want) for row in Y)


if __name__ == "__main__":
    globals()[sys.argv[2]]()
    print("ok", flush=True)
