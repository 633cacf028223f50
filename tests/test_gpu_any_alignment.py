"""Calls off the 16-byte grid on the matrix-core kernels of the general family: odd sizes, leading dimensions and base
addresses in every layout and type, around the edges of tiles, slabs and chunks, whole and in k slices.  Integer data, so every
element is exact; what lies behind a row (NaN) reaches no result and the padding of C keeps its contents."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_16465_amd as lg
import workloads as wl
from gpu_harness import BatchedDeviceProblem, DeviceProblem, c_bits_as_uint, decode_c, expected_bits_exact

pytestmark = pytest.mark.gpu
SHAPES = [(8, 8, 1), (9, 15, 7), (127, 129, 63), (131, 9, 65), (257, 263, 191), (264, 13, 200), (40, 521, 1031)]


@pytest.fixture(scope="module")
def handle():
    h = lg.gemm_create()
    yield h
    torch.cuda.synchronize()
    lg.gemm_destroy(h)


def poisoned(inp, key, rows, cols, ld, dtype):
    x = inp[key].reshape(rows, ld).copy()
    x[:, cols:] = wl.to_bits(np.full((1,), np.nan, dtype=np.float32), dtype)[0]
    return x.reshape(-1)


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("ta,tb", [(0, 1), (0, 0), (1, 1), (1, 0)])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_variant(handle, shape, ta, tb, dtype):
    M, N, K = shape
    cfg = wl.Config("any", M, N, K, ta, tb, dtype, wl.F32 if (M + N) % 2 else dtype, alpha=1.0, beta=-1.0, bias_dist=("normal", 1.0),
                    bias_dtype=wl.F32, lda=(M if ta else K) + 3, ldb=(K if tb else N) + 1, ldc=N + 2)
    inp, _ = wl.make_integer_inputs(cfg, 7 * M + N, -2, 2)
    want = oracle.decode(cfg.out_dtype, expected_bits_exact(cfg, inp)).reshape(M, N)
    a_rows, a_cols = cfg.a_shape()
    b_rows, b_cols = cfg.b_shape()
    inp["A"], inp["B"] = poisoned(inp, "A", a_rows, a_cols, cfg.ld_a(), dtype), poisoned(inp, "B", b_rows, b_cols, cfg.ld_b(), dtype)
    plans = [None] + [(v, s) for v in ((2,) if dtype == wl.F32 else (1,)) for s in (1, 3)] + [(0, 1)]
    for plan in plans:
        print(shape, ta, tb, dtype, plan, flush=True)
        if plan is None:
            lg.gemm_set_plan(handle)
        else:
            lg.gemm_set_plan(handle, lg.GEMM_KERNEL_GENERAL, *plan)
        p = DeviceProblem(cfg, inp, a_offset_elems=1, b_offset_elems=3)
        before = p.result_bits().copy()
        p.run(handle)
        got_plan = lg.gemm_get_last_plan(handle)
        lg.gemm_set_plan(handle)
        assert got_plan[0] == lg.GEMM_KERNEL_GENERAL and (plan is None or got_plan[1] == plan[0]), (plan, got_plan)
        after = p.result_bits()
        got = oracle.decode(cfg.out_dtype, c_bits_as_uint(cfg, after))
        assert np.array_equal(got, want), f"{plan}: {np.argwhere(got != want)[:4]} of {int((got != want).sum())}"
        if M > 1:
            assert np.array_equal(before[:-1, N:].view(np.uint8), after[:-1, N:].view(np.uint8)), "padding of C written"


@pytest.mark.parametrize("dtype,variant", [(wl.BF16, 1), (wl.F32, 2)])
def test_odd_batch(handle, dtype, variant):
    cfg = wl.Config("any", 170, 245, 133, 0, 0, dtype, wl.F32)
    p = BatchedDeviceProblem(cfg, 5, cfg.stride_a() + 1, cfg.stride_b() + 3, cfg.stride_c() + 1, seed=3, integer=True)
    lg.gemm_set_plan(handle, lg.GEMM_KERNEL_GENERAL, variant, 1)
    p.run(handle)
    lg.gemm_set_plan(handle)
    assert lg.gemm_get_last_plan(handle) == (lg.GEMM_KERNEL_GENERAL, variant, 1)
    p.check("odd batch", exact=True)


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("M,N,K", [(1, 1, 8), (4, 3, 520), (6, 5, 512), (16, 7, 1032), (1, 9, 8), (1, 4097, 520), (3, 1031, 1032), (4, 12301, 264), (5, 4095, 256), (8, 4099, 1288), (16, 1025, 776)])
def test_few_rows_and_columns_that_are_no_multiple_of_eight(handle, M, N, K, dtype):
    cfg = wl.Config("ragged", M, N, K, 0, 1, dtype, wl.F32 if N % 4 == 1 else dtype, alpha=1.0, beta=1.0, bias_dist=("normal", 1.0),
                    bias_dtype=wl.F32, lda=K + 8, ldb=K + 24, ldc=N + 3)
    inp, _ = wl.make_integer_inputs(cfg, M + N, -2, 2)
    want = oracle.decode(cfg.out_dtype, expected_bits_exact(cfg, inp)).reshape(M, N)
    inp["A"], inp["B"] = poisoned(inp, "A", M, K, cfg.ld_a(), dtype), poisoned(inp, "B", N, K, cfg.ld_b(), dtype)
    p = DeviceProblem(cfg, inp)
    before = p.result_bits().copy()
    p.run(handle)
    assert lg.gemm_get_last_plan(handle) == (lg.GEMM_KERNEL_SKINNY, 4 if M <= 4 else 5, 1)
    after = p.result_bits()
    assert np.array_equal(oracle.decode(cfg.out_dtype, c_bits_as_uint(cfg, after)), want)
    if M > 1:
        assert np.array_equal(before[:-1, N:].view(np.uint8), after[:-1, N:].view(np.uint8)), "padding of C written"
    # the reported plan can be forced, any other of the family is refused as it always was
    lg.gemm_set_plan(handle, *lg.gemm_get_last_plan(handle))
    again = DeviceProblem(cfg, inp)
    again.run(handle)
    assert np.array_equal(again.result_bits().view(np.uint8), after.view(np.uint8))
    lg.gemm_set_plan(handle, lg.GEMM_KERNEL_SKINNY, -1, 0)
    assert p.run(handle, check=False) == lg.GEMM_ERR_UNSUPPORTED
    lg.gemm_set_plan(handle)


@pytest.mark.parametrize("K", [40, 65, 129, 1025])
def test_fp32_error_is_no_larger_than_that_of_the_plain_kernel(handle, K):
    M, N = 261, 131
    g = torch.Generator(device="cuda").manual_seed(K)
    A, B = torch.randn(M, K, generator=g, device="cuda"), torch.randn(K, N, generator=g, device="cuda")
    want, errors = A.double() @ B.double(), {}
    for plan in ((2, 1), (0, 1)):
        lg.gemm_set_plan(handle, lg.GEMM_KERNEL_GENERAL, *plan)
        C = torch.empty(M, N, device="cuda")
        lg.gemm_run(handle, M, N, K, 0, 0, wl.F32, 1.0, A.data_ptr(), K, B.data_ptr(), N, 0.0, C.data_ptr(), N, lg.make_epilogue(wl.F32),
                    torch.cuda.current_stream().cuda_stream)
        assert lg.gemm_get_last_plan(handle) == (lg.GEMM_KERNEL_GENERAL, *plan)
        errors[plan[0]] = ((C.double() - want).norm() / want.norm()).item()
    lg.gemm_set_plan(handle)
    # one rounding per 32 elements of k at the sum's magnitude against one per 16
    assert errors[2] <= errors[0], errors


def run_problem(p, handle, noalloc=False, check=True):
    c = p.cfg
    return (lg.gemm_run_noalloc if noalloc else lg.gemm_run)(
        handle, c.M, c.N, c.K, c.transA, c.transB, c.dtype, c.alpha, p.A.data_ptr(), c.ld_a(), p.B.data_ptr(), c.ld_b(), c.beta,
        p.C.data_ptr(), c.ld_c(), p.epilogue(), torch.cuda.current_stream().cuda_stream, check=check)


# A call that is cut in slices gives the same bits wherever its partial results go: the handle's workspace, the static scratch,
# or nowhere (captured on a handle without a workspace: the slices one after another).
@pytest.mark.parametrize("dtype,out", [(wl.BF16, wl.BF16), (wl.F16, wl.F32), (wl.F32, wl.F32)])
@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 0), (0, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,plan", [(16, 2047, 4095, None), (131, 257, 1001, (5,)), (130, 141, 333, (3,))])
@pytest.mark.parametrize("beta,act", [(0.0, wl.ACT_SILU), (-1.3, wl.ACT_NONE)])
def test_slices_give_the_same_bits_with_and_without_a_workspace(M, N, K, plan, ta, tb, dtype, out, beta, act):
    if dtype != wl.F32 and ta and M % 8:
        M += 8 - M % 8
    cfg = wl.Config("slices", M, N, K, ta, tb, dtype, out, alpha=0.7, beta=beta, a_dist=("normal", 1.0), b_dist=("normal", 0.05), c_dist=("normal", 1.0),
                    bias_dist=("normal", 0.1), bias_dtype=wl.F32, act=act, lda=(M if ta else K) + 1, ldb=(K if tb else N) + 3, ldc=N + 1)
    inputs = wl.make_inputs(cfg, M + K)
    handles = [lg.gemm_create() for _ in range(3)]
    problems = [DeviceProblem(cfg, inputs) for _ in range(3)]
    try:
        if plan:
            for h in handles:
                lg.gemm_set_plan(h, lg.GEMM_KERNEL_GENERAL, 2 if dtype == wl.F32 else 1, plan[0])
        run_problem(problems[0], handles[0])
        run_problem(problems[1], handles[1], noalloc=True)
        torch.cuda.synchronize()
        assert lg.gemm_get_last_plan(handles[0])[2] > 1 and lg.gemm_workspace_size(handles[0]) > 0 and lg.gemm_workspace_size(handles[1]) == 0
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run_problem(problems[2], handles[2])
        assert lg.gemm_workspace_size(handles[2]) == 0
        plans = [lg.gemm_get_last_plan(h) for h in handles]
        assert plans[0] == plans[1] == plans[2]
        want = problems[0].result_bits()
        assert np.array_equal(problems[1].result_bits().view(np.uint8), want.view(np.uint8)), "static scratch"
        for replay in range(3):
            problems[2].reset_c()
            graph.replay()
            got = problems[2].result_bits()
            assert np.array_equal(got.view(np.uint8), want.view(np.uint8)), (replay, int((got != want).sum()))
            problems[0].reset_c()
            run_problem(problems[0], handles[0])          # eager work between the replays
            assert np.array_equal(problems[0].result_bits().view(np.uint8), want.view(np.uint8))
    finally:
        torch.cuda.synchronize()
        for h in handles:
            lg.gemm_destroy(h)


def test_a_forced_split_beyond_the_static_scratch_is_refused(handle):
    cfg = wl.Config("limit", 1025, 1027, 1029, 0, 1, wl.BF16, wl.F32)
    p = DeviceProblem(cfg, wl.make_integer_inputs(cfg, 1, -2, 2)[0])
    before = p.result_bits().copy()
    lg.gemm_set_plan(handle, lg.GEMM_KERNEL_GENERAL, 1, 16)
    assert run_problem(p, handle, noalloc=True, check=False) == lg.GEMM_ERR_SCRATCH_LIMIT
    assert np.array_equal(p.result_bits().view(np.uint8), before.view(np.uint8))
    assert run_problem(p, handle) == lg.GEMM_OK and lg.gemm_get_last_plan(handle) == (lg.GEMM_KERNEL_GENERAL, 1, 11)
    lg.gemm_set_plan(handle)


def error_of(handle, M, N, K, ta, tb, A, B, dtype, plan):
    lg.gemm_set_plan(handle, *plan)
    C = torch.empty(M, N, device="cuda")
    lg.gemm_run(handle, M, N, K, ta, tb, dtype, 1.0, A.data_ptr(), M if ta else K, B.data_ptr(), K if tb else N, 0.0, C.data_ptr(), N,
                lg.make_epilogue(wl.F32), torch.cuda.current_stream().cuda_stream)
    lg.gemm_set_plan(handle)
    want = (A.t() if ta else A).double() @ (B.t() if tb else B).double()
    return lg.gemm_get_last_plan(handle), ((C.double() - want).norm() / want.norm()).item()


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 0), (0, 0), (1, 1)])
@pytest.mark.parametrize("K", [41, 65, 129, 257, 513, 1025, 4095])
def test_error_of_16_bit_products_with_an_fp32_result_is_no_larger_than_that_of_the_plain_kernel(handle, K, ta, tb, dtype):
    M, N = 261, 517
    g = torch.Generator(device="cuda").manual_seed(K)
    t = torch.bfloat16 if dtype == wl.BF16 else torch.float16
    A, B = (torch.randn(*s, generator=g, device="cuda").to(t) for s in ((K, M) if ta else (M, K), (N, K) if tb else (K, N)))
    plain = error_of(handle, M, N, K, ta, tb, A, B, dtype, (lg.GEMM_KERNEL_GENERAL, 0, 1))[1]
    for slices in (1, 3):
        plan, error = error_of(handle, M, N, K, ta, tb, A, B, dtype, (lg.GEMM_KERNEL_GENERAL, 1, slices))
        assert plan[:2] == (lg.GEMM_KERNEL_GENERAL, 1)
        # a sum rounded at full magnitude once per 32 elements of k (and slice) against one per 16
        assert error <= plain, (slices, error, plain)
