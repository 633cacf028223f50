"""GPU parity of the tiles whose k range is divided among the waves (64x64 and 16x64): edges of a tile, k ranges that give some waves
no slab or a partial one, every layout, type, epilogue and a strided batch, forced and as an automatic call launches them; and
that a forced plan runs the kernel it names."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_16465_amd as lg
import workloads as wl
from gpu_harness import BatchedDeviceProblem, DeviceProblem, check_full, expected_bits_exact, c_bits_as_uint

pytestmark = pytest.mark.gpu

TILE = lg.GEMM_KERNEL_MFMA_TILE
WAVE = {n: v for v in range(64) if (n := lg.gemm_variant_name(TILE, v) or "").startswith("wavek_")}


@pytest.fixture(scope="module")
def handle():
    h = lg.gemm_create()
    yield h
    torch.cuda.synchronize()
    lg.gemm_destroy(h)


def run(handle, cfg, inp, plan):
    lg.gemm_set_plan(handle, *plan) if plan else lg.gemm_set_plan(handle)
    try:
        p = DeviceProblem(cfg, inp)
        p.run(handle)
        return p.result_bits(), lg.gemm_get_last_plan(handle)
    finally:
        lg.gemm_set_plan(handle)


@pytest.mark.parametrize("name", sorted(WAVE))
@pytest.mark.parametrize("ta,tb", [(0, 1), (0, 0), (1, 1), (1, 0)])
@pytest.mark.parametrize("K", [8, 64, 72, 200, 256, 328, 1000])
def test_edges_of_tiles_and_of_the_k_range(handle, name, ta, tb, K):
    """Integer data, one right answer; C padded, its padding untouched."""
    for M, N, dtype, out in [(64, 64, wl.BF16, wl.BF16), (72, 136, wl.F16, wl.F32), (8, 8, wl.BF16, wl.F32), (136, 72, wl.F16, wl.F16)] + (
            [] if ta else [(1, 200, wl.BF16, wl.BF16), (17, 64, wl.F16, wl.F16), (65, 56, wl.BF16, wl.F32)]) + (
            [(24, 61, wl.BF16, wl.BF16), (72, 67, wl.F16, wl.F32)] if tb else []):
        cfg = wl.Config("w", M, N, K, ta, tb, dtype, out, lda=(M if ta else K) + 8, ldb=(K if tb else N) + 8 + (0 if tb else -N % 8), ldc=N + 3)
        inp, _ = wl.make_integer_inputs(cfg, 40 + K, -2, 2)
        got, plan = run(handle, cfg, inp, (TILE, WAVE[name], 1))
        assert plan == (TILE, WAVE[name], 1)
        assert np.array_equal(c_bits_as_uint(cfg, got), c_bits_as_uint(cfg, expected_bits_exact(cfg, inp).reshape(M, N))), (M, N, K)
        assert np.all(np.isnan(oracle.decode(out, np.ascontiguousarray(got[:-1, N:]))))


@pytest.mark.parametrize("name", sorted(WAVE))
@pytest.mark.parametrize("N,tb", [(200, 0), (199, 1), (68, 1)])
def test_epilogues(handle, name, N, tb):
    for dtype, out, act, bias_dtype, beta in [(wl.BF16, wl.BF16, wl.ACT_GELU_ERF, wl.BF16, 0.0), (wl.F16, wl.F16, wl.ACT_SILU, wl.F32, 0.5),
                                              (wl.BF16, wl.F32, wl.ACT_NONE, wl.F32, 1.0), (wl.F16, wl.F32, wl.ACT_RELU, wl.F16, 0.0)]:
        cfg = wl.Config("w", 83, N, 520, 0, tb, dtype, out, alpha=0.75, beta=beta, a_dist=("normal", 1.0), b_dist=("normal", 0.05),
                        c_dist=("normal", 1.0), bias_dist=("normal", 0.1), bias_dtype=bias_dtype, act=act, ldc=N + 5)
        inp = wl.make_inputs(cfg, 9)
        got, _ = run(handle, cfg, inp, (TILE, WAVE[name], 1))
        check_full(cfg, inp, got, f"{name} act={act}")


def test_automatic_calls_take_them_in_place_of_whole_128_tiles_and_of_a_split(handle):
    """What an automatic call is launched on is reported, and gives the same bits when forced."""
    for M, N, K, ta, tb in [(200, 264, 776, 0, 1), (520, 392, 136, 1, 0), (30, 1096, 2056, 0, 0)]:
        cfg = wl.Config("w", M, N, K, ta, tb, wl.BF16, wl.F32, beta=1.0, a_dist=("normal", 1.0), b_dist=("normal", 0.05), c_dist=("normal", 1.0))
        inp = wl.make_inputs(cfg, 3)
        got, plan = run(handle, cfg, inp, None)
        launched = lg.gemm_get_last_launch(handle)
        assert plan[2] == 1 and launched[0] == TILE and launched[1] in WAVE.values() and launched[2] == 1, (plan, launched)
        again, _ = run(handle, cfg, inp, launched)
        check_full(cfg, inp, got, str(plan))
        assert np.array_equal(got.view(np.uint32), again.view(np.uint32))


# (the kernel, another of the same sums, one that adds in another order) on a call that an automatic plan would launch as a wave tile
NAMED = [(200, 264, 776, 0, 1, wl.BF16, (TILE, 5, 1), (TILE, 12, 1), (TILE, 18, 1)), (520, 392, 136, 1, 0, wl.F16, (TILE, 12, 1), (TILE, 5, 1), (TILE, 18, 1)),
         (196, 132, 100, 0, 1, wl.F32, (TILE, 13, 1), None, (TILE, 21, 1)), (64, 460, 1152, 0, 1, wl.F32, (TILE, 13, 2), None, (TILE, 21, 1)),
         (16, 3032, 264, 0, 1, wl.BF16, (lg.GEMM_KERNEL_SKINNY, 5, 1), None, (TILE, 19, 1)), (58, 728, 688, 0, 1, wl.BF16, (TILE, 16, 4), None, (TILE, 19, 1))]


@pytest.mark.parametrize("M,N,K,ta,tb,dtype,plan,same,other", NAMED)
def test_a_forced_plan_runs_the_kernel_that_it_names(handle, M, N, K, ta, tb, dtype, plan, same, other):
    """Gaussian data and a 32-bit result: another order of the sums shows in the bits."""
    cfg = wl.Config("named", M, N + (-N % 8 if plan[2] > 1 else 0), K, ta, tb, dtype, wl.F32, a_dist=("normal", 1.0), b_dist=("normal", 0.05))
    inp = wl.make_inputs(cfg, 7)
    got, last = run(handle, cfg, inp, plan)
    assert last == plan and not np.array_equal(got.view(np.uint32), run(handle, cfg, inp, other)[0].view(np.uint32)), (plan, other)
    assert same is None or np.array_equal(got.view(np.uint32), run(handle, cfg, inp, same)[0].view(np.uint32)), (plan, same)
    check_full(cfg, inp, got, str(plan))
    run(handle, cfg, inp, plan)
    assert lg.gemm_get_last_launch(handle) == plan


def test_a_forced_plan_of_the_unaligned_tiles_runs_the_kernel_that_it_names(handle):
    """16-bit results: of 90 000 elements a few round the other way when they are added in another order."""
    cfg = wl.Config("named", 301, 303, 519, 0, 1, wl.F16, wl.F16, lda=520, ldb=521, ldc=303, a_dist=("normal", 1.0), b_dist=("normal", 0.05))
    inp = wl.make_inputs(cfg, 7)
    bits = {}
    for variant in (1, 3, 4):
        bits[variant], last = run(handle, cfg, inp, (lg.GEMM_KERNEL_GENERAL, variant, 1))
        assert last == (lg.GEMM_KERNEL_GENERAL, variant, 1)
        check_full(cfg, inp, bits[variant], str(variant))
    assert not np.array_equal(bits[1], bits[3]) and not np.array_equal(bits[1], bits[4])
    got, _ = run(handle, cfg, inp, None)
    launched = lg.gemm_get_last_launch(handle)
    assert launched[0] == lg.GEMM_KERNEL_GENERAL and launched[1] in (3, 4) and np.array_equal(got, bits[launched[1]])


@pytest.mark.parametrize("name", sorted(WAVE))
def test_strided_batch(handle, name):
    cfg = wl.Config("w", 72, 80, 136, 0, 0, wl.BF16, wl.BF16, alpha=1.0)
    lg.gemm_set_plan(handle, TILE, WAVE[name], 1)
    try:
        p = BatchedDeviceProblem(cfg, 5, cfg.stride_a() + 8, cfg.stride_b(), cfg.stride_c() + 16, seed=5, integer=True)
        p.run(handle)
        p.check(name, exact=True)
    finally:
        lg.gemm_set_plan(handle)


@pytest.mark.parametrize("ta,tb", [(0, 1), (0, 0), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(9, 200, 9), (65, 131, 63), (130, 73, 65), (200, 139, 201), (19, 67, 1031), (301, 453, 519), (8, 75, 127)])
def test_off_the_grid(handle, ta, tb, M, N, K):
    """The movers that need no alignment: rows that start on any element and end inside a chunk, the last slab of a k range, tiles with fewer
    than eight columns or rows inside C.  What lies outside the operands is NaN; integer data, one right answer."""
    M = max(M, 8) if ta else M
    for dtype in (wl.BF16, wl.F16):
        cfg = wl.Config("w", M, N, K, ta, tb, dtype, dtype, lda=(M if ta else K) + 3, ldb=(K if tb else N) + 1, ldc=N + 1)
        inp, _ = wl.make_integer_inputs(cfg, M + K, -2, 2)
        want = c_bits_as_uint(cfg, expected_bits_exact(cfg, inp).reshape(M, N))
        for key, (rows, cols), ld in (("A", cfg.a_shape(), cfg.ld_a()), ("B", cfg.b_shape(), cfg.ld_b())):
            x = inp[key].reshape(rows, ld).copy()
            x[:, cols:] = wl.to_bits(np.full((1,), np.nan, dtype=np.float32), dtype)[0]
            inp[key] = x.reshape(-1)
        for variant in (1, 3, 4):                               # the 128x128 tile, the 64x64 and (row-major A) the 16x64 wave tile
            if variant == 4 and ta:
                continue
            lg.gemm_set_plan(handle, lg.GEMM_KERNEL_GENERAL, variant, 1)
            try:
                p = DeviceProblem(cfg, inp, a_offset_elems=1, b_offset_elems=3)
                p.run(handle)
                assert lg.gemm_get_last_launch(handle) == (lg.GEMM_KERNEL_GENERAL, variant, 1)
                assert np.array_equal(c_bits_as_uint(cfg, p.result_bits()), want), variant
            finally:
                lg.gemm_set_plan(handle)


WAVE_F32 = {n: v for v in range(64) if (n := lg.gemm_variant_name(TILE, v) or "").endswith("_wk8")}


@pytest.mark.parametrize("name", sorted(WAVE_F32))
@pytest.mark.parametrize("ta,tb", [(0, 1), (0, 0), (1, 1), (1, 0)])
@pytest.mark.parametrize("K", [4, 32, 36, 100, 256, 324, 1000])
def test_fp32_edges_of_tiles_and_of_the_k_range(handle, name, ta, tb, K):
    for M, N in [(32, 32), (36, 68), (4, 8), (16, 100)] + ([] if ta else [(1, 36), (33, 32), (17, 64)]) + ([(32, 33), (16, 31)] if tb else []):
        cfg = wl.Config("w", M, N, K, ta, tb, wl.F32, wl.F32, lda=(M if ta else K) + 4, ldb=(K if tb else N) + 4 + (0 if tb else -N % 4), ldc=N + 3)
        inp, _ = wl.make_integer_inputs(cfg, 40 + K, -5, 5)
        got, plan = run(handle, cfg, inp, (TILE, WAVE_F32[name], 1))
        assert plan == (TILE, WAVE_F32[name], 1)
        assert np.array_equal(c_bits_as_uint(cfg, got), c_bits_as_uint(cfg, expected_bits_exact(cfg, inp).reshape(M, N))), (M, N, K)
        assert np.all(np.isnan(oracle.decode(wl.F32, np.ascontiguousarray(got[:-1, N:]))))


@pytest.mark.parametrize("name", sorted(WAVE_F32) + ["f32_64x64x32_w2x2"])
@pytest.mark.parametrize("M,N,K,tb,batch", [(45, 75, 333, 1, 1), (83, 100, 520, 0, 1), (1100, 1060, 72, 0, 1), (20, 44, 100, 0, 5)])
def test_fp32_epilogues_batches_and_grids_that_stay_on_the_64x64_tile(handle, name, M, N, K, tb, batch):
    K = K // 4 * 4
    variant = next(v for v in range(64) if lg.gemm_variant_name(TILE, v) == name)
    for act, bias_dtype, beta in [(wl.ACT_SILU, wl.F32, 1.0), (wl.ACT_NONE, wl.F32, 0.0)]:
        cfg = wl.Config("w", M, N, K, 0, tb, wl.F32, wl.F32, alpha=0.75, beta=beta, a_dist=("normal", 1.0), b_dist=("normal", 0.05),
                        c_dist=("normal", 1.0), bias_dist=("normal", 0.1) if batch == 1 else None, bias_dtype=bias_dtype, act=act, ldc=N + 5)
        if batch > 1:
            lg.gemm_set_plan(handle, TILE, variant, 1)
            try:
                p = BatchedDeviceProblem(cfg, batch, cfg.stride_a() + 4, cfg.stride_b(), cfg.stride_c() + 3, seed=5)
                p.run(handle)
                p.check(name)
            finally:
                lg.gemm_set_plan(handle)
            continue
        inp = wl.make_inputs(cfg, 9)
        got, _ = run(handle, cfg, inp, (TILE, variant, 1))
        check_full(cfg, inp, got, f"{name} act={act}")


@pytest.mark.parametrize("name", sorted(WAVE_F32))
@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 0)])
def test_fp32_values_outside_the_split(handle, name, ta, tb):
    """Products and sums beyond the scaled range, infinities and NaN, in the share of one wave only or of all: computed again on the fp32
    instruction.  Exact integers times powers of two, one right answer."""
    rng = np.random.default_rng(3)
    M, N, K = 36, 40, 300
    a, b = rng.integers(-7, 8, (M, K)).astype(np.float64), rng.integers(-3, 4, (K, N)).astype(np.float64)
    a[1] *= 2.0 ** 100
    a[2, 70] = np.inf
    a[3, K - 1] = np.nan
    a[4] = rng.integers(-7, 8, K) * 2.0 ** -149
    a[M - 1, :32] *= 2.0 ** 90
    b[:, 1] *= 2.0 ** 12
    A, B = (np.ascontiguousarray(x, dtype=np.float32) for x in (a.T if ta else a, b.T if tb else b))
    cfg = wl.Config("w", M, N, K, ta, tb, wl.F32, wl.F32)
    inp = {"A": wl.to_bits(A.reshape(-1), wl.F32), "B": wl.to_bits(B.reshape(-1), wl.F32), "C": None, "bias": None}
    with np.errstate(invalid="ignore"):
        want = oracle.decode(wl.F32, expected_bits_exact(cfg, inp)).reshape(M, N)
    got, _ = run(handle, cfg, inp, (TILE, WAVE_F32[name], 1))
    got = oracle.decode(wl.F32, np.ascontiguousarray(got[:, :N]))
    assert np.array_equal(got, want, equal_nan=True), np.argwhere(~((got == want) | (np.isnan(got) & np.isnan(want))))[:4]


SKINNY = lg.GEMM_KERNEL_SKINNY


@pytest.mark.parametrize("kernel,variant,M,N,K,tb,launched", [
    (SKINNY, 5, 16, 3032, 264, 1, 19), (SKINNY, 5, 16, 4093, 264, 1, 19), (SKINNY, 0, 16, 13088, 5128, 0, 19), (SKINNY, 1, 14, 13128, 5112, 1, 19),
    (TILE, 16, 58, 728, 688, 1, 19), (TILE, 16, 60, 884, 728, 1, 19), (TILE, 16, 54, 1000, 688, 0, 19), (TILE, 16, 38, 5552, 1200, 1, 18),
    (TILE, 16, 34, 5584, 1192, 0, 18)])
def test_few_rows_whose_plan_runs_on_a_wave_tile(handle, kernel, variant, M, N, K, tb, launched):
    for dtype, out, act, bias_dtype, beta in [(wl.BF16, wl.F32, wl.ACT_NONE, wl.BF16, 1.0), (wl.F16, wl.F16, wl.ACT_GELU_ERF, wl.F32, 0.0)]:
        cfg = wl.Config("w", M, N, K, 0, tb, dtype, out, alpha=0.5, beta=beta, a_dist=("normal", 1.0), b_dist=("normal", 0.05), c_dist=("normal", 1.0),
                        bias_dist=("normal", 0.1), bias_dtype=bias_dtype, act=act, ldb=(K if tb else (N + 7) // 8 * 8) + 8, ldc=N + 3)
        inp = wl.make_inputs(cfg, 21)
        got, plan = run(handle, cfg, inp, None)
        assert plan[:2] == (kernel, variant) and lg.gemm_get_last_launch(handle) == (TILE, launched, 1), plan
        check_full(cfg, inp, got, f"{plan} {M}x{N}x{K}")


@pytest.mark.parametrize("K,launched", [(1272, 5), (1280, 16), (1304, 16)])
def test_whole_128x128_tiles_of_a_long_k(handle, K, launched):
    M, N = 2085, 1051      # beyond two rounds of wave tiles, ragged on both sides
    cfg = wl.Config("w", M, N, K, 0, 1, wl.BF16, wl.F32, lda=K + 8, ldb=K + 16, ldc=N + 3)
    inp, _ = wl.make_integer_inputs(cfg, 77 + K, -5, 5)
    for forced in (None, (TILE, 5, 1), (TILE, 16, 1)):
        got, plan = run(handle, cfg, inp, forced)
        assert plan == (forced or (TILE, 5, 1)) and lg.gemm_get_last_launch(handle) == (forced or (TILE, launched, 1))
        assert np.array_equal(c_bits_as_uint(cfg, got), c_bits_as_uint(cfg, expected_bits_exact(cfg, inp).reshape(M, N)))
        assert np.all(np.isnan(oracle.decode(wl.F32, np.ascontiguousarray(got[:-1, N:]))))


@pytest.mark.parametrize("M,N,K,dtype", [(2085, 1051, 1304, wl.BF16), (200, 328, 4104, wl.F16)])
def test_the_two_pipelines_of_the_128x128_tile_give_the_same_bits(handle, M, N, K, dtype):
    """The ring of four (variant 5, products of 16 along k) and the quartered kernel (16, of 32): Gaussian data and a 32-bit result."""
    cfg = wl.Config("w", M, N, K, 0, 1, dtype, wl.F32, a_dist=("normal", 1.0), b_dist=("normal", 0.05), ldb=K + 16, ldc=N + 3)
    inp = wl.make_inputs(cfg, K)
    a, b = (np.ascontiguousarray(run(handle, cfg, inp, (TILE, v, 1))[0][:, :N]).view(np.uint32) for v in (5, 16))
    assert np.array_equal(a, b), int((a != b).sum())


@pytest.mark.parametrize("K,N,tb,launched", [(760, 64, 0, 5), (768, 64, 0, 18), (776, 48, 0, 18), (776, 37, 1, 18)])
def test_batches_of_up_to_64_columns_beyond_two_rounds(handle, K, N, tb, launched):
    M, batch = 1093, 31
    cfg = wl.Config("w", M, N, K, 0, tb, wl.BF16, wl.BF16, a_dist=("normal", 1.0), b_dist=("normal", 0.05), c_dist=("normal", 1.0), beta=0.5)
    p = BatchedDeviceProblem(cfg, batch, cfg.stride_a(), cfg.stride_b() + 8, cfg.stride_c() + 3, seed=5)
    p.run(handle)
    assert lg.gemm_get_last_plan(handle) == (TILE, 5, 1) and lg.gemm_get_last_launch(handle) == (TILE, launched, 1)
    p.check("narrow batch")
