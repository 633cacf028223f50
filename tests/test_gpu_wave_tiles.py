"""GPU parity of the tiles whose k range is divided among the waves (64x64 and 16x64): edges of a tile, k ranges that give some waves
no slab or a partial one, every layout, type, epilogue and a strided batch, forced and as the automatic plan launches them."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_16465_amd as lg
import workloads as wl
from gpu_harness import BatchedDeviceProblem, DeviceProblem, check_full, expected_bits_exact, c_bits_as_uint

pytestmark = pytest.mark.gpu

TILE = lg.GEMM_KERNEL_MFMA_TILE
WAVE = {n: v for v in range(64) if (n := lg.gemm_variant_name(TILE, v) or "").startswith("wavek")}


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


def test_automatic_calls_take_them_under_the_plan_of_the_128_tile_and_in_place_of_a_split(handle):
    """A whole 128x128 tile plan, reported and forced, is launched on them; so is a call that used to be split."""
    for M, N, K, ta, tb in [(200, 264, 776, 0, 1), (520, 392, 136, 1, 0), (30, 1096, 2056, 0, 0)]:
        cfg = wl.Config("w", M, N, K, ta, tb, wl.BF16, wl.F32, beta=1.0, a_dist=("normal", 1.0), b_dist=("normal", 0.05), c_dist=("normal", 1.0))
        inp = wl.make_inputs(cfg, 3)
        got, plan = run(handle, cfg, inp, None)
        assert plan[2] == 1
        again, _ = run(handle, cfg, inp, plan)
        check_full(cfg, inp, got, str(plan))
        assert np.array_equal(got.view(np.uint32), again.view(np.uint32))
        if not (ta and M % 64):
            tiles = [run(handle, cfg, inp, (TILE, v, 1))[0].view(np.uint32) for n, v in sorted(WAVE.items()) if not (ta and n.startswith("wavek_16"))]
            assert any(np.array_equal(got.view(np.uint32), t) for t in tiles), plan


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
        lg.gemm_set_plan(handle, lg.GEMM_KERNEL_GENERAL, 1, 1)
        try:
            p = DeviceProblem(cfg, inp, a_offset_elems=1, b_offset_elems=3)
            p.run(handle)
            assert np.array_equal(c_bits_as_uint(cfg, p.result_bits()), want)
        finally:
            lg.gemm_set_plan(handle)
