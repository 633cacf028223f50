"""The fp32 tile kernels form their products from bf16 pieces; values that the pieces cannot hold are found and multiplied
as fp32.  Rows of every such kind between ordinary ones, all data exact, in each tile form: bit for bit the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_16465_amd as lg
import workloads as wl
from gpu_harness import DeviceProblem, decode_c, oracle_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def handle():
    h = lg.gemm_create()
    yield h
    torch.cuda.synchronize()
    lg.gemm_destroy(h)


def stored(a, b, ta, tb, odd):
    """The operands as a call and its inputs; `odd`: rows three and one elements longer, filled with NaN."""
    (M, K), N = a.shape, b.shape[1]
    a, b = (np.pad(np.ascontiguousarray(x, dtype=np.float32), ((0, 0), (0, pad if odd else 0)), constant_values=np.nan)
            for x, pad in ((a.T if ta else a, 3), (b.T if tb else b, 1)))
    cfg = wl.Config("split", M, N, K, ta, tb, wl.F32, wl.F32, lda=a.shape[1], ldb=b.shape[1])
    return cfg, {"A": wl.to_bits(a.reshape(-1), wl.F32), "B": wl.to_bits(b.reshape(-1), wl.F32), "C": None, "bias": None}


def run_plan(handle, plan, cfg, inp, odd=False):
    lg.gemm_set_plan(handle, *plan)
    p = DeviceProblem(cfg, inp, a_offset_elems=int(odd), b_offset_elems=3 * int(odd))
    p.run(handle)
    lg.gemm_set_plan(handle)
    assert lg.gemm_get_last_plan(handle)[:2] == plan[:2]
    return decode_c(cfg, p.result_bits())


# 64x64 tiles, one 128x128 tile per workgroup, pairs of them (more than 256 tiles); a partial slab, ragged edges
@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 0), (0, 0), (1, 1)])
@pytest.mark.parametrize("variant,M,N,K", [(13, 196, 132, 100), (11, 196, 260, 100), (11, 2100, 2068, 72)])
def test_values_outside_the_split(handle, variant, M, N, K, ta, tb):
    check_values_outside(handle, (lg.GEMM_KERNEL_MFMA_TILE, variant, 1), M, N, K, ta, tb)


# the folded tiles of the general family (odd sizes, leading dimensions and base addresses), and k slices, of which only some
# hold such values
@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 0), (0, 0), (1, 1)])
@pytest.mark.parametrize("plan,M,N,K", [((lg.GEMM_KERNEL_GENERAL, 2, 1), 197, 131, 99), ((lg.GEMM_KERNEL_GENERAL, 2, 3), 197, 131, 99),
                                        ((lg.GEMM_KERNEL_MFMA_TILE, 13, 3), 196, 136, 100), ((lg.GEMM_KERNEL_MFMA_TILE, 11, 3), 196, 136, 100)])
def test_values_outside_the_split_off_the_grid_and_in_slices(handle, plan, M, N, K, ta, tb):
    check_values_outside(handle, plan, M, N, K, ta, tb, odd=plan[0] == lg.GEMM_KERNEL_GENERAL)


def check_values_outside(handle, plan, M, N, K, ta, tb, odd=False):
    rng = np.random.default_rng([7, M])
    a = rng.integers(-7, 8, (M, K)).astype(np.float64)
    b = rng.integers(-3, 4, (K, N)).astype(np.float64)
    a[0] = 0.0
    a[1] = rng.integers(-7, 8, K) * 2.0 ** -149                 # subnormals: lost by every piece
    a[2] = rng.integers(-7, 8, K) * 2.0 ** -130
    a[3] *= 2.0 ** -108                                          # just inside
    a[4, K - 1] = np.inf
    a[5, 0] = np.nan
    a[6] *= 2.0 ** 80                                            # (every partial sum: at most 100 * 7 * 3 * 2^(80 + 30) < 2^122, no order of addition overflows)
    a[7, 3], a[7, 4] = 2.0 ** -149, 0.0                          # one lost element among ordinary ones: below rounding
    a[M - 1] = rng.integers(-7, 8, K) * 2.0 ** -140
    b[:, 1] *= 2.0 ** 24
    b[:, N - 1] *= 2.0 ** 30
    b[:, 2] = 0.0
    cfg, inp = stored(a, b, ta, tb, odd)
    with np.errstate(invalid="ignore"):
        want = oracle.decode(wl.F32, oracle.encode(wl.F32, oracle.gemm_full(oracle_problem(cfg, inp))))
    assert np.any(want[1] != 0) and np.all(np.isnan(want[5])) and np.any(np.isinf(want[4]))
    got = run_plan(handle, plan, cfg, inp, odd)
    bad = ~((got == want) | (np.isnan(got) & np.isnan(want)))
    # row 7: its lost element is a rounding away from every sum (|sum| >= 1 against 2^-149 * 2^31)
    assert not bad.any(), (plan, sorted(set(np.argwhere(bad)[:, 0]))[:8], int(bad.sum()))


# what lies behind the rows of an operand (padding, or the neighbouring columns of a larger matrix) decides nothing: the bits
# are those of a run with zeros there
@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 0), (0, 0), (1, 1)])
@pytest.mark.parametrize("kernel,variant,M,N,K,pad", [(lg.GEMM_KERNEL_MFMA_TILE, 13, 100, 68, 96, 60), (lg.GEMM_KERNEL_MFMA_TILE, 13, 196, 132, 100, 36),
                                                      (lg.GEMM_KERNEL_MFMA_TILE, 11, 196, 260, 128, 60), (lg.GEMM_KERNEL_MFMA_TILE, 11, 2100, 2068, 72, 60),
                                                      (lg.GEMM_KERNEL_GENERAL, 2, 99, 69, 96, 59), (lg.GEMM_KERNEL_GENERAL, 2, 130, 67, 101, 61)])
def test_memory_outside_the_operands_decides_nothing(handle, kernel, variant, M, N, K, pad, ta, tb):
    rng = np.random.default_rng([11, M, K])
    a_shape, b_shape = ((K, M) if ta else (M, K)), ((N, K) if tb else (K, N))
    a, b = (np.zeros((s[0], s[1] + pad), np.float32) for s in (a_shape, b_shape))
    a[:, :a_shape[1]], b[:, :b_shape[1]] = rng.standard_normal(a_shape), rng.standard_normal(b_shape)
    cfg = wl.Config("padding", M, N, K, ta, tb, wl.F32, wl.F32, lda=a.shape[1], ldb=b.shape[1])
    results = []
    for outside in (0.0, np.inf, 1e30, 1e-40):
        a[:, a_shape[1]:], b[:, b_shape[1]:] = outside, outside
        lg.gemm_set_plan(handle, kernel, variant, 1)
        p = DeviceProblem(cfg, {"A": wl.to_bits(a.reshape(-1), wl.F32), "B": wl.to_bits(b.reshape(-1), wl.F32), "C": None, "bias": None})
        p.run(handle)
        lg.gemm_set_plan(handle)
        assert lg.gemm_get_last_plan(handle) == (kernel, variant, 1)
        results.append(p.result_bits().copy())
    for outside, got in zip((np.inf, 1e30, 1e-40), results[1:]):
        assert np.array_equal(got.view(np.uint32), results[0].view(np.uint32)), (outside, int((got != results[0]).sum()))


# What sends a tile to its second look or its second computation: zeros of every origin, large values whose products stay in range
# or do not, products below the normal range.  All sums exact, bit for bit the oracle's.
@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 0)])
@pytest.mark.parametrize("plan,M,N,K", [((lg.GEMM_KERNEL_MFMA_TILE, 13, 1), 132, 136, 100), ((lg.GEMM_KERNEL_MFMA_TILE, 11, 1), 260, 136, 292),
                                        ((lg.GEMM_KERNEL_MFMA_TILE, 11, 1), 2100, 2068, 72), ((lg.GEMM_KERNEL_GENERAL, 2, 1), 131, 135, 261)])
@pytest.mark.parametrize("kind", ["zero_row", "cancelling", "triangular", "wide", "near_overflow", "tiny_and_cancelling", "subnormal_products"])
def test_second_look(handle, kind, plan, M, N, K, ta, tb):
    rng = np.random.default_rng([3, M, K])
    a, b = rng.integers(-7, 8, (M, K)).astype(np.float64), rng.integers(-3, 4, (K, N)).astype(np.float64)
    if kind == "zero_row":
        a[5], b[:, 7], a[M - 1] = 0.0, 0.0, 0.0
    elif kind == "cancelling":
        a, b = np.sign(a), np.sign(b)
    elif kind == "triangular":
        a *= np.arange(K) <= np.arange(M)[:, None]
        b *= np.arange(N) <= np.arange(K)[:, None]
    elif kind == "wide":                       # 2^100 * 2^10 * K
        a[3] *= 2.0 ** 97
        b[:, 4] *= 2.0 ** 8
    elif kind == "near_overflow":              # results up to 7 * 3 * 292 * 2^113 < 2^126, bounded by more than 2^126
        a[2] *= 2.0 ** 60
        b[:, 9] *= 2.0 ** 53
        b[0, 9] = 2.0 ** 63
        a[2, 0] = 0.0
    elif kind == "tiny_and_cancelling":
        a, b = np.sign(a), np.sign(b)
        a[6] *= 2.0 ** -120
        b[:, 1] = rng.integers(-3, 4, K) * 2.0 ** -140
        a[7] = 1.0
    else:
        a = rng.integers(-2047, 2048, (M, K)) * 2.0 ** -75
        b = rng.integers(-3, 4, (K, N)) * 2.0 ** -74
    odd = plan[0] == lg.GEMM_KERNEL_GENERAL
    cfg, inp = stored(a, b, ta, tb, odd)
    want = oracle.decode(wl.F32, oracle.encode(wl.F32, oracle.gemm_full(oracle_problem(cfg, inp))))
    assert np.all(np.isfinite(want))
    got = run_plan(handle, plan, cfg, inp, odd)
    assert np.array_equal(got, want), (kind, np.argwhere(got != want)[:4], int((got != want).sum()))
