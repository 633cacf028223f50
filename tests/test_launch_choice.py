"""CPU-only: which kernel an automatic plan is launched on, through gemm_launch_query (host arithmetic, no device)."""
import random

import paper_2512_16465_amd as lg
import workloads as wl

TILE, SKINNY, GENERAL = lg.GEMM_KERNEL_MFMA_TILE, lg.GEMM_KERNEL_SKINNY, lg.GEMM_KERNEL_GENERAL
LAYOUT = {"NT": (0, 1), "NN": (0, 0), "TT": (1, 1), "TN": (1, 0)}


def both(M, N, K, layout="NN", dtype=wl.BF16, out=None, batch=1, pad=0, reads_c=False, act=wl.ACT_NONE, cus=256):
    """Name and slices of the plan and of the kernel that it is launched on."""
    ta, tb = LAYOUT[layout]
    call = (cus, batch, M, N, K, ta, tb, dtype, dtype if out is None else out, (M if ta else K) + pad, (K if tb else N) + pad, N)
    plan, launched = lg.gemm_plan_query(*call), lg.gemm_launch_query(*call, reads_c, act)
    return tuple((lg.gemm_variant_name(k, v), s) for k, v, s in (plan, launched))


def test_plans_that_are_launched_as_wave_tiles():
    small, short, f32 = "dma_128x128x32_w2x2_s4", "dma_128x128x32_w2x2_s3", "f32_64x64x32_w2x2"
    w64, w16 = ("wavek_64x64x64_w4", 1), ("wavek_16x64x64_w4", 1)
    assert both(1024, 1024, 1024) == ((small, 1), w64) and both(200, 264, 776, "NT") == ((small, 1), w16)
    assert both(520, 392, 136, "TN") == ((short, 1), w64)
    assert both(8192, 8192, 256) == ((short, 1), (short, 1))                        # more than two 64x64 tiles to a unit
    assert both(2085, 1051, 1280, "NT", pad=8) == ((small, 1), ("dma16p_128x128x32_w2x2_s5", 1))
    assert both(1856, 80, 1856, "NT", batch=39) == ((small, 1), (small, 1))         # 585 tiles: a thin third round of them
    assert both(1856, 80, 1856, "NT", batch=44) == ((small, 1), ("dma16p_128x128x32_w2x2_s5", 1))
    assert both(1093, 64, 768, batch=31) == ((small, 1), w64) and both(1093, 64, 760, batch=31) == ((small, 1), (small, 1))
    assert both(256, 256, 256, dtype=wl.F32) == ((f32, 1), ("f32_16x32x32_wk8", 1))
    plan, launched = both(268, 228, 3592, "TN", dtype=wl.F32)
    assert plan[0] == f32 and launched == ("f32_16x32x32_wk8", 1)
    assert both(512, 512, 512, dtype=wl.F32)[1] == ("f32_32x32x32_wk8", 1)
    assert both(1024, 1024, 1024, dtype=wl.F32) == ((f32, 1), (f32, 1))             # four 32x32 tiles to a unit
    assert both(16, 3032, 264, "NT") == (("skinny_nt_16x16_w4", 1), w16)
    plan, launched = both(38, 5552, 1200, "NT", pad=8)
    assert plan[0] == "dma16p_128x128x32_w2x2_s5" and plan[1] > 1 and launched == w64
    plan, launched = both(335, 75, 629, "NN")
    assert plan == ("general_128x128x64_w2x2", 4) and launched[0].startswith("general_wavek_") and launched[1] == 1
    assert both(335, 75, 629, "NN", out=wl.F32)[1][0] == "general_128x128x64_w2x2"      # a 32-bit result keeps slices and folds


def test_whole_tiles_that_leave_straight_from_the_registers():
    """C = alpha A B on whole 128x128 tiles: the wave tiles only with a k loop long enough to pay for the sums' way through LDS."""
    w64 = ("wavek_64x64x64_w4", 1)
    for call, batch in [((256, 256, 64, "NT"), 21), ((512, 512, 128, "NT"), 5), ((512, 128, 512, "NN"), 17), ((3072, 384, 256, "NT"), 1), ((512, 2560, 256, "NT"), 1)]:
        plan, launched = both(*call, batch=batch)
        assert launched == plan and plan[0].startswith("dma_128x128x32"), (call, plan, launched)
        assert both(*call, batch=batch, act=wl.ACT_SILU)[1][0].startswith("wavek_") and both(*call, batch=batch, reads_c=True)[1][0].startswith("wavek_"), call
    assert both(512, 512, 136, "NT", batch=4)[1] == w64 and both(512, 640, 128, "NT", batch=4)[1] != w64      # up to one tile to a unit: K > 128
    assert both(1536, 1024, 512)[1] == w64 and both(1536, 1024, 504)[1] != w64                                # beyond: from 512 on, TN 1024
    assert both(1536, 1024, 1024, "TN")[1] == w64 and both(1536, 1024, 1016, "TN")[1] != w64
    assert both(512, 128, 1536, "NT", batch=17)[1] == w64 and both(512, 128, 1528, "NT", batch=17)[1] != w64  # a batch: 1536
    assert both(504, 512, 64, "NT", batch=5)[1] == w64                                                        # ragged


def test_narrow_streams_of_a_long_k_on_few_units():
    """5 to 16 rows on a weight stored N x K: fewer workgroups than half the units draw too little from memory for a long k."""
    narrow, w16 = ("skinny_nt_16x16_w4", 1), ("wavek_16x64x64_w4", 1)
    for call in [(16, 6696, 4112), (9, 6693, 4656), (13, 4045, 3848), (7, 7703, 2552), (8, 4000, 2560), (10, 3999, 3584)]:
        assert both(*call, "NT") == (narrow, narrow), call
    for call in [(16, 6696, 1496), (8, 8200, 3336), (8, 4096, 2560), (8, 4000, 2496), (10, 3999, 1032)]:
        assert both(*call, "NT") == (narrow, w16), call


def test_shares_of_a_long_k_stay():
    """Where few workgroups would stream a row-major weight, and with A stored K x M."""
    quarter, w64 = "dma16p_128x128x32_w2x2_s5", ("wavek_64x64x64_w4", 1)
    for call in [(16, 1000, 4936, "NN"), (30, 2048, 5184, "NN"), (40, 2504, 4168, "NN"), (3584, 256, 6144, "TN"), (904, 1024, 5632, "TT")]:
        plan, launched = both(*call)
        assert plan[0] == quarter and plan[1] > 1 and launched == plan, (call, plan, launched)
    for call in [(10, 2560, 3328, "NN"), (6, 2560, 3072, "NN"), (5, 1024, 4864, "NN")]:                # rows of the weight 512 bytes apart, or a multiple
        plan, launched = both(*call)
        assert plan[0] == quarter and plan[1] > 1 and launched == plan, (call, plan, launched)
    assert both(10, 2568, 3328, "NN")[1] == ("wavek_16x64x64_w4", 1) and both(10, 2560, 2944, "NN")[1] == ("wavek_16x64x64_w4", 1)
    assert both(30, 2040, 4096, "NN")[1] == ("wavek_16x64x64_w4", 1) and both(904, 1024, 4096, "TT")[1] == w64


def test_straddling_rows_with_a_stored_k_by_m():
    """A stored K x M, B row-major, rows of both inside a 128-byte line: more than one 64x64 tile to a unit and a long k
    stay with a C of 16 bits that is only written."""
    small, w64 = ("dma_128x128x32_w2x2_s4", 1), ("wavek_64x64x64_w4", 1)
    for call in [(264, 5904, 2824, "TN"), (296, 4968, 2456, "TN"), (416, 4208, 3776, "TN")]:
        assert both(*call) == (small, small) and both(*call, out=wl.F32, reads_c=True)[1] == w64, call
    for call in [(264, 5888, 2824, "TN"), (264, 5904, 2392, "TN"), (264, 2600, 2824, "TN"), (264, 5904, 2824, "TT")]:
        assert both(*call)[1] == w64, call


def test_calls_off_the_grid_that_stay_on_the_128_tile():
    tiles = "general_128x128x64_w2x2"
    for call in [(2711, 1985, 131, "NN"), (1711, 2679, 157, "NT")]:                       # more than two rounds of 64x64 tiles, a promise of less than 10 %
        assert both(*call) == ((tiles, 1), (tiles, 1)), call
    for call in [(9, 6015, 4201, "NT"), (5, 5501, 4101, "NT"), (5, 6079, 5001, "NT")]:   # few workgroups on a long k
        plan, launched = both(*call)
        assert plan[0] == tiles and plan[1] > 1 and launched == plan, (call, plan, launched)
    for call in [(57, 982, 3883, "NT"), (56, 1474, 5045, "NT"), (64, 330, 5030, "NN"), (125, 734, 3956, "NT"), (43, 1817, 4960, "NN")]:   # in sixteen slices
        assert both(*call) == ((tiles, 16), (tiles, 16)), call
    for call in [(57, 982, 3585, "NT"), (60, 3781, 3989, "NN"), (129, 500, 3989, "NN")]:
        assert both(*call)[1][0] == "general_wavek_16x64x64_w4", call
    assert both(9, 6079, 4095, "NT")[1][0] == "general_wavek_16x64x64_w4" and both(5, 6145, 5001, "NT")[1][0] == "general_wavek_16x64x64_w4"


def test_the_substitution_counts_the_units_of_the_device():
    """The same tiles on half or an eighth of the part: more of them to a unit than the wave tiles are ahead with, and no few-row rule, whose
    limits are workgroups on 256 units."""
    assert both(1016, 1024, 1024, cus=128)[1] == ("wavek_64x64x64_w4", 1)                     # 256 tiles of 64x64, two to a unit
    assert both(1528, 1024, 1024, cus=256)[1] == ("wavek_64x64x64_w4", 1)
    for cus in (32, 128):
        plan, launched = both(1528, 1024, 1024, cus=cus)
        assert launched == plan, (cus, launched)
        for call in [(16, 3032, 264, "NT"), (54, 1000, 688, "NN"), (38, 5552, 1200, "NT"), (14, 13128, 5112, "NT")]:
            plan, launched = both(*call, cus=cus, pad=8)
            assert launched == plan or plan[0].startswith("dma_"), (cus, call, plan, launched)
    assert both(512, 512, 512, dtype=wl.F32, cus=64)[1] == ("f32_64x64x32_w2x2", both(512, 512, 512, dtype=wl.F32, cus=64)[0][1])


def test_query_argument_errors():
    ok = (256, 1, 64, 64, 64, 0, 0, wl.BF16, wl.BF16, 64, 64, 64)
    assert isinstance(lg.gemm_launch_query(*ok, check=False), tuple)
    assert lg.gemm_launch_query(*ok, False, 9, check=False) == lg.GEMM_ERR_INVALID_ARG
    assert lg.gemm_launch_query(0, *ok[1:], check=False) == lg.GEMM_ERR_INVALID_ARG
    assert lg.gemm_launch_query(*ok[:8], wl.F16, *ok[9:], check=False) == lg.GEMM_ERR_UNSUPPORTED


def test_invariants_over_random_calls():
    """Either the plan itself or one launch of a kernel that serves the call: its operand types, a row-major A for the 16-row tiles."""
    rng = random.Random(11)
    dims = [1, 7, 8, 16, 24, 64, 100, 128, 136, 250, 520, 1024, 1368, 2056, 4096, 6696]
    for _ in range(4000):
        M, N, K = rng.choice(dims), rng.choice(dims), rng.choice(dims)
        ta, tb = rng.randint(0, 1), rng.randint(0, 1)
        dtype = rng.choice([wl.BF16, wl.F16, wl.F32])
        out, batch, pad = rng.choice([dtype, wl.F32]), rng.choice([1, 1, 5]), rng.choice([0, 0, 8, 3])
        call = (256, batch, M, N, K, ta, tb, dtype, out, (M if ta else K) + pad, (K if tb else N) + pad, N)
        plan, launched = lg.gemm_plan_query(*call), lg.gemm_launch_query(*call)
        if launched == plan:
            continue
        name = lg.gemm_variant_name(*launched[:2])
        assert launched[2] == 1 and (plan[0] == GENERAL) == (launched[0] == GENERAL), call
        assert name.startswith("f32_") == (dtype == wl.F32), call
        assert not (ta and "wavek_16x" in name), call
        assert launched[0] != GENERAL or (out != wl.F32 and (M >= 8 if ta else K >= 8) and (K >= 8 if tb else N >= 8)), call


def test_the_plan_does_not_depend_on_the_epilogue():
    """A call that was made without reading C, and whose workspace is there therefore, is not cut along k, and needs none, where
    it reads C or has an activation: captured, it could not get any."""
    known = [(112, 6664, 2712, 1, 1), (120, 5656, 2728, 0, 1), (152, 2720, 2920, 0, 1), (1720, 136, 2232, 0, 0), (704, 1424, 7536, 0, 1)]
    rng = random.Random(23)
    some = [(8 * rng.randint(1, 260), 8 * rng.randint(8, 900), 8 * rng.randint(60, 900), rng.randint(0, 1), rng.randint(0, 1)) for _ in range(6000)]
    for M, N, K, ta, tb in known + some:
        for out in (wl.BF16, wl.F32):
            call = (256, 1, M, N, K, ta, tb, wl.BF16, out, M if ta else K, K if tb else N, N)
            plan = lg.gemm_plan_query(*call)
            if plan[0] == TILE and plan[2] == 1:
                assert lg.gemm_launch_query(*call, True)[2] == 1 and lg.gemm_launch_query(*call, True, wl.ACT_GELU_ERF)[2] == 1, call
    plan, launched = both(2048, 2048, 128, "NT", batch=32, reads_c=True)      # (the persistent kernel, but for a C that is read)
    assert plan[0].startswith("shortk_") and launched == ("dma_128x128x32_w2x2_s3", 1)


def test_batches_whose_matrices_the_wave_tiles_spread_over_more_l2s():
    small, w64 = ("dma_128x128x32_w2x2_s4", 1), ("wavek_64x64x64_w4", 1)
    for call, batch in [((360, 120, 1696, "NN"), 42), ((120, 264, 1544, "TN"), 29), ((240, 96, 736, "TT"), 48), ((80, 256, 1888, "NN"), 45),
                        ((152, 176, 888, "TN"), 34)]:
        assert both(*call, batch=batch) == (small, small), call
    for call, batch in [((360, 120, 1696, "NN"), 20), ((360, 120, 256, "TT"), 42), ((568, 64, 568, "NN"), 51), ((592, 64, 1888, "NT"), 37),
                        ((512, 512, 1696, "TT"), 6)]:
        assert both(*call, batch=batch)[1][0].startswith("wavek_"), (call, both(*call, batch=batch))
