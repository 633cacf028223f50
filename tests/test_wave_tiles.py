"""CPU checks of the tiles whose k range is divided among the waves: the loads of their movers stay inside the operand and put
every element where the fragment reads look for it (the arithmetic of tile_wavek_kernel.hpp, restated), and the generated code
touches no fragment register before its wait.  (Which lanes of a read the LDS serves together, and so its bank conflicts, is not
checked here.)"""
import os

import numpy as np
import pytest

from asm_inflight import check_listing

LANES = np.arange(64)


def kc_hash(r):
    return (r ^ ((r >> 3) & 1)) & 7


def mc_swizzle(k):
    return (k & 2) | (((k >> 3) & 1) << 2)


def slab_loads(kc, rows, valid, ld, K, slab):
    """(byte offset in the operand, LDS byte, fetched) of every lane's 16 bytes of one slab."""
    k_left = K - slab * 64
    for q in range(rows // 8):
        if kc:
            row = 8 * q + (LANES >> 3)
            c = (LANES & 7) ^ kc_hash(row)
            off = np.minimum(row, valid - 1) * ld * 2 + c * 16 + slab * 128
            k = c * 8
        else:
            k = 8 * (q % 8) + (LANES >> 3)
            c = ((LANES & 7) ^ mc_swizzle(k)) + 8 * (q // 8)
            off = (k * ld + np.where(c * 8 + 8 <= valid, c * 8, valid - 8)) * 2 + slab * 128 * ld
        yield off, q * 1024 + LANES * 16, k < k_left


@pytest.mark.parametrize("kc,rows", [(True, 64), (True, 16), (False, 64)])
@pytest.mark.parametrize("K", [8, 64, 72, 136, 256])
def test_loads_stay_inside_and_the_fragments_find_their_elements(kc, rows, K):
    for valid in (8, 24, 56, 64) if not kc else (1, 7, 16, 63, 64):
        if valid > rows:
            continue
        for ld in ((K if kc else valid), (K if kc else valid) + 8):
            # the operand as its elements' own indices
            n = (valid - 1) * ld + K if kc else (K - 1) * ld + valid
            for slab in range((K + 63) // 64):
                lds = np.full(rows * 64, -1, np.int64)          # element index held by every 16-bit place, -1: zero
                for off, at, fetched in slab_loads(kc, rows, valid, ld, K, slab):
                    assert np.all(off[fetched] + 16 <= n * 2)
                    for o, a, f in zip(off, at, fetched):
                        lds[a // 2: a // 2 + 8] = np.arange(8) + o // 2 if f else -1
                r, g = LANES & 15, LANES >> 4
                for tile in range(rows // 16):
                    for ks in range(2):
                        for e in range(8):
                            k = 32 * ks + 8 * g + e
                            row = 16 * tile + r
                            if kc:
                                place = tile * 2048 + r * 128 + (((4 * ks + g) ^ kc_hash(r)) << 4) + 2 * e
                            else:
                                # a transposing read: lane i of 16 receives column i of the four k-rows that lanes 4j .. 4j+3 address
                                col = 16 * tile + 4 * (r >> 2)
                                place = k * 128 + (((col >> 3) ^ mc_swizzle(k)) << 4) + (col & 7) * 2 + 2 * (r & 3)
                            got = lds[place // 2]
                            inside = (row < valid) & (slab * 64 + k < K)
                            want = row * ld + slab * 64 + k if kc else (slab * 64 + k) * ld + row
                            assert np.array_equal(got[inside], want[inside])
                            past_k = slab * 64 + k >= K
                            assert np.all(got[past_k] == -1)                   # zeros


def any_loads(kc, rows, first, valid, ld, K, slab):
    """(element index relative to the operand, LDS byte, fetched, elements dropped) of every lane's load off the grid."""
    k_left = K - slab * 64
    for q in range(rows // 8):
        if kc:
            row = 8 * q + (LANES >> 3)
            k = ((LANES & 7) ^ kc_hash(row)) * 8
            drop = np.where((k + 8 > k_left) & (k_left < 64), -k_left % 8, 0)
            off = (first + np.minimum(row, valid - 1)) * ld + slab * 64 + k - drop
            yield off, q * 1024 + LANES * 16, k < k_left, drop
        else:
            k = 8 * q + (LANES >> 3)
            c8 = ((LANES & 7) ^ mc_swizzle(k)) * 8
            off = (slab * 64 + k) * ld + first + np.where(c8 + 8 <= valid, c8, valid - 8)
            yield off, q * 1024 + LANES * 16, k < k_left, np.where((c8 == valid // 8 * 8) & (valid % 8 != 0), -valid % 8, 0)


@pytest.mark.parametrize("kc,rows", [(True, 64), (True, 16), (False, 64)])
@pytest.mark.parametrize("K", [9, 63, 65, 131])
def test_loads_off_the_grid_stay_inside_and_land_in_place(kc, rows, K):
    for total in (9, 63, 64, 67, 129):
        ld = (K if kc else total) + 1
        n = (total - 1) * ld + K if kc else (K - 1) * ld + total
        for first in range(0, total, rows):
            valid = min(rows, total - first)
            for slab in range((K + 63) // 64):
                lds = np.full(rows * 64, -1, np.int64)
                for off, at, fetched, drop in any_loads(kc, rows, first, valid, ld, K, slab):
                    assert np.all(off[fetched] >= 0) and np.all(off[fetched] + 8 <= n), (total, first, slab)
                    for o, a, f, d in zip(off, at, fetched, drop):
                        lds[a // 2: a // 2 + 8] = -1
                        if f:
                            lds[a // 2: a // 2 + 8 - d] = np.arange(d, 8) + o
                for row in range(valid):
                    for k in range(64):
                        if kc:
                            place = row * 128 + (((k // 8) ^ kc_hash(np.int64(row))) << 4) + k % 8 * 2
                        else:
                            place = k * 128 + (((row // 8) ^ mc_swizzle(np.int64(k))) << 4) + row % 8 * 2
                        inside = slab * 64 + k < K
                        want = ((first + row) * ld + slab * 64 + k if kc else (slab * 64 + k) * ld + first + row) if inside else -1
                        assert lds[place // 2] == want, (total, first, slab, row, k)


def f32_mc_row(rows, q):
    position = q * (256 // rows) + LANES // (rows // 4)
    return position, 8 * (position & 3) + (position >> 2)


def f32_loads(kc, rows, valid, ld, K, slab):
    """(element in the operand, LDS dword, fetched) of every lane's 16 bytes of one fp32 slab."""
    k_left = K - slab * 32
    for q in range(rows // 8):
        if kc:
            row = 8 * q + (LANES >> 3)
            k = ((LANES & 7) ^ kc_hash(row)) * 4
            off = np.minimum(row, valid - 1) * ld + slab * 32 + k
        else:
            position, k = f32_mc_row(rows, q)
            c = (LANES % (rows // 4)) ^ (((position & 2) << 1) if rows == 32 else 0)
            off = (slab * 32 + k) * ld + np.where(c * 4 + 4 <= valid, c * 4, valid - 4)
        yield off, q * 256 + LANES * 4, k < k_left


@pytest.mark.parametrize("kc", [True, False])
@pytest.mark.parametrize("rows", [16, 32])
@pytest.mark.parametrize("K", [4, 32, 36, 100])
def test_fp32_loads_stay_inside_and_the_fragments_find_their_elements(kc, rows, K):
    for valid in (4, 12, 16, 28, 32) if not kc else (1, 7, 16, 31, 32):
        if valid > rows:
            continue
        ld = (K if kc else valid) + 4
        n = (valid - 1) * ld + K if kc else (K - 1) * ld + valid
        for slab in range((K + 31) // 32):
            lds = np.full(rows * 32, -1, np.int64)
            for off, at, fetched in f32_loads(kc, rows, valid, ld, K, slab):
                assert np.all(off[fetched] >= 0) and np.all(off[fetched] + 4 <= n)
                for o, a, f in zip(off, at, fetched):
                    lds[a: a + 4] = np.arange(4) + o if f else -1
            r, g = LANES & 15, LANES >> 4
            for tile in range(rows // 16):
                for e in range(8):
                    if kc:
                        byte = tile * 2048 + r * 128 + (((2 * g + e // 4) ^ kc_hash(r)) << 4) + e % 4 * 4
                    else:
                        byte = g * rows * 4 + (((tile ^ (g >> 1)) << 6) if rows == 32 else 0) + r * 4 + e * (rows * 4 // 64) * 256
                    k, row = slab * 32 + 8 * g + e, 16 * tile + r
                    got = lds[byte // 4]
                    inside = (row < valid) & (k < K)
                    assert np.array_equal(got[inside], (row * ld + k if kc else k * ld + row)[inside])
                    assert np.all(got[k >= K] == -1)


def test_no_fragment_register_is_touched_before_its_wait(tmp_path):
    from paper_2512_16465_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    for unit, kernels in (("tile_variant_18", 8), ("tile_variant_19", 4), ("tile_wave_any", 12), ("tile_variant_20", 4), ("tile_variant_21", 4)):
        path = build.device_assembly(unit + ".hip", str(tmp_path / (unit + ".s")))
        with open(path) as f:
            n, found = check_listing(f, only="tile_wavek")
        assert n == kernels and not found, (n, found[:1])
