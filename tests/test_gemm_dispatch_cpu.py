"""The GEMM launcher's choice of a tile (host code only; no device)."""
import ctypes
import random

import numpy as np
import pytest

from paper_2605_10793_amd import binding

EPI_SIGN, EPI_ACT, EPI_F32, EPI_GRAMW, EPI_XOUT, EPI_SQUARE = 0, 1, 2, 3, 4, 5


def tile(epi, f16, symmetric, M, N, K, nseg=1, batch=1):
    """(rows, columns, wavefronts, workgroups per batch entry, mirrored)"""
    out = (ctypes.c_int * 5)()
    binding.load().conqur_gemm_tile_for_tests(epi, f16, symmetric, M, N, K, nseg, batch, out)
    return tuple(out)


def test_segments_count_as_k_steps():
    """A product of n segments runs n times the K steps: it takes the tile one segment of n K elements takes."""
    rng = random.Random(5)
    for _ in range(500):
        M, N, K = rng.randint(1, 9000), 16 * rng.randint(1, 300), 64 * rng.randint(1, 64)
        nseg, batch = rng.choice([2, 3, 4, 6]), rng.choice([1, 1, 4, 16])
        for epi, f16 in ((EPI_ACT, 0), (EPI_SIGN, 0), (EPI_F32, 0)):
            assert tile(epi, f16, 0, M, N, K, nseg, batch) == tile(epi, f16, 0, M, N, K * nseg, 1, batch), (M, N, K, nseg, batch)


@pytest.mark.parametrize("T,heads,dh,nseg", [(815, 8, 384, 6), (279, 32, 256, 6), (7654, 1, 336, 6), (6250, 1, 448, 6), (393, 16, 384, 1)])
def test_many_small_tiles_give_way_to_larger_ones(T, heads, dh, nseg):
    """Rotations whose 64 x 64 tiles share the compute units three at a time: 128 x 128 was measured 1.2 to 1.6 times as fast."""
    assert tile(EPI_ACT, 0, 0, T, dh, dh, nseg, heads)[:2] == (128, 128)


@pytest.mark.parametrize("d", [2048, 4256, 5120, 5632, 7424, 8192])
def test_epilogues_without_the_registers_stay_off_the_largest_tile(d):
    for nseg in (1, 2, 4, 6):
        for epi, sym in ((EPI_SQUARE, 1), (EPI_GRAMW, 1), (EPI_XOUT, 0)):
            assert tile(epi, 0, sym, d, d, d, nseg)[:2] != (256, 256)


def test_workgroups_cover_the_output():
    rng = random.Random(6)
    for _ in range(300):
        M, N, K = rng.randint(1, 9000), 16 * rng.randint(1, 300), 8 * rng.randint(1, 600)
        bm, bn, waves, wg, mirrored = tile(EPI_ACT, 0, 0, M, N, K)
        assert wg == -(-M // bm) * -(-N // bn) and not mirrored and waves in (4, 8)
        bm, bn, waves, wg, mirrored = tile(EPI_GRAMW, 1, 1, N, N, N)
        side = -(-N // bm)
        assert wg == (side * (side + 1) // 2 if mirrored else side * -(-N // bn)) and (not mirrored or (bm == bn and side >= 8))


@pytest.mark.parametrize("sym", [0, 1])
def test_every_tile_of_a_grid_is_one_workgroups(sym):
    """Whole and mirrored grids, along lines and in bands: each tile is computed by exactly one workgroup."""
    L = binding.load()
    rng = np.random.default_rng(0)
    grids = [(1, 1), (1, 9), (9, 1), (7, 8), (16, 16), (43, 16), (13, 17), (33, 5), (64, 64), (65536, 1), (3000, 700)]
    grids += [tuple(int(v) for v in rng.integers(1, 70, 2)) for _ in range(60)]
    for m, n in grids:
        if sym:
            m = n = min(m, 1000)
        count = m * (m + 1) // 2 if sym else m * n
        for epi in (1, 4):
            for batch, steps in ((1, 4), (1, 64), (32, 64)):
                tm, tn = np.full(count, -1, np.int32), np.full(count, -1, np.int32)
                L.conqur_gemm_order_for_tests(epi, sym, m, n, 128, 192, batch, steps, tm.ctypes.data_as(ctypes.c_void_p), tn.ctypes.data_as(ctypes.c_void_p))
                assert tm.min() >= 0 and tm.max() < m and tn.min() >= 0 and tn.max() < n
                assert not sym or (tm <= tn).all()
                assert np.unique(tm.astype(np.int64) * n + tn).size == count


@pytest.mark.parametrize("dh,heads,T,one_launch", [
    (16, 2, 65536, 1), (32, 256, 16384, 1), (64, 32, 2048, 1), (48, 2, 65536, 0), (64, 2, 1024, 1), (64, 4, 16384, 0), (80, 4, 8192, 0), (80, 40, 8192, 1),
    (96, 2, 512, 1), (96, 16, 16384, 0), (96, 48, 512, 1), (96, 48, 4096, 0), (96, 128, 4096, 1), (112, 2, 1024, 1), (112, 2, 4096, 0), (112, 4, 65536, 0),
    (112, 8, 8192, 0), (112, 40, 200, 1), (112, 40, 2048, 0), (112, 40, 8192, 0), (112, 256, 64, 0), (64, 1, 2048, 0), (128, 8, 512, 0)])
def test_narrow_heads_take_the_faster_statistics_step(dh, heads, T, one_launch):
    """One launch or the general path's three, as measured: each of these is at least 1.1 times as fast the way stated.  (One head
    and heads of width 128 have other ways.)"""
    L = binding.load()
    assert L.conqur_head_step_narrow_for_tests(dh, heads, ctypes.c_int64(T)) == one_launch


def in_bands(T, d, heads, nseg):
    """Whether a rotation's tiles are taken in bands, not along the rows or columns of its grid."""
    bm, bn = tile(EPI_ACT, 0, 0, T, d, d, nseg, heads)[:2]
    m, n = -(-T // bm), -(-d // bn)
    buf = np.empty((2, m * n), np.int32)
    bands = binding.load().conqur_gemm_order_for_tests(EPI_ACT, 0, m, n, bm, bn, heads, -(-d // 64) * nseg, buf[0].ctypes.data_as(ctypes.c_void_p),
                                                       buf[1].ctypes.data_as(ctypes.c_void_p))
    return 1 < bands < m   # (1: down the columns; m: along the rows)


@pytest.mark.parametrize("T,d,heads,nseg,bands", [
    (1936, 1040, 1, 6, 0), (4000, 1040, 1, 6, 0), (1100, 480, 1, 6, 0), (1500, 800, 1, 6, 0), (1936, 400, 1, 6, 0), (6000, 2096, 1, 1, 0), (603, 2096, 1, 1, 0),
    (9190, 3344, 1, 1, 0), (9190, 304, 8, 1, 0), (12000, 304, 8, 1, 0), (777, 1040, 1, 6, 1), (872, 944, 1, 6, 1), (868, 1152, 1, 6, 1), (9190, 4096, 1, 1, 1),
    (11008, 4096, 1, 1, 1), (4045, 4480, 1, 1, 1), (12000, 5120, 1, 1, 1)])
def test_rotations_take_the_faster_order_of_tiles(T, d, heads, nseg, bands):
    """As measured: each of these rotations is 3 to 18 % faster in the order stated than in the other."""
    assert in_bands(T, d, heads, nseg) == bool(bands)


@pytest.mark.parametrize("epi,m,n,bm,bn,rows", [(EPI_F32, 16, 16, 256, 256, 4), (EPI_F32, 32, 32, 256, 256, 4), (EPI_F32, 16, 16, 128, 128, 4),
                                                (EPI_F32, 16, 16, 64, 64, 4), (EPI_F32, 16, 16, 192, 192, 4), (EPI_XOUT, 32, 32, 256, 256, 4),
                                                (EPI_ACT, 32, 8, 256, 256, 4), (EPI_ACT, 16, 32, 64, 64, 8)])
def test_the_wider_of_two_blocks_that_read_the_same(epi, m, n, bm, bn, rows):
    """Whole 4 x 8 or 8 x 4 blocks: the tiles an XCD takes at a time span so many tile rows (as measured, 1 to 6 % of a launch)."""
    buf = np.empty((2, m * n), np.int32)
    binding.load().conqur_gemm_order_for_tests(epi, 0, m, n, bm, bn, 1, 32, buf[0].ctypes.data_as(ctypes.c_void_p), buf[1].ctypes.data_as(ctypes.c_void_p))
    for xcd in range(8):
        mine = buf[:, xcd::8][:, :32]
        assert len(set(mine[0])) == rows and len(set(mine[1])) == 32 // rows


def test_a_grid_of_no_whole_blocks_keeps_the_taller_one():
    """11008 x 4096 rotated in 256 x 256 tiles: bands of 7 and 8 rows (as measured, 1.5 % of the launch)."""
    buf = np.empty((2, 43 * 16), np.int32)
    assert binding.load().conqur_gemm_order_for_tests(EPI_ACT, 0, 43, 16, 256, 256, 1, 64, buf[0].ctypes.data_as(ctypes.c_void_p),
                                                      buf[1].ctypes.data_as(ctypes.c_void_p)) == 6
