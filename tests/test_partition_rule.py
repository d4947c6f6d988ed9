"""What a run launches (ws_gemm_plan_launches), on the host: whatever the rule
chooses, the launches compute every element of C exactly once, with kernels
whose elements take the same products in the same order as the requested
tile's, in a ring that fits."""
import random

import numpy as np
import pytest

from paper_2506_11209_amd import wsgemm as w
from paper_2506_11209_amd.build import MODE_GEMM, instances

CUS = 256
CONFIGS = sorted({(tm, tn, tk, nc, np_, split) for (tm, tn, tk, nc, np_, split, bf16, trace, mode, general)
                  in instances() if mode == MODE_GEMM and not trace})


def depths(tm, tn, tk, np_):
    lo, hi = (1, 2) if np_ == 0 else (2, 8)
    return [P for P in range(lo, hi + 1) if 256 + P * 2 * tk * (tm + tn) <= 163840]


def launches(M, N, K, cfg, general=0):
    s, out = w.ws_gemm_plan_launches(M, N, K, cfg, CUS, general)
    assert s == w.WS_OK, w.ws_gemm_status_str(s)
    return out


def check(M, N, K, cfg, general=0):
    ls = launches(M, N, K, cfg, general)
    _, whole = w.ws_gemm_plan(M, N, K, cfg, CUS, 0)
    assert 1 <= len(ls) <= 2
    unit = min(min(l.tile_m, l.tile_n) for l in ls)
    cover = np.zeros((-(-M // unit), -(-N // unit)), np.int32)
    for l in ls:
        assert (l.tile_k, l.split) == (cfg.tile_k, whole.split)
        assert cfg.tile_m % l.tile_m == 0 and cfg.tile_n % l.tile_n == 0
        if l.general == 0:  # the plain kernel: whole tiles only, and no other epilogue
            assert general == 0 and K % l.tile_k == 0
        assert l.lds_bytes == 256 + l.stages * 2 * l.tile_k * (l.tile_m + l.tile_n) <= 163840
        assert l.stages in depths(l.tile_m, l.tile_n, l.tile_k, l.producer_waves) and l.stages >= cfg.stages
        assert cfg.producer_waves or l.stages == cfg.stages  # synchronous: the depth says whether it overlaps
        assert l.iters == -(-K // l.tile_k) and l.block == 64 * (l.producer_waves + l.consumer_waves)
        assert l.tiles == l.tiles_m * l.tiles_n - l.skip_m * l.skip_n
        assert 1 <= l.grid <= l.tiles and l.rounds == -(-l.tiles // l.grid)
        a, b = l.tile_m // unit, l.tile_n // unit
        mark = np.zeros((l.tiles_m * a, l.tiles_n * b), np.int32)
        mark[:] = 1
        mark[:l.skip_m * a, :l.skip_n * b] = 0
        if l.general == 0:
            assert l.tiles_m * l.tile_m <= M and l.tiles_n * l.tile_n <= N
        r, c = min(mark.shape[0], cover.shape[0]), min(mark.shape[1], cover.shape[1])
        cover[:r, :c] += mark[:r, :c]
    assert np.all(cover == 1)
    if len(ls) == 1 and (ls[0].tile_m, ls[0].tile_n) == (cfg.tile_m, cfg.tile_n):
        assert ls[0].stages == cfg.stages and ls[0].consumer_waves == cfg.consumer_waves
    return ls


@pytest.mark.parametrize("c", CONFIGS, ids=lambda c: "%dx%dx%d-nc%d-np%d-%d" % c)
def test_launches_cover_c_once(c):
    tm, tn, tk, nc, np_, split = c
    rng = random.Random(repr(c))
    kinds = set()
    for _ in range(60):
        cfg = w.config((tm, tn, tk), rng.choice(depths(tm, tn, tk, np_)), np_, nc, rng.choice(("bf16", "f16")),
                       rng.choice(("registers", "dma")), split)
        if rng.random() < 0.5 or np_ == 0:  # whole tiles
            M, N, K = (t * rng.choice((1, 2, 3, 7, 15, 16, 17, 33)) for t in (tm, tn, tk))
        else:
            M = rng.randrange(1, 40 * tm)
            N, K = 8 * rng.randrange(1, 5 * tn), 8 * rng.randrange(1, 5 * tk)
        ls = check(M, N, K, cfg, int(np_ > 0 and rng.random() < 0.3))
        kinds.add("rest" if len(ls) == 2 else "whole" if ls[0].tile_m * ls[0].tile_n == tm * tn else "parts")
    assert "whole" in kinds
    assert (tm * tn > (1024 if nc == 1 else 4096)) == ("parts" in kinds)


@pytest.mark.parametrize("M,N,K,launch,tiles", [
    (256, 256, 256, ((64, 64, 32), 2, 1, 1), [(32, 32, 4)]),
    (1024, 1024, 1024, ((128, 128, 64), 3, 4, 4), [(64, 64, 6)]),
    (2048, 2048, 4096, ((256, 256, 64), 2, 4, 8), [(128, 128, 4)]),
    (4100, 4104, 4104, ((256, 256, 64), 2, 4, 8), [(256, 256, 2), (64, 64, 8)]),
    (4096, 4096, 4096, ((128, 128, 32), 3, 4, 4), [(128, 128, 3)]),
    (8192, 8192, 8192, ((256, 256, 64), 2, 4, 8), [(256, 256, 2)]),
    (2056, 1160, 5120, ((128, 64, 64), 4, 8, 4), [(128, 64, 4), (64, 64, 6)]),
    # no rest where it shares one round with the block: launches of one round, one consumer wave
    (640, 3520, 5376, ((128, 64, 32), 2, 4, 4), [(128, 64, 2)]),
    (1337, 872, 5992, ((64, 64, 64), 3, 1, 1), [(64, 64, 3)]),
    (1100, 1032, 5120, ((64, 64, 64), 3, 1, 1), [(64, 64, 3)]),
    # synchronous, two buffers, alone on its CU: whole once every CU has a tile, unless K is short
    (19200, 1024, 2048, ((256, 256, 32), 2, 0, 4), [(256, 256, 2)]),
    (4096, 1024, 2048, ((256, 256, 32), 2, 0, 4), [(128, 128, 2)]),
    (2816, 6144, 160, ((256, 256, 32), 2, 0, 4), [(128, 128, 2)]),
])
def test_choices_of_the_rule(M, N, K, launch, tiles):
    assert [(l.tile_m, l.tile_n, l.stages) for l in check(M, N, K, w.config(*launch))] == tiles


def test_refusals_are_those_of_the_plan():
    for M, N, K, cfg in ((100, 100, 100, w.config((64, 64, 64), 3, 4, 4)),       # rows of 16 bytes
                         (100, 128, 128, w.config((64, 64, 64), 2, 0, 4)),       # synchronous: whole tiles
                         (128, 128, 128, w.config((256, 256, 64), 4, 4, 8)),     # LDS
                         (128, 128, 128, w.config((128, 128, 64), 9, 4, 4)),
                         (128, 128, 128, w.config((128, 128, 128), 2, 4, 4)),    # no such kernel
                         (-1, 128, 128, w.config((64, 64, 64), 3, 4, 4))):
        s, _ = w.ws_gemm_plan_launches(M, N, K, cfg, CUS)
        assert s == w.ws_gemm_plan(M, N, K, cfg, CUS, 0)[0] != w.WS_OK
    s, ls = w.ws_gemm_plan_launches(0, 64, 64, w.config((64, 64, 64), 3, 4, 4), CUS)
    assert s == w.WS_OK and ls == []
