"""The generated asm K loops in every configuration that runs them: the streaming
consumer (ws_stream_loop.inc: one and four consumer waves, in the plain and the
general kernels) and the register-lean loop of eight consumer waves
(ws_deep_loop.inc).  Their prologues, loop bodies and last k-steps (1-8
K-iterations per tile; fewer than a loop body takes the compiler-scheduled
consumer instead), slot wrap-around at ring depths two to four, several output
tiles per workgroup, both producer load paths, the polling and draining paths
(late producers), the consumer delay hook and the watchdog.

Operands are small integers, so every product is exact: C is compared with
the oracle on sampled rows and, over all of C, by an exact checksum
C x == A (B x) for a random +-1 vector x (fp64, integer-valued sums)."""
import os
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle.check import compare_exact
from paper_2506_11209_amd import inputs
from tests.gpu_helpers import log, sample_rows

w = pytest.importorskip("paper_2506_11209_amd.wsgemm")

pytestmark = pytest.mark.gpu

sys.path.insert(0, os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                                "paper_2506_11209_amd", "csrc"))
import gen_deep_loop  # noqa: E402  (the lists of configurations with a generated loop)
import gen_stream_loop  # noqa: E402

LDS_LIMIT = 163840
# (tm, tn, tk, consumer waves, producer waves, split)
CONFIGS = ([(tm, tn, tk, nc, np_, split) for (tm, tn, tk, nc, np_) in gen_stream_loop.CONFIGS
            for split in ((1, 2) if (nc, np_) == (4, 4) else (np_ // nc,))] +
           [(tm, tn, tk, nc, np_, split) for (tm, tn, tk, nc, np_) in gen_deep_loop.ROLL_CONFIGS if nc == 8
            for split in (1, 2)])


def cfg_id(t):
    return "%dx%dx%d-nc%d-np%d-%d:1" % t


def max_stages(tile):
    tm, tn, tk = tile
    return (LDS_LIMIT - 256) // (2 * (tm * tk + tk * tn))


def several_rounds(cfg, iters):
    """M, N, K of more tiles than workgroups at every ring depth, the last round not full."""
    tm, tn, tk, nc, np_, split = cfg
    cols = 17
    while True:
        M, N, K = 33 * tm, cols * tn, iters * tk
        plans = [w.ws_gemm_plan(M, N, K, w.config((tm, tn, tk), P, np_, nc, split=split), 256)[1]
                 for P in range(2, min(4, max_stages((tm, tn, tk))) + 1)]
        if all(p.tiles > 2 * p.grid for p in plans):
            return M, N, K
        cols *= 2


class Product:
    """Integer operands of one product on the GPU, its rows from the oracle and
    its exact checksum."""

    def __init__(self, M, N, K, tm, dtype="bf16", seed=0):
        self.shape, self.dtype = (M, N, K), dtype
        A, B = inputs.make_operands(M, N, K, dtype, "int4", seed)
        self.rows = sample_rows(M, tm, n_random=16, seed=seed)
        self.ref, _ = oracle.gemm_rows(inputs.bits(A), inputs.bits(B), dtype, self.rows)
        self.A, self.B = A.cuda(), B.cuda()
        x = np.random.default_rng(seed).choice([-1.0, 1.0], size=N)
        self.x = torch.from_numpy(x).cuda()
        self.sum = self.A.double() @ (self.B.double() @ self.x)

    def check(self, C):
        r = compare_exact(C[torch.as_tensor(self.rows, device="cuda")].cpu().numpy(), self.ref)
        assert r["ok"], r
        assert torch.equal(C.double() @ self.x, self.sum), "checksum over all of C differs"


def run_and_check(p, tile, stages, load_path="registers", debug=None, split=1, nc=4, np_=None):
    M, N, K = p.shape
    np_ = 4 * split if np_ is None else np_
    g = w.WsGemm(M, N, K, tile, stages, np_, nc, p.dtype, load_path, split=split, whole_tiles=True)
    try:
        if debug:
            g.set_debug(*debug)
        C = torch.full((M, N), float("nan"), device="cuda")
        g(p.A, p.B, C)
        st = g.sync_status()
        assert st == w.WS_OK, w.ws_gemm_status_str(st)
        p.check(C)
        return g.info.as_dict()
    finally:
        g.close()


@pytest.mark.parametrize("load_path", ["registers", "dma"])
@pytest.mark.parametrize("iters", [1, 2, 3, 4, 7, 8])
@pytest.mark.parametrize("cfg", CONFIGS, ids=cfg_id)
def test_k_iterations_and_ring_depths(cfg, iters, load_path):
    tm, tn, tk, nc, np_, split = cfg
    tile = (tm, tn, tk)
    p = Product(*several_rounds(cfg, iters), tm, seed=100 * iters)
    for stages in range(2, min(4, max_stages(tile)) + 1):
        log("case deep %s nc=%d np=%d %d:1 S=%d P=%d %s" % (tile, nc, np_, split, iters, stages, load_path))
        info = run_and_check(p, tile, stages, load_path=load_path, split=split, nc=nc, np_=np_)
        assert info["iters"] == iters and info["general"] == 0  # the plain kernel
        assert info["rounds"] > 2, "each workgroup must take several tiles"


@pytest.mark.parametrize("cfg", CONFIGS, ids=cfg_id)
def test_general_kernel_takes_several_ragged_tiles(cfg):
    tm, tn, tk, nc, np_, split = cfg
    M, N, K = several_rounds(cfg, 5)
    p = Product(M - 3, N - 8, K - 8, tm, seed=3)
    for stages in (2, min(3, max_stages((tm, tn, tk)))):
        log("case deep general %s nc=%d np=%d %d:1 P=%d" % ((tm, tn, tk), nc, np_, split, stages))
        assert run_and_check(p, (tm, tn, tk), stages, split=split, nc=nc, np_=np_)["general"] == 1


@pytest.mark.parametrize("cfg", CONFIGS, ids=cfg_id)
def test_f16(cfg):
    tm, tn, tk, nc, np_, split = cfg
    log("case deep f16 %s nc=%d np=%d %d:1" % ((tm, tn, tk), nc, np_, split))
    run_and_check(Product(8 * tm, 8 * tn, 640, tm, dtype="f16", seed=7), (tm, tn, tk), 2, split=split, nc=nc, np_=np_)


@pytest.mark.parametrize("load_path", ["registers", "dma"])
@pytest.mark.parametrize("pdelay,cdelay", [(3, 0), (0, 3), (2, 2)])
@pytest.mark.parametrize("cfg", [c for c in CONFIGS if c[3] < 8], ids=cfg_id)
def test_delays_of_the_streaming_consumer(cfg, pdelay, cdelay, load_path):
    # late producers make the consumer's peek come up short, so it drains (rings of
    # two and three slots at T_K = 64) or polls; a late consumer fills the ring
    tm, tn, tk, nc, np_, split = cfg
    p = Product(2 * tm, 2 * tn, 7 * tk, tm, seed=13)
    for stages in range(2, min(4, max_stages((tm, tn, tk))) + 1):
        log("case deep delays %s nc=%d np=%d %d:1 p=%d c=%d P=%d %s" % ((tm, tn, tk), nc, np_, split, pdelay, cdelay,
                                                                      stages, load_path))
        run_and_check(p, (tm, tn, tk), stages, load_path, debug=(0, pdelay, cdelay), split=split, nc=nc, np_=np_)


@pytest.mark.parametrize("pdelay,cdelay", [(3, 0), (0, 3), (2, 2)])
def test_late_producers_and_consumer_delay(pdelay, cdelay):
    log("case deep delays p=%d c=%d" % (pdelay, cdelay))
    run_and_check(Product(1024, 512, 768, 256, seed=13), (256, 128, 64), 3, debug=(0, pdelay, cdelay))


@pytest.mark.parametrize("split", [1, 2])
@pytest.mark.parametrize("pdelay,cdelay", [(3, 0), (0, 3), (2, 2)])
def test_late_producers_and_consumer_delay_eight_consumers(pdelay, cdelay, split):
    log("case roll delays p=%d c=%d split=%d" % (pdelay, cdelay, split))
    run_and_check(Product(1024, 512, 768, 256, seed=14), (256, 256, 64), 2, debug=(0, pdelay, cdelay), split=split,
                  nc=8, np_=4)


def test_watchdog_eight_consumers():
    A, B = inputs.make_operands(1024, 512, 1024, "bf16", "int4", 18)
    log("case roll watchdog")
    g = w.WsGemm(1024, 512, 1024, (256, 256, 64), 2, 4, 8, "bf16", whole_tiles=True)
    try:
        Ad, Bd = A.cuda(), B.cuda()
        g.set_debug(1, 20, 0)  # one poll allowed, producers ~160k cycles late
        g(Ad, Bd)
        assert g.sync_status() == w.WS_ERR_TIMEOUT
        assert g.sync_status() == w.WS_OK
        g.set_debug(0, 0, 0)
        C = g(Ad, Bd)
        assert g.sync_status() == w.WS_OK
        Cref, _ = oracle.gemm(inputs.bits(A), inputs.bits(B), "bf16", with_abs=False)
        assert compare_exact(C.cpu().numpy(), Cref)["ok"]
    finally:
        g.close()


def test_watchdog_reports_timeout_then_recovers():
    A, B = inputs.make_operands(1024, 512, 1024, "bf16", "int4", 17)
    log("case deep watchdog")
    g = w.WsGemm(1024, 512, 1024, (256, 128, 64), 3, 4, 4, "bf16", whole_tiles=True)
    try:
        Ad, Bd = A.cuda(), B.cuda()
        g.set_debug(1, 20, 0)  # one poll allowed, producers ~160k cycles late
        g(Ad, Bd)
        assert g.sync_status() == w.WS_ERR_TIMEOUT
        assert g.sync_status() == w.WS_OK
        g.set_debug(0, 0, 0)
        C = g(Ad, Bd)
        assert g.sync_status() == w.WS_OK
        Cref, _ = oracle.gemm(inputs.bits(A), inputs.bits(B), "bf16", with_abs=False)
        assert compare_exact(C.cpu().numpy(), Cref)["ok"]
    finally:
        g.close()
