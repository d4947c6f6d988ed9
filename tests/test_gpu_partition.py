"""Problems whose tiles are computed in parts, or as a block of whole tiles and
a rest (ws_gemm_run's choice where whole tiles leave the GPU idle): sizes
around the block's edges, both tile regions of the rest, every entry point.
Which launches a case takes is asserted.  Integer operands: every compared
element is exact; C is pre-filled with NaN and guarded behind its end, so a
tile left out or written twice past an edge shows."""
import numpy as np
import pytest
import torch

import oracle
from oracle.check import compare_exact
from paper_2506_11209_amd import inputs
from tests.gpu_helpers import log, sample_rows

w = pytest.importorskip("paper_2506_11209_amd.wsgemm")

pytestmark = pytest.mark.gpu

T128 = ((128, 128, 64), 3, 4, 4)
T256 = ((256, 256, 64), 2, 4, 8)
# (M, N, K), launch, dtype, load path
PARTS = [
    # every tile in parts: few whole tiles, ragged ones, both ends of the sizes
    ((1024, 1024, 256), T128, "bf16", "registers"),
    ((128, 128, 64), T128, "bf16", "dma"),
    ((1, 8, 8), T128, "f16", "registers"),
    ((520, 264, 136), T256, "bf16", "registers"),
    ((2048, 512, 128), ((256, 128, 32), 4, 8, 4), "bf16", "registers"),
    ((256, 256, 64), ((64, 64, 32), 2, 1, 1), "f16", "registers"),
    ((100, 72, 200), ((64, 64, 64), 2, 2, 1), "bf16", "registers"),
    ((544, 416, 96), ((64, 64, 32), 4, 1, 1), "bf16", "dma"),
]
RESTS = [
    # a block of whole tiles (16 x 16 or more) and the rest below / right / both
    ((2049, 2048, 1280), T128, "bf16", "registers"),
    ((2048, 2056, 1280), T128, "f16", "registers"),
    ((2056, 2056, 1304), T128, "bf16", "registers"),
    ((2176, 2048, 1280), T128, "bf16", "dma"),          # whole tiles: a last round of one tile row
    ((2048, 2176, 1280), ((128, 128, 32), 3, 8, 4), "bf16", "registers"),
    ((4100, 4104, 264), T256, "bf16", "registers"),
    ((4100, 4104, 1288), T256, "f16", "registers"),
    ((4100, 2056, 1280), ((256, 128, 64), 3, 4, 4), "bf16", "registers"),
    ((2056, 1160, 5128), ((128, 64, 64), 4, 8, 4), "f16", "registers"),
]
WHOLE = [
    # one consumer wave: the tiles past the last whole round share the CUs with the others
    ((1100, 1032, 5120), ((64, 64, 64), 3, 1, 1), "bf16", "registers"),
]
CASES = [c + (1,) for c in PARTS] + [c + (2,) for c in RESTS] + [c + (0,) for c in WHOLE]
GUARD, SENTINEL = 4096, -7.0


def rows_of(M, tm):
    return sample_rows(M, tm, 12) if M > 600 else np.arange(M)


def check(C, A, B, dtype, tm, scale=1.0):
    assert np.all(np.isfinite(C)), "elements of C not written"
    rows = np.unique(np.concatenate([rows_of(C.shape[0], tm), np.array([C.shape[0] // tm * tm - 1]).clip(0)]))
    ref, _ = oracle.gemm_rows(inputs.bits(A), inputs.bits(B), dtype, rows, with_abs=False)
    r = compare_exact(C[rows], scale * ref)
    assert r["ok"], r


def tile_of(launch):
    return launch.tile_m, launch.tile_n, launch.tile_k


@pytest.mark.parametrize("shape,launch,dtype,path,count", CASES, ids=str)
def test_partitioned_products_are_exact(shape, launch, dtype, path, count):
    M, N, K = shape
    tile, P, np_, nc = launch
    log("case partition %s %s %s %s" % (shape, launch, dtype, path))
    A, B = inputs.make_operands(M, N, K, dtype, "int4", M + N + K)
    Ad, Bd = A.cuda(), B.cuda()
    g = w.WsGemm(M, N, K, tile, P, np_, nc, dtype, path)
    try:
        ls = g.launches()
        assert len(ls) == max(count, 1)
        assert (tile_of(ls[-1]) == tile) == (count == 0)  # in parts, or a block and the rest in parts
        assert count == 1 or tile_of(ls[0]) == tile
        _, planned = w.ws_gemm_plan_launches(M, N, K, g.cfg, torch.cuda.get_device_properties(0).multi_processor_count)
        assert [x.as_dict() for x in planned] == [x.as_dict() for x in ls]
        buf = torch.full((M * N + GUARD,), float("nan"), device="cuda")
        buf[M * N:] = SENTINEL
        st = torch.cuda.current_stream().cuda_stream
        g.run_ptrs(Ad.data_ptr(), Bd.data_ptr(), buf.data_ptr(), st)
        assert g.sync_status() == w.WS_OK
        out = buf.cpu().numpy()
        assert np.all(out[M * N:] == SENTINEL), "wrote past the end of C"
        C = out[:M * N].reshape(M, N)
        check(C, A, B, dtype, tile[0])
        # the entry point that allocates nothing: the same bits
        C2 = torch.full((M, N), float("nan"), device="cuda")
        assert w.ws_gemm_run_noalloc(M, N, K, g.cfg, Ad.data_ptr(), Bd.data_ptr(), C2.data_ptr(), st) == w.WS_OK
        assert np.array_equal(C2.cpu().numpy().view(np.uint32), C.view(np.uint32))
        # another epilogue of the same handle, and back
        g.set_epilogue(2.0, 1.0, "f32")
        old = torch.ones((M, N), device="cuda")
        g(Ad, Bd, old)
        assert torch.equal(old, 2.0 * torch.from_numpy(C).cuda() + 1.0)
        g.set_epilogue()
        again = g(Ad, Bd)
        torch.cuda.synchronize()
        assert np.array_equal(again.cpu().numpy().view(np.uint32), C.view(np.uint32))
        # whole tiles, by the requested kernel and ring: the same bits
        assert w.ws_gemm_set_partition(g._h, w.WS_PARTITION_WHOLE) == w.WS_OK
        one, = g.launches()
        assert tile_of(one) == tile and one.stages == P and one.consumer_waves == nc and one.grid == g.info.grid
        again = g(Ad, Bd, torch.full((M, N), float("nan"), device="cuda"))
        assert g.sync_status() == w.WS_OK
        assert np.array_equal(again.cpu().numpy().view(np.uint32), C.view(np.uint32))
        assert w.ws_gemm_set_partition(g._h, w.WS_PARTITION_AUTO) == w.WS_OK and len(g.launches()) == max(count, 1)
        assert w.ws_gemm_set_partition(g._h, 2) == w.WS_ERR_INVALID_ARG
    finally:
        g.close()


@pytest.mark.parametrize("shape,tile,P,nc", [((768, 512, 192), (256, 128, 64), 1, 4),
                                             ((512, 512, 128), (256, 256, 64), 1, 4),
                                             ((384, 1024, 96), (128, 128, 32), 2, 4),
                                             ((256, 192, 64), (64, 64, 32), 2, 1)], ids=str)
def test_synchronous_parts_are_exact(shape, tile, P, nc):
    M, N, K = shape
    log("case synchronous parts %s %s" % (shape, tile))
    A, B = inputs.make_operands(M, N, K, "bf16", "int4", M + K)
    g = w.WsGemm(M, N, K, tile, P, 0, nc, "bf16")
    try:
        part, = g.launches()
        assert tile_of(part) != tile and part.stages == P
        C = torch.full((M, N), float("nan"), device="cuda")
        g(A.cuda(), B.cuda(), C)
        assert g.sync_status() == w.WS_OK
        check(C.cpu().numpy(), A, B, "bf16", tile[0])
    finally:
        g.close()


def test_two_launch_run_under_capture_and_the_launch_clock():
    M, N, K = 2056, 2056, 1304
    log("case partition capture")
    A, B = inputs.make_operands(M, N, K, "bf16", "int4", 3)
    Ad, Bd = A.cuda(), B.cuda()
    g = w.WsGemm(M, N, K, T128[0], T128[1], T128[2], T128[3], "bf16")
    try:
        assert len(g.launches()) == 2
        eager = g(Ad, Bd)
        torch.cuda.synchronize()
        assert g.clock_mhz()[1] == 1  # one sample per run
        C = torch.empty_like(eager)
        side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            g.run_ptrs(Ad.data_ptr(), Bd.data_ptr(), C.data_ptr(), side.cuda_stream)
        for _ in range(3):
            C.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(C, eager)
        del graph
    finally:
        g.close()
