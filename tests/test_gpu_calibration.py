"""Calibration kernels of the performance model (ws_gemm_create_calibration).

Each kind must finish without a wait timing out, and touch C only as its
contract says: the epilogue-only kernel stores a zero tile over every output
tile, the others leave C alone.  The bench-size case runs the launch the
calibration uses (8192 x 8192, full grid).
"""
from __future__ import annotations

import pytest
import torch

from tests.gpu_helpers import log

w = pytest.importorskip("paper_2506_11209_amd.wsgemm")

pytestmark = pytest.mark.gpu

SENTINEL = 12345.0


def run_kind(M, N, K, tile, stages, np_, nc, kind, load_path="registers", repeats=2):
    g = w.WsGemm(M, N, K, tile, stages, np_, nc, "bf16", load_path, calibration=kind)
    try:
        A = torch.randn(M, K, device="cuda").to(torch.bfloat16)
        B = torch.randn(K, N, device="cuda").to(torch.bfloat16)
        C = torch.full((M, N), SENTINEL, dtype=torch.float32, device="cuda")
        for _ in range(repeats):
            g(A, B, C)
        st = g.sync_status()
        return st, C
    finally:
        g.close()


CASES = [
    ((128, 128, 64), 3, 4, 4, 1024, 1024, 1024),
    ((256, 128, 64), 3, 4, 4, 1024, 1024, 2048),
    ((128, 256, 32), 4, 8, 4, 1024, 1024, 1024),
    ((64, 64, 64), 2, 8, 4, 512, 512, 512),
    ((256, 128, 64), 3, 8, 4, 768, 512, 512),
]


@pytest.mark.parametrize("load_path", ["registers", "dma"])
@pytest.mark.parametrize("kind", ["empty", "load_a", "load_b", "math", "epilogue", "load_ab"])
@pytest.mark.parametrize("tile,stages,np_,nc,M,N,K", CASES)
def test_calibration_kernel_contract(tile, stages, np_, nc, M, N, K, kind, load_path):
    log("calibration %s %s P=%d %d:%d %dx%dx%d %s" % (kind, tile, stages, np_, nc, M, N, K, load_path))
    st, C = run_kind(M, N, K, tile, stages, np_, nc, kind, load_path)
    assert st == w.WS_OK, w.ws_gemm_status_str(st)
    if kind == "epilogue":
        assert bool((C == 0).all()), "epilogue-only kernel must store a zero tile everywhere"
    else:
        assert bool((C == SENTINEL).all()), "%s kernel must not write C" % kind


@pytest.mark.parametrize("kind", ["load_a", "math", "epilogue"])
def test_calibration_at_bench_launch(kind):
    log("calibration %s at 8192^3 launch" % kind)
    st, C = run_kind(8192, 8192, 1024, (256, 128, 64), 3, 4, 4, kind, repeats=3)
    assert st == w.WS_OK
    if kind == "epilogue":
        assert bool((C == 0).all())


@pytest.mark.parametrize("kind", ["empty", "load_a", "load_b", "math", "epilogue", "load_ab"])
@pytest.mark.parametrize("tile,stages,np_,nc,split,M,N,K", [
    ((128, 128, 64), 3, 4, 4, 1, 1024, 1024, 512),     # few tiles: the GEMM itself runs parts
    ((256, 256, 64), 2, 4, 8, 2, 2048, 2048, 512),
    ((128, 128, 64), 3, 4, 4, 1, 2176, 2048, 1280),    # the GEMM runs a block and the rest
])
def test_calibration_runs_the_plan_it_reports(tile, stages, np_, nc, split, M, N, K, kind):
    """T_INIT, T_EPILOGUE and the costs per K-iteration are differences and
    quotients over the plan's rounds and grid: every kind launches that plan."""
    log("calibration launch %s %s" % (kind, tile))
    gemm = w.WsGemm(M, N, K, tile, stages, np_, nc, "bf16", split=split)
    g = w.WsGemm(M, N, K, tile, stages, np_, nc, "bf16", calibration=kind, split=split)
    try:
        assert gemm.launches()[-1].tile_m < tile[0]
        launch, = g.launches()
        assert (launch.tile_m, launch.tile_n, launch.tile_k) == tile and launch.stages == stages
        assert (launch.grid, launch.rounds, launch.tiles) == (g.info.grid, g.info.rounds, g.info.tiles)
        assert w.ws_gemm_set_partition(gemm._h, w.WS_PARTITION_WHOLE) == w.WS_OK
        assert gemm.launches()[0].as_dict() == launch.as_dict()
        A = torch.zeros(M, K, device="cuda", dtype=torch.bfloat16)
        B = torch.zeros(K, N, device="cuda", dtype=torch.bfloat16)
        g(A, B, torch.zeros(M, N, device="cuda"))
        assert g.sync_status() == w.WS_OK
    finally:
        g.close()
        gemm.close()


def test_tools_measure_the_launch_point_they_name(monkeypatch, tmp_path):
    """The sweep, the optimizer, the model's evaluation and the event trace time
    the tile and ring they report (and predict) also where a run would take
    parts; the benchmark's line names the kernel that ran."""
    import json

    from paper_2506_11209_amd import model_eval, optimize, sweep, trace
    from paper_2506_11209_amd.workloads import Workload
    seen = []
    run = w.ws_gemm_run

    def spy(h, *a):
        seen.append([(l.tile_m, l.tile_n, l.tile_k, l.stages) for l in w.ws_gemm_query_launches(h)[1]])
        return run(h, *a)

    monkeypatch.setattr(w, "ws_gemm_run", spy)
    point = (128, 128, 64, 3, 4, 4)
    wl = Workload("few_tiles", 512, 512, 256, "bf16", "normal", 1, False, (point,))
    A = torch.randn(512, 256, device="cuda").bfloat16()
    B = torch.randn(256, 512, device="cuda").bfloat16()
    log("case tools sweep")
    assert sweep.measure_point(wl, point, A, B, torch.empty(512, 512, device="cuda"), 2, 1,
                               min_warmup_s=0.0)["status"] == "ok"
    log("case tools optimizer")
    optimize.measure([{"tile": (128, 128, 64), "stages": 3, "producer_waves": 4, "consumer_waves": 4, "split": 1,
                       "time_us": 1.0}], 512, 512, 256, "registers", 2, 1)
    log("case tools trace")
    trace.run_traced(wl, point, wgs=1, Ad=A, Bd=B)
    log("case tools model")
    params = dict(t_init=1.0, t_epilogue=1.0, compute_throughput=1.0, compute_latency=1.0, load_throughput=1.0,
                  load_latency=1.0)
    calib = tmp_path / "calib.json"
    calib.write_text(json.dumps({"calibrations": [{"split": 1, "load_path": "registers", "params": params}]}))
    monkeypatch.setattr(model_eval, "paper_grid", lambda: [(512, 512, 256, (128, 128, 64), 3, 1)])
    model_eval.main(["--calib", str(calib), "--grid", "paper", "--steps", "2", "--warmup", "1", "--fixed", "launch"])
    assert len(seen) > 12 and all(x == [(128, 128, 64, 3)] for x in seen), seen


def test_calibration_handles_refuse_tracing():
    g = w.WsGemm(512, 512, 512, (128, 128, 64), 3, 4, 4, "bf16", calibration="math")
    try:
        buf = torch.zeros(1 << 16, dtype=torch.int32, device="cuda")
        s = w.library().ws_gemm_set_trace(g._h, w._p(buf.data_ptr()), buf.numel() * 4, 1, 4)
        assert s == w.WS_ERR_UNSUPPORTED
    finally:
        g.close()
