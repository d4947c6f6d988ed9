"""The launches whose speed this library is judged by.

Each case is one GEMM launch through the public Python entry points: a
``WsGemm`` handle called on torch tensors, or ``ws_gemm_run_noalloc``.  A
launch point (tile, ring depth, wave counts, load path) belongs to the case,
as it does to every call of the library.
"""
from __future__ import annotations

import math

import torch

from paper_2506_11209_amd import wsgemm as w

TORCH = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"f16": 2, "bf16": 2, "f32": 4}


def _case(M, N, K, tile, stages, producers, consumers, dtype="bf16", path="registers", entry="handle",
          dist="normal", alpha=1.0, beta=0.0, out="f32", name=None):
    c = {"M": M, "N": N, "K": K, "tile_m": tile[0], "tile_n": tile[1], "tile_k": tile[2], "stages": stages,
         "producers": producers, "consumers": consumers, "dtype": dtype, "path": path, "entry": entry,
         "dist": dist, "alpha": alpha, "beta": beta, "out": out}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: 16 one-consumer-wave workgroups, eight K-iterations;
        # its time is launch and pipeline latency.  Integer operands.
        _case(256, 256, 256, (64, 64, 32), 2, 1, 1, "f16", dist="int4", name="small_256_f16"),
        # The largest problem of the paper's own evaluation grid, at its tile.
        _case(1024, 1024, 1024, (128, 128, 64), 3, 4, 4, name="paper_grid_1024"),
        # The default launch of a handle on an ordinary square product.
        _case(4096, 4096, 4096, (128, 128, 32), 3, 4, 4, name="cube_4096_default"),
        # The benchmark: the largest product, at the library's fastest launch.
        _case(8192, 8192, 8192, (256, 256, 64), 2, 4, 8, name="cube_8192"),
        # Skinny, memory-bound product with two producers per consumer.
        _case(16384, 256, 8192, (128, 64, 64), 4, 8, 4, dist="uniform", name="skinny_16384x256x8192"),
        # Deep K: a long steady state of the ring, one tile per CU.
        _case(2048, 2048, 32768, (128, 128, 64), 4, 4, 4, dist="normal_k", name="deep_2048x2048x32768"),
        # Sizes the tiles do not divide, a little over whole tiles.
        _case(4100, 4104, 4104, (256, 256, 64), 2, 4, 8, name="ragged_4100x4104x4104"),
        # A small ragged product in fp16.
        _case(1000, 1000, 1000, (64, 64, 64), 3, 4, 4, "f16", name="ragged_1000_f16"),
        # A linear layer that accumulates into a 16-bit output in place.
        _case(8192, 4096, 4096, (256, 128, 64), 3, 4, 4, dist="normal_k", alpha=0.5, beta=0.5, out="bf16",
              name="accumulate_bf16_out"),
        # A serving loop: few rows against a weight matrix, by the entry point
        # that allocates nothing.
        _case(48, 4096, 4096, (64, 64, 64), 3, 4, 4, "f16", entry="noalloc", name="few_rows_noalloc"),
        # The synchronous baseline that warp specialisation is compared with.
        _case(4096, 4096, 4096, (128, 256, 32), 1, 0, 4, "f16", name="synchronous_4096_f16"),
        # Producers that load straight into LDS, two groups of them.
        _case(4096, 8192, 2048, (128, 256, 32), 3, 8, 4, path="dma", name="dma_4096x8192x2048"),
    ]


# Launch points that draw() takes: (tile, stages, producers, consumers).
POINTS_SMALL = [((64, 64, 32), 2, 1, 1), ((64, 64, 64), 3, 2, 1), ((64, 64, 64), 3, 4, 4),
                ((64, 64, 32), 4, 4, 4), ((128, 64, 64), 3, 4, 4), ((64, 128, 64), 3, 8, 4)]
POINTS_LARGE = [((128, 128, 32), 3, 4, 4), ((128, 128, 64), 3, 4, 4), ((128, 128, 64), 4, 8, 4),
                ((128, 64, 64), 4, 8, 4), ((128, 256, 32), 4, 4, 4), ((256, 128, 64), 3, 4, 4),
                ((256, 256, 64), 2, 4, 8), ((256, 256, 32), 4, 4, 8)]
POINTS_SYNC = [((128, 128, 32), 1, 0, 4), ((128, 256, 32), 1, 0, 4), ((256, 128, 64), 1, 0, 4),
               ((256, 128, 64), 2, 0, 4)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("plain", "plain", "ragged", "ragged", "epilogue", "noalloc", "dma", "synchronous"))
    small = kind in ("plain", "ragged", "noalloc") and rng.random() < 0.5
    tile, stages, producers, consumers = rng.choice(
        POINTS_SYNC if kind == "synchronous" else POINTS_SMALL if small else POINTS_LARGE)
    hi = 2048 if small else 16384
    while True:
        M = _log_int(rng, 16 if kind in ("ragged", "noalloc") else tile[0], hi)
        N, K = _log_int(rng, 256, hi), _log_int(rng, 256, hi)
        if kind in ("ragged", "epilogue", "noalloc"):  # any M; rows of 16 bytes
            N, K = N // 8 * 8, K // 8 * 8
        else:
            M, N, K = (max(t, x // t * t) for t, x in zip(tile, (M, N, K)))
        if 1.0 * M * N * K <= 8192.0 ** 3 and 2 * (M * K + K * N) + 4 * M * N <= 1 << 29:
            break
    dtype = rng.choice(("bf16", "bf16", "f16"))
    c = _case(M, N, K, tile, stages, producers, consumers, dtype,
              path="dma" if kind == "dma" else "registers",
              entry="noalloc" if kind == "noalloc" else "handle",
              dist="normal_k" if kind == "epilogue" else rng.choice(("normal", "uniform")))
    if kind == "epilogue":
        c["alpha"] = rng.choice((0.5, 1.0))
        c["beta"] = rng.choice((0.0, 0.5))
        c["out"] = rng.choice(("bf16", "f16", "f32"))
    return c


def _draw_matrix(rows, cols, dist, K, dtype, g):
    if dist == "int4":
        return torch.randint(-4, 5, (rows, cols), generator=g, device="cuda").to(dtype)
    if dist == "uniform":
        return (torch.rand((rows, cols), generator=g, device="cuda") * 2.0 - 1.0).to(dtype)
    t = torch.randn((rows, cols), generator=g, device="cuda")
    return (t / math.sqrt(K) if dist == "normal_k" else t).to(dtype)


def _inputs(case, seed):
    """A, B and the old C (zeros where the epilogue does not read it)."""
    M, N, K, dist = case["M"], case["N"], case["K"], case["dist"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = _draw_matrix(M, K, dist, K, TORCH[case["dtype"]], g)
    B = _draw_matrix(K, N, dist, K, TORCH[case["dtype"]], g)
    if case["beta"] != 0.0:
        C = _draw_matrix(M, N, dist, K, TORCH[case["out"]], g)
    else:
        C = torch.zeros((M, N), dtype=TORCH[case["out"]], device="cuda")
    return A, B, C


def prepare(case, seed):
    A, B, C = _inputs(case, seed)
    tile = (case["tile_m"], case["tile_n"], case["tile_k"])
    s = {"A": A, "B": B, "C": C, "shape": (case["M"], case["N"], case["K"])}
    if case["entry"] == "noalloc":
        s["cfg"] = w.config(tile, case["stages"], case["producers"], case["consumers"], case["dtype"], case["path"])
    else:
        s["gemm"] = w.WsGemm(case["M"], case["N"], case["K"], tile, case["stages"], case["producers"],
                             case["consumers"], case["dtype"], case["path"])
        if (case["alpha"], case["beta"], case["out"]) != (1.0, 0.0, "f32"):
            s["gemm"].set_epilogue(case["alpha"], case["beta"], case["out"])
    return s


def run(state):
    if "gemm" in state:
        return state["gemm"](state["A"], state["B"], state["C"])
    st = w.ws_gemm_run_noalloc(*state["shape"], state["cfg"], state["A"].data_ptr(), state["B"].data_ptr(),
                               state["C"].data_ptr(), torch.cuda.current_stream().cuda_stream)
    if st != w.WS_OK:
        raise w.WsGemmError("ws_gemm_run_noalloc", st)
    return state["C"]


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    c_passes = 2 if case["beta"] != 0.0 else 1
    return {"bytes": 2 * (M * K + K * N) + c_passes * SIZE[case["out"]] * M * N, "flops": 2 * M * N * K}


def exact(case, seed):
    A, B, C = _inputs(case, seed)
    r = case["alpha"] * (A.double() @ B.double())
    return r + case["beta"] * C.double() if case["beta"] != 0.0 else r


def tolerance(case):
    if case["dist"] == "int4":
        return "exact"
    if case["out"] != "f32":
        # one rounding to the output type, 2^-9 (bf16) or 2^-12 (f16) at most
        rel = 7e-3 if case["out"] == "bf16" else 9e-4
        return {"rel": rel, "max": 4 * rel}
    # binary32 sums of K exact products; about four times the error against 64 bits
    rel = 1e-7 * math.sqrt(case["K"]) / 4 + 5e-7
    return {"rel": rel, "max": 10 * rel}
