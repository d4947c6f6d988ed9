// C ABI of the warp-specialised GEMM: validation, kernel selection, launch.
#include "ws_gemm.h"

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <atomic>
#include <mutex>
#include <new>

#include "ws_gemm_kernel.hpp"
#include "ws_gemm_plan.hpp"
#include "ws_gemm_registry.hpp"

// Device memory of ws_gemm_run_noalloc: the wait watchdog's word (the only
// scratch its kernels use), one copy per GPU, held until the process ends.
// The kernels write word 0 only.  Host code reaches a device's copy through
// the address hipGetSymbolAddress returns for it (static_device below).
static __device__ __align__(256) int32_t scratch[64];

// Generated by the build: declares the instance tables and defines
// kAllTables / kNumTables.
#include "ws_gemm_instances.inc"

namespace {

constexpr int kDefaultSpinLimit = 1 << 22;
// The handle's 256-byte device word block: the watchdog word at 0, the
// launch clock accumulators (3 x uint64) at kClockOffset.
constexpr int kClockOffset = 64;

thread_local char g_last_error[256] = "";

// Records the failing HIP call for ws_gemm_last_error() and maps it to WS_ERR_HIP.
ws_status hip_fail(const char* what, hipError_t e) {
  snprintf(g_last_error, sizeof(g_last_error), "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
  return WS_ERR_HIP;
}

#define WSG_HIP(call)                                 \
  do {                                                \
    hipError_t e_ = (call);                           \
    if (e_ != hipSuccess) return hip_fail(#call, e_); \
  } while (0)

ws_status from_plan(int s) {
  switch (s) {
    case wsg::kPlanOk: return WS_OK;
    case wsg::kPlanNotDivisible: return WS_ERR_NOT_DIVISIBLE;
    case wsg::kPlanUnsupported: return WS_ERR_UNSUPPORTED;
    case wsg::kPlanLdsOverflow: return WS_ERR_LDS_OVERFLOW;
    default: return WS_ERR_INVALID_ARG;
  }
}

// DMA warps per MATH warp of c (0 for the synchronous kernel, -1 if none).
int split_of(const ws_gemm_config& c) {
  return wsg::arrangement_split(c.consumer_waves, c.producer_waves, c.split);
}

#include "ws_gemm_resources.inc"

// The compiled kernels by configuration: position in `table` of the key below,
// built once.  A call of ws_gemm_run_noalloc looks several kernels up (walking
// the tables took 1 us a call).
struct KernelIndex {
  static constexpr int kKeys = 4 * 4 * 3 * 3 * 5 * 3 * 2 * 2 * 6 * 2;
  struct Slot {
    const wsg::KernelEntry* kernel;
    int16_t vgprs, agprs;
  };
  Slot slots[1024];
  int16_t at[kKeys];  // index into slots, -1: not compiled
  int count = 0;

  static int log2_of(int x, int lo, int hi) {  // position of x among the powers of two lo .. hi, -1 if it is none
    for (int i = 0, p = lo; p <= hi; ++i, p *= 2)
      if (p == x) return i;
    return -1;
  }
  static int key(int tm, int tn, int tk, int nc, int np, int split, int bf16, int trace, int mode, int general) {
    const int a = log2_of(tm, 32, 256), b = log2_of(tn, 32, 256), c = log2_of(tk, 32, 128);
    const int d = nc == 1 ? 0 : nc == 4 ? 1 : nc == 8 ? 2 : -1;
    const int e = np == 0 ? 0 : log2_of(np, 1, 8) < 0 ? -1 : log2_of(np, 1, 8) + 1;
    if (a < 0 || b < 0 || c < 0 || d < 0 || e < 0 || split < 0 || split > 2 || mode < 0 || mode > 5) return -1;
    return ((((((((a * 4 + b) * 3 + c) * 3 + d) * 5 + e) * 3 + split) * 2 + bf16) * 2 + trace) * 6 + mode) * 2 + general;
  }
  KernelIndex() {
    for (int i = 0; i < kKeys; ++i) at[i] = -1;
    for (int t = 0; t < kNumTables; ++t)
      for (int i = 0; i < kAllTables[t].count && count < 1024; ++i) {
        const wsg::KernelEntry& e = kAllTables[t].entries[i];
        const int k = key(e.tm, e.tn, e.tk, e.nc, e.np, e.split, e.bf16, e.trace, e.mode, e.general);
        if (k < 0) continue;
        slots[count] = Slot{&e, 0, 0};
        at[k] = (int16_t)count++;
      }
    for (int i = 0; i < kNumResources; ++i) {
      const wsg::KernelResources& r = kResources[i];
      const int k = key(r.tm, r.tn, r.tk, r.nc, r.np, r.split, r.bf16, r.trace, r.mode, r.general);
      if (k < 0 || at[k] < 0) continue;
      slots[at[k]].vgprs = r.vgprs;
      slots[at[k]].agprs = r.agprs;
    }
  }
};

const KernelIndex::Slot* find_slot(const ws_gemm_config& c, int trace, int mode, int general) {
  static const KernelIndex index;
  const int k = KernelIndex::key(c.tile_m, c.tile_n, c.tile_k, c.consumer_waves, c.producer_waves, split_of(c),
                                 c.dtype == WS_BF16 ? 1 : 0, trace, mode, general);
  return k < 0 || index.at[k] < 0 ? nullptr : &index.slots[index.at[k]];
}

const wsg::KernelEntry* find_kernel(const ws_gemm_config& c, int trace = 0, int mode = wsg::kModeGemm,
                                   int general = 0) {
  const KernelIndex::Slot* s = find_slot(c, trace, mode, general);
  return s ? s->kernel : nullptr;
}

// Registers per wave of the GEMM kernel of c or of its general twin (0, 0 if
// not in the table).
void kernel_regs(const ws_gemm_config& c, int general, int* vgprs, int* agprs) {
  const KernelIndex::Slot* s = find_slot(c, 0, wsg::kModeGemm, general);
  *vgprs = s ? s->vgprs : 0;
  *agprs = s ? s->agprs : 0;
}

wsg::PlanIn plan_in(int64_t M, int64_t N, int64_t K, const ws_gemm_config& c, int32_t cus,
                    int32_t occ, int general = 0) {
  wsg::PlanIn in{};
  in.M = M;
  in.N = N;
  in.K = K;
  in.tile_m = c.tile_m;
  in.tile_n = c.tile_n;
  in.tile_k = c.tile_k;
  in.producer_waves = c.producer_waves;
  in.consumer_waves = c.consumer_waves;
  in.stages = c.stages;
  in.dtype = c.dtype;
  in.load_path = c.load_path;
  in.split = c.split;
  in.num_cus = cus;
  in.wgs_per_cu = occ;
  kernel_regs(c, general, &in.vgprs, &in.agprs);
  return in;
}

// Lets `fn` use a CU's whole LDS on the current device.  Remembered per
// kernel and device (the setting belongs to the loaded kernel and is never
// lowered), so that a run does not pay for it again.
ws_status allow_lds(const void* fn) {
  int dev = 0;
  WSG_HIP(hipGetDevice(&dev));
  constexpr int kSlots = 2048;  // open addressing by the kernel's address; 420 kernels
  struct Known {
    std::atomic<const void*> fn;
    std::atomic<uint64_t> devices;
  };
  static Known known[kSlots];
  Known* k = nullptr;
  if (dev >= 0 && dev < 64) {
    size_t h = ((uintptr_t)fn >> 4) % kSlots;
    for (int i = 0; i < kSlots && !k; ++i, h = (h + 1) % kSlots) {
      const void* at = known[h].fn.load(std::memory_order_acquire);
      if (!at && known[h].fn.compare_exchange_strong(at, fn, std::memory_order_acq_rel)) at = fn;
      if (at == fn) k = &known[h];
    }
    if (k && (k->devices.load(std::memory_order_acquire) >> dev & 1)) return WS_OK;
  }
  WSG_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, wsg::kLdsLimit));
  if (k) k->devices.fetch_or(1ull << dev, std::memory_order_acq_rel);
  return WS_OK;
}

// A kernel and the grid it is launched with; corner_m >= 0: of the plan's tiles
// only those outside the block of the first corner_m rows and corner_n columns.
struct Launch {
  const void* fn;
  ws_gemm_config cfg;  // of the kernel: its tile, waves and ring
  int32_t general;
  wsg::PlanOut plan;
  int32_t corner_m, corner_n;
};
// What one run launches, in stream order.
struct Run {
  Launch launch[2];
  int count;
};
static_assert(sizeof(Run::launch) / sizeof(Launch) == WS_MAX_LAUNCHES, "header and library agree");

// One launch of every tile.
Run whole_run(const void* fn, const ws_gemm_config& c, int general, const wsg::PlanOut& plan) {
  return Run{{{fn, c, general, plan, -1, -1}, {}}, 1};
}

int64_t tiles_of(int64_t M, int64_t N, const ws_gemm_config& k) {
  return ((M + k.tile_m - 1) / k.tile_m) * ((N + k.tile_n - 1) / k.tile_n);
}

// The configuration of a part of a tile of c: the same T_K, dtype and split
// (four consumer waves for parts of the eight-consumer 256 x 256 tile).
ws_gemm_config part_of(const ws_gemm_config& c, int tm, int tn) {
  ws_gemm_config k = c;
  k.tile_m = tm;
  k.tile_n = tn;
  if (c.producer_waves > 0) k.split = split_of(c);  // 0 for the synchronous kernel
  if (c.consumer_waves == 8 && (tm < c.tile_m || tn < c.tile_n)) k.consumer_waves = 4;
  return k;
}

// Calls f(config, cost) for every compiled part of c's tile (the whole tile
// left out) that is cheaper than `limit`: `count(config)` tiles of it.
// 32 x 32 parts have one consumer wave and are for tiles of one consumer wave
// only: its one loading wave takes 390 ns for 64 of K, four loading waves 280 ns
// for a 64 x 64 tile (48x4096x4096: 256 such parts 28.9 us, 64 tiles 22.9 us).
template <typename Count, typename F>
void each_part(const ws_gemm_config& c, int cus, int general, int64_t limit, Count count, F f) {
  const int least = c.consumer_waves == 1 ? 32 : 64;
  for (int tm = c.tile_m; tm >= least; tm /= 2)
    for (int tn = c.tile_n; tn >= least; tn /= 2) {
      if (tm == c.tile_m && tn == c.tile_n) continue;
      const ws_gemm_config k = part_of(c, tm, tn);
      const int64_t cost = wsg::tiles_cost(count(k), tm, tn, cus);
      if (cost < limit && find_kernel(k, 0, wsg::kModeGemm, general)) {
        f(k, cost);
        limit = cost;
      }
    }
}

// Workgroups of k's kernel that a CU runs when there are `tiles` of them.
int per_cu(const ws_gemm_config& k, int general, int64_t tiles, int cus) {
  int v = 0, a = 0;
  kernel_regs(k, general, &v, &a);
  const int waves = k.consumer_waves + k.producer_waves;
  const int64_t fit = 4 * wsg::waves_per_simd_by_regs(v, a) / waves, want = (tiles + cus - 1) / cus;
  return (int)(want < fit ? want : fit);
}

// Plan of `tiles` tiles of part k of c on the M x N x K problem.
bool plan_part(int64_t M, int64_t N, int64_t K, const ws_gemm_config& c, ws_gemm_config k, int64_t tiles, int cus,
               int general, Launch* l) {
  if (c.producer_waves > 0)  // the synchronous kernel's depth says whether it overlaps: kept
    k.stages = wsg::part_stages(c.stages, 2ll * c.tile_k * (c.tile_m + c.tile_n),
                                2ll * c.tile_k * (k.tile_m + k.tile_n), per_cu(k, general, tiles, cus));
  wsg::PlanOut plan;
  if (wsg::plan_launch(plan_in(M, N, K, k, cus, 0, general), &plan) != wsg::kPlanOk) return false;
  *l = Launch{find_kernel(k, 0, wsg::kModeGemm, general)->fn, k, general, plan, -1, -1};
  return true;
}

// Chooses how to compute the problem with the (general) kernel of c:
// whole tiles (as `out` comes in), every tile in parts, or a block of whole
// tiles and, in a second launch, the rest in parts - the rest being partial
// edge tiles, which would multiply padding for a round of their own, or what a
// nearly empty last round would take.  plain_block: the block's tiles may run
// the plain kernel (default epilogue; they are whole).  The synchronous kernel
// walks one tile region: whole tiles or parts.
//
// Measured, whole tiles -> block and rest: 4100x4104x4104 with 256x256x64 tiles
// (289 tiles, 33 of them almost all padding) 199 -> 148 us, as 128x128 parts
// 269 us.
void choose_run(int64_t M, int64_t N, int64_t K, const ws_gemm_config& c, int cus, int general, bool plain_block,
                Run* out) {
  const Launch& whole = out->launch[0];
  // costs of the whole problem: part_cost units are ns per 64 of K
  const int64_t slabs = (K + 63) / 64;
  const int64_t whole_cost = wsg::tiles_cost(whole.plan.tiles, c.tile_m, c.tile_n, cus) * slabs;
  int64_t best = whole_cost * wsg::kPartitionGainNum / wsg::kPartitionGainDen;  // what another partition must not exceed
  ws_gemm_config part{}, rest{};
  // A double-buffered synchronous workgroup that has its CU to itself overlaps
  // its own loads; parts of it do so no better once every CU has a tile
  // (256x256x32 at 19200x1024x2048, 300 tiles: whole 197 us, in parts 244 us).
  // With fewer than eight K-iterations the stores count for more, and parts win
  // (2816x6144x160 by 1.2).
  int vgprs = 0, agprs = 0;
  kernel_regs(c, general, &vgprs, &agprs);
  const int waves = c.consumer_waves + c.producer_waves;
  const bool alone = 2 * whole.plan.lds_bytes > wsg::kLdsLimit ||
                     4 * wsg::waves_per_simd_by_regs(vgprs, agprs) < 2 * waves;
  if (!(c.producer_waves == 0 && c.stages == 2 && alone && whole.plan.tiles > cus && whole.plan.iters >= 8))
    each_part(c, cus, general, best / slabs + 1, [&](const ws_gemm_config& k) { return tiles_of(M, N, k); },
              [&](const ws_gemm_config& k, int64_t cost) {
                part = k;
                best = cost * slabs;
              });
  // A block and the rest: not where the tiles past the last whole round share
  // their CUs with the others in one round, which costs far less than the round
  // of its own that the cost counts (128x64x32 at 640x3520x5376, 275 tiles: whole
  // 79 us, block and rest 105 us), and so not for one consumer wave, of which
  // four or more tiles share a CU (64x64x64 at 1337x872x5992: 61 and 93 us).
  int rows_best = 0, cols_best = 0;
  if (c.producer_waves > 0 && c.consumer_waves > 1 && whole.plan.rounds > 1) {
    const int64_t rows = M / c.tile_m, cols = N / c.tile_n, rounds = rows * cols / cus;
    for (int t = 0; t < 3 && rows > 0 && cols > 0; ++t) {
      // all whole tiles, or as many rows (columns) of them as whole rounds hold
      const int64_t r = t == 1 ? rounds * cus / cols : rows, q = t == 2 ? rounds * cus / rows : cols;
      if (r < 1 || q < 1 || (r * c.tile_m >= M && q * c.tile_n >= N)) continue;
      const int64_t block = wsg::tiles_cost(r * q, c.tile_m, c.tile_n, cus) * slabs + wsg::kSecondLaunchNs;
      if (block >= best) continue;
      each_part(c, cus, general, (best - block) / slabs,
                [&](const ws_gemm_config& k) {
                  return tiles_of(M, N, k) - r * q * (c.tile_m / k.tile_m) * (c.tile_n / k.tile_n);
                },
                [&](const ws_gemm_config& k, int64_t cost) {
                  rest = k;
                  rows_best = (int)r;
                  cols_best = (int)q;
                  best = block + cost * slabs;
                });
    }
  }
  Run run = *out;
  if (rows_best > 0) {
    run.count = 2;
    Launch& m = run.launch[0];
    Launch& e = run.launch[1];
    if (wsg::plan_launch(plan_in((int64_t)rows_best * c.tile_m, (int64_t)cols_best * c.tile_n, K, c, cus, 0),
                         &m.plan) != wsg::kPlanOk)
      return;
    const wsg::KernelEntry* plain = plain_block && K % c.tile_k == 0 ? find_kernel(c, 0, wsg::kModeGemm, 0) : nullptr;
    if (plain) {
      m.fn = plain->fn;
      m.general = 0;
    }
    const int cm = rows_best * (c.tile_m / rest.tile_m), cn = cols_best * (c.tile_n / rest.tile_n);
    const int64_t tiles = tiles_of(M, N, rest) - (int64_t)cm * cn;
    if (!plan_part(M, N, K, c, rest, tiles, cus, general, &e)) return;
    e.corner_m = cm;
    e.corner_n = cn;
    e.plan.tiles = (int32_t)tiles;
    if (tiles < e.plan.grid) e.plan.grid = (int32_t)tiles;
    e.plan.rounds = (int32_t)((tiles + e.plan.grid - 1) / e.plan.grid);
    e.plan.xcd_remap = e.plan.grid % 8 == 0;
  } else if (part.tile_m > 0) {
    if (!plan_part(M, N, K, c, part, tiles_of(M, N, part), cus, general, &run.launch[0])) return;
  } else {
    return;
  }
  *out = run;
}

// The run of a GEMM (general: by the general kernel) planned without a device:
// resident workgroups from the compiled kernel's registers, which is what the
// runtime's occupancy query gives.
ws_status plan_run(int64_t M, int64_t N, int64_t K, const ws_gemm_config& c, int cus, int general, bool plain_block,
                   Run* out) {
  wsg::PlanOut p;
  const int s = wsg::plan_launch(plan_in(M, N, K, c, cus, 0, general), &p);
  if (s != wsg::kPlanOk) return from_plan(s);
  const wsg::KernelEntry* k = find_kernel(c, 0, wsg::kModeGemm, general);
  if (!k) return WS_ERR_UNSUPPORTED;
  *out = whole_run(k->fn, c, general, p);
  if (p.grid == 0) out->count = 0;  // an empty problem launches no GEMM kernel
  else choose_run(M, N, K, c, cus, general, plain_block, out);
  return WS_OK;
}

ws_status allow_lds(const Run& run) {
  for (int i = 0; i < run.count; ++i) {
    const ws_status st = allow_lds(run.launch[i].fn);
    if (st != WS_OK) return st;
  }
  return WS_OK;
}

// Enqueues a run; `a` has everything but what a launch decides.
ws_status launch_run(const Run& run, wsg::KernelArgs a, hipStream_t stream) {
  for (int i = 0; i < run.count; ++i) {
    const Launch& l = run.launch[i];
    const wsg::TileRegions r =
        wsg::tile_regions(l.plan.tiles_m, l.plan.tiles_n, l.plan.group_m, l.corner_m, l.corner_n);
    a.tiles_m = r.tiles_m;
    a.tiles_n = r.tiles_n;
    a.group_m = r.group_m;
    a.region2 = r.region2;
    a.row1 = r.row1;
    a.tiles2_m = r.tiles2_m;
    a.tiles2_n = r.tiles2_n;
    a.col2 = r.col2;
    a.num_tiles = r.num_tiles;
    a.iters = l.plan.iters;
    a.stages = l.cfg.stages;
    a.xcd_remap = l.plan.xcd_remap;
    if (i > 0) a.clock = nullptr;  // one clock sample per run, of its main launch
    void* params[] = {&a};
    WSG_HIP(hipLaunchKernel(l.fn, dim3(l.plan.grid), dim3(l.plan.block), params, (size_t)l.plan.lds_bytes, stream));
  }
  return WS_OK;
}

void to_info(const wsg::PlanOut& p, ws_gemm_plan_info* o) {
  o->grid = p.grid;
  o->block = p.block;
  o->lds_bytes = p.lds_bytes;
  o->tiles_m = p.tiles_m;
  o->tiles_n = p.tiles_n;
  o->tiles = p.tiles;
  o->rounds = p.rounds;
  o->iters = p.iters;
  o->split = p.split;
  o->group_m = p.group_m;
  o->xcd_remap = p.xcd_remap;
  o->ragged = p.ragged;
  o->general = p.ragged;
}

void to_launches(const Run& run, ws_gemm_launch_info* out, int32_t* count) {
  *count = run.count;
  for (int i = 0; i < run.count; ++i) {
    const Launch& l = run.launch[i];
    out[i] = ws_gemm_launch_info{l.cfg.tile_m, l.cfg.tile_n, l.cfg.tile_k, l.cfg.stages, l.cfg.producer_waves,
                                 l.cfg.consumer_waves, l.plan.split, l.general, l.plan.grid, l.plan.block,
                                 l.plan.lds_bytes, l.plan.tiles_m, l.plan.tiles_n, l.plan.tiles, l.plan.rounds,
                                 l.plan.iters, l.corner_m < 0 ? 0 : l.corner_m, l.corner_m < 0 ? 0 : l.corner_n};
  }
}

bool default_epilogue(const ws_gemm_epilogue& e) {
  return e.alpha == 1.0f && e.beta == 0.0f && e.out_dtype == WS_OUT_F32;
}

// Per device: the address of that device's copy of `scratch` (from
// hipGetSymbolAddress, taken once with the device current) and its compute
// unit count.  The host-side name `scratch` is not a device address and is
// never passed to a kernel or a copy.
constexpr int kMaxDevices = 64;
struct StaticDevice {
  void* scratch;
  int cus;
};
StaticDevice g_static[kMaxDevices];
std::mutex g_static_mu;

// Looks up device `dev`'s copy of the scratch array with that device
// current (the current device is restored afterwards).
ws_status scratch_address(int dev, void** ptr, int* cus) {
  int cur = 0;
  WSG_HIP(hipGetDevice(&cur));
  if (cur != dev) WSG_HIP(hipSetDevice(dev));
  hipError_t e = hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch));
  if (e == hipSuccess && !*ptr) e = hipErrorInvalidSymbol;
  if (e == hipSuccess) e = hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (cur != dev) {
    const hipError_t e2 = hipSetDevice(cur);
    if (e == hipSuccess) e = e2;
  }
  if (e != hipSuccess) return hip_fail("hipGetSymbolAddress(scratch)", e);
  return WS_OK;
}

ws_status static_device(int dev, StaticDevice* out) {
  if (dev < 0 || dev >= kMaxDevices) return WS_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_static_mu);
  if (!g_static[dev].scratch) {
    void* ptr = nullptr;
    int cus = 0;
    const ws_status s = scratch_address(dev, &ptr, &cus);
    if (s != WS_OK) return s;
    g_static[dev].cus = cus;
    g_static[dev].scratch = ptr;
  }
  *out = g_static[dev];
  return WS_OK;
}

}  // namespace

struct ws_gemm_handle {
  int64_t M, N, K;
  ws_gemm_config cfg;
  wsg::PlanOut plan;
  const wsg::KernelEntry* traced;  // instrumented variant (null if none was compiled)
  const wsg::KernelEntry* general; // general twin (partial tiles, epilogue options), or null
  wsg::PlanOut plan_plain, plan_general;  // whole-tile plans of the plain and the general kernel
  Run run_plain, run_general;      // what ws_gemm_run launches for the default / another epilogue
  Run whole_plain, whole_general;  // the same with every tile whole
  bool whole;                      // WS_PARTITION_WHOLE is set
  bool use_general;                // another epilogue is set
  ws_gemm_epilogue epi;
  bool calibration;
  int device;
  int32_t* d_err;
  ws_gemm_debug dbg;
  uint32_t* trace;
  int32_t trace_wgs, trace_iters;
};

namespace {

const Run& current_run(const ws_gemm_handle* h) {
  if (h->whole || (h->trace && h->traced)) return h->use_general ? h->whole_general : h->whole_plain;
  return h->use_general ? h->run_general : h->run_plain;
}

}  // namespace

extern "C" {

int32_t ws_gemm_abi_version(void) { return WS_GEMM_ABI_VERSION; }

const char* ws_gemm_last_error(void) { return g_last_error; }

const char* ws_gemm_status_str(ws_status s) {
  switch (s) {
    case WS_OK: return "ok";
    case WS_ERR_INVALID_ARG: return "invalid argument";
    case WS_ERR_UNSUPPORTED: return "unsupported configuration";
    case WS_ERR_LDS_OVERFLOW: return "LDS ring does not fit in 160 KiB";
    case WS_ERR_HIP: return "HIP runtime error";
    case WS_ERR_TIMEOUT: return "producer/consumer wait timed out";
    case WS_ERR_NOT_DIVISIBLE: return "tile sizes do not divide the problem";
  }
  return "unknown status";
}

ws_status ws_gemm_plan(int64_t M, int64_t N, int64_t K, const ws_gemm_config* cfg,
                       int32_t num_cus, int32_t wgs_per_cu, ws_gemm_plan_info* out) {
  if (!cfg || !out) return WS_ERR_INVALID_ARG;
  wsg::PlanOut p;
  const int s = wsg::plan_launch(plan_in(M, N, K, *cfg, num_cus, wgs_per_cu), &p);
  if (s != wsg::kPlanOk) return from_plan(s);
  if (!find_kernel(*cfg, 0, wsg::kModeGemm, p.ragged)) return WS_ERR_UNSUPPORTED;
  to_info(p, out);
  return WS_OK;
}

ws_status ws_gemm_plan_launches(int64_t M, int64_t N, int64_t K, const ws_gemm_config* cfg, int32_t num_cus,
                                int32_t general, ws_gemm_launch_info* out, int32_t* count) {
  if (!cfg || !out || !count) return WS_ERR_INVALID_ARG;
  wsg::PlanOut p;
  const int s = wsg::plan_launch(plan_in(M, N, K, *cfg, num_cus, 1), &p);
  if (s != wsg::kPlanOk) return from_plan(s);
  Run run;
  const ws_status st = plan_run(M, N, K, *cfg, num_cus, general || p.ragged, !general, &run);
  if (st == WS_OK) to_launches(run, out, count);
  return st;
}

ws_status ws_gemm_schedule(const ws_gemm_plan_info* info, int32_t wg, int32_t round,
                           int32_t* tile_m_idx, int32_t* tile_n_idx) {
  if (!info || !tile_m_idx || !tile_n_idx) return WS_ERR_INVALID_ARG;
  if (info->grid <= 0 || info->tiles_m <= 0 || info->tiles_n <= 0 || info->group_m <= 0)
    return WS_ERR_INVALID_ARG;
  wsg::PlanOut p{};
  p.grid = info->grid;
  p.tiles_m = info->tiles_m;
  p.tiles_n = info->tiles_n;
  p.tiles = info->tiles;
  p.group_m = info->group_m;
  p.xcd_remap = info->xcd_remap;
  int ti = -1, tj = -1;
  if (!wsg::scheduled_tile(p, wg, round, &ti, &tj)) return WS_ERR_INVALID_ARG;
  *tile_m_idx = ti;
  *tile_n_idx = tj;
  return WS_OK;
}

}  // extern "C"

namespace {

// Shared by ws_gemm_create and ws_gemm_create_calibration: the plan (grid,
// occupancy) always comes from the GEMM kernel of cfg, so a calibration
// kernel runs under the launch it calibrates.
ws_status create_handle(int64_t M, int64_t N, int64_t K, const ws_gemm_config* cfg, int kind,
                        ws_gemm_t* out) {
  if (!cfg || !out) return WS_ERR_INVALID_ARG;
  *out = nullptr;
  // Validate everything that does not need the device first.
  wsg::PlanOut p;
  int s = wsg::plan_launch(plan_in(M, N, K, *cfg, 1, 1), &p);
  if (s != wsg::kPlanOk) return from_plan(s);
  // Ragged shapes run the general variant (no calibration or traced twins);
  // empty problems launch no GEMM kernel at all.
  if ((p.ragged || p.grid == 0) && kind != WS_CALIB_NONE) return WS_ERR_UNSUPPORTED;
  const wsg::KernelEntry* k = find_kernel(*cfg, 0, wsg::kModeGemm, p.ragged);
  if (!k) return WS_ERR_UNSUPPORTED;
  const wsg::KernelEntry* general =
      kind == WS_CALIB_NONE ? find_kernel(*cfg, 0, wsg::kModeGemm, 1) : nullptr;
  const void* launch_fn = k->fn;
  if (kind == WS_CALIB_EMPTY) {
    launch_fn = reinterpret_cast<const void*>(&wsg::ws_empty_kernel<0>);
  } else if (kind != WS_CALIB_NONE) {
    const int mode = kind == WS_CALIB_LOAD_A    ? wsg::kModeLoadA
                     : kind == WS_CALIB_LOAD_B  ? wsg::kModeLoadB
                     : kind == WS_CALIB_MATH    ? wsg::kModeMath
                     : kind == WS_CALIB_LOAD_AB ? wsg::kModeLoadAB
                                                : wsg::kModeEpilogue;
    const wsg::KernelEntry* calib = find_kernel(*cfg, 0, mode);
    if (!calib) return WS_ERR_UNSUPPORTED;
    launch_fn = calib->fn;
  }

  WSG_HIP(hipInit(0));
  int dev = 0;
  WSG_HIP(hipGetDevice(&dev));
  WSG_HIP(hipSetDevice(dev));
  int cus = 0;
  WSG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  ws_status sl = allow_lds(k->fn);
  if (sl != WS_OK) return sl;
  int occ = 0;
  WSG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k->fn, p.block, p.lds_bytes));
  if (occ < 1) return WS_ERR_UNSUPPORTED;
  s = wsg::plan_launch(plan_in(M, N, K, *cfg, cus, occ), &p);
  if (s != wsg::kPlanOk) return from_plan(s);
  if (launch_fn != k->fn)
    if ((sl = allow_lds(launch_fn)) != WS_OK) return sl;
  // The general twin may allocate more registers: its own launch.
  wsg::PlanOut pg = p;
  if (general && general != k) {
    if ((sl = allow_lds(general->fn)) != WS_OK) return sl;
    int occ_g = 0;
    WSG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ_g, general->fn, p.block, p.lds_bytes));
    if (occ_g < 1) general = nullptr;
    else if (wsg::plan_launch(plan_in(M, N, K, *cfg, cus, occ_g), &pg) != wsg::kPlanOk)
      general = nullptr;
  }

  // Empty problems launch no GEMM kernel.
  const Run whole_plain = whole_run(launch_fn, *cfg, p.ragged, p);
  const Run whole_general = whole_run(general ? general->fn : nullptr, *cfg, 1, pg);
  Run run_plain = whole_plain, run_general = whole_general;
  // Calibration kernels take the whole tiles that the plan they report counts.
  if (p.grid > 0 && kind == WS_CALIB_NONE) {
    choose_run(M, N, K, *cfg, cus, p.ragged, true, &run_plain);
    if ((sl = allow_lds(run_plain)) != WS_OK) return sl;
    if (general) {
      choose_run(M, N, K, *cfg, cus, 1, false, &run_general);
      if ((sl = allow_lds(run_general)) != WS_OK) return sl;
    }
  }

  const wsg::KernelEntry* traced = (kind == WS_CALIB_NONE && !p.ragged) ? find_kernel(*cfg, 1) : nullptr;
  if (traced && (sl = allow_lds(traced->fn)) != WS_OK) return sl;

  ws_gemm_handle* h = new (std::nothrow) ws_gemm_handle();
  if (!h) return WS_ERR_INVALID_ARG;
  h->M = M;
  h->N = N;
  h->K = K;
  h->cfg = *cfg;
  h->plan = p;
  h->general = general;
  h->plan_plain = p;
  h->plan_general = pg;
  h->run_plain = run_plain;
  h->run_general = run_general;
  h->whole_plain = whole_plain;
  h->whole_general = whole_general;
  h->whole = false;
  h->use_general = false;
  h->epi = ws_gemm_epilogue{1.0f, 0.0f, WS_OUT_F32};
  h->calibration = kind != WS_CALIB_NONE;
  h->traced = traced;
  h->device = dev;
  h->dbg = ws_gemm_debug{0, 0, 0};
  h->trace = nullptr;
  h->trace_wgs = 0;
  h->trace_iters = 0;
  hipError_t e = hipMalloc((void**)&h->d_err, 256);
  if (e != hipSuccess) {
    delete h;
    return hip_fail("hipMalloc", e);
  }
  e = hipMemset(h->d_err, 0, 256);
  if (e != hipSuccess) {
    (void)hipFree(h->d_err);
    delete h;
    return hip_fail("hipMemset", e);
  }
  *out = h;
  return WS_OK;
}

}  // namespace

extern "C" {

ws_status ws_gemm_create(int64_t M, int64_t N, int64_t K, const ws_gemm_config* cfg,
                         ws_gemm_t* out) {
  return create_handle(M, N, K, cfg, WS_CALIB_NONE, out);
}

ws_status ws_gemm_create_calibration(int64_t M, int64_t N, int64_t K, const ws_gemm_config* cfg,
                                     int32_t kind, ws_gemm_t* out) {
  if (kind < WS_CALIB_EMPTY || kind > WS_CALIB_LOAD_AB) return WS_ERR_INVALID_ARG;
  return create_handle(M, N, K, cfg, kind, out);
}

ws_status ws_gemm_run(ws_gemm_t h, const void* A, const void* B, void* C, hipStream_t stream) {
  if (!h) return WS_ERR_INVALID_ARG;
  // Pointers that the problem does not read or write may be NULL: nothing
  // at all when C is empty, A and B when K = 0.
  const bool c_used = h->M > 0 && h->N > 0;
  const bool a_used = c_used && h->K > 0, b_used = a_used;
  if ((a_used && !A) || (b_used && !B) || (c_used && !C)) return WS_ERR_INVALID_ARG;
  const uintptr_t c_align = h->epi.out_dtype == WS_OUT_F32 ? 3 : 1;
  if ((a_used && ((uintptr_t)A & 15)) || (b_used && ((uintptr_t)B & 15)) ||
      (c_used && ((uintptr_t)C & c_align)))
    return WS_ERR_INVALID_ARG;
  if (h->plan.grid == 0) {  // empty problem
    if (!c_used) return WS_OK;
    // K = 0: C <- alpha 0 + beta C
    const int64_t n = h->M * h->N;
    const int64_t want = (n + 255) / 256;
    const int blocks = (int)(want < 8192 ? want : 8192);
    const void* fn = reinterpret_cast<const void*>(&wsg::ws_scale_kernel<float>);
    if (h->epi.out_dtype == WS_OUT_BF16) fn = reinterpret_cast<const void*>(&wsg::ws_scale_kernel<__bf16>);
    if (h->epi.out_dtype == WS_OUT_F16) fn = reinterpret_cast<const void*>(&wsg::ws_scale_kernel<_Float16>);
    void* c = C;
    int64_t count = n;
    float beta = h->epi.beta;
    void* params[] = {&c, &count, &beta};
    WSG_HIP(hipLaunchKernel(fn, dim3(blocks), dim3(256), params, 0, stream));
    return WS_OK;
  }
  wsg::KernelArgs a;
  a.A = (const uint16_t*)A;
  a.B = (const uint16_t*)B;
  a.C = C;
  a.M = (int32_t)h->M;
  a.N = (int32_t)h->N;
  a.K = (int32_t)h->K;
  a.spin_limit = h->dbg.spin_limit > 0 ? h->dbg.spin_limit : kDefaultSpinLimit;
  a.producer_delay = h->dbg.producer_delay;
  a.consumer_delay = h->dbg.consumer_delay;
  a.err = h->d_err;
  a.trace = h->trace;
  a.trace_wgs = h->trace_wgs;
  a.trace_iters = h->trace_iters;
  a.load_path = h->cfg.load_path;
  a.alpha = h->epi.alpha;
  a.beta = h->epi.beta;
  a.out_dtype = h->epi.out_dtype;
  a.clock = (unsigned long long*)((char*)h->d_err + kClockOffset);
  // the traced twin runs the whole-tile plan, which its records describe
  if (h->trace && h->traced) return launch_run(whole_run(h->traced->fn, h->cfg, 0, h->plan), a, stream);
  return launch_run(current_run(h), a, stream);
}

ws_status ws_gemm_sync_status(ws_gemm_t h, hipStream_t stream) {
  if (!h) return WS_ERR_INVALID_ARG;
  WSG_HIP(hipStreamSynchronize(stream));
  int32_t v = 0;
  WSG_HIP(hipMemcpy(&v, h->d_err, sizeof(v), hipMemcpyDeviceToHost));
  if (v != 0) {
    WSG_HIP(hipMemset(h->d_err, 0, sizeof(int32_t)));
    return WS_ERR_TIMEOUT;
  }
  return WS_OK;
}

ws_status ws_gemm_clock(ws_gemm_t h, hipStream_t stream, uint64_t* shader_cycles,
                        uint64_t* ref_ticks, int64_t* launches) {
  if (!h || !shader_cycles || !ref_ticks || !launches) return WS_ERR_INVALID_ARG;
  WSG_HIP(hipStreamSynchronize(stream));
  uint64_t v[3] = {0, 0, 0};
  char* p = (char*)h->d_err + kClockOffset;
  WSG_HIP(hipMemcpy(v, p, sizeof(v), hipMemcpyDeviceToHost));
  WSG_HIP(hipMemset(p, 0, sizeof(v)));
  *shader_cycles = v[0];
  *ref_ticks = v[1];
  *launches = (int64_t)v[2];
  return WS_OK;
}

ws_status ws_gemm_query(ws_gemm_t h, ws_gemm_plan_info* out) {
  if (!h || !out) return WS_ERR_INVALID_ARG;
  to_info(h->plan, out);
  out->general = (h->plan.ragged || (h->use_general && h->plan.grid > 0)) ? 1 : 0;  // empty: no GEMM kernel
  return WS_OK;
}

ws_status ws_gemm_set_partition(ws_gemm_t h, int32_t partition) {
  if (!h || (partition != WS_PARTITION_AUTO && partition != WS_PARTITION_WHOLE)) return WS_ERR_INVALID_ARG;
  h->whole = partition == WS_PARTITION_WHOLE;
  return WS_OK;
}

ws_status ws_gemm_query_launches(ws_gemm_t h, ws_gemm_launch_info* out, int32_t* count) {
  if (!h || !out || !count) return WS_ERR_INVALID_ARG;
  *count = 0;
  if (h->plan.grid > 0) to_launches(current_run(h), out, count);
  return WS_OK;
}

ws_status ws_gemm_set_epilogue(ws_gemm_t h, const ws_gemm_epilogue* epi) {
  if (!h) return WS_ERR_INVALID_ARG;
  const ws_gemm_epilogue e = epi ? *epi : ws_gemm_epilogue{1.0f, 0.0f, WS_OUT_F32};
  if (!__builtin_isfinite(e.alpha) || !__builtin_isfinite(e.beta) || e.out_dtype < WS_OUT_F32 ||
      e.out_dtype > WS_OUT_F16)
    return WS_ERR_INVALID_ARG;
  const bool dflt = default_epilogue(e);
  if (h->calibration) return dflt ? WS_OK : WS_ERR_UNSUPPORTED;
  // Empty problems launch no GEMM kernel (K = 0 runs the epilogue alone), and
  // shapes the tiles do not divide run the general kernel whatever the
  // epilogue.
  if (h->plan_plain.grid == 0 || h->plan_plain.ragged) {
    h->epi = e;
    h->use_general = !dflt;
    return WS_OK;
  }
  if (dflt) {
    h->epi = e;
    h->use_general = false;
    h->plan = h->plan_plain;
    return WS_OK;
  }
  if (!h->general) return WS_ERR_UNSUPPORTED;
  if (h->trace) return WS_ERR_UNSUPPORTED;  // the traced twin has the plain epilogue
  h->epi = e;
  h->use_general = true;
  h->plan = h->plan_general;
  return WS_OK;
}

ws_status ws_gemm_set_debug(ws_gemm_t h, const ws_gemm_debug* dbg) {
  if (!h) return WS_ERR_INVALID_ARG;
  if (!dbg) {
    h->dbg = ws_gemm_debug{0, 0, 0};
    return WS_OK;
  }
  if (dbg->spin_limit < 0 || dbg->producer_delay < 0 || dbg->consumer_delay < 0 ||
      dbg->producer_delay > 1000 || dbg->consumer_delay > 1000)
    return WS_ERR_INVALID_ARG;
  h->dbg = *dbg;
  return WS_OK;
}

ws_status ws_gemm_set_trace(ws_gemm_t h, void* buffer, int64_t bytes, int32_t wgs,
                            int32_t iters) {
  if (!h) return WS_ERR_INVALID_ARG;
  if (!buffer) {
    h->trace = nullptr;
    h->trace_wgs = 0;
    h->trace_iters = 0;
    return WS_OK;
  }
  if (((uintptr_t)buffer & 3) || wgs <= 0 || iters <= 0 || wgs > h->plan.grid) return WS_ERR_INVALID_ARG;
  if (!h->traced || !default_epilogue(h->epi)) return WS_ERR_UNSUPPORTED;
  if ((int64_t)wgs * iters * wsg::kTraceEvents * 4 > bytes) return WS_ERR_INVALID_ARG;
  h->trace = (uint32_t*)buffer;
  h->trace_wgs = wgs;
  h->trace_iters = iters;
  return WS_OK;
}

ws_status ws_gemm_destroy(ws_gemm_t h) {
  if (!h) return WS_OK;
  ws_status s = WS_OK;
  if (h->d_err && hipFree(h->d_err) != hipSuccess) s = WS_ERR_HIP;
  delete h;
  return s;
}

ws_status ws_gemm_run_noalloc(int64_t M, int64_t N, int64_t K, const ws_gemm_config* cfg,
                              const void* A, const void* B, float* C, hipStream_t stream) {
  if (!cfg) return WS_ERR_INVALID_ARG;
  // Everything that needs no device: validation and the kernel.
  wsg::PlanOut p;
  int s = wsg::plan_launch(plan_in(M, N, K, *cfg, 1, 1), &p);
  if (s != wsg::kPlanOk) return from_plan(s);
  const bool c_used = M > 0 && N > 0;
  const bool a_used = c_used && K > 0, b_used = a_used;
  if ((a_used && !A) || (b_used && !B) || (c_used && !C)) return WS_ERR_INVALID_ARG;
  if ((a_used && ((uintptr_t)A & 15)) || (b_used && ((uintptr_t)B & 15)) || (c_used && ((uintptr_t)C & 3)))
    return WS_ERR_INVALID_ARG;
  if (p.grid == 0) {  // empty problem
    if (!c_used) return WS_OK;
    // K = 0: C = 0 (the product of an empty sum)
    const int64_t n = M * N;
    const int64_t want = (n + 255) / 256;
    const int blocks = (int)(want < 8192 ? want : 8192);
    void* c = C;
    int64_t count = n;
    float beta = 0.0f;
    void* params[] = {&c, &count, &beta};
    WSG_HIP(hipLaunchKernel(reinterpret_cast<const void*>(&wsg::ws_scale_kernel<float>), dim3(blocks),
                            dim3(256), params, 0, stream));
    return WS_OK;
  }
  if (!find_kernel(*cfg, 0, wsg::kModeGemm, p.ragged)) return WS_ERR_UNSUPPORTED;
  // The device the launch goes to (the stream's), its scratch and size.
  int dev = 0;
  if (stream) {
    WSG_HIP(hipStreamGetDevice(stream, &dev));
  } else {
    WSG_HIP(hipGetDevice(&dev));
  }
  StaticDevice sd;
  const ws_status st = static_device(dev, &sd);
  if (st != WS_OK) return st;
  Run run;
  ws_status ls = plan_run(M, N, K, *cfg, sd.cus, p.ragged, true, &run);
  if (ls == WS_OK) ls = allow_lds(run);
  if (ls != WS_OK) return ls;
  wsg::KernelArgs a{};
  a.A = (const uint16_t*)A;
  a.B = (const uint16_t*)B;
  a.C = C;
  a.M = (int32_t)M;
  a.N = (int32_t)N;
  a.K = (int32_t)K;
  a.spin_limit = kDefaultSpinLimit;
  a.err = (int32_t*)sd.scratch;  // this device's copy of the scratch array
  a.load_path = cfg->load_path;
  a.alpha = 1.0f;
  a.beta = 0.0f;
  a.out_dtype = WS_OUT_F32;
  return launch_run(run, a, stream);
}

}  // extern "C"
