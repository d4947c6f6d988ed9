// Warp-specialised tiled GEMM kernel for gfx950 (MI355X).
//
// C (M x N, fp32) = A (M x K) * B (K x N), A and B fp16 or bf16, all row-major
// (the general variant below also stores alpha A B + beta C as fp32, bf16 or
// fp16, and handles partial edge tiles).
// The kernel follows the producer/consumer structure of the GeMM-WS kernel the
// paper models (Section 1.3, Algorithm 1): inside each workgroup, producer
// ("DMA") wavefronts move A and B tiles from global memory into a circular
// buffer of `stages` slots in LDS, and consumer ("MATH") wavefronts take the
// tiles out, run the contraction on the matrix cores and write the output
// tile (the epilogue).  The two sides synchronise through wait/signal
// counters, one pair per slot (Section 1.3: the buffer blocks producers when
// full and consumers when empty).
//
// gfx950 mapping
//  * Roles are chosen per wavefront from the wave index, so no wave diverges
//    (Section 1.2).  Waves [0, NC) are consumers, waves [NC, NC + NP) are
//    producers.  With NC = 4 the consumers sit one per SIMD and tile the
//    output block 2 x 2; with NC = 8 (256 x 256 tiles, four producer waves)
//    two per SIMD, 2 x 4.
//  * Producers move a tile in 16-byte chunks, 1 KiB per wave instruction,
//    either staged through VGPRs several K-iterations ahead
//    (buffer_load_dwordx4, then ds_write_b128 once the slot is free; the
//    default) or with buffer_load_dwordx4 ... lds straight into the slot.  The
//    LDS placement of every chunk is fixed by the lane; the layout below is
//    produced by choosing which global chunk each lane fetches.
//  * 1:1 split (NP == NC): every producer loads a share of the A tile and then
//    a share of the B tile, in that order (one DMA warp loading both tiles).
//    2:1 split (NP == 2 NC): the first half of the producers loads A, the
//    second half loads B, concurrently (two DMA warps, one tile each).  With
//    four consumer waves the waves that load a tile form two groups that take
//    the K-iterations in turn.
//  * Consumers read operands with ds_read_b128 (A, K-contiguous) and
//    ds_read_b64_tr_b16 (B, N-contiguous, transposed by the read) and
//    accumulate with v_mfma_f32_32x32x16_{bf16,f16} in fp32.  The K loop of a
//    tile is a generated asm block, in the plain and in the general kernels:
//    with one or four consumer waves the streaming loop (consumer_stream,
//    ws_stream_loop.inc, configurations in gen_stream_loop.py), with eight
//    (two per SIMD) the register-lean roll loop (consumer_roll,
//    ws_deep_loop.inc, gen_deep_loop.py; also in its event-traced twin and in
//    that of the four-consumer 128 x 128 x 32 kernel).  The other traced twins
//    run compiler-scheduled consumers.
//  * The grid is persistent: at most one workgroup per CU slot, each walking
//    output tiles in dispatch rounds (Section 2.1, "Wave").  The tile order
//    places the tiles that run at the same time on one XCD next to each
//    other so that they share A row panels and B column panels in that XCD's
//    L2.
//  * Variants of one template: the plain GEMM, its event-traced twin, the
//    calibration kernels of the performance model (KernelMode), and the
//    general variant (GENERAL: partial tiles and the alpha / beta epilogue).
//    Slot and counter arithmetic is in ws_ring.hpp.
//
// LDS layout (dynamic shared memory)
//   [0, 256)            counters: full[8], empty[8], abort
//   [256 + s * STAGE)   slot s: A tile (TM x TK) then B tile (TK x TN)
// A tile: row-major, each row split in 16-byte chunks (8 elements); chunk c of
//   row r is stored at position c ^ swz_a(r).
// B tile: 4 x 32 element blocks of 256 bytes; block (kq, nd) holds rows
//   4 kq .. 4 kq + 3 and columns 32 nd .. 32 nd + 31, row-major inside the
//   block (64 bytes a row); blocks are ordered kq-major.  A 16-lane
//   transposed read takes one 16-column half of a block (32 bytes of each
//   row), two neighbouring groups the whole block.  Why 32 columns: chunk q
//   goes to byte 16 q of the tile on every load path, so four neighbouring
//   lanes fetch the 64 bytes of one block row.  The address unit takes four
//   16-byte lanes per clock when they lie in one cache line and twice as long
//   when they do not: with 16-column blocks (two rows per four lanes) B loads
//   ran at 31.9 bytes per clock and CU, with these at 63.8, the rate of the A
//   loads and of linear ones (L2-resident panel, one workgroup per CU).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ws_ring.hpp"

#include "ws_gemm_plan.hpp"

namespace wsg {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(4))) short i16x4_t;
typedef __attribute__((ext_vector_type(8))) short i16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

#define WSG_LDS __attribute__((address_space(3)))

constexpr int kHeaderBytes = 256;
constexpr int kMaxStages = 8;

struct KernelArgs {
  const uint16_t* A;
  const uint16_t* B;
  void* C;             // fp32, or the general variant's output type
  int32_t M, N, K;
  int32_t tiles_m, tiles_n, num_tiles;
  int32_t iters;       // S = K / TK
  int32_t stages;      // ring slots P
  int32_t group_m;     // tile rows per raster group
  int32_t xcd_remap;   // 1: remap workgroup ids so one XCD gets consecutive tiles
  int32_t spin_limit;  // bounded waits: give up after this many polls
  int32_t producer_delay;  // debug: s_sleep bursts per K-iteration in producers
  int32_t consumer_delay;  // debug: s_sleep bursts per K-iteration in consumers
  int32_t* err;            // set to 1 when a bounded wait gives up
  uint32_t* trace;         // event trace (null: off), [trace_wgs][trace_iters][kTraceEvents]
  int32_t trace_wgs;       // workgroups 0 .. trace_wgs-1 are traced
  int32_t trace_iters;     // K-iterations recorded per workgroup
  int32_t load_path;       // producer load path: 0 register-staged, 1 LDS-DMA
  // General variant only: C <- alpha * (A B) + beta * C, C of type out_dtype.
  float alpha, beta;
  int32_t out_dtype;       // OutType
  // Launch clock (null: off): workgroup 0's first wave adds the shader-clock
  // cycles and the 100 MHz reference ticks it spans to clock[0] and clock[1],
  // and 1 to clock[2]; their ratio is the average shader clock of the launch.
  unsigned long long* clock;
  // Second tile region (see TileRegions).
  int32_t region2, row1, tiles2_m, tiles2_n, col2;
};

// Output element type of the general variant's epilogue.
enum OutType { kOutF32 = 0, kOutBF16 = 1, kOutF16 = 2 };

// Event trace: one record of kTraceEvents 32-bit shader-clock stamps per
// K-iteration q of a traced workgroup (the paper's event analysis, Section
// 2.2: S_a(i), S_b(i), S_m(i)).
//   0  producer starts issuing the A tile of q            (S_a)
//   1  producer starts issuing the B tile of q            (S_b)
//   2  the A tile of q has landed in LDS (signal)
//   3  the B tile of q has landed in LDS (signal)
//   4  consumer wave 0 observes slot q full
//   5  consumer wave 0 starts the MFMAs of q              (S_m)
//   6  consumer wave 0 releases slot q
//   7  consumer wave 0 finished the epilogue (last K-iteration of a tile), else 0
constexpr int kTraceEvents = 8;
// LDS header words holding the producer stamps of each slot (indices 24..55).
constexpr int kStampIssueA = 24, kStampIssueB = 32, kStampLandA = 40, kStampLandB = 48;

// Launch clock (KernelArgs::clock), taken by one wave at the start and the
// end of the kernel.  Both counters are read with scalar loads that are
// waited for at once, so nothing of theirs is in flight afterwards.
struct LaunchClock {
  uint64_t c0 = 0, r0 = 0;
  bool on = false;
  __device__ __forceinline__ void start(const KernelArgs& args, int wave) {
    on = args.clock != nullptr && blockIdx.x == 0 && wave == 0;  // wave-uniform
    if (on) {
      c0 = __builtin_amdgcn_s_memtime();
      r0 = __builtin_amdgcn_s_memrealtime();
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
  }
  __device__ __forceinline__ void stop(const KernelArgs& args, int lane) {
    if (on) {
      const uint64_t c1 = __builtin_amdgcn_s_memtime();
      const uint64_t r1 = __builtin_amdgcn_s_memrealtime();
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (lane == 0) {
        atomicAdd(&args.clock[0], (unsigned long long)(c1 - c0));
        atomicAdd(&args.clock[1], (unsigned long long)(r1 - r0));
        atomicAdd(&args.clock[2], 1ull);
      }
    }
  }
};

// Low 32 bits of the shader-clock counter (s_memtime).
__device__ __forceinline__ uint32_t cycles32() {
  return (uint32_t)__builtin_amdgcn_s_memtime();
}

// XOR swizzle of the 16-byte chunks of A-tile row r.  It depends on r & 31
// only, so rows 32 apart share it and the consumer can fold whole 32-row
// blocks into instruction offsets.  The operand read (lane l: row l & 31,
// chunk l / 32, or that chunk XOR 2 for the next k-step) is free of LDS bank
// conflicts with these choices, as measured with SQ_LDS_BANK_CONFLICT on
// gfx950 at every block and slot base the kernels use; at TK = 32,
// ((r >> 1) ^ (r >> 3)) & 3 and (r >> 1) & 3 cost four conflict cycles per
// read and no swizzle twelve.
template <int TK>
__host__ __device__ constexpr int swz_a(int r) {
  if constexpr (TK == 32) return (r ^ (r >> 2)) & 3;
  else if constexpr (TK == 64) return (r ^ ((r >> 3) & 1)) & 7;
  else return r & 15;
}

template <int TK>
constexpr bool swz_a_period32() {
  for (int r = 0; r < 256; ++r)
    if (swz_a<TK>(r) != swz_a<TK>(r & 31) || swz_a<TK>(r) < 0 || swz_a<TK>(r) >= TK / 8)
      return false;
  return true;
}
static_assert(swz_a_period32<32>() && swz_a_period32<64>() && swz_a_period32<128>(),
              "A swizzle must repeat every 32 rows and stay inside the row");

// True when rows r and r + step of an A tile use the same swizzle for every r.
template <int TK>
constexpr bool swz_a_step_invariant(int step) {
  for (int r = 0; r < 64; ++r)
    if (swz_a<TK>(r + step) != swz_a<TK>(r)) return false;
  return true;
}

// B tile layout: k-row and first column, inside the tile, of the 16-byte chunk
// stored at byte 16 q.
template <int TN>
__host__ __device__ constexpr int b_chunk_row(int q) {
  return (q >> 4) / (TN / 32) * 4 + ((q >> 2) & 3);
}
template <int TN>
__host__ __device__ constexpr int b_chunk_col(int q) {
  return (q >> 4) % (TN / 32) * 32 + (q & 3) * 8;
}

// Byte offset, inside the B tile, of a lane's transposed 8-byte read of
// k-step 0 in the 32 columns from `col` (a multiple of 32): 16-lane group g
// takes k-rows 8 (g / 2) .. 8 (g / 2) + 3 and the column half g % 2, lane j of
// the group 8 bytes (columns 4 (j % 4) ..) of row j / 4.
template <int TN>
__host__ __device__ constexpr uint32_t b_read_off(int lane, int col) {
  const int g = lane >> 4, j = lane & 15;
  return (uint32_t)(((2 * (g >> 1)) * (TN / 32) + col / 32) * 256 + (j >> 2) * 64 + (g & 1) * 32 + (j & 3) * 8);
}

// Every read lands on the chunk that holds its row and columns.
template <int TN>
constexpr bool b_layout_consistent() {
  for (int lane = 0; lane < 64; ++lane)
    for (int col = 0; col < TN; col += 32) {
      const int off = (int)b_read_off<TN>(lane, col), q = off >> 4;
      const int row = 8 * (lane >> 5) + ((lane & 15) >> 2);
      const int c = col + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      if (b_chunk_row<TN>(q) != row || b_chunk_col<TN>(q) + (off & 15) / 2 != c) return false;
    }
  return true;
}
static_assert(b_layout_consistent<32>() && b_layout_consistent<64>() && b_layout_consistent<128>() &&
                  b_layout_consistent<256>(),
              "B chunks and B reads must agree");

__device__ __forceinline__ uint32_t lds_peek(WSG_LDS uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Compiler-only fence: no memory access moves across it.
__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}

// signal(): add one to an LDS counter from lane 0 only, after every earlier
// LDS access of this wave has completed.  Done in one asm block with the exec
// mask narrowed to lane 0, so the surrounding code stays branch-free.
// YOUNGER: how many of this wave's most recent LDS operations may still be
// outstanding (LDS operations of a wave complete in order, so every older
// one has completed).  Scalar-memory loads share the counter and complete
// out of order, but one in flight only makes the wait stricter: the count
// bounds LDS and scalar operations together, so when it is at most YOUNGER
// at most YOUNGER LDS operations are outstanding, and those are the youngest.
template <int YOUNGER = 0, int COUNT = 1>
__device__ __forceinline__ void lds_signal(WSG_LDS uint32_t* p) {
  static_assert(YOUNGER >= 0 && YOUNGER <= 15, "lgkmcnt range");
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t addr = (uint32_t)(uintptr_t)p;
  const uint32_t one = COUNT;
  uint64_t saved;
  asm volatile(
      "s_waitcnt lgkmcnt(%3)\n\t"
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, 1\n\t"
      "ds_add_u32 %1, %2\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "v"(addr), "v"(one), "n"(YOUNGER)
      : "memory");
#endif
}

// signal() of the counter at p, together with a read of the counter at
// `peek`: the read goes out before the wait that the signal needs anyway (for
// the wave's own LDS writes), so it costs no LDS round trip of its own.
// Returns the value read (wave-uniform); the counters are monotonic, so a
// value that already satisfies a later wait stays valid.
template <int COUNT = 1>
__device__ __forceinline__ uint32_t lds_signal_peek(WSG_LDS uint32_t* p, WSG_LDS uint32_t* peek) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t addr = (uint32_t)(uintptr_t)p;
  const uint32_t paddr = (uint32_t)(uintptr_t)peek;
  const uint32_t one = COUNT;
  uint64_t saved;
  uint32_t v;
  asm volatile(
      "ds_read_b32 %1, %3\n\t"
      "s_waitcnt lgkmcnt(0)\n\t"
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, 1\n\t"
      "ds_add_u32 %2, %4\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved), "=&v"(v)
      : "v"(addr), "v"(paddr), "v"(one)
      : "memory");
  return __builtin_amdgcn_readfirstlane(v);
#else
  *p += COUNT;
  return *peek;
#endif
}

// signal() when `enable` (wave-uniform) is non-zero, as one asm block, so
// the caller's control flow gets no join.
template <int YOUNGER = 0>
__device__ __forceinline__ void lds_signal_if(WSG_LDS uint32_t* p, uint32_t enable) {
  static_assert(YOUNGER >= 0 && YOUNGER <= 15, "lgkmcnt range");
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t addr = (uint32_t)(uintptr_t)p;
  const uint32_t one = 1u;
  uint64_t saved;
  asm volatile(
      "s_cmp_eq_u32 %4, 0\n\t"
      "s_cbranch_scc1 1f\n\t"
      "s_waitcnt lgkmcnt(%3)\n\t"
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, 1\n\t"
      "ds_add_u32 %1, %2\n\t"
      "s_mov_b64 exec, %0\n"
      "1:"
      : "=&s"(saved)
      : "v"(addr), "v"(one), "n"(YOUNGER), "s"(__builtin_amdgcn_readfirstlane(enable))
      : "memory", "scc");
#endif
}

// Blocking read of an LDS counter, issued from asm so that the compiler does
// not order it behind outstanding LDS-DMA loads (it cannot prove the counter
// and the DMA destination are disjoint).  Result is wave-uniform.
__device__ __forceinline__ uint32_t lds_read_now(WSG_LDS uint32_t* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t addr = (uint32_t)(uintptr_t)p;
  uint32_t v;
  asm volatile(
      "ds_read_b32 %0, %1\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=v"(v)
      : "v"(addr)
      : "memory");
  return __builtin_amdgcn_readfirstlane(v);
#else
  return *p;
#endif
}

// Store a wave-uniform value to an LDS word from lane 0 (asm, so the producer's
// vmcnt accounting and the compiler's LDS ordering are untouched).
__device__ __forceinline__ void lds_stamp(WSG_LDS uint32_t* p, uint32_t value) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t addr = (uint32_t)(uintptr_t)p;
  uint64_t saved;
  asm volatile(
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, 1\n\t"
      "ds_write_b32 %1, %2\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "v"(addr), "v"(value)
      : "memory");
#endif
}

// wait(): poll *ctr until it reaches target (wrap-safe).  Returns true when
// it did; false when the workgroup aborted or this wait exceeded the poll
// limit (it then raises the workgroup abort flag and the device error word,
// so every wave drains quickly).  The result is wave-uniform.  The poll loop
// itself issues no vector-memory instruction, so it does not disturb the
// compiler's accounting of outstanding loads around it.
__device__ __forceinline__ void report_timeout(WSG_LDS uint32_t* abort_flag, int32_t* err) {
  if ((threadIdx.x & 63) == 0) {
    __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__device__ __forceinline__ bool wait_counter(WSG_LDS uint32_t* ctr, uint32_t target,
                                             WSG_LDS uint32_t* abort_flag, int spin_limit,
                                             int32_t* err) {
  int spins = 0;
  int status = 0;  // 0 reached, 1 aborted elsewhere, 2 timed out here
  while (true) {
    const uint32_t v = lds_read_now(ctr);
    if ((int32_t)(v - target) >= 0) break;
    if (lds_read_now(abort_flag)) {
      status = 1;
      break;
    }
    if (++spins > spin_limit) {
      status = 2;
      break;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  compiler_fence();
  status = __builtin_amdgcn_readfirstlane(status);
  if (status == 2) report_timeout(abort_flag, err);
  return status == 0;
}

// The same wait as one asm block, so that it adds no join to the caller's
// control flow (the consumer's K loop stays a single basic block and its
// operand registers are not shuffled around a join).  `seen` is a value of
// *ctr read earlier: when it already satisfies the target, nothing is read.
// Returns 0 when the counter reached the target, 1 when the workgroup abort
// flag is up, 2 after `limit` polls; wave-uniform.
__device__ __forceinline__ uint32_t wait_until(uint32_t seen, WSG_LDS uint32_t* ctr,
                                               WSG_LDS uint32_t* abort_flag, uint32_t target,
                                               int32_t limit, uint32_t enable = 1) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t ca = (uint32_t)(uintptr_t)ctr, aa = (uint32_t)(uintptr_t)abort_flag;
  uint32_t st, spins, v0, v1;
  asm volatile(
      "s_mov_b32 %[st], 0\n\t"
      "s_cmp_eq_u32 %[en], 0\n\t"
      "s_cbranch_scc1 2f\n\t"
      "v_readfirstlane_b32 %[st], %[seen]\n\t"
      "s_sub_u32 %[st], %[st], %[target]\n\t"
      "s_cmp_ge_i32 %[st], 0\n\t"
      "s_mov_b32 %[st], 0\n\t"
      "s_cbranch_scc1 2f\n\t"
      "s_mov_b32 %[spins], 0\n"
      "1:\n\t"
      "ds_read_b32 %[v0], %[ca]\n\t"
      "ds_read_b32 %[v1], %[aa]\n\t"
      "s_waitcnt lgkmcnt(0)\n\t"
      "v_readfirstlane_b32 %[st], %[v0]\n\t"
      "s_sub_u32 %[st], %[st], %[target]\n\t"
      "s_cmp_ge_i32 %[st], 0\n\t"
      "s_mov_b32 %[st], 0\n\t"
      "s_cbranch_scc1 2f\n\t"
      "v_readfirstlane_b32 %[st], %[v1]\n\t"
      "s_cmp_lg_u32 %[st], 0\n\t"
      "s_mov_b32 %[st], 1\n\t"
      "s_cbranch_scc1 2f\n\t"
      "s_add_u32 %[spins], %[spins], 1\n\t"
      "s_cmp_gt_i32 %[spins], %[limit]\n\t"
      "s_mov_b32 %[st], 2\n\t"
      "s_cbranch_scc1 2f\n\t"
      "s_sleep 1\n\t"
      "s_branch 1b\n"
      "2:"
      : [st] "=&s"(st), [spins] "=&s"(spins), [v0] "=&v"(v0), [v1] "=&v"(v1)
      : [seen] "v"(seen), [target] "s"(__builtin_amdgcn_readfirstlane(target)), [ca] "v"(ca),
        [aa] "v"(aa), [limit] "s"(limit), [en] "s"(__builtin_amdgcn_readfirstlane(enable))
      : "memory", "scc");
  return st;
#else
  if (!enable) return 0u;
  return (int32_t)(*ctr - target) >= 0 ? 0u : (*abort_flag ? 1u : 2u);
#endif
}

// Test hook: n bursts of ~8k-cycle sleeps (n wave-uniform; 0 in production),
// as one asm block so that the caller's loop gets no join.
__device__ __forceinline__ void debug_delay(int n) {
#if defined(__HIP_DEVICE_COMPILE__)
  uint32_t left;
  asm volatile(
      "s_mov_b32 %0, %1\n\t"
      "s_cmp_le_i32 %0, 0\n\t"
      "s_cbranch_scc1 2f\n"
      "1:\n\t"
      "s_sleep 127\n\t"
      "s_sub_u32 %0, %0, 1\n\t"
      "s_cmp_lg_u32 %0, 0\n\t"
      "s_cbranch_scc1 1b\n"
      "2:"
      : "=&s"(left)
      : "s"(__builtin_amdgcn_readfirstlane(n))
      : "scc");
#else
  (void)n;
#endif
}

template <bool BF16>
__device__ __forceinline__ f32x16_t mfma32x32x16(const i16x8_t& a, const i16x8_t& b,
                                                 const f32x16_t& c) {
  if constexpr (BF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a),
                                                  __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16>
struct Cfg {
  static constexpr int NP = NPW;                     // producer waves
  static constexpr int NW = NC + NP;                 // waves per workgroup
  static constexpr int WGM = (NC >= 4) ? 2 : 1;      // consumer grid rows
  static constexpr int WGN = (NC == 8) ? 4 : (NC == 4) ? 2 : 1;  // consumer grid cols
  static constexpr int WM = TM / WGM;                // wave tile rows
  static constexpr int WN = TN / WGN;                // wave tile cols
  static constexpr int BM = WM / 32;                 // 32x32 blocks per wave (rows)
  static constexpr int BN = WN / 32;
  static constexpr int KS = TK / 16;                 // MFMA k-steps per K-iteration
  static constexpr int A_BYTES = TM * TK * 2;
  static constexpr int B_BYTES = TK * TN * 2;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int A_INSTR = A_BYTES / 1024;     // 1 KiB DMA instructions per A tile
  static constexpr int B_INSTR = B_BYTES / 1024;
  static constexpr int CA = TK / 8;                  // 16-byte chunks per A row
  static constexpr int NQ = TN / 16;                 // 16-column halves of B blocks per block-row
  static_assert(NC == 1 || NC == 4 || NC == 8, "consumer waves must be 1, 4 or 8");
  static_assert(SPLIT == 1 || SPLIT == 2, "split must be 1:1 or 2:1");
  // producer waves: one group of NC (1:1) or two of NC (2:1); with NC = 4 also
  // two groups of 2 (2:1 at eight waves); with NC = 8 one group of 4 (1:1) or
  // two of 2 (2:1), twelve waves in all.
  static_assert((NP == NC * SPLIT && NC != 8) || (NC == 4 && NP == 4) || (NC == 8 && NP == 4),
                "unsupported producer / consumer arrangement");
  static_assert(SPLIT == 1 || NP % 2 == 0, "two producer groups need an even number of waves");
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile must be a multiple of 32x32");
  static_assert(TK == 32 || TK == 64 || TK == 128, "TK must be 32, 64 or 128");
  static_assert(A_BYTES % 1024 == 0 && B_BYTES % 1024 == 0, "tiles must be whole KiB");
};

// What a kernel instance runs.  kModeGemm is the GEMM; the others are the
// calibration kernels of the paper's evaluation (Section 4.2), built from the
// same code so that they measure this kernel's own costs:
//   kModeLoadA / kModeLoadB  the producers load only the A (B) tiles of every
//                            K-iteration; the consumers take each slot and
//                            release it without reading it; C is not written.
//   kModeMath                the producers release slots without loading; the
//                            consumers read and multiply whatever the slots
//                            hold; C is not written.
//   kModeEpilogue            no K loop: the consumers store one zero tile per
//                            output tile, the producers exit.
//   kModeLoadAB              the producers load both tiles as in the GEMM; the
//                            consumers release every slot unread.
enum KernelMode {
  kModeGemm = 0, kModeLoadA = 1, kModeLoadB = 2, kModeMath = 3, kModeEpilogue = 4, kModeLoadAB = 5
};

typedef __attribute__((ext_vector_type(4))) int i32x4_t;

// Producer loads and the epilogue's stores go through a raw buffer resource
// over a tile panel: the base sits in SGPRs and each lane adds a 32-bit byte
// offset (panel offsets stay below 2^31, checked by the plan), so an access
// needs no 64-bit address arithmetic on the vector ALU of a SIMD whose other
// waves issue MFMAs.  Word 3 of the descriptor: data format
// 32 bits (field at bits 15-18 = 4), every other field zero (no swizzle, no
// index stride); the record count is the largest, so no offset is clipped.
constexpr int kRawBufferWord3 = 0x00020000;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t panel_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, -1, kRawBufferWord3);
}
// Cache-policy operand of the raw buffer builtins that marks an access
// non-temporal (the `nt` bit).
constexpr int kBufferNonTemporal = 2;
__device__ __forceinline__ i32x4_t panel_load16(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_bit_cast(i32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, 0));
}
// The general variant's producers read through resources whose record count
// ends at the end of the matrix (at most 2^31 bytes: the plan keeps panel
// offsets under 2^31).  A chunk outside A or B lies past the record count or
// is read from offset kOutsidePanel = 2^31; the range check of a raw buffer
// load returns zeros for it without touching memory.
constexpr uint32_t kOutsidePanel = 0x80000000u;
// Record count: the bytes from the panel base to the end of the matrix, at
// most 2^31; a row-major panel's rows past the matrix's last row read as
// zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t panel_rsrc_to_end(const void* base, int64_t bytes_left) {
  const uint32_t n = bytes_left < (int64_t)kOutsidePanel ? (uint32_t)bytes_left : kOutsidePanel;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)n, kRawBufferWord3);
}
// 16 bytes per lane straight into LDS: lane l's bytes land at dst + 16 l.
__device__ __forceinline__ void panel_load16_lds(__amdgpu_buffer_rsrc_t r, WSG_LDS void* dst, uint32_t byte_off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, byte_off, 0, 0, 0);
}
// Epilogue: the fp32 tile of consumer wave (wm, wn) to C.  acc[mb][nb][e] is
// row 8(e/4) + 4(lane/32) + e%4, column lane%32 of the 32x32 block.  The row
// pitch is made opaque so that the address arithmetic stays here instead of
// being hoisted (and spilled) out of the caller's K loop.
//
// GENERAL: elements outside C (partial edge tiles) are not stored, and the
// epilogue is the BLAS one, C <- alpha * (A B) + beta * C, rounded once to
// the output type (round to nearest even); beta == 0 does not read C.
template <typename T>
__device__ __forceinline__ float load_out(const T* p) {
  return (float)*p;
}
// One specialisation per output type T, READ_C (beta != 0) and MASK (the
// wave tile crosses an edge of C).  The old C of EG consecutive k-step rows
// is loaded before any of them is stored, so those loads overlap.
template <int TM, int TN, int WM, int WN, int BM, int BN, int EG, typename T, bool READ_C, bool MASK>
__device__ __forceinline__ void store_tile_general(const KernelArgs& args,
                                                   const f32x16_t (&acc)[BM][BN], int ti, int tj,
                                                   int wm, int wn, int lane) {
  static_assert(16 % EG == 0, "row groups split the 16 accumulator rows");
  constexpr uint32_t ES = sizeof(T);
  const float alpha = args.alpha, beta = args.beta;
  uint32_t ldc = (uint32_t)args.N * ES;
  asm volatile("" : "+s"(ldc));
  // Lane-derived offsets are computed here, not hoisted into the caller's
  // prologue and kept (or spilled) across its K loop.
  asm volatile("" : "+v"(lane));
  const int r0 = ti * TM + wm * WM, c0 = tj * TN + wn * WN;
  char* cbase = (char*)args.C + ((int64_t)r0 * args.N + c0) * ES;
  const uint32_t lane_off = (uint32_t)(4 * (lane >> 5)) * ldc + (uint32_t)(lane & 31) * ES;
  // rows / columns of C left from this lane's first element
  const int rows_left = args.M - r0 - 4 * (lane >> 5);
  const int cols_left = args.N - c0 - (lane & 31);
#pragma unroll
  for (int mb = 0; mb < BM; ++mb)
#pragma unroll
    for (int e0 = 0; e0 < 16; e0 += EG) {
      float old[EG][BN];
      if constexpr (READ_C) {
#pragma unroll
        for (int i = 0; i < EG; ++i) {
          const int e = e0 + i, dr = mb * 32 + 8 * (e >> 2) + (e & 3);
#pragma unroll
          for (int nb = 0; nb < BN; ++nb) {
            old[i][nb] = 0.0f;
            if (!MASK || (dr < rows_left && nb * 32 < cols_left))
              old[i][nb] = load_out((const T*)(cbase + (uint32_t)dr * ldc + lane_off + nb * 32 * ES));
          }
        }
      }
#pragma unroll
      for (int i = 0; i < EG; ++i) {
        const int e = e0 + i, dr = mb * 32 + 8 * (e >> 2) + (e & 3);
#pragma unroll
        for (int nb = 0; nb < BN; ++nb) {
          if (!MASK || (dr < rows_left && nb * 32 < cols_left)) {
            float v = alpha * acc[mb][nb][e];
            if constexpr (READ_C) v = __builtin_fmaf(beta, old[i][nb], v);
            *(T*)(cbase + (uint32_t)dr * ldc + lane_off + nb * 32 * ES) = (T)v;
          }
        }
      }
    }
}

template <int TM, int TN, int WM, int WN, int BM, int BN, int EG, typename T>
__device__ __forceinline__ void store_tile_general_t(const KernelArgs& args,
                                                     const f32x16_t (&acc)[BM][BN], int ti, int tj,
                                                     int wm, int wn, int lane) {
  const bool read_c = args.beta != 0.0f;
  const bool mask = ti * TM + wm * WM + WM > args.M || tj * TN + wn * WN + WN > args.N;
  if (read_c) {
    if (mask)
      store_tile_general<TM, TN, WM, WN, BM, BN, EG, T, true, true>(args, acc, ti, tj, wm, wn, lane);
    else
      store_tile_general<TM, TN, WM, WN, BM, BN, EG, T, true, false>(args, acc, ti, tj, wm, wn, lane);
  } else {
    if (mask)
      store_tile_general<TM, TN, WM, WN, BM, BN, EG, T, false, true>(args, acc, ti, tj, wm, wn, lane);
    else
      store_tile_general<TM, TN, WM, WN, BM, BN, EG, T, false, false>(args, acc, ti, tj, wm, wn, lane);
  }
}

// EG: k-step rows whose old C values are loaded together by the general
// epilogue (fewer when registers are tight).
template <int TM, int TN, int WM, int WN, int BM, int BN, bool GENERAL = false, int EG = 16>
__device__ __forceinline__ void store_tile(const KernelArgs& args, const f32x16_t (&acc)[BM][BN],
                                           int ti, int tj, int wm, int wn, int lane) {
  if constexpr (GENERAL) {
    const int od = __builtin_amdgcn_readfirstlane(args.out_dtype);
    if (od == kOutBF16)
      store_tile_general_t<TM, TN, WM, WN, BM, BN, EG, __bf16>(args, acc, ti, tj, wm, wn, lane);
    else if (od == kOutF16)
      store_tile_general_t<TM, TN, WM, WN, BM, BN, EG, _Float16>(args, acc, ti, tj, wm, wn, lane);
    else
      store_tile_general_t<TM, TN, WM, WN, BM, BN, EG, float>(args, acc, ti, tj, wm, wn, lane);
  } else {
    uint32_t ldc = (uint32_t)args.N * 4u;
    asm volatile("" : "+s"(ldc));
    const char* cbase = (const char*)args.C +
                        (((int64_t)ti * TM + wm * WM) * (int64_t)args.N + (int64_t)tj * TN + wn * WN) * 4;
    // the wave tile's rows lie below T_M * N * 4 < 2^31 bytes from cbase
    const __amdgpu_buffer_rsrc_t crs = panel_rsrc(cbase);
    const uint32_t lane_off = (uint32_t)(4 * (lane >> 5)) * ldc + (uint32_t)(lane & 31) * 4u;
#pragma unroll
    for (int mb = 0; mb < BM; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t row_off = (uint32_t)(mb * 32 + 8 * (e >> 2) + (e & 3)) * ldc;  // wave-uniform
#pragma unroll
        for (int nb = 0; nb < BN; ++nb) {  // non-temporal: C is not read again here, the panels are
          // copy the element out first: a bit cast of a vector element lvalue reads element 0
          const float v = acc[mb][nb][e];
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), crs, (int)(lane_off + nb * 128),
                                                (int)row_off, kBufferNonTemporal);
        }
      }
  }
}

// ---------------------------------------------------------------------------
// Per-workgroup tile sequence (identical in both roles).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void tile_at(const KernelArgs& args, int v, int* ti, int* tj) {
  const TileRegions r{args.tiles_m, args.tiles_n, args.group_m, args.region2, args.row1, args.tiles2_m, args.tiles2_n,
                      args.col2, args.num_tiles};
  region_tile(r, v, ti, tj);
}
__device__ __forceinline__ int first_slot(const KernelArgs& args) {
  const int G = gridDim.x;
  return args.xcd_remap ? xcd_slot(blockIdx.x, G) : (int)blockIdx.x;
}

// Events of one kind that a producer wave stores into its workgroup's trace
// record, batched: lane k of `vals` holds the event of K-iteration base + k
// (events arrive for consecutive K-iterations), and 64 of them go out in one
// store.  A store sits in the same vector-memory counter as the loads the
// wave waits for before it writes a slot, so one store per K-iteration would
// hold every slot back behind its write acknowledgement.
struct StampBatch {
  uint32_t vals = 0;
  uint32_t base = 0, n = 0;
};
// Adds the event of K-iteration iq; true when the batch is full.
__device__ __forceinline__ bool stamp_put(StampBatch& b, uint32_t iq, uint32_t value, int lane) {
  if (b.n == 0) b.base = iq;
  b.vals = ((uint32_t)lane == b.n) ? value : b.vals;
  return ++b.n == 64;
}
__device__ __forceinline__ void stamp_store(const StampBatch& b, __amdgpu_buffer_rsrc_t rec, int ev,
                                            uint32_t limit, int lane) {
  const uint32_t iq = b.base + (uint32_t)lane;
  if ((uint32_t)lane < b.n && iq < limit)
    __builtin_amdgcn_raw_buffer_store_b32(b.vals, rec, (int)((iq * kTraceEvents + (uint32_t)ev) * 4u), 0, 0);
}

// Events 0-3 of a producer wave (issue of its A / B loads of K-iteration q,
// their landing in the slot); A and B share one clock reading each.  With
// DIRECT (the eight-consumer arrangement, whose consumer does not copy stamps
// out of the LDS header) they go straight into the workgroup's trace record,
// batched; otherwise into the LDS header for consumer wave 0 to copy.
template <bool DIRECT>
struct ProducerStamps {
  // Bit 0: this wave stamps the A events, bit 1: the B events.  Kept as a
  // scalar integer, not as bools (those would be materialised as lane masks
  // through vector instructions).
  uint32_t who;
  int lane;
  uint32_t limit;
  __amdgpu_buffer_rsrc_t rec;
  StampBatch iss, land;
  __device__ ProducerStamps(const KernelArgs& args, bool stamps_a, bool stamps_b, int lane_)
      : who(__builtin_amdgcn_readfirstlane((stamps_a ? 1u : 0u) | (stamps_b ? 2u : 0u))), lane(lane_),
        limit(DIRECT ? (uint32_t)args.trace_iters : 0u),
        rec(panel_rsrc(DIRECT ? args.trace + (size_t)blockIdx.x * args.trace_iters * kTraceEvents : nullptr)) {}
  __device__ void flush(StampBatch& b, int ev_a, int ev_b) {
    if (who & 1u) stamp_store(b, rec, ev_a, limit, lane);
    if (who & 2u) stamp_store(b, rec, ev_b, limit, lane);
    b.n = 0;
  }
  __device__ void put(StampBatch& b, int ev_a, int ev_b, uint32_t q, uint32_t t, WSG_LDS uint32_t* hdr_a,
                      WSG_LDS uint32_t* hdr_b) {
    if constexpr (DIRECT) {
      if (who != 0u && stamp_put(b, q, t, lane)) flush(b, ev_a, ev_b);
    } else {
      if (who & 1u) lds_stamp(hdr_a, t);
      if (who & 2u) lds_stamp(hdr_b, t);
    }
  }
  __device__ void issued(uint32_t q, uint32_t t, WSG_LDS uint32_t* hdr_a, WSG_LDS uint32_t* hdr_b) {
    put(iss, 0, 1, q, t, hdr_a, hdr_b);
  }
  __device__ void landed(uint32_t q, uint32_t t, WSG_LDS uint32_t* hdr_a, WSG_LDS uint32_t* hdr_b) {
    put(land, 2, 3, q, t, hdr_a, hdr_b);
  }
  __device__ void finish() {
    if constexpr (DIRECT) {
      flush(iss, 0, 1);
      flush(land, 2, 3);
    }
  }
};

// A traced kernel runs its producer loop's traced instance only in the
// workgroups that record events; the others run the plain instance.
__device__ __forceinline__ bool traced_workgroup(const KernelArgs& args) {
  return args.trace != nullptr && (int)blockIdx.x < args.trace_wgs;
}

// A wave's place in the ring as LDS byte addresses: the slot it reads, the
// full counter (and target) of the K-iteration it looks at next and the empty
// counter it signals next, each wrapping at the end of its range.
struct RingCursor {
  uint32_t slot, full, target, empty;
  uint32_t ring, ring_end, full0, full_end, empty0, empty_end, abort_flag;
};

#include "ws_stream_loop.inc"

// ---------------------------------------------------------------------------
// Producer (DMA warp).  Waits for a free slot, streams its share of the A
// and/or B tile of one K-iteration into that slot, and signals the slot full
// once the data has landed.  Up to `lag` + 1 K-iterations are in flight per
// wave: iteration q is signalled once iteration q + lag has been issued.
// Before blocking on a slot that is still in use, every pending iteration is
// published (oldest first), so a consumer never waits on data that landed.
//
// GROUPS: the waves that load a tile are split into that many groups; group g
// takes the K-iterations q with q % GROUPS == g, and each of its waves adds
// GROUPS to full[], so a use of a slot still counts NP signals.  What bounds a
// single group is its own chain (wait for the slot, issue, wait for the data,
// signal): with P = 3 slots it kept one K-iteration in flight while it waited
// for the landing of the one before.  Two groups run that chain side by side:
// the load-only kernel of 128x256x32 (2:1, three slots, 4096x8192x2048) went
// from 134 to 91 us and the GEMM from 168 to 151 us, 128x64x64 (2:1, four
// slots, 16384x256x8192) from 145 to 112 us, 128x128x32 (three slots, 4096^3)
// from 165 to 151 us.
// ---------------------------------------------------------------------------

// Block until at most n of this wave's most recent K-iterations (LOADS DMA
// instructions each) are still in flight.
template <int LOADS>
__device__ __forceinline__ void wait_landed(uint32_t n) {
  switch (n) {
    case 0: wait_vmcnt<0>(); break;
    case 1: wait_vmcnt<(LOADS * 1 <= 63 ? LOADS * 1 : 0)>(); break;
    case 2: wait_vmcnt<(LOADS * 2 <= 63 ? LOADS * 2 : 0)>(); break;
    case 3: wait_vmcnt<(LOADS * 3 <= 63 ? LOADS * 3 : 0)>(); break;
    case 4: wait_vmcnt<(LOADS * 4 <= 63 ? LOADS * 4 : 0)>(); break;
    case 5: wait_vmcnt<(LOADS * 5 <= 63 ? LOADS * 5 : 0)>(); break;
    default: wait_vmcnt<(LOADS * 6 <= 63 ? LOADS * 6 : 0)>(); break;
  }
}

template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, bool TRACE, bool DO_A, bool DO_B,
          int GROUPS>
__device__ __forceinline__ void producer_loop(const KernelArgs& args, WSG_LDS char* smem,
                                              int a_rank, int b_rank, int lane) {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  // waves sharing the A (B) tile of one K-iteration
  constexpr int A_GROUP = ((SPLIT == 1) ? G::NP : G::NP / 2) / GROUPS;
  constexpr int B_GROUP = A_GROUP;
  constexpr int A_PER = DO_A ? G::A_INSTR / A_GROUP : 0;     // DMA instructions per wave
  constexpr int B_PER = DO_B ? G::B_INSTR / B_GROUP : 0;
  constexpr int LOADS = A_PER + B_PER;
  constexpr int MAX_LAG = (63 / LOADS) < 6 ? (63 / LOADS) : 6;
  static_assert(G::A_INSTR % A_GROUP == 0 && G::B_INSTR % B_GROUP == 0, "even DMA split");
  static_assert(LOADS > 0 && MAX_LAG >= 1, "vmcnt range");

  WSG_LDS uint32_t* full = (WSG_LDS uint32_t*)smem;
  WSG_LDS uint32_t* empty = full + kMaxStages;
  WSG_LDS uint32_t* abort_flag = full + 2 * kMaxStages;
  const int K = args.K, N = args.N;
  const uint32_t grp = (uint32_t)(DO_A ? a_rank : b_rank) / (uint32_t)A_GROUP;  // this wave's group
  a_rank %= A_GROUP;
  b_rank %= B_GROUP;

  // Byte offset, inside the tile, of the 16-byte chunk this lane fetches for
  // each of its DMA instructions (the LDS side is fixed: lane l writes bytes
  // 16 l .. 16 l + 15 of the instruction's KiB).
  uint32_t a_goff[A_PER > 0 ? A_PER : 1];
  uint32_t b_goff[B_PER > 0 ? B_PER : 1];
#pragma unroll
  for (int n = 0; n < A_PER; ++n) {
    const int q = (a_rank + n * A_GROUP) * 64 + lane;  // chunk index in the LDS tile
    const int r = q / G::CA, p = q % G::CA;
    a_goff[n] = (uint32_t)(r * K + 8 * (p ^ swz_a<TK>(r))) * 2u;
  }
#pragma unroll
  for (int n = 0; n < B_PER; ++n) {
    const int q = (b_rank + n * B_GROUP) * 64 + lane;
    b_goff[n] = (uint32_t)(b_chunk_row<TN>(q) * N + b_chunk_col<TN>(q)) * 2u;
  }

  // TRACE: this instance runs only in workgroups that record events.
  constexpr bool tracing = TRACE;
  static_assert(!TRACE || GROUPS == 1, "the traced producers take every K-iteration");
  ProducerStamps<TRACE && NC == 8> stamps(args, DO_A && a_rank == 0, DO_B && b_rank == 0, lane);
  const int Gd = gridDim.x;
  const uint32_t P = (uint32_t)args.stages;
  // signal() of K-iteration q_sig, whose data has landed (landing time stamped
  // first when tracing).
  uint32_t q_sig = grp, s_slot = grp;  // next K-iteration to signal and its slot
  auto publish = [&]() {
    if constexpr (tracing) stamps.landed(q_sig, cycles32(), &full[kStampLandA + s_slot], &full[kStampLandB + s_slot]);
    lds_signal<0, GROUPS>(&full[s_slot]);
    q_sig += GROUPS;
    s_slot += GROUPS;
    if (s_slot >= P) s_slot -= P;
  };
  const uint32_t S = (uint32_t)args.iters;
  // K-iterations of this wave issued ahead of the one it signals
  uint32_t lag = GROUPS > 1 ? P / GROUPS - 1 : (P > 3 ? P - 2 : 1);
  if (lag > (uint32_t)MAX_LAG) lag = MAX_LAG;
  const int g0 = first_slot(args);
  const int my_tiles = g0 < args.num_tiles ? (args.num_tiles - g0 + Gd - 1) / Gd : 0;
  const uint32_t total = (uint32_t)my_tiles * S;
  // next K-iteration to issue, its slot and the empty[] value that use needs
  // (0 for a slot's first use)
  uint32_t q = grp, slot = grp, need = 0;
  uint32_t kk = grp;
  for (int v = g0; q < total; v += Gd) {
    if (GROUPS > 1 && kk >= S) {  // a tile without K-iterations of this group
      kk -= S;
      continue;
    }
    int ti, tj;
    tile_at(args, v, &ti, &tj);
    const uint16_t* a_tile = args.A + (int64_t)ti * TM * K;
    const uint16_t* b_tile = args.B + (int64_t)tj * TN;
    for (; kk < S; kk += GROUPS, q += GROUPS) {
      if (need > 0) {
        // wait(): the slot is free once every consumer wave released its previous use.
        if ((int32_t)(lds_read_now(&empty[slot]) - need) < 0) {
          while (q_sig < q) {  // publish pending iterations first, oldest first
            wait_landed<LOADS>((q - q_sig) / GROUPS - 1);
            publish();
          }
          if (!wait_counter(&empty[slot], need, abort_flag, args.spin_limit, args.err)) {
            wait_vmcnt<0>();  // no DMA into LDS may outlive the wave
            return;
          }
        }
      }
      debug_delay(args.producer_delay);
      compiler_fence();
      if constexpr (tracing) stamps.issued(q, cycles32(), &full[kStampIssueA + slot], &full[kStampIssueB + slot]);
      WSG_LDS char* a_dst = smem + kHeaderBytes + slot * G::STAGE;
      WSG_LDS char* b_dst = a_dst + G::A_BYTES;
      if constexpr (DO_A) {
        const __amdgpu_buffer_rsrc_t src = panel_rsrc(a_tile + kk * TK);
#pragma unroll
        for (int n = 0; n < A_PER; ++n)
          panel_load16_lds(src, (WSG_LDS void*)(a_dst + (a_rank + n * A_GROUP) * 1024), a_goff[n]);
      }
      if constexpr (DO_B) {
        const __amdgpu_buffer_rsrc_t src = panel_rsrc(b_tile + (int64_t)kk * TK * N);
#pragma unroll
        for (int n = 0; n < B_PER; ++n)
          panel_load16_lds(src, (WSG_LDS void*)(b_dst + (b_rank + n * B_GROUP) * 1024), b_goff[n]);
      }
      // signal(): iteration q - lag has landed once at most `lag` newer ones are in flight.
      if ((q - q_sig) / GROUPS + 1 > lag) {
        wait_landed<LOADS>(lag);
        publish();
      }
      slot += GROUPS;
      if (slot >= P) {  // P >= 2 = the most groups: one lap at most
        slot -= P;
        need += NC;
      }
    }
    kk -= S;
  }
  while (q_sig < q) {
    wait_landed<LOADS>((q - q_sig) / GROUPS - 1);
    publish();
  }
  stamps.finish();
}

// ---------------------------------------------------------------------------
// Register-staged producer (DMA warp).  The wave loads its share of the tiles
// of K-iteration q + L into VGPRs (buffer_load_dwordx4) while K-iteration q
// waits in registers for its slot; once the slot is free it writes q with
// ds_write_b128 and signals.  Bytes in flight per wave are L iterations'
// worth, independent of the LDS ring depth: producer waves get the kernel's
// full VGPR allocation (sized for the consumers) and would otherwise leave
// it idle.  The LDS layout is the one the LDS-DMA producer writes.
//
// GROUPS as in producer_loop.  A wave's writes (1 KiB in 13 clocks for the
// whole CU), its signal and its loads (1 KiB in 16 clocks of the CU's address
// unit) follow each other, and waves that wait for the same slot do them in
// step, so the LDS idles while they load and the address unit while they
// write.  Two groups are in different phases: 128x128x64 (four slots, 4 + 4
// waves, 2048x2048x32768) took 1161 clocks per K-iteration with one group and
// 968 with two (292 -> 269 us), 128x128x32 at 4096^3 159 -> 156 us, 128x256x32
// (four slots) 134.6 -> 129.6 us, 128x64x64 2:1 (16384x256x8192)
// 111 -> 103 us; its general twin, whose loads test their chunks, 122 -> 109.
// ---------------------------------------------------------------------------
template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, bool TRACE, bool DO_A, bool DO_B,
          bool GENERAL, int GROUPS>
__device__ __forceinline__ void producer_loop_reg(const KernelArgs& args, WSG_LDS char* smem,
                                                  int a_rank, int b_rank, int lane) {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  // Waves sharing the A (B) tile of one K-iteration: of the waves that load
  // A (B), one of GROUPS groups, which take the K-iterations in turn.
  constexpr int A_GROUP = ((SPLIT == 1) ? G::NP : G::NP / 2) / GROUPS;
  constexpr int B_GROUP = A_GROUP;
  constexpr int A_PER = DO_A ? G::A_INSTR / A_GROUP : 0;
  constexpr int B_PER = DO_B ? G::B_INSTR / B_GROUP : 0;
  constexpr int LOADS = A_PER + B_PER;
  // VGPRs for staged tiles: what the consumers' allocation leaves (256 a wave
  // with eight waves, 168 with twelve; the 128 x 128 x 32 kernel held to 128
  // registers stages its cap of six K-iterations in 96)
  constexpr int REGS = StreamLoop<TM, TN, TK, NC, NPW, BF16>::kVgprs;
  constexpr int STAGE_VGPRS = REGS == 80    ? (GENERAL ? 32 : 48)
                              : REGS == 128 ? (GENERAL && NC == 4 ? 64 : 96)
                              : G::NW <= 8  ? 152
                                            : (NC == 8 ? 128 : 96);
  constexpr int L0 = STAGE_VGPRS / (4 * LOADS);
  constexpr int L1 = (63 / LOADS) < L0 ? (63 / LOADS) : L0;
  constexpr int LCAP = 6 / GROUPS;
  constexpr int L = L1 < 1 ? 1 : (L1 > LCAP ? LCAP : L1);  // of its K-iterations, staged in VGPRs
  // With one K-iteration staged, each register is loaded again right behind
  // the write that empties it, so that the loads in flight never run out; with
  // more, the loads follow the signal, which they would only delay.
  constexpr bool CHUNKWISE = L == 1;
  static_assert(G::A_INSTR % A_GROUP == 0 && G::B_INSTR % B_GROUP == 0, "even split");

  WSG_LDS uint32_t* full = (WSG_LDS uint32_t*)smem;
  WSG_LDS uint32_t* empty = full + kMaxStages;
  WSG_LDS uint32_t* abort_flag = full + 2 * kMaxStages;
  const int K = args.K, N = args.N;
  const uint32_t grp = (uint32_t)(DO_A ? a_rank : b_rank) / (uint32_t)A_GROUP;  // this wave's group
  a_rank %= A_GROUP;
  b_rank %= B_GROUP;

  uint32_t goff[LOADS];  // byte offset of this lane's 16-byte chunk in the A / B tile
#pragma unroll
  for (int n = 0; n < A_PER; ++n) {
    const int q = (a_rank + n * A_GROUP) * 64 + lane;
    const int r = q / G::CA, p = q % G::CA;
    goff[n] = (uint32_t)(r * K + 8 * (p ^ swz_a<TK>(r))) * 2u;
  }
#pragma unroll
  for (int n = 0; n < B_PER; ++n) {
    const int q = (b_rank + n * B_GROUP) * 64 + lane;
    goff[A_PER + n] = (uint32_t)(b_chunk_row<TN>(q) * N + b_chunk_col<TN>(q)) * 2u;
  }
  // The general variant needs registers for its edge tests: where a wave's
  // successive A (B) instructions lie a whole number of swizzle periods
  // (block rows) apart, it keeps only the first instruction's offset and
  // adds the (wave-uniform) step between instructions.
  constexpr int A_STEP = (64 / G::CA) * A_GROUP;  // A rows from one of a wave's instructions to the next
  constexpr bool kStrided = GENERAL && swz_a_step_invariant<TK>(A_STEP) && (8 * B_GROUP) % G::NQ == 0;
  constexpr int B_STEP = (8 * B_GROUP) / G::NQ;   // B block rows (4 K rows each) between instructions
  const uint32_t a_step = (uint32_t)A_STEP * (uint32_t)K * 2u;      // bytes, wave-uniform
  const uint32_t b_step = (uint32_t)(B_STEP * 4) * (uint32_t)N * 2u;
  // kStrided: the lane's K chunk of A and column chunk of B (the same for
  // all of its instructions)
  int a_kc0 = 0, b_nc0 = 0;
  if constexpr (kStrided) {
    const int qa = a_rank * 64 + lane;
    a_kc0 = 8 * ((qa % G::CA) ^ swz_a<TK>(qa / G::CA));
    const int qb = b_rank * 64 + lane;
    b_nc0 = b_chunk_col<TN>(qb);
  }
  const uint32_t lane16 = (uint32_t)lane * 16u;

  // TRACE: this instance runs only in workgroups that record events.
  constexpr bool tracing = TRACE;
  static_assert(!TRACE || GROUPS == 1, "the traced producers take every K-iteration");
  ProducerStamps<TRACE && NC == 8> stamps(args, DO_A && a_rank == 0, DO_B && b_rank == 0, lane);
  const int Gd = gridDim.x;
  const int g0 = first_slot(args);
  const int my_tiles = (args.num_tiles - g0 + Gd - 1) / Gd;
  const uint32_t S = (uint32_t)args.iters;
  const uint32_t total = (uint32_t)my_tiles * S;
  const uint32_t P = (uint32_t)args.stages;

  // Issue cursor: the next K-iteration whose loads go out (its A and B panel
  // addresses move with it).
  int v_i = g0, ti_i = 0, tj_i = 0;
  uint32_t kk_i = 0, q_iss = grp;
  const char* a_src = nullptr;
  const char* b_src = nullptr;
  const int64_t a_adv = (int64_t)TK * 2 * GROUPS, b_adv = (int64_t)TK * 2 * GROUPS * N;
  auto point = [&]() {
    tile_at(args, v_i, &ti_i, &tj_i);
    a_src = (const char*)(args.A + (int64_t)ti_i * TM * K + kk_i * TK);
    b_src = (const char*)(args.B + (int64_t)kk_i * TK * N + (int64_t)tj_i * TN);
  };
  if (GROUPS > 1 && q_iss < total) {
    kk_i = q_iss;
    while (kk_i >= S) {
      kk_i -= S;
      v_i += Gd;
    }
  }
  point();

  i32x4_t stage[L][LOADS];
  // Traced: one clock reading per K-iteration, taken once K-iteration q is in
  // its slot, stands for the landing of q and the issue of q + L (the loads
  // go out right after q's signal).
  uint32_t t_issue[L], t_now = 0;
  __amdgpu_buffer_rsrc_t ra, rb;
  uint32_t ab = 0, bb = 0;
  int k_left = 0, cols_left = 0;
  // Descriptors of the K-iteration under the issue cursor.
  auto aim = [&]() {
    if constexpr (GENERAL) {
      // rows, columns and K left from this K-iteration's tile origin
      // (wave-uniform; the origin is always inside A and B); the record
      // counts end at the last row of A (the last K row of B); offsets stay
      // 16-byte multiples, so no chunk straddles the end
      const int rows_left = args.M - ti_i * TM;
      cols_left = N - tj_i * TN;
      k_left = K - (int)kk_i * TK;
      ra = panel_rsrc_to_end(a_src, ((int64_t)rows_left * K - (int64_t)kk_i * TK) * 2);
      rb = panel_rsrc_to_end(b_src, ((int64_t)k_left * N - (int64_t)tj_i * TN) * 2);
      if constexpr (kStrided) {
        ab = goff[0];
        bb = goff[A_PER];
        asm volatile("" : "+v"(ab), "+v"(bb));
        ab = a_kc0 < k_left ? ab : kOutsidePanel;
        bb = b_nc0 < cols_left ? bb : kOutsidePanel;
      }
    } else {
      ra = panel_rsrc(a_src);
      rb = panel_rsrc(b_src);
    }
  };
  auto load = [&](int u, int n) {
    if constexpr (GENERAL) {
      if constexpr (kStrided) {
        stage[u][n] = n < A_PER ? panel_load16(ra, ab + (uint32_t)n * a_step)
                                : panel_load16(rb, bb + (uint32_t)(n - A_PER) * b_step);
      } else if (n < A_PER) {
        const int q = (a_rank + n * A_GROUP) * 64 + lane;
        const int kc = 8 * ((q % G::CA) ^ swz_a<TK>(q / G::CA));
        stage[u][n] = panel_load16(ra, kc < k_left ? goff[n] : kOutsidePanel);
      } else {
        const int q = (b_rank + (n - A_PER) * B_GROUP) * 64 + lane;
        const int nc8 = b_chunk_col<TN>(q);
        stage[u][n] = panel_load16(rb, nc8 < cols_left ? goff[n] : kOutsidePanel);
      }
    } else {
      stage[u][n] = panel_load16(n < A_PER ? ra : rb, goff[n]);
    }
  };
  // Loads go out unconditionally (past the last K-iteration they re-read the
  // last valid tile and are never written to LDS), so every path through the
  // loop has the same number of loads in flight and the compiler's vmcnt
  // waits before each ds_write allow exactly the newer ones.
  auto advance = [&]() {
    if (q_iss + GROUPS < total) {
      q_iss += GROUPS;
      kk_i += GROUPS;
      a_src += a_adv;
      b_src += b_adv;
      if (kk_i >= S) {
        do {
          kk_i -= S;
          v_i += Gd;
        } while (GROUPS > 1 && kk_i >= S);
        point();
      }
    }
  };

  if constexpr (tracing) t_now = cycles32();
#pragma unroll
  for (int u = 0; u < L; ++u) {
    if constexpr (tracing) t_issue[u] = t_now;
    aim();
#pragma unroll
    for (int n = 0; n < LOADS; ++n) load(u, n);
    advance();
  }

  // Slot of the next K-iteration to write, the empty[] value its use needs
  // (0 for a slot's first use), and the value of that counter read with the
  // previous signal: when the consumers are ahead it already satisfies the
  // wait, and the wave skips an LDS round trip.
  uint32_t w_slot = grp, w_need = 0, seen = 0;
  for (uint32_t q0 = grp; q0 < total; q0 += L * GROUPS) {
#pragma unroll
    for (int u = 0; u < L; ++u) {
      const uint32_t q = q0 + u * GROUPS;
      aim();
      if (q < total) {
      const uint32_t slot = w_slot;
      // No early exit when the wait fails (workgroup aborted, or this wait
      // timed out and raised the abort): the wave runs its remaining
      // K-iterations without waiting (every later wait sees the abort flag
      // at once) and leaves at the loop's end.  A return from inside the
      // loop would join the loop header in the compiler's control flow, and
      // its wait-count analysis would then drain every load in flight at the
      // first register stage of each pass through the stages.
      if ((int32_t)(seen - w_need) < 0)
        (void)wait_counter(&empty[slot], w_need, abort_flag, args.spin_limit, args.err);
      debug_delay(args.producer_delay);
      compiler_fence();
      WSG_LDS char* base = smem + kHeaderBytes + slot * G::STAGE + lane16;
#pragma unroll
      for (int n = 0; n < LOADS; ++n) {
        if (n < A_PER) *(WSG_LDS i32x4_t*)(base + (a_rank + n * A_GROUP) * 1024) = stage[u][n];
        else *(WSG_LDS i32x4_t*)(base + G::A_BYTES + (b_rank + (n - A_PER) * B_GROUP) * 1024) = stage[u][n];
        if constexpr (CHUNKWISE) {
          __builtin_amdgcn_sched_barrier(0);
          load(u, n);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if constexpr (tracing) {
        t_now = cycles32();
        stamps.issued(q, t_issue[u], &full[kStampIssueA + slot], &full[kStampIssueB + slot]);
        stamps.landed(q, t_now, &full[kStampLandA + slot], &full[kStampLandB + slot]);
        t_issue[u] = t_now;
      }
      w_slot += GROUPS;
      if (w_slot >= P) {
        w_slot -= P;
        w_need += NC;
      }
      // waits for the LDS writes, signals, and reads the next slot's empty[]
      seen = lds_signal_peek<GROUPS>(&full[slot], &empty[w_slot]);
      } else if constexpr (CHUNKWISE) {
#pragma unroll
        for (int n = 0; n < LOADS; ++n) load(u, n);
      }
      if constexpr (!CHUNKWISE) {
#pragma unroll
        for (int n = 0; n < LOADS; ++n) load(u, n);  // refill this register stage
      }
      advance();
    }
  }
  stamps.finish();
  wait_vmcnt<0>();
}

// Producer that loads nothing: waits for each slot to be free and signals it
// full (the calibration MATH kernel, and the idle half of a two-DMA split in
// the load calibration kernels).
template <int NC>
__device__ __forceinline__ void producer_signal_only(const KernelArgs& args, WSG_LDS char* smem) {
  WSG_LDS uint32_t* full = (WSG_LDS uint32_t*)smem;
  WSG_LDS uint32_t* empty = full + kMaxStages;
  WSG_LDS uint32_t* abort_flag = full + 2 * kMaxStages;
  const int Gd = gridDim.x;
  const int g0 = first_slot(args);
  const int my_tiles = g0 < args.num_tiles ? (args.num_tiles - g0 + Gd - 1) / Gd : 0;
  const uint32_t total = (uint32_t)my_tiles * (uint32_t)args.iters;
  const uint32_t P = (uint32_t)args.stages;
  uint32_t slot = 0, need = 0;  // empty[] value this use of the slot needs
  for (uint32_t q = 0; q < total; ++q) {
    if (need > 0 && !wait_counter(&empty[slot], need, abort_flag, args.spin_limit, args.err)) return;
    lds_signal(&full[slot]);
    if (++slot == P) {
      slot = 0;
      need += NC;
    }
  }
}

// One producer wave's loop on the configured load path; STAMP: it records
// trace events.
template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, bool STAMP, bool DO_A, bool DO_B,
          bool GENERAL>
__device__ __forceinline__ void producer_run(const KernelArgs& args, WSG_LDS char* smem, int a_rank, int b_rank,
                                             int lane) {
  // Producer groups (see producer_loop_reg).  One where a wave group cannot be
  // halved (one consumer wave), where a stamp stands for every K-iteration
  // (tracing), and on the register path of the eight-consumer arrangement:
  // there a group of two waves could stage only one K-iteration, and the two
  // ring slots leave one free at a time (256x256x64 at 8192^3: 838 us with one
  // group, 852 with two; its LDS-DMA path gains 0-2 %).
  constexpr int GR = (STAMP || NC != 4) ? 1 : 2;
  constexpr int GD = (STAMP || NC == 1) ? 1 : 2;
  if constexpr (GENERAL) {  // partial tiles possible: always register-staged
    producer_loop_reg<TM, TN, TK, NC, NPW, SPLIT, BF16, STAMP, DO_A, DO_B, true, GR>(args, smem, a_rank, b_rank,
                                                                                lane);
  } else if (args.load_path == 1) {  // wave-uniform: 0 = register-staged, 1 = LDS-DMA
    producer_loop<TM, TN, TK, NC, NPW, SPLIT, BF16, STAMP, DO_A, DO_B, GD>(args, smem, a_rank, b_rank, lane);
  } else {
    producer_loop_reg<TM, TN, TK, NC, NPW, SPLIT, BF16, STAMP, DO_A, DO_B, false, GR>(args, smem, a_rank, b_rank,
                                                                                 lane);
  }
}

template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, bool TRACE, bool DO_A, bool DO_B,
          bool GENERAL>
__device__ __forceinline__ void producer_share(const KernelArgs& args, WSG_LDS char* smem, int a_rank,
                                               int b_rank, int lane) {
  if constexpr (!DO_A && !DO_B) {
    producer_signal_only<NC>(args, smem);
  } else if (TRACE && traced_workgroup(args)) {
    producer_run<TM, TN, TK, NC, NPW, SPLIT, BF16, TRACE, DO_A, DO_B, GENERAL>(args, smem, a_rank, b_rank, lane);
  } else {
    producer_run<TM, TN, TK, NC, NPW, SPLIT, BF16, false, DO_A, DO_B, GENERAL>(args, smem, a_rank, b_rank, lane);
  }
}

template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, bool TRACE, int MODE, bool GENERAL>
__device__ __forceinline__ void producer(const KernelArgs& args, WSG_LDS char* smem, int pw,
                                         int lane) {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  constexpr bool LA = MODE == kModeGemm || MODE == kModeLoadA || MODE == kModeLoadAB;  // A loaded
  constexpr bool LB = MODE == kModeGemm || MODE == kModeLoadB || MODE == kModeLoadAB;  // B loaded
  if constexpr (MODE == kModeEpilogue) {
    return;
  } else if constexpr (SPLIT == 1) {
    producer_share<TM, TN, TK, NC, NPW, SPLIT, BF16, TRACE, LA, LB, GENERAL>(args, smem, pw, pw, lane);
  } else {
    if (pw < G::NP / 2)
      producer_share<TM, TN, TK, NC, NPW, SPLIT, BF16, TRACE, LA, false, GENERAL>(args, smem, pw, 0, lane);
    else
      producer_share<TM, TN, TK, NC, NPW, SPLIT, BF16, TRACE, false, LB, GENERAL>(args, smem, 0,
                                                                           pw - G::NP / 2, lane);
  }
}

// ---------------------------------------------------------------------------
// Consumer (MATH wave).  One K-iteration is KS MFMA k-steps of 16.  Inside a
// k-step the MFMAs run M-major: every column block nb of row block mb, then
// the next row block.  Operands for k-step s + 1 are read while k-step s
// multiplies:
//   * the B fragments of k-step s + 1 go to the other of two buffers at the
//     start of k-step s;
//   * A fragment mb is single-buffered and refilled right after its row of
//     MFMAs, (BM - 1) * BN MFMAs before its next use.
// The last k-step of a K-iteration reads k-step 0 of the next slot: the slot's
// full[] counter was peeked one k-step earlier, so the wait costs nothing
// when the producers are ahead.  The slot is released (empty[] signal) right
// after that k-step's reads are issued, once the older reads have completed.
// ---------------------------------------------------------------------------
template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16>
struct ConsumerOps {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  static constexpr int kReads = G::BM + 2 * G::BN;  // LDS reads per k-step
  // A operand of row block mb: 16 bytes per lane at a_src + a_off + mb * 32 rows.
  static __device__ __forceinline__ void load_a(i16x8_t& fa, WSG_LDS char* a_src, uint32_t a_off,
                                                int mb) {
    fa = *(WSG_LDS i16x8_t*)(a_src + a_off + mb * 32 * TK * 2);
  }
  // B operand of column block nb at k-step s: two transposed 8-byte reads.
  static __device__ __forceinline__ void load_b(i16x8_t& fb, WSG_LDS char* b_src, uint32_t b_off,
                                                int s, int nb) {
    WSG_LDS char* p = b_src + b_off + ((4 * s) * G::NQ + 2 * nb) * 128;
    const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((WSG_LDS i16x4_t*)p);
    const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((WSG_LDS i16x4_t*)(p + G::NQ * 128));
    fb = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, bool TRACE, int MODE, bool GENERAL>
__device__ __forceinline__ void consumer(const KernelArgs& args, WSG_LDS char* smem, int cw,
                                         int lane) {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  using Ops = ConsumerOps<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  static_assert(G::KS >= 2, "a K-iteration holds at least two k-steps");
  WSG_LDS uint32_t* full = (WSG_LDS uint32_t*)smem;
  WSG_LDS uint32_t* empty = full + kMaxStages;
  WSG_LDS uint32_t* abort_flag = full + 2 * kMaxStages;

  const int wm = cw / G::WGN, wn = cw % G::WGN;
  // A: lane reads row wm*WM + mb*32 + lane%32, chunk 2s + lane/32 (swizzled;
  // the swizzle repeats every 32 rows, so it depends only on the lane).
  uint32_t a_off[G::KS];
  {
    const int r = wm * G::WM + (lane & 31);
#pragma unroll
    for (int s = 0; s < G::KS; ++s)
      a_off[s] = (uint32_t)(r * TK * 2 + (((2 * s + (lane >> 5)) ^ swz_a<TK>(r)) << 4));
  }
  // B: 16-lane group g reads its half of block (kq = 4s + 2(g>>1) + h, nd = (wn*WN)/32 + nb).
  const uint32_t b_off = b_read_off<TN>(lane, wn * G::WN);

  const int Gd = gridDim.x;
  const int g0 = first_slot(args);
  if (g0 >= args.num_tiles) return;
  const int my_tiles = (args.num_tiles - g0 + Gd - 1) / Gd;
  const uint32_t S = (uint32_t)args.iters;
  const uint32_t total = (uint32_t)my_tiles * S;
  const uint32_t P = (uint32_t)args.stages;

  int v = g0;
  int ti, tj;
  tile_at(args, v, &ti, &tj);

  f32x16_t acc[G::BM][G::BN];
#pragma unroll
  for (int mb = 0; mb < G::BM; ++mb)
#pragma unroll
    for (int nb = 0; nb < G::BN; ++nb) acc[mb][nb] = f32x16_t{};
  i16x8_t fa[G::BM];
  i16x8_t fb[2][G::BN];

  // Event trace (consumer wave 0 of traced workgroups writes the records).
  const bool tracing = TRACE && args.trace != nullptr && cw == 0 && (int)blockIdx.x < args.trace_wgs;
  uint32_t* trec = tracing ? args.trace + (size_t)blockIdx.x * args.trace_iters * kTraceEvents : nullptr;
  auto record = [&](uint32_t iq, int ev, uint32_t value) {
    if (tracing && iq < (uint32_t)args.trace_iters && lane == 0) trec[iq * kTraceEvents + ev] = value;
  };
  // Slot `ps` of K-iteration iq is full: copy the producer stamps, stamp "ready".
  auto record_ready = [&](uint32_t iq, uint32_t ps) {
    if (tracing) {
      const uint32_t t = cycles32();
      record(iq, 0, lds_read_now(&full[kStampIssueA + ps]));
      record(iq, 1, lds_read_now(&full[kStampIssueB + ps]));
      record(iq, 2, lds_read_now(&full[kStampLandA + ps]));
      record(iq, 3, lds_read_now(&full[kStampLandB + ps]));
      record(iq, 4, t);
    }
  };

  // Prologue: wait for K-iteration 0 and read k-step 0.
  if (!wait_counter(&full[ring_slot(0, P)], ring_full_target(0, P, G::NP), abort_flag,
                    args.spin_limit, args.err))
    return;
  record_ready(0, 0);
#pragma unroll
  for (int mb = 0; mb < G::BM; ++mb) Ops::load_a(fa[mb], smem + kHeaderBytes, a_off[0], mb);
#pragma unroll
  for (int nb = 0; nb < G::BN; ++nb)
    Ops::load_b(fb[0][nb], smem + kHeaderBytes + G::A_BYTES, b_off, 0, nb);

  uint32_t q = 0, kk = 0;
  while (true) {
    const uint32_t slot = ring_slot(q, P);
    WSG_LDS char* a_src = smem + kHeaderBytes + slot * G::STAGE;
    WSG_LDS char* b_src = a_src + G::A_BYTES;
    const bool has_next = (q + 1) < total;
    // After the last K-iteration the next-slot reads re-read this slot (and
    // are never used), so every path issues the same LDS operations.
    const uint32_t nslot = has_next ? ring_slot(q + 1, P) : slot;
    const uint32_t ntarget = has_next ? ring_full_target(q + 1, P, G::NP) : 0u;
    WSG_LDS char* na_src = smem + kHeaderBytes + nslot * G::STAGE;
    WSG_LDS char* nb_src = na_src + G::A_BYTES;
    uint32_t peek = 0;
    debug_delay(args.consumer_delay);
    if (tracing) record(q, 5, cycles32());
#pragma unroll
    for (int s = 0; s < G::KS; ++s) {
      const int cur = s & 1, nxt = cur ^ 1;
      const bool last = (s == G::KS - 1);
      if (s == G::KS - 2) {
        peek = lds_peek(&full[nslot]);  // before this k-step's reads
        __builtin_amdgcn_sched_barrier(0);
      }
      if (last) {
        const uint32_t st = wait_until(peek, &full[nslot], abort_flag, ntarget, args.spin_limit);
        if (st != 0) {
          if (st == 2) report_timeout(abort_flag, args.err);
          return;
        }
        compiler_fence();
        if (tracing && has_next) record_ready(q + 1, nslot);
      }
      WSG_LDS char* ra = last ? na_src : a_src;
      WSG_LDS char* rb = last ? nb_src : b_src;
      const int ts = last ? 0 : s + 1;
#pragma unroll
      for (int nb = 0; nb < G::BN; ++nb) Ops::load_b(fb[nxt][nb], rb, b_off, ts, nb);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mb = 0; mb < G::BM; ++mb) {
#pragma unroll
        for (int nb = 0; nb < G::BN; ++nb)
          acc[mb][nb] = mfma32x32x16<BF16>(fa[mb], fb[cur][nb], acc[mb][nb]);
        Ops::load_a(fa[mb], ra, a_off[ts], mb);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (last) {
        // Every read of this slot is older than the kReads just issued.
        lds_signal<Ops::kReads>(&empty[slot]);
        if (tracing) record(q, 6, cycles32());
      }
    }
    ++q;
    if (++kk == S) {
      // The calibration MATH kernel keeps its products (the store below is
      // never taken: M > 0) without writing C.
      if (MODE != kModeMath || args.M < 0)
        store_tile<TM, TN, G::WM, G::WN, G::BM, G::BN, GENERAL, (G::NW > 8 ? 1 : (G::BN > 2 ? 32 / G::BN : 16))>(args, acc, ti, tj, wm, wn, lane);
      if (tracing) record(q - 1, 7, cycles32());
      if (!has_next) break;
      kk = 0;
      v += Gd;
      tile_at(args, v, &ti, &tj);
#pragma unroll
      for (int mb = 0; mb < G::BM; ++mb)
#pragma unroll
        for (int nb = 0; nb < G::BN; ++nb) acc[mb][nb] = f32x16_t{};
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

#include "ws_deep_loop.inc"

// ---------------------------------------------------------------------------
// Streaming consumer: the generated StreamLoop block (ws_stream_loop.inc,
// gen_stream_loop.py) runs the K loop of a tile.  What bounds a consumer wave
// that is alone on its SIMD is issue: everything between two MFMAs beyond
// seven instructions leaves the matrix core idle.  Math-only kernels, clocks
// per K-iteration against the MFMAs' own (one wave per SIMD unless said), for
// the loops this one replaced and now: 128x128x64 859 -> 644 (512), 256x128x64
// 1357 -> 1175 (1024), 128x256x32 2:1 (single-buffered) 1756 -> 789 (512),
// 128x128x32 with two workgroups per CU 866 -> 722 (512), 64x64x64 with two
// 1277 -> 747 (256).  The GEMM of 128x256x32 2:1 on the LDS-DMA path
// (4096x8192x2048) went from 210 to 164 us, of 64x64x64 at 4096^3 from 317 to
// 277 us.
// ---------------------------------------------------------------------------
template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, int MODE, bool GENERAL>
__device__ __forceinline__ void consumer_stream(const KernelArgs& args, WSG_LDS char* smem, int cw,
                                                int lane) {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  using Loop = StreamLoop<TM, TN, TK, NC, NPW, BF16>;
  constexpr int BM = G::BM, BN = G::BN;
  // old C rows the general epilogue loads together: as registers allow
  constexpr int EG = G::NW > 8 ? 1 : Loop::kVgprs <= 128 ? 4 : (BN > 2 ? 32 / BN : 16);
  WSG_LDS uint32_t* full = (WSG_LDS uint32_t*)smem;
  WSG_LDS uint32_t* empty = full + kMaxStages;
  WSG_LDS uint32_t* abort_flag = full + 2 * kMaxStages;

  const int wm = cw / G::WGN, wn = cw % G::WGN;
  uint32_t a_off[G::KS];
  const int r = wm * G::WM + (lane & 31);
#pragma unroll
  for (int s = 0; s < G::KS; ++s)
    a_off[s] = (uint32_t)(r * TK * 2 + (((2 * s + (lane >> 5)) ^ swz_a<TK>(r)) << 4));
  const uint32_t b_off = G::A_BYTES + b_read_off<TN>(lane, wn * G::WN);

  const uint32_t S = (uint32_t)args.iters;
  // T_K = 32 in a ring of two slots takes the block with two fragment sets
  // (see gen_stream_loop.py).  Four sets -> two: 128x64x32 at 2048x2048x4096
  // 93.0 -> 67.0 us, 256x128x32 (2:1, eight waves) at 2048x4096x4096 117.7 ->
  // 80.5 us, 32x32x32 at 256x256x4096 57.9 -> 34.0 us; three slots keep four.
  const bool short_ring = Loop::kShort && args.stages < 3;  // wave-uniform
  if (Loop::kMinIters > 1 && S < (uint32_t)Loop::kMinIters && !short_ring) {
    consumer<TM, TN, TK, NC, NPW, SPLIT, BF16, false, MODE, GENERAL>(args, smem, cw, lane);
    return;
  }
  const int Gd = gridDim.x;
  const int g0 = first_slot(args);
  if (g0 >= args.num_tiles) return;
  const int my_tiles = (args.num_tiles - g0 + Gd - 1) / Gd;
  const uint32_t P = (uint32_t)args.stages;
  RingCursor rc;
  rc.slot = rc.ring = (uint32_t)(uintptr_t)(smem + kHeaderBytes);
  rc.ring_end = rc.ring + P * (uint32_t)G::STAGE;
  rc.full = rc.full0 = (uint32_t)(uintptr_t)full;
  rc.full_end = rc.full0 + 4 * P;
  rc.empty = rc.empty0 = (uint32_t)(uintptr_t)empty;
  rc.empty_end = rc.empty0 + 4 * P;
  rc.abort_flag = (uint32_t)(uintptr_t)abort_flag;
  rc.target = (uint32_t)G::NP;

  int v = g0, ti, tj;
  tile_at(args, v, &ti, &tj);
  f32x16_t acc[BM][BN];
  for (int t = 0; t < my_tiles; ++t) {
#pragma unroll
    for (int mb = 0; mb < BM; ++mb)
#pragma unroll
      for (int nb = 0; nb < BN; ++nb) acc[mb][nb] = f32x16_t{};
    if (!wait_counter((WSG_LDS uint32_t*)(uintptr_t)rc.full, rc.target, abort_flag, args.spin_limit, args.err))
      return;
    uint32_t st;
    if constexpr (Loop::kShort) {
      st = short_ring ? Loop::tile_short(acc, a_off, b_off, rc, S, args.spin_limit, args.consumer_delay)
                      : Loop::tile(acc, a_off, b_off, rc, S, args.spin_limit, args.consumer_delay);
      // the two blocks' scalar results meet here; the compiler does not see that they are uniform
      rc.slot = __builtin_amdgcn_readfirstlane(rc.slot);
      rc.full = __builtin_amdgcn_readfirstlane(rc.full);
      rc.target = __builtin_amdgcn_readfirstlane(rc.target);
      rc.empty = __builtin_amdgcn_readfirstlane(rc.empty);
      st = __builtin_amdgcn_readfirstlane(st);
    } else {
      st = Loop::tile(acc, a_off, b_off, rc, S, args.spin_limit, args.consumer_delay);
    }
    if (st != 0) {
      if (st == 2) report_timeout(abort_flag, args.err);
      return;
    }
    // The calibration MATH kernel keeps its products (the store below is
    // never taken: M > 0) without writing C.
    if (MODE != kModeMath || args.M < 0)
      store_tile<TM, TN, G::WM, G::WN, BM, BN, GENERAL, EG>(args, acc, ti, tj, wm, wn, lane);
    v += Gd;
    tile_at(args, v, &ti, &tj);
  }
}

// ---------------------------------------------------------------------------
// Consumer with two consumer waves per SIMD: the eight-consumer arrangement
// (2 x 4 grid of 128 x 64 wave tiles next to four producer waves) and the
// event-traced four-consumer 128 x 128 x 32 kernel held to 128 registers a wave
// (2 x 2 grid of 64 x 64 wave tiles, two workgroups per CU).  The K loop of a tile is
// the generated RollLoop block (ws_deep_loop.inc).  Its fragments are
// single-buffered and refilled right after their last MFMA of the k-step; the
// other consumer wave of the SIMD covers the read latency.
// ---------------------------------------------------------------------------
template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, bool TRACE, int MODE, bool GENERAL>
__device__ __forceinline__ void consumer_roll(const KernelArgs& args, WSG_LDS char* smem, int cw,
                                              int lane) {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  using Loop = RollLoop<TM, TN, TK, NC, NPW, BF16>;
  static_assert(Loop::kAvailable, "roll consumer configuration");
  constexpr int BM = G::BM, BN = G::BN;
  WSG_LDS uint32_t* full = (WSG_LDS uint32_t*)smem;
  WSG_LDS uint32_t* empty = full + kMaxStages;
  WSG_LDS uint32_t* abort_flag = full + 2 * kMaxStages;

  const int wm = cw / G::WGN, wn = cw % G::WGN;
  // A operand of k-step 0: row r, 16-byte chunk (lane / 32) ^ swz(r); the
  // block moves it to k-step s by XORing 32 s into the byte offset.
  const int r = wm * G::WM + (lane & 31);
  const uint32_t a_off0 = (uint32_t)(r * TK * 2 + (((lane >> 5) ^ swz_a<TK>(r)) << 4));
  const uint32_t b_off = G::A_BYTES + b_read_off<TN>(lane, wn * G::WN);
  static_assert(kHeaderBytes % 128 == 0 && G::STAGE % 128 == 0, "slots on 128-byte boundaries");

  const int Gd = gridDim.x;
  const int g0 = first_slot(args);
  if (g0 >= args.num_tiles) return;
  const int my_tiles = (args.num_tiles - g0 + Gd - 1) / Gd;
  const uint32_t P = (uint32_t)args.stages;
  const uint32_t S = (uint32_t)args.iters;
  const uint32_t ring = (uint32_t)(uintptr_t)(smem + kHeaderBytes);
  const uint32_t fullb = (uint32_t)(uintptr_t)full;
  const uint32_t emptyb = (uint32_t)(uintptr_t)empty;
  const uint32_t abortb = (uint32_t)(uintptr_t)abort_flag;

  // Event trace: consumer wave 0 of the traced workgroups runs the block's
  // traced twin, which stores events 4-6 of every K-iteration; the first
  // K-iteration's event 4 and each tile's event 7 are stored here.
  const bool tracing = TRACE && args.trace != nullptr && cw == 0 && (int)blockIdx.x < args.trace_wgs;
  uint32_t* trec = tracing ? args.trace + (size_t)blockIdx.x * args.trace_iters * kTraceEvents : nullptr;
  auto record = [&](uint32_t iq, int ev, uint32_t value) {
    if (tracing && iq < (uint32_t)args.trace_iters && lane == 0) trec[iq * kTraceEvents + ev] = value;
  };

  int v = g0, ti, tj;
  tile_at(args, v, &ti, &tj);
  f32x16_t acc[BM][BN];
  uint32_t slot = 0, ftarget = (uint32_t)G::NP;  // K-iteration 0: ring_slot 0, ring_full_target NP
  for (int t = 0; t < my_tiles; ++t) {
#pragma unroll
    for (int mb = 0; mb < BM; ++mb)
#pragma unroll
      for (int nb = 0; nb < BN; ++nb) acc[mb][nb] = f32x16_t{};
    if (!wait_counter(&full[slot], ftarget, abort_flag, args.spin_limit, args.err)) return;
    const uint32_t q0 = (uint32_t)t * S;  // the tile's first K-iteration in this workgroup's sequence
    if (tracing) record(q0, 4, cycles32());  // the tile's first slot seen full
    const uint32_t base = ring + slot * (uint32_t)G::STAGE;
    uint32_t st;
    if (tracing)
      st = Loop::tile_traced(acc, base + a_off0, base + b_off, slot, ftarget, P, S, ring, fullb, emptyb,
                             abortb, args.spin_limit, args.consumer_delay, trec, q0,
                             (uint32_t)args.trace_iters);
    else
      st = Loop::tile(acc, base + a_off0, base + b_off, slot, ftarget, P, S, ring, fullb, emptyb, abortb,
                      args.spin_limit, args.consumer_delay);
    if (st != 0) {
      if (st == 2) report_timeout(abort_flag, args.err);
      return;
    }
    // The calibration MATH kernel keeps its products (the store below is
    // never taken: M > 0) without writing C.
    if (MODE != kModeMath || args.M < 0)
      store_tile<TM, TN, G::WM, G::WN, BM, BN, GENERAL, 1>(args, acc, ti, tj, wm, wn, lane);
    if (tracing) record(q0 + S - 1, 7, cycles32());
    v += Gd;
    tile_at(args, v, &ti, &tj);
  }
}

// ---------------------------------------------------------------------------
// Compiler-scheduled register-lean consumer for three waves per SIMD (the
// event-traced twins of the largest four-consumer tiles with eight producer
// waves): every operand fragment is single-buffered and
// refilled right after its last MFMA of the k-step, and the loop body is one
// k-step, so each fragment has a single load site and keeps its registers.
// Waits and releases are branch-free asm blocks enabled on the last k-step
// of a K-iteration.  Same synchronisation as consumer().
// ---------------------------------------------------------------------------
template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, bool TRACE, int MODE, bool GENERAL>
__device__ __forceinline__ void consumer_rolling(const KernelArgs& args, WSG_LDS char* smem, int cw,
                                                 int lane) {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  using Ops = ConsumerOps<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  WSG_LDS uint32_t* full = (WSG_LDS uint32_t*)smem;
  WSG_LDS uint32_t* empty = full + kMaxStages;
  WSG_LDS uint32_t* abort_flag = full + 2 * kMaxStages;

  const int wm = cw / G::WGN, wn = cw % G::WGN;
  // A operand of k-step s: a_off0 ^ (32 s).  The chunk of k-step s is
  // (2 s + lane / 32) ^ swz, and XOR acts bit by bit, so only bits 5.. of the
  // in-row byte offset change with s.
  const int r = wm * G::WM + (lane & 31);
  const uint32_t a_off0 = (uint32_t)(r * TK * 2 + (((lane >> 5) ^ swz_a<TK>(r)) << 4));
  const uint32_t b_off = b_read_off<TN>(lane, wn * G::WN);
  const uint32_t ring = (uint32_t)(uintptr_t)smem + kHeaderBytes;

  const int Gd = gridDim.x;
  const int g0 = first_slot(args);
  if (g0 >= args.num_tiles) return;
  const int my_tiles = (args.num_tiles - g0 + Gd - 1) / Gd;
  const uint32_t S = (uint32_t)args.iters;
  const uint32_t total = (uint32_t)my_tiles * S;
  const uint32_t P = (uint32_t)args.stages;

  int v = g0;
  int ti, tj;
  tile_at(args, v, &ti, &tj);

  f32x16_t acc[G::BM][G::BN];
#pragma unroll
  for (int mb = 0; mb < G::BM; ++mb)
#pragma unroll
    for (int nb = 0; nb < G::BN; ++nb) acc[mb][nb] = f32x16_t{};
  i16x8_t fa[G::BM];
  i16x8_t fb[G::BN];

  const bool tracing = TRACE && args.trace != nullptr && cw == 0 && (int)blockIdx.x < args.trace_wgs;
  uint32_t* trec = tracing ? args.trace + (size_t)blockIdx.x * args.trace_iters * kTraceEvents : nullptr;
  auto record = [&](uint32_t iq, int ev, uint32_t value) {
    if (tracing && iq < (uint32_t)args.trace_iters && lane == 0) trec[iq * kTraceEvents + ev] = value;
  };
  auto record_ready = [&](uint32_t iq, uint32_t ps) {
    if (tracing) {
      const uint32_t t = cycles32();
      record(iq, 0, lds_read_now(&full[kStampIssueA + ps]));
      record(iq, 1, lds_read_now(&full[kStampIssueB + ps]));
      record(iq, 2, lds_read_now(&full[kStampLandA + ps]));
      record(iq, 3, lds_read_now(&full[kStampLandB + ps]));
      record(iq, 4, t);
    }
  };

  if (!wait_counter(&full[ring_slot(0, P)], ring_full_target(0, P, G::NP), abort_flag,
                    args.spin_limit, args.err))
    return;
  record_ready(0, 0);
  // full[] of the slot the next wait is for, read one k-step before that
  // wait.  Read here before the first operand loads, so that on every path
  // into the loop a whole k-step of loads is younger than it and the wait
  // for it does not drain them.
  uint32_t peek = lds_peek(&full[ring_slot(1, P)]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int mb = 0; mb < G::BM; ++mb) Ops::load_a(fa[mb], smem + kHeaderBytes, a_off0, mb);
#pragma unroll
  for (int nb = 0; nb < G::BN; ++nb)
    Ops::load_b(fb[nb], smem + kHeaderBytes + G::A_BYTES, b_off, 0, nb);

  uint32_t q = 0, kk = 0, s = 0;
  // (nslot, ntarget): slot and full[] target of K-iteration q + 1.
  uint32_t slot = 0, nslot = ring_slot(1, P);
  uint32_t ntarget = ring_full_target(1, P, G::NP);
  while (true) {
    const uint32_t last = (s == (uint32_t)G::KS - 1) ? 1u : 0u;
    const bool has_next = (q + 1) < total;
    const uint32_t do_wait = (last && has_next) ? 1u : 0u;
    debug_delay(s == 0 ? args.consumer_delay : 0);
    if (tracing && s == 0) record(q, 5, cycles32());
    const uint32_t st = wait_until(peek, &full[nslot], abort_flag, ntarget, args.spin_limit, do_wait);
    if (st != 0) {
      if (st == 2) report_timeout(abort_flag, args.err);
      return;
    }
    compiler_fence();
    if (tracing && do_wait) record_ready(q + 1, nslot);
    {
      const uint32_t pslot = last ? ((nslot + 1 == P) ? 0u : nslot + 1) : nslot;
      peek = lds_peek(&full[pslot]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // Source of the next k-step: k-step s + 1 of this slot, or k-step 0 of
    // the next slot (this slot again after the last K-iteration; never used).
    const uint32_t ts = last ? 0u : s + 1;
    const uint32_t src = ring + (do_wait ? nslot : slot) * (uint32_t)G::STAGE;
    WSG_LDS char* ra = (WSG_LDS char*)(uintptr_t)(src);
    WSG_LDS char* rb = (WSG_LDS char*)(uintptr_t)(src + G::A_BYTES + ts * (uint32_t)(4 * G::NQ * 128));
    const uint32_t a_off = a_off0 ^ (32u * ts);
#pragma unroll
    for (int nb = 0; nb < G::BN; ++nb) {
#pragma unroll
      for (int mb = 0; mb < G::BM; ++mb) {
        acc[mb][nb] = mfma32x32x16<BF16>(fa[mb], fb[nb], acc[mb][nb]);
        if (nb == G::BN - 1) Ops::load_a(fa[mb], ra, a_off, mb);
        __builtin_amdgcn_sched_barrier(0);
      }
      Ops::load_b(fb[nb], rb, b_off, 0, nb);
      __builtin_amdgcn_sched_barrier(0);
    }
    // Every read of this slot is older than the kReads just issued.
    lds_signal_if<Ops::kReads>(&empty[slot], last);
    if (!last) {
      ++s;
      continue;
    }
    if (tracing) record(q, 6, cycles32());
    s = 0;
    slot = nslot;
    ring_advance(nslot, ntarget, P, G::NP);
    ++q;
    if (++kk == S) {
      // The calibration MATH kernel keeps its products (the store below is
      // never taken: M > 0) without writing C.
      if (MODE != kModeMath || args.M < 0)
        store_tile<TM, TN, G::WM, G::WN, G::BM, G::BN, GENERAL, 1>(args, acc, ti, tj, wm, wn, lane);
      if (tracing) record(q - 1, 7, cycles32());
      if (!has_next) break;
      kk = 0;
      v += Gd;
      tile_at(args, v, &ti, &tj);
#pragma unroll
      for (int mb = 0; mb < G::BM; ++mb)
#pragma unroll
        for (int nb = 0; nb < G::BN; ++nb) acc[mb][nb] = f32x16_t{};
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Calibration consumers.  Release-only: take every slot in order and free it
// without reading it (load calibration).  Epilogue-only: store a zero tile
// for every output tile of the workgroup, with no K loop.
template <int NP, int NC>
__device__ __forceinline__ void consumer_release_only(const KernelArgs& args, WSG_LDS char* smem) {
  WSG_LDS uint32_t* full = (WSG_LDS uint32_t*)smem;
  WSG_LDS uint32_t* empty = full + kMaxStages;
  WSG_LDS uint32_t* abort_flag = full + 2 * kMaxStages;
  const int Gd = gridDim.x;
  const int g0 = first_slot(args);
  const int my_tiles = g0 < args.num_tiles ? (args.num_tiles - g0 + Gd - 1) / Gd : 0;
  const uint32_t total = (uint32_t)my_tiles * (uint32_t)args.iters;
  const uint32_t P = (uint32_t)args.stages;
  uint32_t slot = 0, target = ring_full_target(0, P, NP);
  for (uint32_t q = 0; q < total; ++q) {
    if (!wait_counter(&full[slot], target, abort_flag, args.spin_limit, args.err)) return;
    lds_signal(&empty[slot]);
    ring_advance(slot, target, P, NP);
  }
}

template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16>
__device__ __forceinline__ void consumer_epilogue_only(const KernelArgs& args, int cw, int lane) {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  const int wm = cw / G::WGN, wn = cw % G::WGN;
  f32x16_t acc[G::BM][G::BN];
#pragma unroll
  for (int mb = 0; mb < G::BM; ++mb)
#pragma unroll
    for (int nb = 0; nb < G::BN; ++nb) acc[mb][nb] = f32x16_t{};
  for (int v = first_slot(args); v < args.num_tiles; v += (int)gridDim.x) {
    int ti, tj;
    tile_at(args, v, &ti, &tj);
    store_tile<TM, TN, G::WM, G::WN, G::BM, G::BN>(args, acc, ti, tj, wm, wn, lane);
  }
}

// The epilogue of a product with K = 0 (nothing to multiply): C <- beta C
// over n elements of type T; zeros when beta == 0 (C is then not read).
template <typename T>
__global__ void __launch_bounds__(256) ws_scale_kernel(void* C, int64_t n, float beta) {
  T* c = (T*)C;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    c[i] = beta == 0.0f ? (T)0.0f : (T)(beta * load_out(c + i));
}

// Calibration of the launch itself (T_INIT): an empty kernel launched with
// the GEMM's grid, block and LDS size.  A template so that every translation
// unit including this header may instantiate it.
template <int UNUSED = 0>
__global__ void __launch_bounds__(1024) ws_empty_kernel(KernelArgs) {}

// Waves per SIMD a kernel's register allocation must leave room for: what its
// streaming K loop is laid out for (kVgprs: 256, 168, 128 or 80 registers a wave
// are two, three, four or six waves per SIMD; the traced twin of a kernel held to
// 128 runs the roll loop, laid out for the same), else one workgroup (what the
// compiler assumes without the bound).
template <int TM, int TN, int TK, int NC, int NPW, bool BF16, bool TRACE>
constexpr int kernel_waves_per_simd() {
  using Loop = StreamLoop<TM, TN, TK, NC, NPW, BF16>;
  if (Loop::kAvailable && !TRACE) return 512 / Loop::kVgprs;
  if (NC == 4 && RollLoop<TM, TN, TK, NC, NPW, BF16>::kAvailable) return 4;
  return (NC + NPW + 3) / 4;
}

template <int TM, int TN, int TK, int NC, int NPW, int SPLIT, bool BF16, bool TRACE, int MODE, bool GENERAL>
__global__ void __launch_bounds__((NC + NPW) * 64, (kernel_waves_per_simd<TM, TN, TK, NC, NPW, BF16, TRACE>()))
    ws_gemm_kernel(KernelArgs args) {
  using G = Cfg<TM, TN, TK, NC, NPW, SPLIT, BF16>;
  extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
  WSG_LDS char* smem = (WSG_LDS char*)smem_generic;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  LaunchClock clk;
  clk.start(args, wave);
  if (threadIdx.x < 2 * kMaxStages + 1) ((WSG_LDS uint32_t*)smem)[threadIdx.x] = 0u;
  __syncthreads();
  if (wave < NC) {
    if constexpr (MODE == kModeLoadA || MODE == kModeLoadB || MODE == kModeLoadAB) {
      consumer_release_only<G::NP, NC>(args, smem);
    } else if constexpr (MODE == kModeEpilogue) {
      consumer_epilogue_only<TM, TN, TK, NC, NPW, SPLIT, BF16>(args, wave, lane);
    } else if constexpr (!TRACE && StreamLoop<TM, TN, TK, NC, NPW, BF16>::kAvailable) {
      // One or four consumer waves: the streaming K loop, in the general
      // variant too (its producers zero-fill what lies outside A and B, so
      // only the epilogue differs).
      consumer_stream<TM, TN, TK, NC, NPW, SPLIT, BF16, MODE, GENERAL>(args, smem, wave, lane);
    } else if constexpr (RollLoop<TM, TN, TK, NC, NPW, BF16>::kAvailable) {
      // Two consumer waves per SIMD: the generated register-lean K loop, its
      // general variant and its event-traced twin.
      consumer_roll<TM, TN, TK, NC, NPW, SPLIT, BF16, TRACE, MODE, GENERAL>(args, smem, wave, lane);
    } else if constexpr (G::NW > 8 && G::BM * G::BN >= 8) {
      // Traced; three waves per SIMD leave 168 VGPRs: the largest wave tiles
      // then take the single-buffered consumer.
      consumer_rolling<TM, TN, TK, NC, NPW, SPLIT, BF16, TRACE, MODE, GENERAL>(args, smem, wave, lane);
    } else {
      consumer<TM, TN, TK, NC, NPW, SPLIT, BF16, TRACE, MODE, GENERAL>(args, smem, wave, lane);
    }
  } else {
    producer<TM, TN, TK, NC, NPW, SPLIT, BF16, TRACE, MODE, GENERAL>(args, smem, wave - NC, lane);
  }
  clk.stop(args, lane);
}

}  // namespace wsg
