// Fused single-launch sp_score for long prompts: every K row is read from HBM
// exactly once (paper: Appendix A.1.1; Algorithm 1 "AggregateMaxMean").
//
// The exact softmax needs each row's normaliser (a reduction over all L keys)
// before any probability can be formed, and the head maximum must be taken on
// normalised values. Reading K a second time would halve the achievable rate,
// so this kernel keeps K on chip between the two uses:
//
//  * one persistent workgroup per compute unit (8 waves) owns 512 consecutive
//    keys for the whole call; a "phase" is one (layer, kv head) pair, and the
//    workgroup's share of a phase is a 512 x 64 bf16 tile (64 KB);
//  * tiles stream HBM -> LDS with direct-to-LDS loads about one and a half
//    phases ahead. K is wave-private: each wave loads its own 64 keys, in two
//    32-key sub-tiles, into a ring of three sub-tile slots, and later lifts them
//    into MFMA fragments, so the K path needs no barrier. The fragments of four
//    phases live in registers (a ring of 4 x 32 VGPRs);
//  * a vector-memory instruction blocks its wave while the compute unit's memory
//    pipe is full, and the pipe drains at the unit's share of HBM bandwidth, so
//    the eight tile loads of an iteration are spread over its MFMA steps, one
//    or two at a time (two tiles a workgroup: four, behind what the step waits
//    for): while one wave waits for a slot the other waves compute;
//  * phase p: the statistics pass computes the partial (max, sum exp) of every
//    query row over the workgroup's keys and publishes it to global memory;
//  * some workgroup (rotating "duty") combines the partials of four consecutive
//    rows over all workgroups in a fixed order and publishes their normalisers:
//    one wave, or two with two rows each (see kDutyWaves);
//  * three phases later the workgroup picks the normalisers up and runs the
//    probability pass of phase p from the fragments still in its registers:
//    logits again with -lse folded into the MFMA accumulator, maximum over
//    heads on logits, one exp per (lookahead row, key), accumulation over
//    lookahead rows and layers in registers. Scores are stored once at the end;
//  * Q tiles, per-wave statistics and accumulator seeds are double-buffered in
//    LDS so that one workgroup barrier per phase orders everything shared.
//
// The exchange uses no read-modify-write atomics and no cache-wide fences:
// every exchanged word is written and read with device-scope relaxed atomics,
// readiness travels inside the data (the sign bit of the always-positive sum
// carries the parity of the slot's use; normalisers carry the phase number),
// and all waits are bounded. The grid never exceeds the number of compute units
// (one workgroup fits per unit), so every workgroup is resident on an idle device.
// A wait that gives up makes the whole call fail: the workgroup raises the
// call's status word at once, a duty that could not be completed publishes a
// poison entry that fails every workgroup reading it, and every workgroup
// reads the status word before it stores its scores (once any workgroup of a
// prompt has passed that point all exchanged data of the prompt is out, so none
// of them can fail after it; the entries of a table can, one after another has
// stored its scores, so the caller looks at the word once more in a later launch).
//
// Variants of the same loop: head_dim 128 (256 keys per workgroup, a wave's two
// sub-tiles are the two halves of its 32 keys' rows: see the kernel's template
// flag W; with two blocks of query rows Q takes twice the LDS and the transit
// ring has two slots), two tiles a workgroup (flag PAIR), paged keys and lookahead keys in the normaliser, and
// launches that carry a table of (prompt, layer range) entries (see Kind: each
// entry has its own workgroups, duty blocks and row of normalisers).
// Entries are the prompts of a ragged batch, and the layer ranges of prompts
// that fill only part of the device: a step takes about as long whether 64 or
// 256 compute units take part (the exchange and a wave's chain of dependent
// work set it), so a prompt of 98 workgroups runs its 16 layers as two ranges of
// 8 on 196 of them, in half the steps; a small launch then adds the ranges up.
#include "sp_score_fused.hpp"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <type_traits>

namespace {

using namespace sp_dev;
using sp_fused::FusedArgs;
using sp_fused::GroupTable;

constexpr int kD = 64;
constexpr int kKS = kD / 16;              // MFMA k-steps per row
constexpr int kFWaves = 8;
constexpr int kFThreads = kFWaves * 64;
constexpr int kNS = 2;                    // 32-key sub-tiles per wave
constexpr int kFTile = sp_fused::kTileKeys;   // 512 keys per workgroup per phase
constexpr int kSubInstr = 4;              // tile-load instructions per sub-tile (8 rows, 1 KB each)
constexpr int kSubSlots = 3;              // sub-tile slots in a wave's transit ring
constexpr int kLag = 3;                   // phases between statistics and probability pass
constexpr int kRing = kLag + 1;           // fragment ring: four phases
constexpr int kSlots = sp_fused::kSlots;  // exchange ring depth
constexpr int kMaxRowsF = sp_fused::kMaxRows;   // 64 padded query rows per kv head
constexpr int kPubWave = 0;                // the wave that publishes this workgroup's partials
constexpr int kDutyWave = 1;               // the wave that combines this workgroup's duty rows, or with kDutyWave + 2 two of them each
constexpr int kDutyRows = sp_fused::kDutyRows;   // 4: 32 bytes per source workgroup
constexpr int kLseWave = 2;                // the wave that fetches the normalisers
constexpr uint32_t kPoisonTag = 0xffffffffu;   // normaliser entry of a duty that gave up

// LDS map in bytes. Q comes first and everything read with a compile-time offset sits below 64 KB, so that such reads
// can carry the buffer's place in the instruction's offset field. BIG: two blocks of query rows at head_dim 128; their
// Q tiles take twice the room, and the K transit ring has two slots a wave instead of three (all of a phase's tile
// loads are then issued in the statistics pass, once the lift has emptied both slots).
constexpr int kWideHalf = 4096;                                    // head_dim 128: dims 64..127 of a block's 32 rows sit here
constexpr int kWstatsBytes = kFWaves * kMaxRowsF * 8;              // (max, sum) of 64 rows from 8 waves
constexpr int kSubBytes = 32 * kD * 2;
constexpr int kOffXlook = 1024;                                    // of the lookahead-key terms behind the normaliser entries
template <bool BIG>
struct Map {
    static constexpr int kQTileBytes = kMaxRowsF * kD * 2 * (BIG ? 2 : 1);     // one Q tile: 64 rows x 128 (BIG: 256) bytes
    static constexpr int kQBlock = BIG ? 2 * kWideHalf : kWideHalf;            // 32 rows
    static constexpr int kQ1 = 0;                                  // [2] Q of the statistics pass, by phase parity
    static constexpr int kQ2 = kQ1 + 2 * kQTileBytes;              // [2] Q of the probability pass
    static constexpr int kWstats = kQ2 + 2 * kQTileBytes;          // [2], pairs of tiles: [4]
    static constexpr int kCinit = kWstats + 4 * kWstatsBytes;      // [2][64] accumulator seeds
    static constexpr int kXduty = kCinit + 2 * kMaxRowsF * 4;      // 8 KB: partials of the duty rows (direct exchange: of all rows)
    static constexpr int kXlse = kXduty + 8192;                    // 1 KB: normaliser entries of one phase, 1 KB: lookahead-key terms
    static constexpr int kFail = kXlse + 2048;
    static constexpr int kSeeded = kFail + 4;                      // step_prob_last: phase whose seeds are in kCinit, plus one
    static constexpr int kKring = (kFail + 16 + 1023) / 1024 * 1024;   // [8 waves][slots][32 rows x 128 bytes]
    static constexpr int kSlotsPerWave = BIG ? 2 : kSubSlots;
    static constexpr int kBytes = kKring + kFWaves * kSlotsPerWave * kSubBytes;
    static_assert(kQ2 + 2 * kQTileBytes <= 65536 && kBytes <= 160 * 1024, "offset fields hold 16 bits; 160 KB a compute unit");
};

// The probability pass at the end of a step (see step_late): K stays in the transit ring for the whole step, so a wave
// has four slots (two tiles of two sub-tiles); everything else is sized for 32 rows.
struct LateMap {
    static constexpr int kRows = 32, kWaveStats = kRows * 8;                   // (max, sum) of one wave
    static constexpr int kQTileBytes = kRows * kD * 2;
    static constexpr int kQBlock = kQTileBytes;
    static constexpr int kQ1 = 0;                                  // [2] by step parity
    static constexpr int kQ2 = kQ1 + 2 * kQTileBytes;              // [2]
    static constexpr int kWstats = kQ2 + 2 * kQTileBytes;          // first tile of a phase: [2] by phase parity; second tile
    static constexpr int kCinit = kWstats + 3 * kFWaves * kWaveStats;
    static constexpr int kXduty = kCinit + kRows * 4;              // two waves x 4 KB
    static constexpr int kXlse = kXduty + 8192;                    // normaliser entries
    static constexpr int kXlook = kXlse + kRows * 8;
    static constexpr int kFail = kXlook + kRows * 4;
    static constexpr int kSeeded = kFail + 4;                      // phase whose seeds are in kCinit, plus one
    static constexpr int kKring = (kFail + 16 + 1023) / 1024 * 1024;
    static constexpr int kBytes = kKring + kFWaves * 4 * kSubBytes;
    static_assert(kBytes <= 160 * 1024, "160 KB a compute unit");
    // sub-tile s2 of the tile of a step of parity par
    static __device__ __forceinline__ uint32_t slot(int wave, int par, int s2) { return (uint32_t)(kKring + ((wave * 2 + par) * 2 + s2) * kSubBytes); }
};

#define SP_LPTR(p) ((__attribute__((address_space(3))) void *)(p))

__device__ __forceinline__ uint64_t ld64(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st64(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Workgroup barrier that orders LDS traffic only. Direct-to-LDS loads are
// waited for explicitly (vm_wait) by the wave that issued them, so that younger
// loads can stay in flight across the barrier.
__device__ __forceinline__ void lds_barrier()
{
    __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
}
// Wait until at most N vector-memory operations of this wave are outstanding.
template <int N>
__device__ __forceinline__ void vm_wait()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
    __asm__ volatile("" ::: "memory");
}

// max(a, b, c); built without NaN honouring the compiler emits a single v_max3_f32 for it
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// What a variant of the kernel serves beyond one whole prompt of contiguous keys. Every one carries only its
// own code: shared duties in the variant for ranges would cost the batches 3 %.
enum Kind {
    kPlain,
    kExtra,     // + paged keys, lookahead keys, or the whole prompts of a batch, whose duties rotate over the launch
    kRanges     // + paged keys, lookahead keys, and a table of entries that keep to themselves: layer ranges, short prompts
};

// A workgroup's index, which says which tile it owns and where its partials go. Blocks are handed to the eight dies in
// turn. BY_DIE: consecutive tiles go to one die, whose L2 then waits less for DRAM: 131072 tokens, 8 lookahead rows, the same
// reads (TCC_EA0_RDREQ 1.71e7) and address translations, but TCC_EA0_RDREQ_DRAM_CREDIT_STALL 7.2e6 -> 5.0e6 and TCC_TAG_STALL 8.4e6 ->
// 6.2e6 a launch, token-major 8.2e6 -> 7.0e6 and 10.5e6 -> 8.8e6. Duties go by block, so that the workgroups of a phase's duties sit
// on all dies (with them by tile 262144 tokens took 841 us).
template <bool BY_DIE>
__device__ __forceinline__ int workgroup_index(int n_wg)
{
    const int b = (int)blockIdx.x, die = b & 7;
    return BY_DIE ? die * (n_wg >> 3) + min(die, n_wg & 7) + (b >> 3) : b;
}

// Where a prompt has the launch to itself, contiguous bf16 keys of head_dim 64 (score calls and, *, whole passes, every eighth tile /
// consecutive ones, us, both in turn on one card): one block of query rows, 16 x 8 phases, 131072 tokens 376 / 361, token-major 445 / 423, 100000 291 / 289 and
// 346 / 334, 8 x 8 phases 75324 149 / 144, 2 x 2 33000 17.1 / 16.1; two tiles a workgroup 262144 776 / 773, token-major 851 / 843. With two
// blocks of rows only in the instantiation for all compute units, * 131072 tokens 500 / 496, on another card 478 / 475; elsewhere * 75324 382 / 385, 8 x 8 phases
// 120000 230 / 236, 2 x 4 75324 22.3 / 23.0, two tiles a workgroup * 150000 764 / 770. Not for 8-bit keys * 458 / 460, head_dim 128 two tiles a
// workgroup * 1103 / 1110, sixteen prompts * 999 / 1001; layer ranges * 8192 tokens 55.9 / 59.3 (a range's workgroups on one die).
template <int BLOCKS, Kind KIND, bool W, bool F8, class M>
constexpr bool tiles_by_die = KIND == kPlain && !W && !F8 && (BLOCKS == 1 || M::kWorkgroups > 0);

struct Ring {
    bf16x8 kf[kRing][kNS][kKS];           // K fragments of the phases in flight
};

// Values that depend on the lane only, computed once: they cost a few registers and save the
// address arithmetic of every load and lift.
struct LaneConst {
    uint32_t ld[kKS];       // LDS byte address of this lane's fragment chunk t in a tile at LDS offset 0
    uint32_t ld8[kKS];      // the same in a sub-tile of 8-bit keys (rows of 64 bytes, 8 bytes per chunk)
    uint32_t koff[2];       // byte offset of this lane's chunk in an even / odd tile-load instruction (full tiles)
    int32_t qoff[2];        // byte offset of this lane's chunk of its wave's Q slice in a (layer, kv head) block; < 0: padding (BIG: per row block)
};

// All LDS traffic of the main loop is written as asm: the compiler cannot tell which in-flight
// direct-to-LDS load targets which buffer and would put a full vector-memory wait in front of
// LDS accesses it can see. The kernel waits (vm_wait, barrier) for exactly what it is about to read.
__device__ __forceinline__ uint32_t lds_addr(const void *p) { return (uint32_t)reinterpret_cast<uintptr_t>(SP_LPTR(p)); }

// Direct-to-LDS loads of 64 lanes x 16 bytes into LDS bytes [lds_dst, lds_dst + 1024); lds_dst is
// uniform and travels in M0, which nothing else in this kernel uses. They are asm for the same
// reason, and so that the scalar-base form is used: a uniform 64-bit base plus a 32-bit lane offset.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ uint32_t uniform32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
// The LDS destination is lds_base + LDS_IMM: call sites that differ only in the constant share one
// scalar register for the base.
template <int LDS_IMM>
__device__ __forceinline__ void dma_u(uint32_t lane_off, const void *base, uint32_t lds_base)
{
    const uint64_t b = reinterpret_cast<uintptr_t>(base);
    const uint64_t ub = (uint64_t)uniform32((uint32_t)b) | ((uint64_t)uniform32((uint32_t)(b >> 32)) << 32);
    __asm__ volatile("s_add_i32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     : : "v"(lane_off), "s"(ub), "s"(uniform32(lds_base)), "i"(LDS_IMM) : "memory", "m0", "scc");
}
// Per-lane addresses, bypassing the non-coherent cache levels like the atomic loads of the retry paths do.
__device__ __forceinline__ void dma_v_device(const void *addr, uint32_t lds_dst)
{
    __asm__ volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off sc1"
                     : : "v"(addr), "s"(uniform32(lds_dst)) : "memory", "m0");
}
#pragma clang diagnostic pop

// MFMA fragments of 32 rows of a swizzled 64-wide bf16 tile at compile-time LDS offset OFF:
// lane (col, hf) takes row col, 16-byte chunks 2t + hf.
template <int OFF>
__device__ __forceinline__ void lift_at(const LaneConst &lc, bf16x8 (&f)[kKS])
{
    static_assert(kKS == 4 && OFF >= 0 && OFF < 65536, "layout of the asm block");
    u32x4 r[kKS];
    __asm__ volatile(
        "ds_read_b128 %0, %4 offset:%8\n\t"
        "ds_read_b128 %1, %5 offset:%8\n\t"
        "ds_read_b128 %2, %6 offset:%8\n\t"
        "ds_read_b128 %3, %7 offset:%8\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
        : "v"(lc.ld[0]), "v"(lc.ld[1]), "v"(lc.ld[2]), "v"(lc.ld[3]), "i"(OFF)
        : "memory");
#pragma unroll
    for (int t = 0; t < kKS; ++t) f[t] = __builtin_bit_cast(bf16x8, r[t]);
}
// Both 32-key sub-tiles of a K tile (run-time slot offsets) and one 32-row Q block (compile-time
// offset) in one round trip to LDS.
template <int QOFF>
__device__ __forceinline__ void lift_k_and_q(const LaneConst &lc, uint32_t koff0, uint32_t koff1,
                                             bf16x8 (&kf)[kNS][kKS], bf16x8 (&qf)[kKS])
{
    static_assert(kKS == 4 && kNS == 2 && QOFF >= 0 && QOFF < 65536, "layout of the asm block");
    u32x4 r[12];
    uint32_t a0[kKS], a1[kKS];
#pragma unroll
    for (int t = 0; t < kKS; ++t) { a0[t] = lc.ld[t] + koff0; a1[t] = lc.ld[t] + koff1; }
    __asm__ volatile(
        "ds_read_b128 %0, %12\n\t"
        "ds_read_b128 %1, %13\n\t"
        "ds_read_b128 %2, %14\n\t"
        "ds_read_b128 %3, %15\n\t"
        "ds_read_b128 %8, %20 offset:%24\n\t"
        "ds_read_b128 %9, %21 offset:%24\n\t"
        "ds_read_b128 %10, %22 offset:%24\n\t"
        "ds_read_b128 %11, %23 offset:%24\n\t"
        "ds_read_b128 %4, %16\n\t"
        "ds_read_b128 %5, %17\n\t"
        "ds_read_b128 %6, %18\n\t"
        "ds_read_b128 %7, %19\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]),
          "=&v"(r[8]), "=&v"(r[9]), "=&v"(r[10]), "=&v"(r[11])
        : "v"(a0[0]), "v"(a0[1]), "v"(a0[2]), "v"(a0[3]), "v"(a1[0]), "v"(a1[1]), "v"(a1[2]), "v"(a1[3]),
          "v"(lc.ld[0]), "v"(lc.ld[1]), "v"(lc.ld[2]), "v"(lc.ld[3]), "i"(QOFF)
        : "memory");
#pragma unroll
    for (int t = 0; t < kKS; ++t) {
        kf[0][t] = __builtin_bit_cast(bf16x8, r[t]);
        kf[1][t] = __builtin_bit_cast(bf16x8, r[4 + t]);
        qf[t] = __builtin_bit_cast(bf16x8, r[8 + t]);
    }
}

// head_dim 128: both halves of a 32-row Q block in one round trip to LDS, with the seeds or the K tile that go with it.
template <int QOFF>
__device__ __forceinline__ void lift_q_wide_and_seed(const LaneConst &lc, uint32_t seed_ad, bf16x8 (&q0)[kKS], bf16x8 (&q1)[kKS], f32x16 &seed)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    u32x4 r[8];
    f32x4 c[4];
    __asm__ volatile(
        "ds_read_b128 %8, %16\n\tds_read_b128 %9, %16 offset:16\n\tds_read_b128 %10, %16 offset:32\n\tds_read_b128 %11, %16 offset:48\n\t"
        "ds_read_b128 %0, %12 offset:%17\n\tds_read_b128 %1, %13 offset:%17\n\t"
        "ds_read_b128 %2, %14 offset:%17\n\tds_read_b128 %3, %15 offset:%17\n\t"
        "ds_read_b128 %4, %12 offset:%17+4096\n\tds_read_b128 %5, %13 offset:%17+4096\n\t"
        "ds_read_b128 %6, %14 offset:%17+4096\n\tds_read_b128 %7, %15 offset:%17+4096\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]),
          "=&v"(c[0]), "=&v"(c[1]), "=&v"(c[2]), "=&v"(c[3])
        : "v"(lc.ld[0]), "v"(lc.ld[1]), "v"(lc.ld[2]), "v"(lc.ld[3]), "v"(seed_ad), "i"(QOFF) : "memory");
#pragma unroll
    for (int t = 0; t < kKS; ++t) {
        q0[t] = __builtin_bit_cast(bf16x8, r[t]);
        q1[t] = __builtin_bit_cast(bf16x8, r[4 + t]);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) { seed[4 * v] = c[v].x; seed[4 * v + 1] = c[v].y; seed[4 * v + 2] = c[v].z; seed[4 * v + 3] = c[v].w; }
}
// The K tile's two halves (run-time slot offsets) and both halves of a Q block.
template <int QOFF>
__device__ __forceinline__ void lift_k_and_q_wide(const LaneConst &lc, uint32_t koff0, uint32_t koff1, bf16x8 (&kf)[kNS][kKS],
                                                  bf16x8 (&q0)[kKS], bf16x8 (&q1)[kKS])
{
    u32x4 r[16];
    uint32_t a0[kKS], a1[kKS];
#pragma unroll
    for (int t = 0; t < kKS; ++t) { a0[t] = lc.ld[t] + koff0; a1[t] = lc.ld[t] + koff1; }
    __asm__ volatile(
        "ds_read_b128 %0, %16\n\tds_read_b128 %1, %17\n\tds_read_b128 %2, %18\n\tds_read_b128 %3, %19\n\t"
        "ds_read_b128 %8, %24 offset:%28\n\tds_read_b128 %9, %25 offset:%28\n\tds_read_b128 %10, %26 offset:%28\n\tds_read_b128 %11, %27 offset:%28\n\t"
        "ds_read_b128 %4, %20\n\tds_read_b128 %5, %21\n\tds_read_b128 %6, %22\n\tds_read_b128 %7, %23\n\t"
        "ds_read_b128 %12, %24 offset:%28+4096\n\tds_read_b128 %13, %25 offset:%28+4096\n\t"
        "ds_read_b128 %14, %26 offset:%28+4096\n\tds_read_b128 %15, %27 offset:%28+4096\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]),
          "=&v"(r[8]), "=&v"(r[9]), "=&v"(r[10]), "=&v"(r[11]), "=&v"(r[12]), "=&v"(r[13]), "=&v"(r[14]), "=&v"(r[15])
        : "v"(a0[0]), "v"(a0[1]), "v"(a0[2]), "v"(a0[3]), "v"(a1[0]), "v"(a1[1]), "v"(a1[2]), "v"(a1[3]),
          "v"(lc.ld[0]), "v"(lc.ld[1]), "v"(lc.ld[2]), "v"(lc.ld[3]), "i"(QOFF) : "memory");
#pragma unroll
    for (int t = 0; t < kKS; ++t) {
        kf[0][t] = __builtin_bit_cast(bf16x8, r[t]);
        kf[1][t] = __builtin_bit_cast(bf16x8, r[4 + t]);
        q0[t] = __builtin_bit_cast(bf16x8, r[8 + t]);
        q1[t] = __builtin_bit_cast(bf16x8, r[12 + t]);
    }
}

// One 32-key sub-tile at a run-time offset, both of a tile, and one with a 32-row Q block: one round trip to LDS each.
__device__ __forceinline__ void lift_sub(const LaneConst &lc, uint32_t koff, bf16x8 (&kf)[kKS])
{
    static_assert(kKS == 4, "layout of the asm block");
    u32x4 r[4];
    __asm__ volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
                     : "v"(lc.ld[0] + koff), "v"(lc.ld[1] + koff), "v"(lc.ld[2] + koff), "v"(lc.ld[3] + koff) : "memory");
#pragma unroll
    for (int t = 0; t < kKS; ++t) kf[t] = __builtin_bit_cast(bf16x8, r[t]);
}
__device__ __forceinline__ void lift_tile(const LaneConst &lc, uint32_t koff, bf16x8 (&kf)[kNS][kKS])
{
    static_assert(kKS == 4 && kNS == 2 && kSubBytes == 4096, "layout of the asm block");
    u32x4 r[8];
    __asm__ volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                     "ds_read_b128 %4, %8 offset:4096\n\tds_read_b128 %5, %9 offset:4096\n\t"
                     "ds_read_b128 %6, %10 offset:4096\n\tds_read_b128 %7, %11 offset:4096\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
                     : "v"(lc.ld[0] + koff), "v"(lc.ld[1] + koff), "v"(lc.ld[2] + koff), "v"(lc.ld[3] + koff) : "memory");
#pragma unroll
    for (int t = 0; t < kKS; ++t) {
        kf[0][t] = __builtin_bit_cast(bf16x8, r[t]);
        kf[1][t] = __builtin_bit_cast(bf16x8, r[4 + t]);
    }
}
template <int QOFF>
__device__ __forceinline__ void lift_sub_and_q(const LaneConst &lc, uint32_t koff, bf16x8 (&kf)[kKS], bf16x8 (&qf)[kKS])
{
    static_assert(kKS == 4 && QOFF >= 0 && QOFF < 65536, "layout of the asm block");
    u32x4 r[8];
    __asm__ volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                     "ds_read_b128 %4, %12 offset:%16\n\tds_read_b128 %5, %13 offset:%16\n\t"
                     "ds_read_b128 %6, %14 offset:%16\n\tds_read_b128 %7, %15 offset:%16\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
                     : "v"(lc.ld[0] + koff), "v"(lc.ld[1] + koff), "v"(lc.ld[2] + koff), "v"(lc.ld[3] + koff),
                       "v"(lc.ld[0]), "v"(lc.ld[1]), "v"(lc.ld[2]), "v"(lc.ld[3]), "i"(QOFF) : "memory");
#pragma unroll
    for (int t = 0; t < kKS; ++t) {
        kf[t] = __builtin_bit_cast(bf16x8, r[t]);
        qf[t] = __builtin_bit_cast(bf16x8, r[4 + t]);
    }
}

// 8-bit keys: both 32-key sub-tiles of a K tile (rows of 64 codes; this lane's eight codes of k-step t
// are one 8-byte read) and one 32-row Q block in one round trip to LDS, the codes widened to bf16.
template <int QOFF>
__device__ __forceinline__ void lift_k8_and_q(const LaneConst &lc, uint32_t koff0, uint32_t koff1,
                                              bf16x8 (&kf)[kNS][kKS], bf16x8 (&qf)[kKS])
{
    static_assert(kKS == 4 && kNS == 2 && QOFF >= 0 && QOFF < 65536, "layout of the asm block");
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
    u32x2 r[8];
    u32x4 q[4];
    uint32_t a0[kKS], a1[kKS];
#pragma unroll
    for (int t = 0; t < kKS; ++t) { a0[t] = lc.ld8[t] + koff0; a1[t] = lc.ld8[t] + koff1; }
    __asm__ volatile(
        "ds_read_b64 %0, %12\n\t"
        "ds_read_b64 %1, %13\n\t"
        "ds_read_b64 %2, %14\n\t"
        "ds_read_b64 %3, %15\n\t"
        "ds_read_b128 %8, %20 offset:%24\n\t"
        "ds_read_b128 %9, %21 offset:%24\n\t"
        "ds_read_b128 %10, %22 offset:%24\n\t"
        "ds_read_b128 %11, %23 offset:%24\n\t"
        "ds_read_b64 %4, %16\n\t"
        "ds_read_b64 %5, %17\n\t"
        "ds_read_b64 %6, %18\n\t"
        "ds_read_b64 %7, %19\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]),
          "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3])
        : "v"(a0[0]), "v"(a0[1]), "v"(a0[2]), "v"(a0[3]), "v"(a1[0]), "v"(a1[1]), "v"(a1[2]), "v"(a1[3]),
          "v"(lc.ld[0]), "v"(lc.ld[1]), "v"(lc.ld[2]), "v"(lc.ld[3]), "i"(QOFF)
        : "memory");
#pragma unroll
    for (int t = 0; t < kKS; ++t) {
        kf[0][t] = __builtin_bit_cast(bf16x8, e4m3x8_to_bf16x8(r[t].x, r[t].y));
        kf[1][t] = __builtin_bit_cast(bf16x8, e4m3x8_to_bf16x8(r[4 + t].x, r[4 + t].y));
        qf[t] = __builtin_bit_cast(bf16x8, q[t]);
    }
}

// One 32-row Q block (compile-time offset) and the sixteen accumulator seeds at seed_ad (64-byte
// aligned) in one round trip to LDS.
template <int QOFF>
__device__ __forceinline__ void lift_q_and_seed(const LaneConst &lc, uint32_t seed_ad, bf16x8 (&qf)[kKS], f32x16 &seed)
{
    static_assert(kKS == 4 && QOFF >= 0 && QOFF < 65536, "layout of the asm block");
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    u32x4 r[kKS];
    f32x4 c[4];
    __asm__ volatile(
        "ds_read_b128 %0, %8 offset:%13\n\t"
        "ds_read_b128 %1, %9 offset:%13\n\t"
        "ds_read_b128 %2, %10 offset:%13\n\t"
        "ds_read_b128 %3, %11 offset:%13\n\t"
        "ds_read_b128 %4, %12\n\t"
        "ds_read_b128 %5, %12 offset:16\n\t"
        "ds_read_b128 %6, %12 offset:32\n\t"
        "ds_read_b128 %7, %12 offset:48\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(c[0]), "=&v"(c[1]), "=&v"(c[2]), "=&v"(c[3])
        : "v"(lc.ld[0]), "v"(lc.ld[1]), "v"(lc.ld[2]), "v"(lc.ld[3]), "v"(seed_ad), "i"(QOFF)
        : "memory");
#pragma unroll
    for (int t = 0; t < kKS; ++t) qf[t] = __builtin_bit_cast(bf16x8, r[t]);
#pragma unroll
    for (int v = 0; v < 4; ++v) { seed[4 * v] = c[v].x; seed[4 * v + 1] = c[v].y; seed[4 * v + 2] = c[v].z; seed[4 * v + 3] = c[v].w; }
}

__device__ __forceinline__ void lds_store_f32(uint32_t ad, float v)
{
    __asm__ volatile("ds_write_b32 %0, %1" : : "v"(ad), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_store_u32(uint32_t ad, uint32_t v)
{
    __asm__ volatile("ds_write_b32 %0, %1" : : "v"(ad), "v"(v) : "memory");
}
__device__ __forceinline__ uint32_t lds_load_u32(uint32_t ad)
{
    uint32_t v;
    __asm__ volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(ad) : "memory");
    return uniform32(v);
}
__device__ __forceinline__ void lds_store_f2(uint32_t ad, float2 v)
{
    __asm__ volatile("ds_write_b64 %0, %1" : : "v"(ad), "v"(v) : "memory");
}
// Butterfly reductions with data-parallel-primitive moves: after the three steps every lane of an
// aligned group of 8 holds the group's result; one more step extends it to the row of 16. Every
// lane adds the same two operands in either order, so the results are identical across lanes.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1;          // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;          // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;   // lane i <- lane 7 - i within groups of 8
constexpr int kDppMirror = 0x140;       // lane i <- lane 15 - i within rows of 16

// Maximum and sum over a lane and the one 32 away, the same bits in both (no trip through LDS as shuffles make).
__device__ __forceinline__ float halves_max(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float halves_sum(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp_move<kDppXor1>(v));
    v = fmaxf(v, dpp_move<kDppXor2>(v));
    v = fmaxf(v, dpp_move<kDppHalfMirror>(v));
    v = fmaxf(v, dpp_move<kDppMirror>(v));
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp_move<kDppXor1>(v);
    v += dpp_move<kDppXor2>(v);
    v += dpp_move<kDppHalfMirror>(v);
    v += dpp_move<kDppMirror>(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// (layer, kv head) of a phase, walked step by step instead of divided out every time.
struct PhaseCtr { int layer, kv; };
__device__ __forceinline__ PhaseCtr phase_at(int p, int n_phases, int n_kv)
{
    p = clampi(p, 0, n_phases - 1);
    PhaseCtr r; r.layer = p / n_kv; r.kv = p - r.layer * n_kv; return r;
}
// c holds clamp(p_next - 1, 0, n_phases - 1); make it hold clamp(p_next, 0, n_phases - 1).
__device__ __forceinline__ void phase_advance(PhaseCtr &c, int p_next, int n_phases, int n_kv)
{
    if (p_next > 0 && p_next < n_phases) {
        if (++c.kv == n_kv) { c.kv = 0; ++c.layer; }
    }
}

// 8-bit keys: scale of a phase, through the scalar cache (the array is constant for the whole launch, and the
// constant address space says so). As vector loads these values made the compiler wait for every tile load in
// flight before their first use, in every step.
__device__ __forceinline__ float key_scale(const FusedArgs &a, int phase)
{
    typedef const __attribute__((address_space(4))) float *scalar_ptr;
    return reinterpret_cast<scalar_ptr>(reinterpret_cast<uintptr_t>(a.kscale))[phase];
}

// padded query row -> (group head, lookahead row); see the row order in sp_score.hip
template <int NB>
__device__ __forceinline__ bool row_valid(const FusedArgs &a, int row, int &g, int &n)
{
    const int blk = row >> 5, rho = row & 31;
    const int gblk = blk / NB, nblk = blk - gblk * NB;
    g = 4 * gblk + (rho >> 3);
    n = 8 * nblk + (rho & 7);
    return g < a.group && n < a.n_q;
}

// One wave instruction moves 64 chunks = 8 key rows (1 KB, contiguous in HBM when keys are
// contiguous); a 32-key sub-tile takes four of them: a uniform base that steps by 8 keys, plus the
// lane's constant offset (even / odd instruction).
struct KIssue {
    uint32_t lds_dst;         // LDS byte address of the sub-tile slot being refilled (this wave's)
    const char *base;         // first key of the sub-tile in the (layer, kv head) being fetched (uniform)
    uint32_t step_bytes;      // bytes between the first keys of consecutive instructions (8 keys)
};

// Issues instructions first .. first+COUNT-1 of the sub-tile (first and COUNT compile-time at call sites).
template <int IDX>
__device__ __forceinline__ void k_issue_one(const KIssue &ki, const uint32_t (&voff)[2])
{
    dma_u<IDX * 1024>(voff[IDX & 1], ki.base + (uint32_t)IDX * ki.step_bytes, ki.lds_dst);
}
template <int COUNT>
__device__ __forceinline__ void k_issue(const KIssue &ki, const uint32_t (&voff)[2], int first)
{
    static_assert(kSubInstr == 4, "instruction indices 0..3");
#pragma unroll
    for (int i = 0; i < COUNT; ++i) {
        switch (first + i) {          // compile-time after unrolling
        case 0: k_issue_one<0>(ki, voff); break;
        case 1: k_issue_one<1>(ki, voff); break;
        case 2: k_issue_one<2>(ki, voff); break;
        default: k_issue_one<3>(ki, voff); break;
        }
    }
}

// Sub-tile s2 of phase p lives in slot (2p + s2) mod 3 of its wave's transit ring; slot0 = 2p mod 3.
template <bool BIG>
__device__ __forceinline__ uint32_t sub_slot_off(int wave, int slot0, int s2)
{
    if (BIG) return (uint32_t)(Map<BIG>::kKring + (wave * 2 + s2) * kSubBytes);
    int slot = slot0 + s2;
    slot = slot >= kSubSlots ? slot - kSubSlots : slot;
    return (uint32_t)(Map<BIG>::kKring + (wave * kSubSlots + slot) * kSubBytes);
}

template <int NB>
struct Acc {
    float mx[kNS][NB][4];
    float total[kNS];
};

// ---- probability pass of one phase from the fragment ring; tile loads are issued between the MFMA steps ----
// The four loads of sub-tile 0 (8-bit keys: two) are issued between the MFMA steps of the probability pass. With half of
// them right after the barrier, where every wave also requests its slices of Q, eight waves stood behind each other at
// the unit's memory pipe: sixteen prompts 1017 -> 1002 us.

// F8: logits are in units of the phase's key scale `ks`; a phase's head maximum is brought to common
// units before it meets other phases'. One tile load instead of two (half the bytes per sub-tile).
template <int NB, int GB, int PAR, bool W, bool F8>
__device__ __forceinline__ void prob_pass(const bf16x8 (&kf)[kNS][kKS], const LaneConst &lc, uint32_t cinit_ad,
                                          Acc<NB> &acc, const KIssue &ki, const uint32_t (&voff)[2], float ks)
{
    static_assert(NB * GB == 1 || NB * GB == 2, "one load per row block, or one per step");
    using MP = Map<W && NB * GB == 2>;
    constexpr int kHalf = F8 ? 1 : 2;
    if constexpr (W) {
        // head_dim 128: one chain of eight MFMA steps over both halves of the 32 keys' rows
        static_assert(NB == 1, "one block of lookahead rows");
#pragma unroll
        for (int gb = 0; gb < GB; ++gb) {
            bf16x8 q0[kKS], q1[kKS];
            f32x16 d;
            if (gb == 0) {
                lift_q_and_seed<MP::kQ2 + PAR * MP::kQTileBytes>(lc, cinit_ad, q0, d);
                lift_at<MP::kQ2 + PAR * MP::kQTileBytes + kWideHalf>(lc, q1);
            } else {
                lift_q_and_seed<MP::kQ2 + PAR * MP::kQTileBytes + MP::kQBlock>(lc, cinit_ad + 128, q0, d);
                lift_at<MP::kQ2 + PAR * MP::kQTileBytes + MP::kQBlock + kWideHalf>(lc, q1);
            }
#pragma unroll
            for (int t = 0; t < kKS; ++t) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q0[t], kf[0][t], d, 0, 0, 0);
            if (GB == 1) k_issue<kHalf>(ki, voff, 0);
#pragma unroll
            for (int t = 0; t < kKS; ++t) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q1[t], kf[1][t], d, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (F8) acc.mx[0][0][e] = fmaxf(acc.mx[0][0][e], fmaxf(max3(d[e], d[4 + e], d[8 + e]), d[12 + e]) * ks);
                else acc.mx[0][0][e] = max3(max3(d[e], d[4 + e], d[8 + e]), d[12 + e], acc.mx[0][0][e]);
            }
            if (GB == 1) k_issue<kHalf>(ki, voff, kHalf);
        }
        __builtin_amdgcn_sched_barrier(0);
        return;
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
        for (int gb = 0; gb < GB; ++gb) {
            const int blk = gb * NB + nb;
            bf16x8 qf[kKS];
            f32x16 ci;
            if (blk == 0) lift_q_and_seed<MP::kQ2 + PAR * MP::kQTileBytes>(lc, cinit_ad, qf, ci);
            else lift_q_and_seed<MP::kQ2 + PAR * MP::kQTileBytes + MP::kQBlock>(lc, cinit_ad + 128, qf, ci);
#pragma unroll
            for (int s = 0; s < kNS; ++s) {
                f32x16 d = ci;
#pragma unroll
                for (int t = 0; t < kKS; ++t) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[t], kf[s][t], d, 0, 0, 0);
                // d[r]: group head r/4, lookahead row 8*nb + 4*hf + r%4, key (wave*2+s)*32 + col
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (F8) acc.mx[s][nb][e] = fmaxf(acc.mx[s][nb][e], fmaxf(max3(d[e], d[4 + e], d[8 + e]), d[12 + e]) * ks);
                    else acc.mx[s][nb][e] = max3(max3(d[e], d[4 + e], d[8 + e]), d[12 + e], acc.mx[s][nb][e]);
                }
                if (NB * GB == 1) k_issue<kHalf>(ki, voff, kHalf * s);
                else if (!F8 || blk == 0) k_issue<1>(ki, voff, kNS * blk + s);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

template <int NB, int NSE>
__device__ __forceinline__ void close_layer(Acc<NB> &acc, float c)
{
#pragma unroll
    for (int s = 0; s < NSE; ++s) {
        float sum = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sum += fast_exp2(acc.mx[s][b][e] * c);
                acc.mx[s][b][e] = neg_inf();
            }
        acc.total[s] += sum;
    }
}

// 64 x 16 bytes: the 16-byte pairs 0 .. 63 of a row of 8-byte entries (row 16-byte aligned) that
// holds `pairs` pairs; lanes beyond the row repeat its last pair.
__device__ __forceinline__ void stage_entries(uint32_t lds_dst, const uint64_t *row, int pairs, int lane)
{
    dma_v_device(row + 2 * min(lane, pairs - 1), lds_dst);
}

// The normaliser wave's requests of one step: the rows' lookahead-key terms (when the call has
// them; 4-byte entries, four to a lane) and, behind them, the normaliser entries. Loads return in
// order, so the wait for the normalisers covers both.
__device__ __forceinline__ void stage_exchange_rows(uint32_t xlse_ad, const uint64_t *lse_row, const float *look_row,
                                                    int rows_pad, int lane)
{
    if (look_row != nullptr) dma_v_device(look_row + 4 * min(lane, rows_pad / 4 - 1), xlse_ad + kOffXlook);
    if (lse_row != nullptr) stage_entries(xlse_ad, lse_row, rows_pad / 2, lane);
}

// ---- statistics pass of one phase: per-wave (max, sum exp) of every row into wstats ----
// Logits of 32 keys (one sub-tile) against 32 query rows: d[r] is key 8*(r/4) + 4*hf + r%4 of the
// sub-tile, query row col.
__device__ __forceinline__ f32x16 logits32(const bf16x8 (&kf)[kKS], const bf16x8 (&qf)[kKS])
{
    f32x16 d = {0.f};
#pragma unroll
    for (int t = 0; t < kKS; ++t) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t], qf[t], d, 0, 0, 0);
    return d;
}

// Folds the 16 logits of a lane into its running (max, sum exp), which they start if FIRST (m = -inf, l = 0); only
// keys lo <= key < hi of the sub-tile are this workgroup's (all 32 except in the prompt's last tile).
template <bool FIRST>
__device__ __forceinline__ void fold_logits(const f32x16 &d, float &m, float &l, float c, int lo, int hi, int hf)
{
    if (lo <= 0 && hi >= 32) {
        // running maximum including these 16 logits, as a tree: a chain of eight waits for every one of them
        const float m0 = max3(d[0], d[1], d[2]), m1 = max3(d[3], d[4], d[5]), m2 = max3(d[6], d[7], d[8]);
        const float m3 = max3(d[9], d[10], d[11]), m4 = max3(d[12], d[13], d[14]);
        const float a0 = max3(m0, m1, m2), a1 = max3(m3, m4, d[15]);
        const float mn = FIRST ? fmaxf(a0, a1) : max3(a0, a1, m);
        if (!FIRST) l *= fast_exp2((m - mn) * c);
        m = mn;
        const float mc = mn * c;
        float sum = fast_exp2(fmaf(d[0], c, -mc));
#pragma unroll
        for (int r = 1; r < 16; ++r) sum += fast_exp2(fmaf(d[r], c, -mc));
        l = FIRST ? sum : l + sum;
    } else if (lo < 32 && hi > 0) {
        float tm = neg_inf();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = 8 * (r >> 2) + 4 * hf + (r & 3);
            if (key >= lo && key < hi) tm = fmaxf(tm, d[r]);
        }
        if (tm > neg_inf()) {
            const float mn = fmaxf(m, tm);
            l *= fast_exp2((m - mn) * c);
            m = mn;
            const float mc = mn * c;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = 8 * (r >> 2) + 4 * hf + (r & 3);
                if (key >= lo && key < hi) l += fast_exp2(fmaf(d[r], c, -mc));
            }
        }
    }
}

__device__ __forceinline__ void store_row_stats(uint32_t ad, float m, float l, float c, int hf)
{
    const float mm = halves_max(m);
    l = halves_sum(mm > neg_inf() ? l * fast_exp2((m - mm) * c) : 0.f);
    if (hf == 0) lds_store_f2(ad, make_float2(mm, l));
}

// Lifts the K tile of the phase into kf, then runs the MFMA steps one ahead of the arithmetic on
// their results, so that the matrix pipe works under the exponentials of the previous step. One
// tile load is issued after each of the four steps (with one row block: two per step). late() requests
// exchange data after the first step: late enough for other workgroups' stores to be visible, early
// enough to land before the barrier.
template <int NBLK, bool F8, bool BIG>
constexpr int kLoadsBehindLse = BIG ? 6 : F8 ? 1 : kSubInstr - kSubInstr / (NBLK * kNS);

template <int NBLK, int PAR, bool W, bool F8, class Late, class Advance>
__device__ __forceinline__ void stats_pass(float c, bf16x8 (&kf)[kNS][kKS], const LaneConst &lc, uint32_t koff0,
                                           uint32_t koff1, uint32_t wstats_ad, int lo0, int hi0, int lane,
                                           const KIssue &ki0, const KIssue &ki, const uint32_t (&voff)[2], const Late &late,
                                           const Advance &advance)
{
    // tile-load instructions issued after each MFMA step (8-bit keys: two in all, after the first two steps)
    constexpr int kPerStep = F8 ? 1 : kSubInstr / (NBLK * kNS);
    constexpr int kLate = F8 ? 0 : kPerStep;             // after the third and fourth step
    using MP = Map<W && NBLK == 2>;
    const int hf = lane >> 5;
    if constexpr (W) {
        // head_dim 128: the two sub-tiles are the two halves of the rows of this wave's 32 keys
        bf16x8 q0[kKS], q1[kKS];
        if (F8) lift_k8_and_q<MP::kQ1 + PAR * MP::kQTileBytes>(lc, koff0, koff1, kf, q0);
        else lift_k_and_q<MP::kQ1 + PAR * MP::kQTileBytes>(lc, koff0, koff1, kf, q0);
        lift_at<MP::kQ1 + PAR * MP::kQTileBytes + kWideHalf>(lc, q1);
        f32x16 d = logits32(kf[0], q0);
#pragma unroll
        for (int t = 0; t < kKS; ++t) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[1][t], q1[t], d, 0, 0, 0);
        if (NBLK == 1) advance();
        k_issue<NBLK == 2 ? 2 : kPerStep>(NBLK == 2 ? ki0 : ki, voff, 0);
        late();
        __builtin_amdgcn_sched_barrier(0);
        float m = neg_inf(), l = 0.f;
        if constexpr (NBLK == 2) {
            // BIG: both slots are free now, all eight loads of the next tile go out from here on
            lift_at<MP::kQ1 + PAR * MP::kQTileBytes + MP::kQBlock>(lc, q0);
            lift_at<MP::kQ1 + PAR * MP::kQTileBytes + MP::kQBlock + kWideHalf>(lc, q1);
            f32x16 d1 = logits32(kf[0], q0);
            fold_logits<true>(d, m, l, c, lo0, hi0, hf);
            store_row_stats(wstats_ad, m, l, c, hf);
            k_issue<2>(ki0, voff, 2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < kKS; ++t) d1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[1][t], q1[t], d1, 0, 0, 0);
            k_issue<2>(ki, voff, 0);
            m = neg_inf(); l = 0.f;
            fold_logits<true>(d1, m, l, c, lo0, hi0, hf);
            store_row_stats(wstats_ad + 256, m, l, c, hf);
            k_issue<2>(ki, voff, 2);
            advance();          // 15503 tokens: 119.2 us, up there 119.9; 20001: 146.3 and 146.2
        } else {
            fold_logits<true>(d, m, l, c, lo0, hi0, hf);
            store_row_stats(wstats_ad, m, l, c, hf);
            k_issue<kPerStep>(ki, voff, kPerStep);
        }
        __builtin_amdgcn_sched_barrier(0);
        return;
    }
    const int lo1 = lo0 - 32, hi1 = hi0 - 32;      // this wave's keys lo0 <= key < hi0 (of 64) are the workgroup's
    bf16x8 qf[kKS];
    if (F8) lift_k8_and_q<MP::kQ1 + PAR * MP::kQTileBytes>(lc, koff0, koff1, kf, qf);
    else lift_k_and_q<MP::kQ1 + PAR * MP::kQTileBytes>(lc, koff0, koff1, kf, qf);
    f32x16 da = logits32(kf[0], qf);
    f32x16 db = logits32(kf[1], qf);
    advance();
    float m = neg_inf(), l = 0.f;
    fold_logits<true>(da, m, l, c, lo0, hi0, hf);
    k_issue<kPerStep>(ki, voff, 0);
    late();
    __builtin_amdgcn_sched_barrier(0);
    if (NBLK == 2) {
        lift_at<MP::kQ1 + PAR * MP::kQTileBytes + MP::kQBlock>(lc, qf);
        da = logits32(kf[0], qf);
    }
    fold_logits<false>(db, m, l, c, lo1, hi1, hf);
    store_row_stats(wstats_ad, m, l, c, hf);
    k_issue<kPerStep>(ki, voff, kPerStep);
    __builtin_amdgcn_sched_barrier(0);
    if (NBLK == 2) {
        db = logits32(kf[1], qf);
        m = neg_inf(); l = 0.f;
        fold_logits<true>(da, m, l, c, lo0, hi0, hf);
        k_issue<kLate>(ki, voff, 2 * kPerStep);
        __builtin_amdgcn_sched_barrier(0);
        fold_logits<false>(db, m, l, c, lo1, hi1, hf);
        store_row_stats(wstats_ad + 256, m, l, c, hf);
        k_issue<kLate>(ki, voff, 3 * kPerStep);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The eight per-wave statistics of row `lane` of one buffer, STRIDE bytes apart, one round trip to LDS.
template <int STRIDE>
__device__ __forceinline__ void read_wave_stats(uint32_t buf, int lane, float (&m)[kFWaves], float (&l)[kFWaves])
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    const uint32_t ad = buf + 8u * (uint32_t)lane;
    f32x2 r[kFWaves];
    static_assert(kFWaves == 8, "layout of the asm block");
    __asm__ volatile(
        "ds_read_b64 %0, %8\n\t"
        "ds_read_b64 %1, %8 offset:%9\n\t"
        "ds_read_b64 %2, %8 offset:%9*2\n\t"
        "ds_read_b64 %3, %8 offset:%9*3\n\t"
        "ds_read_b64 %4, %8 offset:%9*4\n\t"
        "ds_read_b64 %5, %8 offset:%9*5\n\t"
        "ds_read_b64 %6, %8 offset:%9*6\n\t"
        "ds_read_b64 %7, %8 offset:%9*7\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
        : "v"(ad), "i"(STRIDE)
        : "memory");
#pragma unroll
    for (int i = 0; i < kFWaves; ++i) { m[i] = r[i].x; l[i] = r[i].y; }
}

// Exchange data requested with direct-to-LDS loads lands in two small staging areas, each private
// to one wave. Partials are stored workgroup-major, part[slot][workgroup][row], so that a workgroup
// publishes all its rows with one contiguous store; a duty covers kDutyRows consecutive rows, i.e.
// one 32-byte piece of every workgroup's line. A wave that combines R of them fetches 16-byte pairs of rows:
// its chunk (q * R / 2 + h) * 64 + lane of xduty holds its rows 2h and 2h+1 from workgroup lane + 64q.
template <int R>
struct DutyRows { uint64_t e[R][4]; };     // [row][workgroup lane + 64q]

template <int R>
__device__ __forceinline__ DutyRows<R> read_duty_staging(uint32_t staging, int lane)
{
    static_assert(R == 2 || R == 4, "layout of the asm blocks");
    typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
    const uint32_t ad = staging + 16u * (uint32_t)lane;
    u64x2 r[2 * R];
#define SP_READ4(I, WAIT)                                                                                     \
    __asm__ volatile("ds_read_b128 %0, %4 offset:" #I "*4096\n\tds_read_b128 %1, %4 offset:" #I "*4096+1024\n\t" \
                     "ds_read_b128 %2, %4 offset:" #I "*4096+2048\n\tds_read_b128 %3, %4 offset:" #I "*4096+3072" WAIT \
                     : "=&v"(r[4 * I]), "=&v"(r[4 * I + 1]), "=&v"(r[4 * I + 2]), "=&v"(r[4 * I + 3]) : "v"(ad) : "memory")
    SP_READ4(0, "\n\ts_waitcnt lgkmcnt(0)");
    if constexpr (R == 4) SP_READ4(1, "\n\ts_waitcnt lgkmcnt(0)");
#undef SP_READ4
    DutyRows<R> d;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int h = 0; h < R / 2; ++h) {
            d.e[2 * h][q] = r[q * (R / 2) + h].x;
            d.e[2 * h + 1][q] = r[q * (R / 2) + h].y;
        }
    return d;
}

__device__ __forceinline__ uint64_t read_lse_staging(uint32_t xlse, int lane)
{
    const uint32_t ad = xlse + 8u * (uint32_t)lane;
    uint64_t v;
    __asm__ volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(ad) : "memory");
    return v;
}

__device__ __forceinline__ float read_look_staging(uint32_t xlook, int lane)
{
    const uint32_t ad = xlook + 4u * (uint32_t)lane;
    float v;
    __asm__ volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(ad) : "memory");
    return v;
}

// Direct exchange: all rows of one exchange slot from every workgroup of the entry, `entries` 8-byte
// entries in one piece (at most 8 KB).
__device__ __forceinline__ void stage_direct(uint32_t xduty, const uint64_t *slot_base, int entries, int lane)
{
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (128 * i < entries) dma_v_device(slot_base + min(128 * i + 2 * lane, entries - 2), xduty + i * 1024);      // uniform
}

// The partials of rows row0 .. row0+R-1 of one exchange slot from every workgroup: R/2 loads for every 64 workgroups,
// of 256 or (SKIP) of those there are.
template <int R, bool SKIP>
__device__ __forceinline__ void stage_duty_rows(uint32_t staging, const uint64_t *slot_base, int rows_pad, int n_wg,
                                                int row0, int lane)
{
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int h = 0; h < R / 2; ++h)
            if (!SKIP || 64 * q < n_wg)
                dma_v_device(slot_base + (size_t)min(lane + 64 * q, n_wg - 1) * rows_pad + row0 + 2 * h, staging + (q * (R / 2) + h) * 1024);
}

// A partial is ready when it carries the parity of this use of its slot and a non-zero sum.
// Entries beyond the last workgroup do not exist, rows outside the mask are padding: both count as ready.
template <int R>
__device__ __forceinline__ bool duty_ready(const DutyRows<R> &d, uint32_t par, int lane, int n_wg, uint32_t row_mask)
{
    uint32_t ok = 1u;           // branch-free: one straight-line test of all entries
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            ok &= (uint32_t)(lane + 64 * q >= n_wg) | (((row_mask >> r) & 1u) ^ 1u) |
                  ((uint32_t)((uint32_t)(d.e[r][q] >> 63) == par) & (uint32_t)(((d.e[r][q] >> 32) & 0x7fffffffu) != 0));
    return ok != 0;
}

// A wait gave up (or met a poison entry): the workgroup stops waiting for anything and the call's
// status word is raised at once, so that every workgroup finds it before storing its scores.
__device__ __forceinline__ void raise_failure(const FusedArgs &a, int *fail)
{
    *fail = 1;
    __hip_atomic_store(a.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Direct exchange: the normaliser (negated) of row `lane` of a phase from the staged partials of the entry's
// src_n workgroups, `src` their place in memory. With 32 rows the two halves of the wave take the even and the
// odd workgroups: entry i of a lane sits 512 i bytes behind its first either way. Fixed order, so every
// workgroup finds the same bits.
template <int NB, int GB>
__device__ __forceinline__ float direct_combine(const FusedArgs &a, const uint64_t *src, int src_n, uint32_t par, uint32_t xduty,
                                                int *fail, int lane, float c, float inv_c)
{
    constexpr int kRowsPad = 32 * NB * GB, kPer = 64 / kRowsPad;      // workgroups per 512 bytes
    static_assert(kRowsPad == 32 || kRowsPad == 64, "one or two row blocks");
    const int row = lane & (kRowsPad - 1);
    const int mine = (src_n - lane / kRowsPad + kPer - 1) / kPer;     // entries of this lane
    int g, n;
    const bool valid_row = row_valid<NB>(a, row, g, n);
    constexpr int kMaxE = (sp_fused::direct_max(kRowsPad) + kPer - 1) / kPer;     // 4 or 15
    uint64_t e[16];
    const uint32_t ad = xduty + 8u * (uint32_t)lane;
    for (unsigned spins = 0;;) {
#define SP_READ4(B)                                                                                                     \
    __asm__ volatile(                                                                                                   \
        "ds_read_b64 %0, %4 offset:" #B "\n\tds_read_b64 %1, %4 offset:" #B "+512\n\t"                                 \
        "ds_read_b64 %2, %4 offset:" #B "+1024\n\tds_read_b64 %3, %4 offset:" #B "+1536\n\ts_waitcnt lgkmcnt(0)"       \
        : "=&v"(e[B / 512]), "=&v"(e[B / 512 + 1]), "=&v"(e[B / 512 + 2]), "=&v"(e[B / 512 + 3])                        \
        : "v"(ad) : "memory")
        SP_READ4(0);
        if (kMaxE > 4) { SP_READ4(2048); SP_READ4(4096); SP_READ4(6144); }
#undef SP_READ4
        uint32_t bad = 0u;
#pragma unroll
        for (int i = 0; i < kMaxE; ++i)
            bad |= (uint32_t)(i < mine) & ((uint32_t)((uint32_t)(e[i] >> 63) != par) | (uint32_t)(((e[i] >> 32) & 0x7fffffffu) == 0));
        if (!__any(valid_row && bad != 0u) && a.force_miss == 0) break;
        if (*fail != 0) break;
        if (++spins > a.spin_max) { raise_failure(a, fail); break; }
        stage_direct(xduty, src, src_n * kRowsPad, lane);        // bounded polling
        vm_wait<0>();
    }
    float m = neg_inf(), l = 0.f;
#pragma unroll
    for (int i = 0; i < kMaxE; ++i) m = i < mine ? fmaxf(m, __uint_as_float((uint32_t)e[i])) : m;
    if (kRowsPad == 32) m = halves_max(m);
#pragma unroll
    for (int i = 0; i < kMaxE; ++i) {
        const float p = __uint_as_float((uint32_t)(e[i] >> 32) & 0x7fffffffu) * fast_exp2((__uint_as_float((uint32_t)e[i]) - m) * c);
        l += i < mine ? p : 0.f;
    }
    if (kRowsPad == 32) l = halves_sum(l);
    return -(m + fast_log2(l) * inv_c);
}

// One duty wave's rows duty_row .. duty_row + R - 1 of phase pd, whose partials from workgroups src_w0 .. src_w0 + src_n - 1
// have been staged: publishes their normalisers in row lse_idx.
template <int NB, int R, bool EXTRA, bool F8>
__device__ __forceinline__ void combine_rows(const FusedArgs &a, uint32_t staging, int pd, int duty_row, int src_w0, int src_n,
                                             int lse_idx, float c_duty, int *fail, int lane)
{
    uint32_t row_mask = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int g, n;
        if (row_valid<NB>(a, duty_row + r, g, n)) row_mask |= 1u << r;
    }
    if (row_mask == 0) return;
    const uint32_t par = (uint32_t)(pd / kSlots) & 1u;
    const uint64_t *src = a.part + ((size_t)(pd % kSlots) * a.n_wg + src_w0) * a.rows_pad + duty_row;
    // fast path: the partials requested before are all there; otherwise poll (bounded)
    DutyRows<R> de = read_duty_staging<R>(staging, lane);
    bool ready = !__any(!duty_ready(de, par, lane, src_n, row_mask)) && a.force_miss == 0;
    if (!ready && *fail == 0) {
        unsigned spins = 0;
        do {
            if (++spins > a.spin_max) { raise_failure(a, fail); break; }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    de.e[r][q] = ld64(src + (size_t)min(lane + 64 * q, src_n - 1) * a.rows_pad + r);
            ready = !__any(!duty_ready(de, par, lane, src_n, row_mask)) && a.force_miss == 0;
        } while (!ready);
    }
    // per row: maximum first, then one exponential per partial (short dependency chains, fixed order)
    float mine = 0.f;       // lane r keeps the normaliser of row r of the wave's
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float pm[4], pl4[4], m = neg_inf();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool valid = lane + 64 * q < src_n;
            pm[q] = valid ? __uint_as_float((uint32_t)de.e[r][q]) : neg_inf();
            pl4[q] = valid ? __uint_as_float((uint32_t)(de.e[r][q] >> 32) & 0x7fffffffu) : 0.f;
            m = fmaxf(m, pm[q]);
        }
        m = wave_max(m);
        float l = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (!EXTRA || 64 * q < src_n) l += pl4[q] * fast_exp2((pm[q] - m) * c_duty);      // uniform
        l = wave_sum(l);
        const float v = -(m + fast_log2(l) * (F8 ? 1.0f / c_duty : a.inv_c));
        if (lane == r) mine = v;
    }
    // a duty that could not be completed (now or because the workgroup has failed before)
    // publishes poison: whoever reads it fails too instead of using a wrong normaliser
    const uint32_t tag = (ready && *fail == 0) ? (uint32_t)(pd + 1) : kPoisonTag;
    if (lane < R && ((row_mask >> lane) & 1u))
        st64(a.lse + ((size_t)(pd % kSlots) * a.n_gp + lse_idx) * a.rows_pad + duty_row + lane,
             (uint64_t)__float_as_uint(mine) | ((uint64_t)tag << 32));
}

// Uniform state that walks along with the steps.
struct Walk {
    PhaseCtr k;       // phase s + 1: next statistics pass (its K tile is being fetched)
    const char *kptr; // this wave's first key of that phase (PAIR: in the first tile)
    PhaseCtr c;       // phase s - 4: this step's probability pass
    int slot0;        // transit slot of sub-tile 0 of phase s: 2s mod 3
    uint64_t pair_off;    // PAIR: bytes from a wave's first key in the first tile to its first key in the second
    int duty_blk;     // this workgroup's block of phase s - 2, or -1
    int dfirst;       // workgroup (of those that share the duties) that combines block 0 of phase s - 2
};

// One step `s` of the software pipeline: everything between two workgroup barriers. Per wave, in
// program order (phase numbers in brackets are skipped when out of range):
//   mid     one wave publishes this workgroup's partials of phase s-1; the duty waves request the
//           partials of their duty rows of phase s-2; every wave requests its slices of Q(s+1) for
//           the next statistics pass and of Q(s-3) for the next probability pass
//   prob    probability pass of phase s-4 from ring slot s%4; loads of sub-tile 0 of K(s+1)
//   lift    wait for sub-tile 1 of K(s); duty waves: combine the duty rows of phase s-2 and publish their
//           normalisers (kDutyAtLift; otherwise at pre); normaliser wave: request of the normalisers of phase s-3
//           (kEarlyLse; otherwise after the first step of stats); lift K(s) into ring slot s%4
//   stats   statistics pass of phase s; loads of sub-tile 1 of K(s+1); scalar state of step s+1 under the first MFMA steps
//   pre     wait for the Q slices (and the exchange data); normaliser wave: seeds of the probability pass of phase s-3
//   barrier
// Vector-memory operations per wave and step, oldest first: [publish store] [4 duty loads on each of two waves, or 8 on
// one] [Q] [Q] 4 K loads (prob), [normalisers' duty stores (kDutyAtLift)], [normaliser load], 4 K loads (stats; kEarlyLse
// false: the normaliser load comes between them, PAIR: the duty loads as well; 8-bit keys: 2 and 2 K loads; BIG: none in
// prob, 8 in stats); the bracketed ones exist on some waves or in some steps only, so every wait counts only operations
// that are certainly issued behind the ones it needs.
// KIND (see there): the plain variant carries none of the others' code or registers.
template <int NB, int GB, int SLOT, int PAR, Kind KIND, bool W, bool F8, bool PAIR, bool BY_DIE>
__device__ __forceinline__ void step(const FusedArgs &args, const LayerPtrs &kp, const GroupTable &gt, int s, int n_phases, Ring &ring,
                                     Acc<NB> (&accs)[PAIR ? 2 : 1], const LaneConst &lc, Walk &wk, unsigned char *lds, uint32_t lds0,
                                     uint64_t wave_off, const int (&r_ranges)[PAIR ? 2 : 1])
{
    constexpr bool EXTRA = KIND != kPlain, RANGES = KIND == kRanges, BIG = W && NB * GB == 2;
    using MP = Map<BIG>;
    // Two blocks of query rows in layer ranges: the compiler keeps what the four unrolled steps compute from these values alive
    // across the loop, 160 to 210 scalars in vector lanes, of which a step read some 250 back, each behind wait states before
    // it can be an address. Opaque copies make every step compute them again (90 to 115 scalars; at head_dim 128 from the
    // pointers and strides on). Whole passes, in turn on one card, runs of one side up to 0.5 % apart: 20001 tokens
    // of 24 x 4 heads of 128 144.3 -> 140.1 us, 30000 201.5 -> 196.2; 16 x 8 heads of 64, 16 lookahead rows 40000 tokens 196.4 -> 190.5,
    // token-major 20000 119.2 -> 116.1, 8-bit keys 20000 127.9 -> 123.5.
    // With one block the step waits for memory, and the added instructions cost 1 %; pointers as well at head_dim 64: 1 %.
    constexpr bool kRecompute = RANGES && NB * GB == 2;
    typename std::conditional<kRecompute, FusedArgs, const FusedArgs &>::type a = args;
    if constexpr (kRecompute) {
        __asm__ volatile("" : "+s"(a.n_wg), "+s"(a.ent_w0), "+s"(a.ent_n), "+s"(a.p_idx), "+s"(a.n_gp), "+s"(a.phase0));
        if constexpr (BIG) __asm__ volatile("" : "+s"(a.part), "+s"(a.lse), "+s"(a.q), "+s"(a.k_stride_token), "+s"(a.k_stride_head),
                                                 "+s"(a.group), "+s"(a.n_q), "+s"(a.rows_pad));
    }
    // Other lane-derived values are recomputed every step instead of being kept in registers across
    // the whole loop (the opaque copy stops the compiler from hoisting them).
    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int w = workgroup_index<BY_DIE>(a.n_wg);
    // Phases this step works on; < 0 or >= n_phases: nothing to do. PAIR: step s handles tile s % 2 (= PAR) of
    // phase s / 2; publishing and duties happen in even steps, when both tiles of a phase have been seen.
    const int ps = PAIR ? s >> 1 : s;                             // statistics pass
    const int pf = PAIR ? (s + 1) >> 1 : s + 1;                   // being fetched: the next step's statistics pass
    const int pp = PAIR ? (PAR == 0 ? (s - 2) >> 1 : -1) : s - 1; // partials are published
    const int pd = PAIR ? pp : s - 2;                             // duty rows are combined
    const int pl = PAIR ? (s - 3) >> 1 : s - kLag;                // normalisers are fetched
    const int pc = PAIR ? (s - 4) >> 1 : s - 1 - kLag;            // probability pass
    const bool do_stats = ps < n_phases, do_prob = pc >= 0 && pc < n_phases;
    Acc<NB> &acc = accs[PAIR ? PAR : 0];
    const int r_range = r_ranges[PAIR ? PAR : 0];
    constexpr int kSI = F8 ? kSubInstr / 2 : kSubInstr;     // tile-load instructions per sub-tile
    constexpr uint32_t kElem = F8 ? 1u : 2u;                // bytes per key element
    const uint32_t stride_bytes = (uint32_t)a.k_stride_token * kElem;
    // 8-bit keys: the exponent's scale of a phase is c times that phase's key scale
    const float c_stats = F8 ? a.c * key_scale(a, clampi(ps, 0, n_phases - 1)) : a.c;
    const float c_pub = F8 ? a.c * key_scale(a, clampi(pp, 0, n_phases - 1)) : a.c;
    const float c_duty = F8 ? a.c * key_scale(a, clampi(pd, 0, n_phases - 1)) : a.c;
    const float c_direct = F8 ? a.c * key_scale(a, clampi(pl, 0, n_phases - 1)) : a.c;
    const float ks_prob = F8 ? key_scale(a, clampi(pc, 0, n_phases - 1)) : 1.f;
    // Duty blocks of a phase: kDutyRows consecutive rows of one entry. Block i goes to workgroup dfirst + i of the
    // launch, so that the duties of small prompts rotate over everybody (that keeps the prompts within a few
    // phases of each other: every phase of one needs a duty workgroup, which needs that phase of it); RANGES: of
    // the entry, so that entries of unequal length share nothing and none waits for another's pace. src_w0 /
    // src_n: the workgroups whose partials the block combines (its entry's), lse_idx: the entry's row of normalisers.
    constexpr int kRowsPad = 32 * NB * GB, kBlocks = kRowsPad / kDutyRows;
    const bool direct = RANGES && a.ent_n <= sp_fused::direct_max(kRowsPad);
    const int duty_w0 = RANGES ? a.ent_w0 : 0, duty_n = RANGES ? a.ent_n : a.n_wg, duty_blocks = RANGES ? kBlocks : kBlocks * a.n_gp;
    int duty_blk = wk.duty_blk;
    int src_w0 = duty_w0, src_n = duty_n, lse_idx = RANGES ? a.p_idx : 0;
    if (KIND == kExtra && a.n_gp > 1 && duty_blk >= 0) {
        lse_idx = duty_blk / kBlocks;
        duty_blk -= lse_idx * kBlocks;
        src_w0 = gt.w0[lse_idx];
        src_n = gt.w0[lse_idx + 1] - src_w0;
    }

    // When the duty rows are combined, and by how many waves. With one block of query rows a step is short (some 4500
    // cycles of work), and two trips through memory that the compute units share with the K stream take three such
    // steps: combined at the end of the step by one wave (2900 cycles for four rows), the normalisers came too late in
    // nine steps of ten, and everybody waited 3000 cycles. Two waves before the statistics pass have them out in time.
    // Whole passes: 32K tokens of head_dim 128 366 -> 332 us, 128K tokens and 8 lookahead rows 465 -> 413, sixteen
    // prompts 1119 -> 1025. With two blocks the pass itself bounds the step: 128K tokens and 16 lookahead rows
    // 494 (one wave, end), 494 (one wave, here), 492 (two, end), 495 (two, here); 8-bit keys 465, 464, 470, 469. In layer
    // ranges 8-bit keys and 16 lookahead rows are better off at the end: 65536 tokens 261 -> 257, 33000 204.5 -> 201.5
    // (all layers in one range, 100000 tokens: 403 here, 414 at the end).
    constexpr bool kTwoBlocks = NB * GB == 2;
    // When the normaliser wave requests the normalisers of phase s-3. After the first MFMA step of the statistics pass it
    // waits for them at the end of a short step (500 to 1100 cycles, everybody else for it); at the top of the step they
    // are often not out yet, and every miss is a trip of its own. Before the lift, against the former: 24 short prompts
    // 329 -> 293 us, 12007 tokens 83.7 -> 79.5, 32K tokens of head_dim 128 326.3 -> 321.5, sixteen prompts 1002 -> 997; at the
    // top 291, 79.8, 349 and 1018. With two blocks the pass is long enough: 20001 tokens 145 -> 148.
    constexpr bool kEarlyLse = !PAIR && !kTwoBlocks;
    constexpr bool kDutyAtLift = !PAIR && (!kTwoBlocks || (F8 && !RANGES));
    constexpr int kDutyWaves = kTwoBlocks && F8 ? 1 : 2, kWaveRows = kDutyRows / kDutyWaves;
    // the duty of this wave: kWaveRows rows of the block from duty_row on
    const bool duty_wave = (wave == kDutyWave || (kDutyWaves == 2 && wave == kDutyWave + 2)) && duty_blk >= 0;
    const int duty_half = kDutyWaves == 2 && wave != kDutyWave ? 1 : 0;
    const int duty_row = duty_blk * kDutyRows + duty_half * kWaveRows;
    const uint32_t staging = lds0 + MP::kXduty + duty_half * (8192 / kDutyWaves);
    int *fail = reinterpret_cast<int *>(lds + MP::kFail);
    auto request_duty = [&]() {
        if (duty_wave)
            stage_duty_rows<kWaveRows, EXTRA>(staging, a.part + ((size_t)(pd % kSlots) * a.n_wg + src_w0) * a.rows_pad, a.rows_pad,
                                              src_n, duty_row, lane);
    };
    auto combine_duty = [&]() {
        combine_rows<NB, kWaveRows, EXTRA, F8>(a, staging, pd, duty_row, src_w0, src_n, lse_idx, c_duty, fail, lane);
    };

    // ---- mid ----
    if (wave == kPubWave) {
        if (pp >= 0 && pp < n_phases) {
            // one wave combines the eight per-wave statistics of every row (lane = row), maximum first,
            // then one exponential per source, and publishes the rows with one contiguous store
            constexpr int kSets = PAIR ? 2 : 1;          // of eight per-wave statistics
            float pm[kSets][kFWaves], pl8[kSets][kFWaves];
            read_wave_stats<kMaxRowsF * 8>(lds0 + MP::kWstats + (PAIR ? (SLOT ^ 2) : 1 - PAR) * kWstatsBytes, lane, pm[0], pl8[0]);
            if constexpr (PAIR) read_wave_stats<kMaxRowsF * 8>(lds0 + MP::kWstats + ((SLOT ^ 2) + 1) % 4 * kWstatsBytes, lane, pm[1], pl8[1]);
            float m = neg_inf();
#pragma unroll
            for (int h = 0; h < kSets; ++h)
#pragma unroll
                for (int i = 0; i < kFWaves; ++i) m = fmaxf(m, pm[h][i]);
            float l = 0.f;
#pragma unroll
            for (int h = 0; h < kSets; ++h)
#pragma unroll
                for (int i = 0; i < kFWaves; ++i) l += pl8[h][i] * fast_exp2((pm[h][i] - m) * c_pub);
            if (lane < a.rows_pad) {
                const uint64_t bits = (uint64_t)__float_as_uint(m) | ((uint64_t)__float_as_uint(l) << 32) |
                                      ((uint64_t)((pp / kSlots) & 1) << 63);
                st64(a.part + ((size_t)(pp % kSlots) * a.n_wg + w) * a.rows_pad + lane, bits);
            }
        }
    } else if (!PAIR && duty_wave) {
        request_duty();
    } else if (RANGES && wave == kLseWave && direct && pl >= 0 && pl < n_phases) {
        stage_direct(lds0 + MP::kXduty, a.part + ((size_t)(pl % kSlots) * a.n_wg + a.ent_w0) * kRowsPad, a.ent_n * kRowsPad, lane);
    }
    const char *kbase = wk.kptr + (PAIR && PAR == 0 ? wk.pair_off : 0);      // PAIR: the second tile is fetched in even steps
    int slot_next = wk.slot0 + 2;         // sub-tile 0 of phase s + 1
    slot_next = slot_next >= kSubSlots ? slot_next - kSubSlots : slot_next;
    // past the last phase the loads shrink to one 16-byte piece per instruction: the count stays fixed
    const uint32_t live = pf < n_phases ? 0xffffffffu : 0u;
    const uint32_t voff[2] = {lc.koff[0] & live, lc.koff[1] & live};
    KIssue ki0;
    ki0.lds_dst = lds0 + sub_slot_off<BIG>(wave, slot_next, 0);
    ki0.base = kbase;
    ki0.step_bytes = (F8 ? 16u : 8u) * stride_bytes;
#pragma unroll
    for (int blk = 0; blk < (BIG ? 2 : 1); ++blk) if (lc.qoff[blk] >= 0) {       // padding rows of the Q tiles stay zero; the Q blocks of consecutive phases are contiguous
        const uint32_t qblock = (uint32_t)(a.group * a.n_q * kD * 2) * (W ? 2u : 1u);
        const char *q1src = reinterpret_cast<const char *>(a.q) + (uint32_t)min(pf, n_phases - 1) * qblock;
        const char *q2src = reinterpret_cast<const char *>(a.q) + (uint32_t)clampi(pl, 0, n_phases - 1) * qblock;
        const uint32_t dst = lds0 + wave * 1024 + blk * MP::kQBlock;
        dma_u<MP::kQ1 + (1 - PAR) * MP::kQTileBytes>((uint32_t)lc.qoff[blk], q1src, dst);
        dma_u<MP::kQ2 + PAR * MP::kQTileBytes>((uint32_t)lc.qoff[blk], q2src, dst);
    }

    // ---- probability pass of phase pc; sub-tile 0 of K(s+1) ----
    {
        if (do_prob) {
            const uint32_t cinit_ad = lds0 + MP::kCinit + (1 - PAR) * (kMaxRowsF * 4) + ((uint32_t)(lane & 32) << 1);
            prob_pass<NB, GB, 1 - PAR, W, F8>(ring.kf[SLOT], lc, cinit_ad, acc, ki0, voff, ks_prob);
            if (wk.c.kv == a.n_kv_heads - 1 && (a.layer_agg == SP_LAYER_MEAN || wk.c.layer == (RANGES ? a.last_layer : a.n_layers - 1)))
                close_layer<NB, W ? 1 : kNS>(acc, a.c);
        } else if (!BIG) {
            k_issue<kSI>(ki0, voff, 0);
        }
    }

    // ---- lift K(s), statistics pass of phase s; sub-tile 1 of K(s+1) ----
    // behind sub-tile 1 of K(s): at least the loads of sub-tile 0 of K(s+1); BIG: nothing that is certain
    if (BIG) vm_wait<0>(); else vm_wait<kSI>();
    // The duty's partials were requested before the loads counted here, so they have landed as well.
    if (kDutyAtLift && duty_wave) combine_duty();
    {
        KIssue ki;
        ki.lds_dst = lds0 + sub_slot_off<BIG>(wave, slot_next, 1);
        ki.base = kbase + (W ? (int64_t)(kD * kElem) : (int64_t)32 * stride_bytes);     // W: the rows' second halves
        ki.step_bytes = (F8 ? 16u : 8u) * stride_bytes;
        const uint64_t *lse_row = wave == kLseWave && !direct ? a.lse + ((size_t)(clampi(pl, 0, n_phases - 1) % kSlots) * a.n_gp + a.p_idx) * a.rows_pad : nullptr;
        const float *look_row = nullptr;
        if (EXTRA && a.look != nullptr && wave == kLseWave) look_row = a.look + (size_t)((RANGES ? a.phase0 : 0) + clampi(pl, 0, n_phases - 1)) * a.rows_pad;
        // requests after the first MFMA step: the normalisers; PAIR: also the duty rows, published at the start of
        // this very step (their normalisers are due at the next one's end)
        auto late = [&]() {
            if (!kEarlyLse) stage_exchange_rows(lds0 + MP::kXlse, lse_row, look_row, a.rows_pad, lane);
            if (PAIR && PAR == 0) request_duty();
        };
        if (kEarlyLse) stage_exchange_rows(lds0 + MP::kXlse, lse_row, look_row, a.rows_pad, lane);
        // Scalar state of the next step. A chain of some thirty scalar instructions: at the end of the step it took 400 to
        // 500 cycles of the waves that everybody waits for; here it runs while the first MFMA steps are under way (whole
        // passes: 8192 tokens 56.4 -> 55.5 us, paged 50021 tokens 205 -> 201.5; BIG: at the end of the pass).
        const int slot0 = wk.slot0;
        auto advance = [&]() {
            if (PAIR ? PAR == 0 && pf + 1 < n_phases : s + 2 < n_phases) {               // K pointer of the next phase to fetch
                wk.kptr += (uint64_t)a.k_stride_head * kElem;
                if (__builtin_expect(++wk.k.kv == a.n_kv_heads, 0)) {
                    wk.k.kv = 0;
                    ++wk.k.layer;
                    wk.kptr = reinterpret_cast<const char *>(kp.p[wk.k.layer]) + wave_off;
                }
            }
            if (!PAIR || PAR == 1) phase_advance(wk.c, pc + 1, n_phases, a.n_kv_heads);
            wk.slot0 = slot_next;
            const int pd_next = PAIR ? (PAR == 1 ? (s - 1) >> 1 : -1) : pd + 1;
            if (pd + 1 > 0 && pd + 1 < n_phases && (!PAIR || PAR == 0)) {
                wk.dfirst += duty_blocks;
                if (wk.dfirst >= duty_n) wk.dfirst -= duty_n;
            }
            const int blk = (BY_DIE ? (int)blockIdx.x : w) - duty_w0 - wk.dfirst;
            wk.duty_blk = blk < 0 ? blk + duty_n : blk;
            if (pd_next < 0 || pd_next >= n_phases || wk.duty_blk >= duty_blocks || direct) wk.duty_blk = -1;
        };
        // r_range = r_lo | r_hi << 16 (r_hi = 512 without EXTRA): this wave's share of it
        constexpr int kWaveKeys = W ? 32 : kNS * 32;
        const int lo0 = (r_range & 0xffff) - wave * kWaveKeys;
        const int hi0 = EXTRA ? (r_range >> 16) - wave * kWaveKeys : kWaveKeys;
        if (do_stats) {
            const uint32_t wstats_ad = lds0 + MP::kWstats + (PAIR ? SLOT : PAR) * kWstatsBytes + wave * (kMaxRowsF * 8) + ((uint32_t)(lane & 31) << 3);
            stats_pass<NB * GB, PAR, W, F8>(c_stats, ring.kf[SLOT], lc, sub_slot_off<BIG>(wave, slot0, 0),
                                     sub_slot_off<BIG>(wave, slot0, 1), wstats_ad, lo0, hi0, lane, ki0, ki, voff, late, advance);
        } else {
            advance();
            late();
            if (BIG) k_issue<kSI>(ki0, voff, 0);
            k_issue<kSI>(ki, voff, 0);
        }
    }

    // ---- pre-barrier: exchange data in, seeds out ----
    if ((wave == kLseWave && !(RANGES && direct && a.look == nullptr)) || (PAIR && PAR == 0 && duty_wave)) vm_wait<kEarlyLse ? kSI : kLoadsBehindLse<NB * GB, F8, BIG>>();
    else vm_wait<2 * kSI>();
    if (duty_wave) {
        if (!kDutyAtLift) combine_duty();
    } else if (wave == kLseWave) {
        float direct_v = 0.f;
        if (RANGES && direct && pl >= 0 && pl < n_phases)
            direct_v = direct_combine<NB, GB>(a, a.part + ((size_t)(pl % kSlots) * a.n_wg + a.ent_w0) * kRowsPad, a.ent_n,
                                              (uint32_t)(pl / kSlots) & 1u, lds0 + MP::kXduty, fail, lane, c_direct, F8 ? 1.0f / c_direct : a.inv_c);
        if (pl >= 0 && pl < n_phases && lane < a.rows_pad) {
            int g, n;
            float v = neg_inf();
            if (row_valid<NB>(a, lane, g, n)) {
              if (RANGES && direct) v = direct_v;
              else {
                const uint64_t *src = a.lse + ((size_t)(pl % kSlots) * a.n_gp + a.p_idx) * a.rows_pad + lane;
                uint64_t entry = read_lse_staging(lds0 + MP::kXlse, lane);
                if ((uint32_t)(entry >> 32) != (uint32_t)(pl + 1) && *fail == 0) {
                    unsigned spins = 0;
                    while ((uint32_t)(entry >> 32) != (uint32_t)(pl + 1)) {
                        if ((uint32_t)(entry >> 32) == kPoisonTag || ++spins > a.spin_max) { raise_failure(a, fail); break; }
                        entry = ld64(src);
                    }
                }
                v = __uint_as_float((uint32_t)entry);
              }
                if (EXTRA && a.look != nullptr) {
                    // the row's softmax also runs over its visible lookahead keys: log-sum-exp of the
                    // prompt's normaliser and theirs (-inf when the row sees none), in raw-logit units
                    const float lp = -v, lk = read_look_staging(lds0 + MP::kXlse + kOffXlook, lane), top = fmaxf(lp, lk);
                    v = -(top + fast_log2(fast_exp2((lp - top) * a.c) + fast_exp2((lk - top) * a.c)) * a.inv_c);
                }
            }
            const int rho = lane & 31;
            lds_store_f32(lds0 + MP::kCinit + PAR * (kMaxRowsF * 4) +
                              4u * (uint32_t)((lane & ~31) + ((rho >> 2) & 1) * 16 + 4 * (rho >> 3) + (rho & 3)), v);
        }
    }

    lds_barrier();
}

// The step of one prompt of head_dim 128, one tile a workgroup, one block of query rows, bf16 keys, where the prompt
// fills the device (see launch): the probability pass comes last. The order of `step` has the normalisers back three steps
// after their partials; with K streaming at the rate of HBM two trips through memory take about that long, and whoever
// finds them missing polls behind its own tile loads. Here the tile of a step waits in registers of its own (head_dim 64
// has none left for that: with spills 50021 tokens took 237 us against 176) until the probability pass of the phase
// four steps earlier has freed its place in the ring, and the normalisers have two thirds of a step more:
//   top     publish the partials of phase s-1; the normaliser wave requests the normalisers of phase s-4; wait for K(s)
//   lift    K(s); requests of the duty rows of phase s-2 and of Q
//   stats   statistics pass of phase s; loads of the rows' second halves of K(s+1)
//   duties  duty rows of phase s-2 combined; seeds of phase s-4, handed over through LDS without a barrier
//   prob    probability pass of phase s-4; loads of the first halves of K(s+2); K(s) into its place in the ring
//   barrier
// Loads return in order: every wait counts the loads certainly issued behind what it needs. Whole passes of 28 x 8
// phases: 50000 tokens 539 -> 521 us, 54000 578 -> 545, 60000 632 -> 594, 65536 692 -> 649, token-major 779 -> 733, paged 50000
// 620 -> 551, lookahead keys 58000 624 -> 579. At 65536 tokens a wave waits 26 % less (SQ_WAIT_ANY 4.4e8 -> 3.2e8 of 7.3e8 and 6.8e8
// SQ_WAVE_CYCLES), and 14000 loads fewer are issued, polls for normalisers that were not there.
template <int SLOT, int PAR, Kind KIND>
__device__ __forceinline__ void step_prob_last(const FusedArgs &a, const LayerPtrs &kp, int s, int n_phases, Ring &ring, Acc<1> &acc,
                                               const LaneConst &lc, Walk &wk, unsigned char *lds, uint32_t lds0, uint64_t wave_off, int r_range)
{
    constexpr bool EXTRA = KIND != kPlain;
    using MP = Map<false>;
    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, hf = lane >> 5;
    const int w = blockIdx.x;
    // phases: fetched, published, combined, of the next step's probability pass, of this one's
    const int pf = s + 1, pp = s - 1, pd = s - 2, pl = s - kLag, pc = s - 1 - kLag;
    const bool do_stats = s < n_phases, do_prob = pc >= 0 && pc < n_phases;
    constexpr int kBlocks = 32 / kDutyRows, kWaveRows = kDutyRows / 2, kHalf = kSubInstr / 2, kWaveKeys = 32;
    const uint32_t stride_bytes = (uint32_t)a.k_stride_token * 2u;
    const int duty_blk = wk.duty_blk;
    const bool duty_wave = (wave == kDutyWave || wave == kDutyWave + 2) && duty_blk >= 0;
    const int duty_half = wave != kDutyWave ? 1 : 0;
    const int duty_row = duty_blk * kDutyRows + duty_half * kWaveRows;
    const uint32_t staging = lds0 + MP::kXduty + duty_half * 4096;
    int *fail = reinterpret_cast<int *>(lds + MP::kFail);
    const PhaseCtr c_now = wk.c;

    // ---- top ----
    const bool publishes = wave == kPubWave && pp >= 0 && pp < n_phases;
    if (publishes) {
        float pm[kFWaves], pl8[kFWaves];
        read_wave_stats<kMaxRowsF * 8>(lds0 + MP::kWstats + (1 - PAR) * kWstatsBytes, lane, pm, pl8);
        float m = neg_inf(), l = 0.f;
#pragma unroll
        for (int i = 0; i < kFWaves; ++i) m = fmaxf(m, pm[i]);
#pragma unroll
        for (int i = 0; i < kFWaves; ++i) l += pl8[i] * fast_exp2((pm[i] - m) * a.c);
        if (lane < a.rows_pad)
            st64(a.part + ((size_t)(pp % kSlots) * a.n_wg + w) * a.rows_pad + lane,
                 (uint64_t)__float_as_uint(m) | ((uint64_t)__float_as_uint(l) << 32) | ((uint64_t)((pp / kSlots) & 1) << 63));
    }
    const bool seeds = wave == kLseWave && do_prob;
    if (seeds)
        stage_exchange_rows(lds0 + MP::kXlse, a.lse + (size_t)(pc % kSlots) * a.rows_pad,
                            EXTRA && a.look != nullptr ? a.look + (size_t)pc * a.rows_pad : nullptr, a.rows_pad, lane);
    // the second halves of K(s): behind them the first halves of K(s+1), and the store or the request just issued
    if (publishes || seeds) vm_wait<kSubInstr + 1>(); else vm_wait<kSubInstr>();

    // ---- lift, statistics pass ----
    const uint32_t live1 = pf < n_phases ? 0xffffffffu : 0u, live2 = s + 2 < n_phases ? 0xffffffffu : 0u;      // past the last phase 16 bytes a load
    const uint32_t voff1[2] = {lc.koff[0] & live1, lc.koff[1] & live1}, voff2[2] = {lc.koff[0] & live2, lc.koff[1] & live2};
    const int slot0 = wk.slot0;
    int slot_next = slot0 + 2;
    slot_next = slot_next >= kSubSlots ? slot_next - kSubSlots : slot_next;
    KIssue k1, k0;
    k1.lds_dst = lds0 + sub_slot_off<false>(wave, slot_next, 1);          // where the first halves of K(s) are
    k1.base = wk.kptr + kD * 2;
    k1.step_bytes = 8u * stride_bytes;
    auto requests = [&]() {
        if (duty_wave)
            stage_duty_rows<kWaveRows, EXTRA>(staging, a.part + (size_t)(pd % kSlots) * a.n_wg * a.rows_pad, a.rows_pad, a.n_wg, duty_row, lane);
        if (lc.qoff[0] >= 0) {
            const uint32_t qblock = (uint32_t)(a.group * a.n_q * kD * 4);
            const char *q1src = reinterpret_cast<const char *>(a.q) + (uint32_t)min(pf, n_phases - 1) * qblock;
            const char *q2src = reinterpret_cast<const char *>(a.q) + (uint32_t)clampi(pl, 0, n_phases - 1) * qblock;
            dma_u<MP::kQ1 + (1 - PAR) * MP::kQTileBytes>((uint32_t)lc.qoff[0], q1src, lds0 + wave * 1024);
            dma_u<MP::kQ2 + PAR * MP::kQTileBytes>((uint32_t)lc.qoff[0], q2src, lds0 + wave * 1024);
        }
    };
    auto advance = [&]() {               // scalar state of the next step, as in `step`
        if (s + 2 < n_phases) {
            wk.kptr += (uint64_t)a.k_stride_head * 2u;
            if (__builtin_expect(++wk.k.kv == a.n_kv_heads, 0)) {
                wk.k.kv = 0;
                ++wk.k.layer;
                wk.kptr = reinterpret_cast<const char *>(kp.p[wk.k.layer]) + wave_off;
            }
        }
        phase_advance(wk.c, pc + 1, n_phases, a.n_kv_heads);
        wk.slot0 = slot_next;
        if (pd + 1 > 0 && pd + 1 < n_phases) {
            wk.dfirst += kBlocks;
            if (wk.dfirst >= a.n_wg) wk.dfirst -= a.n_wg;
        }
        const int blk = w - wk.dfirst;
        wk.duty_blk = blk < 0 ? blk + a.n_wg : blk;
        if (pd + 1 < 0 || pd + 1 >= n_phases || wk.duty_blk >= kBlocks) wk.duty_blk = -1;
    };
    bf16x8 kf[kNS][kKS];
    if (do_stats) {
        const int lo = (r_range & 0xffff) - wave * kWaveKeys, hi = EXTRA ? (r_range >> 16) - wave * kWaveKeys : kWaveKeys;
        bf16x8 q0[kKS], q1[kKS];
        lift_k_and_q_wide<MP::kQ1 + PAR * MP::kQTileBytes>(lc, sub_slot_off<false>(wave, slot0, 0), sub_slot_off<false>(wave, slot0, 1), kf, q0, q1);
        requests();
        f32x16 d = logits32(kf[0], q0);
#pragma unroll
        for (int t = 0; t < kKS; ++t) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[1][t], q1[t], d, 0, 0, 0);
        advance();
        k_issue<kHalf>(k1, voff1, 0);
        __builtin_amdgcn_sched_barrier(0);
        float m = neg_inf(), l = 0.f;
        fold_logits<true>(d, m, l, a.c, lo, hi, hf);
        store_row_stats(lds0 + MP::kWstats + PAR * kWstatsBytes + wave * (kMaxRowsF * 8) + ((uint32_t)(lane & 31) << 3), m, l, a.c, hf);
        k_issue<kHalf>(k1, voff1, kHalf);
    } else {
        requests();
        advance();
        k_issue<kSubInstr>(k1, voff1, 0);
#pragma unroll
        for (int i = 0; i < kNS; ++i)
#pragma unroll
            for (int t = 0; t < kKS; ++t) kf[i][t] = ring.kf[SLOT][i][t];
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- duties, seeds: their data was requested before the loads of the statistics pass ----
    if (duty_wave) {
        vm_wait<kSubInstr>();
        combine_rows<1, kWaveRows, EXTRA, false>(a, staging, pd, duty_row, 0, a.n_wg, 0, a.c, fail, lane);
    } else if (seeds) {
        vm_wait<kSubInstr>();
        if (lane < a.rows_pad) {
            int g, n;
            float v = neg_inf();
            if (row_valid<1>(a, lane, g, n)) {
                const uint64_t *src = a.lse + (size_t)(pc % kSlots) * a.rows_pad + lane;
                uint64_t entry = read_lse_staging(lds0 + MP::kXlse, lane);
                if ((uint32_t)(entry >> 32) != (uint32_t)(pc + 1) && *fail == 0) {
                    unsigned spins = 0;
                    while ((uint32_t)(entry >> 32) != (uint32_t)(pc + 1)) {
                        if ((uint32_t)(entry >> 32) == kPoisonTag || ++spins > a.spin_max) { raise_failure(a, fail); break; }
                        entry = ld64(src);
                    }
                }
                v = __uint_as_float((uint32_t)entry);
                if (EXTRA && a.look != nullptr) {
                    const float lp = -v, lk = read_look_staging(lds0 + MP::kXlse + kOffXlook, lane), top = fmaxf(lp, lk);
                    v = -(top + fast_log2(fast_exp2((lp - top) * a.c) + fast_exp2((lk - top) * a.c)) * a.inv_c);
                }
            }
            lds_store_f32(lds0 + MP::kCinit + 4u * (uint32_t)(((lane >> 2) & 1) * 16 + 4 * (lane >> 3) + (lane & 3)), v);
        }
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        lds_store_u32(lds0 + MP::kSeeded, (uint32_t)(pc + 1));
    }

    // ---- probability pass ----
    k0.lds_dst = lds0 + sub_slot_off<false>(wave, slot0, 1);              // where the second halves of K(s) were
    k0.base = wk.kptr;
    k0.step_bytes = k1.step_bytes;
    if (do_prob) {
        while (lds_load_u32(lds0 + MP::kSeeded) != (uint32_t)(pc + 1)) __builtin_amdgcn_s_sleep(1);      // set in this step, whatever the waits came to
        bf16x8 q0[kKS], q1[kKS];
        f32x16 d;
        lift_q_wide_and_seed<MP::kQ2 + (1 - PAR) * MP::kQTileBytes>(lc, lds0 + MP::kCinit + ((uint32_t)(lane & 32) << 1), q0, q1, d);
#pragma unroll
        for (int t = 0; t < kKS; ++t) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q0[t], ring.kf[SLOT][0][t], d, 0, 0, 0);
        k_issue<kHalf>(k0, voff2, 0);
#pragma unroll
        for (int t = 0; t < kKS; ++t) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q1[t], ring.kf[SLOT][1][t], d, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc.mx[0][0][e] = max3(max3(d[e], d[4 + e], d[8 + e]), d[12 + e], acc.mx[0][0][e]);
        k_issue<kHalf>(k0, voff2, kHalf);
        if (c_now.kv == a.n_kv_heads - 1 && (a.layer_agg == SP_LAYER_MEAN || c_now.layer == a.n_layers - 1)) close_layer<1, 1>(acc, a.c);
    } else {
        k_issue<kSubInstr>(k0, voff2, 0);
    }
#pragma unroll
    for (int i = 0; i < kNS; ++i)
#pragma unroll
        for (int t = 0; t < kKS; ++t) ring.kf[SLOT][i][t] = kf[i][t];
    vm_wait<2 * kSubInstr>();            // Q
    lds_barrier();
}

// The step of two tiles a workgroup, one block of query rows, head_dim 64, bf16 keys. Half as many phases are in flight
// as with one tile, and the exchange's two trips through memory, each behind what the compute units have requested of K,
// take some 16000 cycles: with the order of `step` odd steps waited 5500 of their 9600 cycles for the normalisers. Here
// the probability pass comes last, so that they have most of a step more, and what is exchanged is requested and
// consumed while no tile loads are in flight (loads return in order, and a load issued behind a burst of
// tile loads takes as long as they do):
//   top     even steps: the normaliser wave requests the normalisers of phase P-2; wait for K(s); even steps: publish both
//           tiles' partials of phase P-1, seeds of phase P-2; odd steps: combine the duty rows of phase P-1; requests of Q
//   stats   statistics pass of K(s) from the transit ring; loads of K(s+1), the first sub-tile right after the lift
//   prob    probability pass of this tile of phase P-2 from ring slot s%4, once its seeds are there (even steps wait
//           for the normaliser wave, without a barrier)
//   lift    K(s) into ring slot s%4; even steps: request of the duty rows
//   barrier
// Whole passes of 256K tokens: 924 us before, 980 with the loads and requests where `step` has them, 875 with the duty
// rows requested last, 833 with the tile loads behind the consumption, 802 with the normalisers requested at the top.
// Duty rows requested at the top as well: 898; behind the statistics: 985; combined in even steps: 840 .. 894.
template <int SLOT, int PAR, Kind KIND>
__device__ __forceinline__ void step_late(const FusedArgs &a, const LayerPtrs &kp, int s, int n_phases, Ring &ring, Acc<1> (&accs)[2],
                                          const LaneConst &lc, Walk &wk, unsigned char *lds, uint32_t lds0, uint64_t wave_off,
                                          const int (&r_ranges)[2])
{
    constexpr bool EXTRA = KIND != kPlain;
    using MP = LateMap;
    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int w = workgroup_index<KIND == kPlain>(a.n_wg);
    const int ps = s >> 1, pf = (s + 1) >> 1, pd = (s - 2) >> 1, pc = (s - 4) >> 1;       // pd: published, combined; pc: probability pass
    const uint32_t stride_bytes = (uint32_t)a.k_stride_token * 2u;
    int *fail = reinterpret_cast<int *>(lds + MP::kFail);
    constexpr int kBlocks = MP::kRows / kDutyRows, kWaveRows = kDutyRows / 2;
    const int duty_blk = wk.duty_blk;
    const bool duty_wave = (wave == kDutyWave || wave == kDutyWave + 2) && duty_blk >= 0;
    const int duty_half = wave != kDutyWave ? 1 : 0;
    const PhaseCtr c_now = wk.c;
    // scalar state of the next step, as in `step`
    auto advance = [&]() {
        if (PAR == 0 && pf + 1 < n_phases) {               // K pointer of the next phase to fetch
            wk.kptr += (uint64_t)a.k_stride_head * 2u;
            if (__builtin_expect(++wk.k.kv == a.n_kv_heads, 0)) {
                wk.k.kv = 0;
                ++wk.k.layer;
                wk.kptr = reinterpret_cast<const char *>(kp.p[wk.k.layer]) + wave_off;
            }
        }
        if (PAR == 1) {
            phase_advance(wk.c, pc + 1, n_phases, a.n_kv_heads);
            if (pd + 1 > 0 && pd + 1 < n_phases) {
                wk.dfirst += kBlocks;
                if (wk.dfirst >= a.n_wg) wk.dfirst -= a.n_wg;
            }
            const int blk = (int)blockIdx.x - wk.dfirst;
            wk.duty_blk = blk < 0 ? blk + a.n_wg : blk;
            if (pd + 1 < 0 || pd + 1 >= n_phases || wk.duty_blk >= kBlocks) wk.duty_blk = -1;
        }
    };

    // ---- top ----
    const bool publishes = PAR == 0 && wave == kPubWave && pd >= 0 && pd < n_phases;
    uint64_t partial = 0;
    if (publishes) {
        // the first tile's statistics in one half of the wave, the second's in the other
        float pm[kFWaves], pl8[kFWaves];
        const uint32_t buf = lds0 + MP::kWstats + (lane < 32 ? (1 - (SLOT >> 1)) * kFWaves * MP::kWaveStats : 2 * kFWaves * MP::kWaveStats - MP::kWaveStats);
        read_wave_stats<MP::kWaveStats>(buf, lane, pm, pl8);
        float m = neg_inf(), l = 0.f;
#pragma unroll
        for (int i = 0; i < kFWaves; ++i) m = fmaxf(m, pm[i]);
        m = halves_max(m);
#pragma unroll
        for (int i = 0; i < kFWaves; ++i) l += pl8[i] * fast_exp2((pm[i] - m) * a.c);
        l = halves_sum(l);
        partial = (uint64_t)__float_as_uint(m) | ((uint64_t)__float_as_uint(l) << 32) | ((uint64_t)((pd / kSlots) & 1) << 63);
    }
    const char *kbase = wk.kptr + (PAR == 0 ? wk.pair_off : 0);      // the second tile is fetched in even steps
    const uint32_t live = pf < n_phases ? 0xffffffffu : 0u;          // past the last phase one 16-byte piece per instruction
    const uint32_t voff[2] = {lc.koff[0] & live, lc.koff[1] & live};
    KIssue k0, k1;
    k0.lds_dst = lds0 + MP::slot(wave, 1 - PAR, 0);
    k0.base = kbase;
    k0.step_bytes = 8u * stride_bytes;
    k1.lds_dst = lds0 + MP::slot(wave, 1 - PAR, 1);
    k1.base = kbase + (int64_t)32 * stride_bytes;
    k1.step_bytes = k0.step_bytes;
    const bool do_prob = pc >= 0 && pc < n_phases;
    const bool consumes = PAR == 0 ? wave == kLseWave && do_prob : duty_wave;
    if (PAR == 0 && consumes) {
        if (EXTRA && a.look != nullptr && lane < MP::kRows / 4) dma_v_device(a.look + (size_t)pc * MP::kRows + 4 * lane, lds0 + MP::kXlook);
        if (lane < MP::kRows / 2) dma_v_device(a.lse + (size_t)(pc % kSlots) * MP::kRows + 2 * lane, lds0 + MP::kXlse);
    }
    vm_wait<0>();                    // K(s), and what was requested behind it
    if (publishes && lane < MP::kRows)      // only now: the wait would be for this store as well
        st64(a.part + ((size_t)(pd % kSlots) * a.n_wg + w) * MP::kRows + lane, partial);
    if (PAR == 0 && consumes) {
        if (lane < MP::kRows) {
            int g, n;
            float v = neg_inf();
            if (row_valid<1>(a, lane, g, n)) {
                const uint64_t *src = a.lse + (size_t)(pc % kSlots) * MP::kRows + lane;
                uint64_t entry = read_lse_staging(lds0 + MP::kXlse, lane);
                if ((uint32_t)(entry >> 32) != (uint32_t)(pc + 1) && *fail == 0) {
                    unsigned spins = 0;
                    while ((uint32_t)(entry >> 32) != (uint32_t)(pc + 1)) {
                        if ((uint32_t)(entry >> 32) == kPoisonTag || ++spins > a.spin_max) { raise_failure(a, fail); break; }
                        entry = ld64(src);
                    }
                }
                v = __uint_as_float((uint32_t)entry);
                if (EXTRA && a.look != nullptr) {
                    const float lp = -v, lk = read_look_staging(lds0 + MP::kXlook, lane), top = fmaxf(lp, lk);
                    v = -(top + fast_log2(fast_exp2((lp - top) * a.c) + fast_exp2((lk - top) * a.c)) * a.inv_c);
                }
            }
            lds_store_f32(lds0 + MP::kCinit + 4u * (uint32_t)(((lane >> 2) & 1) * 16 + 4 * (lane >> 3) + (lane & 3)), v);
        }
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        lds_store_u32(lds0 + MP::kSeeded, (uint32_t)(pc + 1));
    }
    if (PAR == 1 && consumes)
        combine_rows<1, kWaveRows, false, false>(a, lds0 + MP::kXduty + duty_half * 4096, pd, duty_blk * kDutyRows + duty_half * kWaveRows, 0,
                                                 a.n_wg, 0, a.c, fail, lane);
    if (lc.qoff[0] >= 0) {
        const uint32_t qblock = (uint32_t)(a.group * a.n_q * kD * 2);
        const char *q1src = reinterpret_cast<const char *>(a.q) + (uint32_t)min(pf, n_phases - 1) * qblock;
        const char *q2src = reinterpret_cast<const char *>(a.q) + (uint32_t)clampi((s - 3) >> 1, 0, n_phases - 1) * qblock;
        dma_u<MP::kQ1 + (1 - PAR) * MP::kQTileBytes>((uint32_t)lc.qoff[0], q1src, lds0 + wave * 1024);
        dma_u<MP::kQ2 + (1 - PAR) * MP::kQTileBytes>((uint32_t)lc.qoff[0], q2src, lds0 + wave * 1024);
    }

    // ---- statistics pass ----
    if (ps < n_phases) {
        const int r_range = r_ranges[PAR];
        const int lo0 = (r_range & 0xffff) - wave * (kNS * 32), hi0 = EXTRA ? (r_range >> 16) - wave * (kNS * 32) : kNS * 32;
        const int hf = lane >> 5;
        const uint32_t wstats_ad = lds0 + MP::kWstats + ((PAR ? 2 : SLOT >> 1) * kFWaves + wave) * MP::kWaveStats + ((uint32_t)(lane & 31) << 3);
        bf16x8 kf[kKS], qf[kKS];
        float m = neg_inf(), l = 0.f;
        lift_sub_and_q<MP::kQ1 + PAR * MP::kQTileBytes>(lc, MP::slot(wave, PAR, 0), kf, qf);
        k_issue<kSubInstr>(k0, voff, 0);
        const f32x16 da = logits32(kf, qf);
        lift_sub(lc, MP::slot(wave, PAR, 1), kf);
        const f32x16 db = logits32(kf, qf);
        advance();
        fold_logits<true>(da, m, l, a.c, lo0, hi0, hf);
        k_issue<2>(k1, voff, 0);
        __builtin_amdgcn_sched_barrier(0);
        fold_logits<false>(db, m, l, a.c, lo0 - 32, hi0 - 32, hf);
        store_row_stats(wstats_ad, m, l, a.c, hf);
        k_issue<2>(k1, voff, 2);
    } else {
        advance();
        k_issue<kSubInstr>(k0, voff, 0);
        k_issue<kSubInstr>(k1, voff, 0);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- probability pass ----
    if (do_prob) {
        if (PAR == 0)       // set in this step, whatever the waits came to
            while (lds_load_u32(lds0 + MP::kSeeded) != (uint32_t)(pc + 1)) __builtin_amdgcn_s_sleep(1);
        Acc<1> &acc = accs[PAR];
        bf16x8 qf[kKS];
        f32x16 seed;
        lift_q_and_seed<MP::kQ2 + PAR * MP::kQTileBytes>(lc, lds0 + MP::kCinit + ((uint32_t)(lane & 32) << 1), qf, seed);
#pragma unroll
        for (int s2 = 0; s2 < kNS; ++s2) {
            f32x16 d = seed;
#pragma unroll
            for (int t = 0; t < kKS; ++t) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[t], ring.kf[SLOT][s2][t], d, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc.mx[s2][0][e] = max3(max3(d[e], d[4 + e], d[8 + e]), d[12 + e], acc.mx[s2][0][e]);
        }
        if (c_now.kv == a.n_kv_heads - 1 && (a.layer_agg == SP_LAYER_MEAN || c_now.layer == a.n_layers - 1)) close_layer<1, kNS>(acc, a.c);
        __builtin_amdgcn_sched_barrier(0);
    }
    lift_tile(lc, MP::slot(wave, PAR, 0), ring.kf[SLOT]);
    if (PAR == 0 && duty_wave)
        stage_duty_rows<kWaveRows, false>(lds0 + MP::kXduty + duty_half * 4096, a.part + (size_t)(pd % kSlots) * a.n_wg * MP::kRows, MP::kRows,
                                          a.n_wg, duty_blk * kDutyRows + duty_half * kWaveRows, lane);

    // Q(s+1): K(s+1) was requested behind it, and on the duty waves their rows
    if (PAR == 0 && duty_wave) vm_wait<2 * kSubInstr + 4>();
    else vm_wait<2 * kSubInstr>();
    lds_barrier();
}

// Model shapes. The kernel takes every dimension at run time (AnyModel); an instantiation for a
// fixed model overwrites its copy of the arguments with the model's constants, which the compiler
// then folds: fewer live scalars (the generic kernel spills some sixty of them) and no address
// arithmetic on run-time dimensions. Prompt length, workgroup count, kv-head stride and pointers
// stay run-time values; the workgroup count is folded too in the instantiations for a prompt that
// fills the device (256 workgroups: 128K tokens), where every exchange slot is in use and the bounds
// checks on workgroup indices fall away.
struct AnyModel {
    static constexpr bool kFixed = false;
    static constexpr int kLayers = 0, kQHeads = 0, kKvHeads = 0, kNq = 0, kWorkgroups = 0;
};
// The 16-layer, 32-query / 8-kv-head, head_dim 64 draft shape (a Llama-3.2-1B-class draft; Table 1 of
// the paper) with NQ lookahead rows, token-contiguous keys and scale 1/8.
template <int NQ, int WORKGROUPS>
struct Draft16x32x8 {
    static constexpr bool kFixed = true;
    static constexpr int kLayers = 16, kQHeads = 32, kKvHeads = 8, kNq = NQ, kWorkgroups = WORKGROUPS;   // 0: run-time count
};
constexpr float kScaleEighthLog2e = 0.125f * 1.44269504088896340736f;    // scale 1/sqrt(64) times log2(e), as the host computes it

template <class M>
__device__ __forceinline__ void fold_model_constants(FusedArgs &a)
{
    if (M::kFixed) {
        a.n_layers = M::kLayers;
        a.n_q_heads = M::kQHeads;
        a.n_kv_heads = M::kKvHeads;
        a.group = M::kQHeads / M::kKvHeads;
        a.n_q = M::kNq;
        a.n_nblk = (M::kNq + 7) / 8;
        a.n_gblk = (M::kQHeads / M::kKvHeads + 3) / 4;
        a.rows_pad = a.n_nblk * a.n_gblk * 32;
        a.k_stride_token = kD;
        a.c = kScaleEighthLog2e;
        a.inv_c = 1.0f / kScaleEighthLog2e;
        if (M::kWorkgroups > 0) a.n_wg = M::kWorkgroups;
    }
}

// W: head_dim 128. A workgroup owns 256 keys, a wave 32; the two "sub-tiles" of a wave are the two
// 64-element halves of its keys' rows (same transit ring, same fragment ring: kf[s][t] holds MFMA
// k-step 4s + t), Q tiles hold 32 rows as two half-tiles, and a logit is one chain of eight MFMA steps.
// F8: 8-bit keys (head_dim 64): rows of 64 codes, sub-tiles of 2 KB fetched by two instructions of 16 rows,
// widened to bf16 at the lift; every phase has its own key scale.
// PAIR: prompts of up to two tiles per compute unit (head_dim 64: 256K tokens, 128: 128K). A workgroup owns two
// tiles and a phase takes two steps, one a tile, on the same fragment ring: two phases instead of four are in
// flight, so the normalisers have to come back within four steps less the two of their own phase. In `step` duties are
// therefore combined in the step in which the partials are published; step_late gives them the next one and takes the
// probability pass last. One read of K instead of the general path's two.
// PROB_LAST: see step_prob_last.
template <int NB, int GB, Kind KIND, class M, bool W = false, bool F8 = false, bool PAIR = false, bool PROB_LAST = false>
__global__ __launch_bounds__(kFThreads, 2) void sp_fused_kernel(FusedArgs a, LayerPtrs kp, GroupTable gt)
{
    static_assert(!W || (NB == 1 && !M::kFixed), "head_dim 128: one block of lookahead rows");
    constexpr bool BIG = W && NB * GB == 2;
    static_assert(!BIG || !F8, "head_dim 128, two blocks of query rows: bf16 keys");
    static_assert(!PROB_LAST || (W && NB * GB == 1 && KIND != kRanges && !F8 && !PAIR), "head_dim 128, one block of query rows, whole prompts");
    constexpr bool LATE = PAIR && !W && !F8 && NB * GB == 1, kByDie = tiles_by_die<NB * GB, KIND, W, F8, M>;
    using MP = typename std::conditional<LATE, LateMap, Map<BIG>>::type;
    static_assert(!F8 || KIND != kExtra, "8-bit keys: contiguous keys of one prompt");
    static_assert(!PAIR || KIND != kRanges, "pairs of tiles: whole prompts");
    constexpr bool EXTRA = KIND != kPlain, RANGES = KIND == kRanges;
    constexpr int kSI = F8 ? kSubInstr / 2 : kSubInstr;
    constexpr uint32_t kElem = F8 ? 1u : 2u;
    constexpr int kTile = W ? kFTile / 2 : kFTile;            // keys per workgroup
    constexpr int kWaveKeys = kTile / kFWaves;
    constexpr int kHeadDim = W ? 2 * kD : kD;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[MP::kBytes];
    fold_model_constants<M>(a);

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, hf = lane >> 5, col = lane & 31;
    const int w = workgroup_index<kByDie>(a.n_wg);
    int n_phases = a.n_layers * a.n_kv_heads;
    // Contiguous keys: the last workgroup's tile is shifted back so that it ends with the prompt (the
    // caller guarantees L >= 512): every workgroup loads 512 real keys; rows below r_lo belong to the
    // previous workgroup. Paged keys: pages are allocated whole and hold a multiple of 512 keys, so the
    // last tile stays where it is and rows from r_hi on (allocated, never written) are ignored.
    // Several entries in one launch (a prompt's layer range each; prompts are packed back to back): entry p owns workgroups gt.w0[p] .. gt.w0[p+1]-1 and is a call of its
    // own in everything below: tile positions count from its prompt's first key, its queries and layers
    // are its own, partials are combined among its workgroups only and its normalisers have their own row.
    const bool paged = EXTRA && a.block_table != nullptr;
    int64_t p_start = 0, p_len = a.L;
    int wl = w;                               // this workgroup's index within its entry
    int layer0 = 0, slice = 0;
    if (EXTRA && gt.n > 0) {
        int p = 0;
        while (p + 1 < gt.n && w >= gt.w0[p + 1]) ++p;
        p_start = gt.start[p];
        p_len = gt.len[p];
        wl = w - gt.w0[p];
        a.q += (size_t)gt.prompt[p] * ((size_t)a.n_layers * a.n_q_heads * a.n_q * kHeadDim);
        a.p_idx = p;
        a.n_gp = gt.n;
        if (RANGES) {
            layer0 = gt.layer0[p];
            n_phases = gt.layers[p] * a.n_kv_heads;
            slice = gt.slice[p];
            a.q += (size_t)layer0 * ((size_t)a.n_q_heads * a.n_q * kHeadDim);
            a.ent_w0 = gt.w0[p];
            a.ent_n = gt.w0[p + 1] - a.ent_w0;
            a.phase0 = layer0 * a.n_kv_heads;
            if (F8) a.kscale += a.phase0;
            // a range of the maximum over layers stays open: its rows' maxima are the result
            a.last_layer = a.split_out != nullptr ? -1 : layer0 + gt.layers[p] - 1;
        }
    } else {
        a.p_idx = 0;
        a.n_gp = 1;
    }
    constexpr int kOwn = PAIR ? 2 * kTile : kTile;            // keys of this workgroup
    int64_t j0l = (paged || (int64_t)(wl + 1) * kOwn <= p_len) ? (int64_t)wl * kOwn : p_len - kOwn;
    // A prompt of a batch that is shorter than a tile: the tile starts with it and the keys of the prompts behind
    // it are ignored; at the end of the packed keys (L of them, at least one tile) it ends with them instead.
    if (RANGES && p_len < kTile && !paged) j0l = p_start + kTile <= a.L ? 0 : a.L - kTile - p_start;
    const int64_t j0 = p_start + j0l;         // first key of the tile in the layer's key array
    // this workgroup's keys r_lo <= key < r_hi of each tile; PAIR, paged: a second tile without keys is the first
    // one again (its own may have no page)
    int r_ranges[PAIR ? 2 : 1];
    const int own_lo = (int)((int64_t)wl * kOwn - j0l), own_hi = (int)(p_len - j0l < kOwn ? p_len - j0l : kOwn);
    const bool second = PAIR && own_hi > kTile;
#pragma unroll
    for (int t = 0; t < (PAIR ? 2 : 1); ++t)
        r_ranges[t] = clampi(own_lo - t * kTile, 0, kTile) | (clampi(own_hi - t * kTile, 0, kTile) << 16);
    const uint32_t lds0 = lds_addr(lds);
    const uint32_t stride_bytes = (uint32_t)a.k_stride_token * kElem;

    // zero the Q tiles (their padding rows are never loaded), seed the accumulator seeds with -inf
    {
        u32x4 *z = reinterpret_cast<u32x4 *>(lds + MP::kQ1);
        const u32x4 zero = {0u, 0u, 0u, 0u};
        for (int i = tid; i < 4 * MP::kQTileBytes / 16; i += kFThreads) z[i] = zero;
        float *ci = reinterpret_cast<float *>(lds + MP::kCinit);
        if (tid < (LATE ? 32 : 2 * kMaxRowsF)) ci[tid] = neg_inf();
        if (tid < (LATE || PROB_LAST ? 2 : 1)) reinterpret_cast<int *>(lds + MP::kFail)[tid] = 0;       // and kSeeded
    }
    __syncthreads();

    LaneConst lc;
#pragma unroll
    for (int t = 0; t < kKS; ++t) lc.ld[t] = lds0 + 16u * (uint32_t)lds_slot<kD>(col, 2 * t + hf);
    // 8-bit sub-tile: row r at 64 r, its four 16-byte chunks XOR-swizzled by (r >> 2) & 3 (eight-byte reads of
    // 64 lanes then spread over all banks twice, which is what 512 bytes need anyway)
#pragma unroll
    for (int t = 0; t < kKS; ++t) lc.ld8[t] = lds0 + 64u * (uint32_t)col + ((((uint32_t)t ^ ((uint32_t)col >> 2)) & 3u) << 4) + 8u * (uint32_t)hf;
    {
        uint32_t rowpart = (uint32_t)(lane >> 3) * stride_bytes;
        const uint32_t swz = (uint32_t)(lane >> 4);               // (row >> 1) & 7 of row = lane >> 3 in an even instruction
        lc.koff[0] = rowpart + (((uint32_t)(lane & 7) ^ swz) << 4);
        lc.koff[1] = rowpart + (((uint32_t)(lane & 7) ^ (swz | 4u)) << 4);
        if (F8) {       // an instruction moves 16 rows of 64 bytes: row lane >> 2, chunk (lane & 3) ^ ((row >> 2) & 3)
            rowpart = (uint32_t)(lane >> 2) * stride_bytes;
            lc.koff[0] = lc.koff[1] = rowpart + ((((uint32_t)lane & 3u) ^ (((uint32_t)lane >> 4) & 3u)) << 4);
        }
        // a wave's slice of a Q tile: 8 rows (W: of one half-tile, waves 4..7 take the second halves)
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            const int row = (BIG ? 32 * blk : 0) + (W ? (wave & 3) : wave) * 8 + (lane >> 3);
            int g, n;
            lc.qoff[blk] = -1;
            if ((BIG || blk == 0) && row < a.rows_pad && row_valid<NB>(a, row, g, n))
                lc.qoff[blk] = ((g * a.n_q + n) * kHeadDim + (W ? (wave >> 2) * kD : 0) + (((lane & 7) ^ ((row >> 1) & 7)) << 3)) * 2;
        }
    }

    Ring ring;
    Acc<NB> accs[PAIR ? 2 : 1];
#pragma unroll
    for (auto &acc : accs)
#pragma unroll
    for (int s = 0; s < kNS; ++s) {
        acc.total[s] = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc.mx[s][b][e] = neg_inf();
    }

    // byte offset of this wave's first key within a (layer, kv head): uniform, kept in scalar registers
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    auto key_offset = [&](int64_t j) -> uint64_t {
        uint64_t off = (uint64_t)(j + wave_u * kWaveKeys) * (uint64_t)a.k_stride_token * kElem;
        if (paged) {
            const int64_t page = j / a.page_tokens;
            off = ((uint64_t)a.block_table[page] * (uint64_t)a.page_stride +
                   (uint64_t)(j - page * a.page_tokens + wave_u * kWaveKeys) * (uint64_t)a.k_stride_token) * 2u;
        }
        return (uint64_t)uniform32((uint32_t)off) | ((uint64_t)uniform32((uint32_t)(off >> 32)) << 32);
    };
    const uint64_t wave_off = key_offset(j0);

    // prologue: this wave's slice of Q(0) and both sub-tiles of K(0); everything lands before step 0
#pragma unroll
    for (int blk = 0; blk < (BIG ? 2 : 1); ++blk)
        if (lc.qoff[blk] >= 0) dma_u<MP::kQ1>((uint32_t)lc.qoff[blk], a.q, lds0 + wave_u * 1024 + blk * MP::kQBlock);
#pragma unroll
    for (int s2 = 0; s2 < kNS; ++s2) {
        KIssue ki;
        ki.lds_dst = lds0 + (LATE ? LateMap::slot(wave_u, 0, s2) : sub_slot_off<BIG>(wave_u, 0, s2));
        ki.base = reinterpret_cast<const char *>(kp.p[layer0]) + wave_off + (W ? (uint64_t)(s2 * kD * kElem) : (uint64_t)(s2 * 32) * stride_bytes);
        ki.step_bytes = (F8 ? 16u : 8u) * stride_bytes;
        k_issue<kSI>(ki, lc.koff, 0);
    }
    vm_wait<0>();
    lds_barrier();

    Walk wk;
    wk.k = phase_at(PAIR ? 0 : 1, n_phases, a.n_kv_heads);
    wk.pair_off = second ? key_offset(j0 + kTile) - wave_off : 0;
    wk.k.layer += layer0;
    wk.kptr = reinterpret_cast<const char *>(kp.p[wk.k.layer]) + (uint64_t)wk.k.kv * (uint64_t)a.k_stride_head * kElem + wave_off;
    wk.c = phase_at(0, n_phases, a.n_kv_heads);
    wk.c.layer += layer0;
    if constexpr (PROB_LAST) {           // the first halves of K(1)
        KIssue ki;
        ki.lds_dst = lds0 + sub_slot_off<BIG>(wave_u, 2, 0);
        ki.base = wk.kptr;
        ki.step_bytes = 8u * stride_bytes;
        k_issue<kSubInstr>(ki, lc.koff, 0);
    }
    wk.slot0 = 0;
    wk.dfirst = 0;
    wk.duty_blk = -1;
    if (!EXTRA) { a.p_idx = 0; a.n_gp = 1; }

    // The body is unrolled four times so that the fragment ring slot (s % 4) and the buffer parity
    // (s % 2) are compile-time; the trip count is rounded up, surplus steps do no work but keep the
    // instruction stream uniform. The last probability pass (phase n_phases - 1) runs in step n_phases + 3.
    const int n_steps = ((PAIR ? 2 * n_phases : n_phases) + kLag + 1 + 3) / 4 * 4;
    if constexpr (LATE) {
        for (int s0 = 0; s0 < n_steps; s0 += 4) {
            step_late<0, 0, KIND>(a, kp, s0 + 0, n_phases, ring, accs, lc, wk, lds, lds0, wave_off, r_ranges);
            step_late<1, 1, KIND>(a, kp, s0 + 1, n_phases, ring, accs, lc, wk, lds, lds0, wave_off, r_ranges);
            step_late<2, 0, KIND>(a, kp, s0 + 2, n_phases, ring, accs, lc, wk, lds, lds0, wave_off, r_ranges);
            step_late<3, 1, KIND>(a, kp, s0 + 3, n_phases, ring, accs, lc, wk, lds, lds0, wave_off, r_ranges);
        }
    } else if constexpr (PROB_LAST) {
        for (int s0 = 0; s0 < n_steps; s0 += 4) {
            step_prob_last<0, 0, KIND>(a, kp, s0 + 0, n_phases, ring, accs[0], lc, wk, lds, lds0, wave_off, r_ranges[0]);
            step_prob_last<1, 1, KIND>(a, kp, s0 + 1, n_phases, ring, accs[0], lc, wk, lds, lds0, wave_off, r_ranges[0]);
            step_prob_last<2, 0, KIND>(a, kp, s0 + 2, n_phases, ring, accs[0], lc, wk, lds, lds0, wave_off, r_ranges[0]);
            step_prob_last<3, 1, KIND>(a, kp, s0 + 3, n_phases, ring, accs[0], lc, wk, lds, lds0, wave_off, r_ranges[0]);
        }
    } else {
        for (int s0 = 0; s0 < n_steps; s0 += 4) {
            step<NB, GB, 0, 0, KIND, W, F8, PAIR, kByDie>(a, kp, gt, s0 + 0, n_phases, ring, accs, lc, wk, lds, lds0, wave_off, r_ranges);
            step<NB, GB, 1, 1, KIND, W, F8, PAIR, kByDie>(a, kp, gt, s0 + 1, n_phases, ring, accs, lc, wk, lds, lds0, wave_off, r_ranges);
            step<NB, GB, 2, 0, KIND, W, F8, PAIR, kByDie>(a, kp, gt, s0 + 2, n_phases, ring, accs, lc, wk, lds, lds0, wave_off, r_ranges);
            step<NB, GB, 3, 1, KIND, W, F8, PAIR, kByDie>(a, kp, gt, s0 + 3, n_phases, ring, accs, lc, wk, lds, lds0, wave_off, r_ranges);
        }
    }
    vm_wait<0>();               // no direct-to-LDS load may outlive the workgroup
    lds_barrier();
    if (RANGES && a.split_out != nullptr) {
        // one layer range of several: MEAN leaves the range's sum per key, MAX the probability of every
        // lookahead row's maximum (exp is monotone: the maximum over ranges can be taken after it). The
        // reduce launch looks at the status word.
#pragma unroll
        for (int s = 0; s < kWaveKeys / 32; ++s) {
            const int key = wave * kWaveKeys + s * 32 + col;
            const bool mine = key >= (r_ranges[0] & 0xffff) && key < (r_ranges[0] >> 16);
            const Acc<NB> &acc = accs[0];
            if (a.layer_agg == SP_LAYER_MEAN) {
                const float both = acc.total[s] + __shfl_xor(acc.total[s], 32);
                if (hf == 0 && mine) a.split_out[slice * a.split_stride + j0 + key] = both;
            } else {
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (mine) a.split_out[((int64_t)slice * (8 * NB) + 8 * b + 4 * hf + e) * a.split_stride + j0 + key] = fast_exp2(acc.mx[s][b][e] * a.c);
            }
        }
        return;
    }
    // the call has failed if any workgroup raised the status word; this workgroup's own failures are in it
    const bool failed = __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
#pragma unroll
    for (int t = 0; t < (PAIR ? 2 : 1); ++t)
#pragma unroll
    for (int s = 0; s < kWaveKeys / 32; ++s) {
        const float both = accs[t].total[s] + __shfl_xor(accs[t].total[s], 32);
        const int key = wave * kWaveKeys + s * 32 + col;
        if (hf == 0 && key >= (r_ranges[t] & 0xffff) && key < (r_ranges[t] >> 16)) a.scores[j0 + t * kTile + key] = failed ? __uint_as_float(0x7fc00000u) : both * a.out_scale;   // quiet NaN marks a failed call
    }
}

// Clears the exchange area and the status word: a zero sum marks a partial as not yet written and
// phase numbers start at 1, so zero normaliser entries are never taken as ready.
__global__ void sp_fused_clear_kernel(uint64_t *p, size_t n, uint32_t *err)
{
    if (err != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *err = 0u;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0;
}

// Test hook (see sp_debug_fused_giveup): polls before a wait gives up, and the launches whose duty waves
// treat their partials as never arriving (0: none, 1: all, 2 + b: those that hold prompt b) or, with -1, whose
// last workgroup is left out. (A miss of one prompt's partials in the kernel would have to know the duty's prompt
// there: up to 29 more scalar spills, 28 layers of six prompts at head_dim 128, 73K tokens, 1177 us instead of 1167.)
std::atomic<uint32_t> g_spin_max{1u << 20};     // about a second
std::atomic<int32_t> g_force_miss{0};

}  // namespace

namespace sp_fused {

void set_giveup(uint32_t spin_max, int32_t force_miss)
{
    g_spin_max.store(spin_max, std::memory_order_relaxed);
    g_force_miss.store(force_miss, std::memory_order_relaxed);
}

bool fits_one_per_cu()
{
    int n1 = 0, n2 = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n1, sp_fused_kernel<1, 1, kRanges, AnyModel>, kFThreads, 0) != hipSuccess) return false;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n2, sp_fused_kernel<2, 1, kRanges, AnyModel>, kFThreads, 0) != hipSuccess) return false;
    return n1 >= 1 && n2 >= 1;
}

sp_status launch(FusedArgs a, const LayerPtrs &kp, const GroupTable *group, bool shared, Clear clear, void *ws,
                 uint32_t *status_word, hipStream_t st)
{
    GroupTable gt;
    std::memset(&gt, 0, sizeof gt);
    if (group) gt = *group;
    // The kernel places workgroup w of a prompt at key w * tile: the grid must be exactly the prompts' tiles
    // (a surplus workgroup of a paged prompt would look up a page the table does not have).
    const int64_t tile = a.tile_keys;
    const int base_tile = a.head_dim == 2 * kD ? kFTile / 2 : kFTile;
    const bool pair = tile == 2 * base_tile;
    if ((a.head_dim != kD && a.head_dim != 2 * kD) || (tile != base_tile && !pair))
        return sp::fail(SP_ERR_INVALID_ARG, "fused score kernel: head_dim %d with %d keys per workgroup", a.head_dim, a.tile_keys);
    if (gt.n == 0) {
        if (a.L < tile || sp::ceil_div(a.L, tile) != a.n_wg)
            return sp::fail(SP_ERR_INVALID_ARG, "fused score kernel: %d workgroups for %lld keys", a.n_wg, (long long)a.L);
    } else {
        if (gt.n < 0 || gt.n > sp_fused::kMaxGroup || gt.w0[0] != 0 || gt.w0[gt.n] != a.n_wg)
            return sp::fail(SP_ERR_INVALID_ARG, "fused score kernel: group table does not cover %d workgroups", a.n_wg);
        for (int i = 0; i < gt.n; ++i) {
            if (gt.len[i] < 1 || (gt.len[i] < tile && (a.L < tile || a.block_table)) || gt.start[i] < 0 ||
                gt.start[i] + gt.len[i] > a.L || sp::ceil_div(gt.len[i], tile) != gt.w0[i + 1] - gt.w0[i])
                return sp::fail(SP_ERR_INVALID_ARG, "fused score kernel: entry %d of the group: %d workgroups for %lld keys", i,
                                gt.w0[i + 1] - gt.w0[i], (long long)gt.len[i]);
            if (shared && (gt.len[i] < tile || gt.layers[i] != a.n_layers))
                return sp::fail(SP_ERR_INVALID_ARG, "fused score kernel: entry %d of the group cannot share duties", i);
            if (gt.layer0[i] < 0 || gt.layers[i] < 1 || gt.layer0[i] + gt.layers[i] > a.n_layers)
                return sp::fail(SP_ERR_INVALID_ARG, "fused score kernel: entry %d of the group: layers %d + %d of %d", i, gt.layer0[i],
                                gt.layers[i], a.n_layers);
        }
        if (shared && gt.n * (a.rows_pad / kDutyRows) > a.n_wg)
            return sp::fail(SP_ERR_INVALID_ARG, "fused score kernel: %d entries of %d rows share %d workgroups", gt.n, a.rows_pad, a.n_wg);
    }
    uint64_t *base = static_cast<uint64_t *>(ws);
    a.part = base;
    a.lse = base + exchange_words(a.rows_pad, a.n_wg, 0);
    a.err = status_word;
    a.spin_max = std::min(a.spin_max, g_spin_max.load(std::memory_order_relaxed));
    const int32_t miss = g_force_miss.load(std::memory_order_relaxed);
    a.force_miss = miss == 1 || (miss == 2 && gt.n == 0);
    for (int i = 0; i < gt.n && miss >= 2; ++i)
        a.force_miss |= gt.prompt[i] == miss - 2;
    if (clear != Clear::kDone) {
        const size_t n_clear = exchange_words(a.rows_pad, a.n_wg, gt.n > 0 ? gt.n : 1);
        hipLaunchKernelGGL(sp_fused_clear_kernel, dim3((unsigned)((n_clear + 255) / 256 > 1024 ? 1024 : (n_clear + 255) / 256)),
                           dim3(256), 0, st, base, n_clear, clear == Clear::kAll ? status_word : (uint32_t *)nullptr);
        SP_HIP_CHECK(hipGetLastError());
    }
    // Every workgroup must be resident for the exchange to make progress: one workgroup fits per
    // compute unit (LDS), so the grid may not exceed the number of compute units. All waits in the
    // kernel are bounded; should residency fail (the device shared with other work), the call ends
    // with NaN scores and the status word set instead of hanging.
    const bool ranges = gt.n > 0 && !shared;
    const bool extra = a.look != nullptr || a.block_table != nullptr || gt.n > 0;
    const dim3 grid(a.n_wg - (miss == -1 && a.n_wg > 1)), block(kFThreads);
#define SP_FUSED(...) hipLaunchKernelGGL((sp_fused_kernel<__VA_ARGS__>), grid, block, 0, st, a, kp, gt)
    // one variant for whole prompts with extras, one for tables of entries, one for plain prompts
#define SP_FUSED_KINDS(NB, GB, ...)                             \
    do {                                                        \
        if (ranges) SP_FUSED(NB, GB, kRanges, __VA_ARGS__);     \
        else if (extra) SP_FUSED(NB, GB, kExtra, __VA_ARGS__);  \
        else SP_FUSED(NB, GB, kPlain, __VA_ARGS__);             \
    } while (0)
    using Draft16 = Draft16x32x8<16, 0>;
    using Draft8 = Draft16x32x8<8, 0>;
    const int blocks = a.n_nblk * 10 + a.n_gblk;
    if (a.head_dim == 2 * kD ? blocks != 11 && (blocks != 12 || a.kscale) : blocks != 11 && blocks != 12 && blocks != 21)
        return sp::fail(SP_ERR_UNSUPPORTED, "fused score kernel, head_dim %d: %d x %d row blocks", a.head_dim, a.n_nblk, a.n_gblk);
    if (a.kscale != nullptr && extra && !(ranges && a.look == nullptr && a.block_table == nullptr))
        return sp::fail(SP_ERR_UNSUPPORTED, "fused score kernel, 8-bit keys: one prompt, contiguous keys only");
    // The fixed-model instantiations apply when every folded constant equals the call's value. Against the generic ones
    // (whole passes): 128K tokens 4 %; in layer ranges 8192 tokens 60.8 -> 58.8 us, paged 50021 tokens 241.4 -> 233.1; two
    // tiles a workgroup, 256K tokens 946.8 -> 932.3, with 16 lookahead rows 150000 tokens 784 -> 764 (262144 1005 / 1003), 8-bit
    // keys 160000 827 -> 805.
    const bool draft = a.head_dim == kD && a.n_layers == 16 && a.n_q_heads == 32 && a.n_kv_heads == 8 && a.k_stride_token == kD &&
                       a.c == kScaleEighthLog2e && a.inv_c == 1.0f / kScaleEighthLog2e;
    if (pair) {
        if (gt.n > 0)
            return sp::fail(SP_ERR_UNSUPPORTED, "fused score kernel, two tiles a workgroup: one prompt");
        if (a.kscale != nullptr) {
            if (a.head_dim == 2 * kD) SP_FUSED(1, 1, kPlain, AnyModel, true, true, true);
            else if (blocks == 12) SP_FUSED(1, 2, kPlain, AnyModel, false, true, true);
            else if (blocks == 21 && draft && a.n_q == 16) SP_FUSED(2, 1, kPlain, Draft16, false, true, true);
            else if (blocks == 21) SP_FUSED(2, 1, kPlain, AnyModel, false, true, true);
            else SP_FUSED(1, 1, kPlain, AnyModel, false, true, true);
        } else
        if (a.head_dim == 2 * kD && blocks == 12 && extra) SP_FUSED(1, 2, kExtra, AnyModel, true, false, true);
        else if (a.head_dim == 2 * kD && blocks == 12) SP_FUSED(1, 2, kPlain, AnyModel, true, false, true);
        else if (a.head_dim == 2 * kD && extra) SP_FUSED(1, 1, kExtra, AnyModel, true, false, true);
        else if (a.head_dim == 2 * kD) SP_FUSED(1, 1, kPlain, AnyModel, true, false, true);
        else if (blocks == 12 && extra) SP_FUSED(1, 2, kExtra, AnyModel, false, false, true);
        else if (blocks == 12) SP_FUSED(1, 2, kPlain, AnyModel, false, false, true);
        else if (blocks == 21 && extra) SP_FUSED(2, 1, kExtra, AnyModel, false, false, true);
        else if (blocks == 21 && draft && a.n_q == 16) SP_FUSED(2, 1, kPlain, Draft16, false, false, true);
        else if (blocks == 21) SP_FUSED(2, 1, kPlain, AnyModel, false, false, true);
        else if (extra) SP_FUSED(1, 1, kExtra, AnyModel, false, false, true);
        else if (draft && a.n_q == 8) SP_FUSED(1, 1, kPlain, Draft8, false, false, true);
        else SP_FUSED(1, 1, kPlain, AnyModel, false, false, true);
    } else if (a.kscale != nullptr) {       // 8-bit keys
        if (ranges && a.head_dim == 2 * kD) SP_FUSED(1, 1, kRanges, AnyModel, true, true);
        else if (ranges && blocks == 21) SP_FUSED(2, 1, kRanges, AnyModel, false, true);
        else if (ranges && blocks == 12) SP_FUSED(1, 2, kRanges, AnyModel, false, true);
        else if (ranges) SP_FUSED(1, 1, kRanges, AnyModel, false, true);
        else if (a.head_dim == 2 * kD) SP_FUSED(1, 1, kPlain, AnyModel, true, true);
        else if (draft && a.n_q == 16 && a.n_wg == 256) SP_FUSED(2, 1, kPlain, Draft16x32x8<16, 256>, false, true);
        else if (draft && a.n_q == 16) SP_FUSED(2, 1, kPlain, Draft16, false, true);
        else if (draft && a.n_q == 8) SP_FUSED(1, 1, kPlain, Draft8, false, true);
        else if (blocks == 21) SP_FUSED(2, 1, kPlain, AnyModel, false, true);
        else if (blocks == 12) SP_FUSED(1, 2, kPlain, AnyModel, false, true);
        else SP_FUSED(1, 1, kPlain, AnyModel, false, true);
    } else if (a.head_dim == 2 * kD && blocks == 12) SP_FUSED_KINDS(1, 2, AnyModel, true);
    // One prompt of head_dim 128 on most of the device. `step` / step_prob_last, 28 x 8 phases: 34000 tokens (133 workgroups) 461 /
    // 463 us, 45000 (176) 492 / 494, 48000 (188) 507 / 510, 50000 (196) 539 / 521, 65536 (256) 692 / 649. Batches stay: 234
    // workgroups of six prompts 558 / 568.
    else if (a.head_dim == 2 * kD && gt.n == 0 && a.n_wg >= 192 && extra) SP_FUSED(1, 1, kExtra, AnyModel, true, false, false, true);
    else if (a.head_dim == 2 * kD && gt.n == 0 && a.n_wg >= 192) SP_FUSED(1, 1, kPlain, AnyModel, true, false, false, true);
    else if (a.head_dim == 2 * kD) SP_FUSED_KINDS(1, 1, AnyModel, true);
    else if (draft && !extra && a.n_q == 16 && a.n_wg == 256) SP_FUSED(2, 1, kPlain, Draft16x32x8<16, 256>);
    else if (draft && !extra && a.n_q == 8 && a.n_wg == 256) SP_FUSED(1, 1, kPlain, Draft16x32x8<8, 256>);
    else if (draft && a.n_q == 16) SP_FUSED_KINDS(2, 1, Draft16);
    else if (draft && a.n_q == 8) SP_FUSED_KINDS(1, 1, Draft8);
    else if (blocks == 21) SP_FUSED_KINDS(2, 1, AnyModel);
    else if (blocks == 12) SP_FUSED_KINDS(1, 2, AnyModel);
    else SP_FUSED_KINDS(1, 1, AnyModel);
#undef SP_FUSED_KINDS
#undef SP_FUSED
    SP_HIP_CHECK(hipGetLastError());
    return SP_OK;
}

}  // namespace sp_fused
