// MFMA main loop shared by the four contractions of the fused LM-head + cross-entropy path
// (logit tile of the chunked forward algorithm, its recomputation in the backward
// algorithm, and the two gradient products dH = G W and dW = G^T H).
//
// One workgroup = 512 threads = 8 wavefronts (256 = 4 for TileDuo) arranged WM x WN, computing a BM x BN fp32 tile
// C[m, n] = sum_k A(m, k) * B(n, k) with v_mfma_f32_32x32x16_bf16.  Each wavefront owns
// TM x TN blocks of 32 x 32 (16 accumulator registers per block and lane).
//
// Operands arrive in one of two global layouts:
//   K-major : element (free f, k) at base[f * ld + k]   (k contiguous)  -- H and W in the
//             logit products, G in dH
//   K-slow  : element (k, free f) at base[k * ld + f]   (f contiguous)  -- W in dH, G and H
//             in dW; fragments are then fetched with the LDS transpose read
//             (ds_read_b64_tr_b16), so no transposed copy of any tensor is ever made.
//
// The gradient chunk G lies in panels (PanelTile) and is read in either way.
//
// K is walked in slices of 64 (32 for TileDuo).  A slice of both operands is brought straight from global
// memory into LDS (global_load_lds_dwordx4: 16 B per lane, a wavefront fills 1 KB of
// consecutive LDS), double buffered: the loads of slice t+1 are issued before the MFMAs of
// slice t.  Because the LDS side of such a load is fixed (lane * 16 B), the
// bank-conflict-avoiding swizzle is applied on the global side: the lane that fills
// physical 16-byte chunk p of a row fetches logical chunk p ^ f(row).
//   K-major stage: [R rows][128 B]; f(row) = (row >> 1) & 7, so that the 16 lanes served
//                  per LDS cycle by a ds_read_b128 (16 rows, same logical chunk) cover all
//                  64 banks.
//   K-slow  stage: [64 k-rows][2R B]; logical chunk c is stored at c ^ ((k & 3) << 2), so
//                  that the 4 k-rows x 64 B touched per cycle by a transpose read fall in
//                  different quarters of the bank space.
// Rows / columns past the edge of a matrix are clamped to the last valid one (their
// products are discarded or meet zero padding in the other operand), so the loop has a
// single code path for full and ragged tiles.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace cce {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int kBK = 64;           // K slice
constexpr int kThreads = 512;     // 8 wavefronts

#define CCE_LDS __attribute__((address_space(3)))
#define CCE_GLOBAL __attribute__((address_space(1)))

// KG_ > 1 splits the k16 steps of every slice between KG_ groups of wavefronts that all work
// on the same output positions (their accumulators are summed once, after the loop): a
// 256 x 128 tile then keeps the 128 x 64 wavefront tile of the 256 x 256 one, i.e. 0.75
// instead of 1 LDS fragment read per MFMA and 8 instead of 4 independent accumulators.
template <int WM_, int WN_, int TM_, int TN_, int STAGES_, int KG_ = 1, int BK_ = 64>
struct TileCfg {
    static constexpr int NW = WM_ * WN_ * KG_;                  // wavefronts per workgroup
    static constexpr int kThreads = NW * 64;
    static constexpr int BK = BK_;                              // K slice
    static_assert(NW == 8 || NW == 4, "eight or four wavefronts per workgroup");
    static_assert(BK_ == 64 || BK_ == 32, "128 or 64 bytes per row of a K-major stage");
    static_assert(KG_ == 1 || KG_ == 2, "one or two K groups");
    static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, STAGES = STAGES_, KG = KG_;
    static constexpr int kSteps = BK_ / 16 / KG_;                      // k16 steps per slice and wavefront
    static constexpr int BM = WM_ * TM_ * 32;
    static constexpr int BN = WN_ * TN_ * 32;
    static constexpr int kAStage = BM * BK * 2;
    static constexpr int kBStage = BN * BK * 2;
    static constexpr int kStage = kAStage + kBStage;
    static constexpr int kLdsBytes = STAGES_ * kStage;
    static constexpr int kLoadsPerSlice = (BM + BN) * BK / 8 / kThreads;   // 16-byte loads per thread
    static_assert(kLdsBytes <= 160 * 1024, "stages must fit the 160 KB LDS");
};
typedef TileCfg<2, 4, 4, 2, 2> TileBig;      // 256 x 256, wave tile 128 x 64, 2 x 64 KB stages
typedef TileCfg<2, 2, 4, 2, 3, 2> TileNarrow; // 256 x 128, wave tile 128 x 64, 2 K groups, 3 x 48 KB stages
// 128 x 128, wave tile 64 x 32, 4 x 32 KB stages: for products of so few larger tiles that many
// compute units would have none (three slices ahead: a slice lasts a third of a 256 x 256 one and no
// other workgroup of the unit covers its latency).  322 x 1856 x 1015, 8 large tiles: forward and
// backward 102.8 -> 58.2 us; 256 x 64 x 1000: 38.9 -> 30.2.
typedef TileCfg<2, 4, 2, 1, 4> TileSmall;
// 256 x 128 by four wavefronts, K slices of 32 in 3 x 24 KB stages: two workgroups to a compute unit, each with half
// of its LDS and registers, so that one's first slice and epilogue run beside the other's main loop.  For contractions
// of many items (see contraction_kind).  Rounds of 256 items, dW: 8 slices of 64 15.3 -> 13.7 us, 32 37.6 -> 33.2,
// 96 94.2 -> 90.3; alone on its unit an item is slower than TileNarrow's (252 items of 48 slices: 51 -> 60 us).
// Not for the logit products: their K-major operands would come in 64-byte rows (forward at D = 896 1.9 -> 2.3 ms).
typedef TileCfg<2, 2, 4, 2, 3, 1, 32> TileDuo;


// Wavefront coordinates inside the workgroup: K group, then position along M and N.
template <class Cfg> __device__ __forceinline__ int wave_kg() { return (threadIdx.x >> 6) / (Cfg::WM * Cfg::WN); }
template <class Cfg> __device__ __forceinline__ int wave_m() { return ((threadIdx.x >> 6) % (Cfg::WM * Cfg::WN)) / Cfg::WN; }
template <class Cfg> __device__ __forceinline__ int wave_n() { return ((threadIdx.x >> 6) % (Cfg::WM * Cfg::WN)) % Cfg::WN; }

__device__ __forceinline__ void load16_to_lds(const char* g, CCE_LDS char* lds_wave_base) {
    // global_load_lds_dwordx4: lane i's 16 bytes land at lds_wave_base + 16 * i
    // (lds_wave_base is wave-uniform and travels in M0).
    // Written as inline assembly on purpose: when the compiler sees this load it makes
    // every later LDS read it cannot disambiguate (the transpose reads in particular) wait
    // for ALL outstanding global->LDS loads (s_waitcnt vmcnt(0)), which serialises the
    // prefetch of the next K slice with the current one.  The main loop orders these
    // loads against the LDS reads itself (barrier_pending_loads).
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds_wave_base);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(g), "s"(m0) : "memory", "m0");
}

// The same load with the address split as the instruction takes it: a wave-uniform 64-bit base in
// scalar registers plus a 32-bit per-lane byte offset; m0_value is the wave-uniform LDS destination.
// With the base advanced per K slice on the scalar unit and the per-lane offsets constant, a load
// costs no vector-ALU instruction at all (the full-address form above needs an offset add, a
// 64-bit add and, for the LDS destination, an add and a readfirstlane per load).
__device__ __forceinline__ void load16_to_lds_sbase(const char* uniform_base, uint32_t lane_offset, uint32_t m0_value) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(lane_offset), "s"(uniform_base), "s"(m0_value) : "memory", "m0");
}

// 4 bytes per lane.
__device__ __forceinline__ void load4_to_lds_sbase(const void* uniform_base, uint32_t lane_offset, uint32_t m0_value) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :: "v"(lane_offset), "s"(uniform_base), "s"(m0_value) : "memory", "m0");
}

// One operand (R = 128 or 256 free indices) of one workgroup tile: global -> LDS.
// MAP (K-slow only): the k-rows are reached through a table in LDS with an entry for every k of whole slices, 1: byte
// offsets of matrix rows (kmap), 2: row numbers in 16 bits (kmap16).  A load then costs one LDS read and one add or
// multiply-add.  (With bounds, rows that map to none and the multiplication in the loop: contractions of 8400 of 12000 rows x
// 1024 x 40000 1.79 ms, now 1.71; of 12288 of 16384 x 2048 x 50000 5.27, now 5.17.)
template <bool KMAJOR, int R, int MAP = 0, int NW = 8, int BK = 64>
struct OperandTile {
    static_assert(!(KMAJOR && MAP), "only a K-slow operand carries a k-row map");
    static constexpr int NL = R * BK / 512 / NW;   // 16-byte loads per thread and K slice
    const char* base;       // matrix base address
    uint32_t ld_bytes;      // leading dimension in bytes
    uint32_t off[NL];       // K-major: clamped row offset + swizzled chunk; K-slow: clamped column offset
    int krow[NL];           // K-slow: k-row inside a slice handled by load i
    uint32_t slow_off[NL];  // K-slow: krow[i] * row pitch + off[i] (full slices are loaded from a uniform base)
    int k_last;             // K-slow: last valid k (rows beyond are clamped to it)
    const CCE_LDS uint32_t* kmap;
    const CCE_LDS uint16_t* kmap16;

    // free0: first free index of the tile; free_n: number of valid free indices in the matrix
    // (a multiple of 8, at least 8, for a K-slow operand); k_n: valid K extent.
    // row_map (K-major operands only): free index f is fetched from matrix row row_map[f] (row 0
    // where the map holds -1; such rows are padding whose products the caller discards).
    __device__ __forceinline__ void init(const void* p, int64_t ld, int free0, int free_n, int k_n,
                                         const int32_t* row_map = nullptr) {
        base = (const char*)p;
        ld_bytes = (uint32_t)(ld * 2);
        k_last = k_n - 1;
        kmap = nullptr;
        kmap16 = nullptr;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (KMAJOR) {
            constexpr int CPR = BK / 8, RPL = 64 / CPR;      // 16-byte chunks per row, rows per wavefront load
            const int r0 = RPL * wave + lane / CPR;          // row inside the tile of load 0
            const int sw = BK == 64 ? (r0 >> 1) & 7 : (r0 >> 2) & 3;
            const int c = (lane % CPR) ^ sw;
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                int row = free0 + RPL * NW * i + r0;
                row = row < free_n ? row : free_n - 1;
                if (row_map) {
                    const int mapped = row_map[row];
                    row = mapped < 0 ? 0 : mapped;
                }
                off[i] = (uint32_t)row * ld_bytes + (uint32_t)c * 16u;
                krow[i] = 0;
                slow_off[i] = 0;
            }
        } else {
            constexpr int CR = R / 8;            // 16-byte chunks per k-row
            constexpr int RPL = 512 / R;         // k-rows per wavefront load
            const int sub = lane / CR;           // k-row inside the wavefront load
            const int k3 = (RPL * wave + sub) & 3;
            const int c = (lane % CR) ^ (k3 << 2);
            int col = free0 + c * 8;
            col = col <= free_n - 8 ? col : free_n - 8;
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                off[i] = (uint32_t)col * 2u;
                krow[i] = (wave + NW * i) * RPL + sub;
                slow_off[i] = (uint32_t)krow[i] * ld_bytes + off[i];
            }
        }
    }

    // K slices [0, full_slices()) lie entirely inside the operand's valid K extent (every slice of a
    // K-major operand does: its extent is padded to the slice).
    __device__ __forceinline__ int full_slices() const { return KMAJOR || MAP ? 0x7fffffff : (k_last + 1) / BK; }

    // Issue this thread's loads of the K slice starting at k0 into `stage` (LDS).  FULL (compile time):
    // the caller knows that the slice is one of full_slices().
    template <bool FULL = false>
    __device__ __forceinline__ void issue(CCE_LDS char* stage, int k0) const {
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const uint32_t lds0 = (uint32_t)(uintptr_t)stage + (uint32_t)wave * 1024u;     // wave-uniform
        if (KMAJOR) {
            // uniform base = matrix base + this slice's K offset; lane offsets are those of init()
            const char* sb = base + (size_t)((uint32_t)k0 * 2u);
#pragma unroll
            for (int i = 0; i < NL; ++i) load16_to_lds_sbase(sb, off[i], lds0 + (uint32_t)i * (NW * 1024u));
            return;
        }
        if constexpr (MAP == 1) {
#pragma unroll
            for (int i = 0; i < NL; ++i) load16_to_lds_sbase(base, kmap[k0 + krow[i]] + off[i], lds0 + (uint32_t)i * (NW * 1024u));
            return;
        }
        if constexpr (MAP == 2) {
#pragma unroll
            for (int i = 0; i < NL; ++i)
                load16_to_lds_sbase(base, __umul24((uint32_t)kmap16[k0 + krow[i]], ld_bytes) + off[i], lds0 + (uint32_t)i * (NW * 1024u));
            return;
        }
        if (FULL || k0 + BK - 1 <= k_last) {
            // a full slice of a K-slow operand: uniform base = row k0, lane offset = its k-row inside
            // the slice times the row pitch plus its column offset
            const char* sb = base + (size_t)k0 * ld_bytes;
#pragma unroll
            for (int i = 0; i < NL; ++i) load16_to_lds_sbase(sb, slow_off[i], lds0 + (uint32_t)i * (NW * 1024u));
            return;
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            int k = k0 + krow[i];                                 // a ragged slice of a K-slow operand
            k = k < k_last ? k : k_last;
            load16_to_lds(base + (size_t)((uint32_t)k * ld_bytes + off[i]), stage + (wave + NW * i) * 1024);
        }
    }
};

// The gradient chunk G as the A operand of the contractions.  It is kept in panels as wide as the K slice of the
// tiles that read it, element (row, col) at (col / BK) * panel + row * BK + col % BK: a K slice of the dH product
// (K = columns) is then one contiguous run, and one of the dW product (K = rows) whole 128-byte lines.  (With rows
// as long as the chunk, K slices of 32 took half of every line: 96 slices of a dH item 104 us, in panels 92; K slices of
// 64 from panels of 32: the 128 x 128 dW items of 16 x 16 tiles at D = 512 34 -> 50 us.)  Rows and columns are padded to
// whole tiles: nothing is clamped.
template <bool KMAJOR, int R, int NW, int BK>
struct PanelTile {
    static constexpr int NL = R * BK / 512 / NW;
    static constexpr int CPP = BK / 8;          // 16-byte chunks across a panel
    const char* base;
    uint32_t panel;         // bytes from one panel to the next
    uint32_t off[NL];
    __device__ __forceinline__ void init(const uint16_t* chunk, uint32_t panel_elements, int free0, int k0) {
        panel = panel_elements * 2u;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (KMAJOR) {
            base = (const char*)chunk + (size_t)(k0 / BK) * panel;
            constexpr int RPL = 64 / CPP;
            const int r0 = RPL * wave + lane / CPP;
            const int sw = BK == 64 ? (r0 >> 1) & 7 : (r0 >> 2) & 3;
            const int c = (lane % CPP) ^ sw;
#pragma unroll
            for (int i = 0; i < NL; ++i) off[i] = (uint32_t)(free0 + RPL * NW * i + r0) * (BK * 2u) + (uint32_t)c * 16u;
        } else {
            base = (const char*)chunk + (size_t)k0 * (BK * 2u);
            constexpr int CR = R / 8, RPL = 512 / R;
            const int sub = lane / CR, k3 = (RPL * wave + sub) & 3;
            const int c = (lane % CR) ^ (k3 << 2);
#pragma unroll
            for (int i = 0; i < NL; ++i)
                off[i] = (uint32_t)((wave + NW * i) * RPL + sub) * (BK * 2u) + (uint32_t)(free0 / BK + c / CPP) * panel + (uint32_t)(c % CPP) * 16u;
        }
    }
    __device__ __forceinline__ int full_slices() const { return 0x7fffffff; }
    template <bool FULL = false>
    __device__ __forceinline__ void issue(CCE_LDS char* stage, int k0) const {
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const uint32_t lds0 = (uint32_t)(uintptr_t)stage + (uint32_t)wave * 1024u;
        const char* sb = base + (KMAJOR ? (size_t)(k0 / BK) * panel : (size_t)k0 * (BK * 2u));
#pragma unroll
        for (int i = 0; i < NL; ++i) load16_to_lds_sbase(sb, off[i], lds0 + (uint32_t)i * (NW * 1024u));
    }
};

// Per-lane LDS byte offsets of the MFMA fragments of one operand, relative to its stage.
// A wavefront of K group kg reads the k16 steps kk = j * KG + kg, j = 0 .. STEPS - 1.
template <bool KMAJOR, int R, int NB, int STEPS, int KG, int BK = 64>
struct FragAddr {
    uint32_t a[KMAJOR ? STEPS : NB];   // K-major: one per step j; K-slow: one per 32-wide block

    // tile_off: first row/column of this wave's sub-tile inside the R-wide tile.
    __device__ __forceinline__ void init(int tile_off, int kg) {
        const int l = threadIdx.x & 63;
        if (KMAJOR) {
            const int row = tile_off + (l & 31);
            const int s = BK == 64 ? ((l & 31) >> 1) & 7 : ((l & 31) >> 2) & 3;
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                const int kk = j * KG + kg;
                a[j] = (uint32_t)(row * (BK * 2) + (((2 * kk + (l >> 5)) ^ s) << 4));
            }
        } else {
            const int q = l >> 4, jj = l & 15;
            const int krow = 16 * kg + 8 * (q >> 1) + (jj >> 2);
            const int within = (jj & 1) * 8;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int col = tile_off + b * 32 + 16 * (q & 1) + 4 * (jj & 3);
                const int pc = (col >> 3) ^ ((jj >> 2) << 2);
                a[b] = (uint32_t)(krow * (2 * R) + pc * 16 + within);
            }
        }
    }

    // Fragment of 32-wide block b for this wave's step j of the slice held at `op` (LDS):
    // lane l gets elements (free = block base + l % 32, k = 16 kk + 8 (l / 32) + 0..7).
    __device__ __forceinline__ bf16x8 load(const CCE_LDS char* op, int b, int j) const {
        if (KMAJOR) {
            return *(const CCE_LDS bf16x8*)(op + a[j] + b * (32 * BK * 2));
        } else {
            const CCE_LDS char* p = op + a[b] + j * (KG * 16 * 2 * R);
            s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CCE_LDS s16x4*)p);
            s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CCE_LDS s16x4*)(p + 4 * 2 * R));
            s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, v);
        }
    }
};

// Scheduling hint: one MFMA, then PER LDS reads, repeated (compile-time recursion because
// the builtin wants constant arguments).
template <int I, int N_MFMA, int N_READS, int PER>
struct SchedInterleave {
    static __device__ __forceinline__ void run() {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (I * PER < N_READS)
            __builtin_amdgcn_sched_group_barrier(0x100, ((I + 1) * PER <= N_READS ? PER : N_READS - I * PER), 0);
        if constexpr (I + 1 < N_MFMA) SchedInterleave<I + 1, N_MFMA, N_READS, PER>::run();
    }
};

// Workgroup barrier that first waits until at most `PENDING` of this thread's global->LDS
// loads are still in flight and all of its LDS reads have returned.  (__syncthreads would
// wait for every outstanding load, which defeats a prefetch distance of more than one
// slice.)  The "memory" clobber keeps the compiler from moving LDS accesses across it.
template <int PENDING>
__device__ __forceinline__ void barrier_pending_loads() {
    static_assert(PENDING >= 0 && PENDING < 64, "vmcnt is a 6-bit counter");
    if constexpr (PENDING == 0) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(PENDING) : "memory");
}

// Workgroup barrier for data exchanged through LDS only: waits for this thread's LDS
// traffic, not for its outstanding global loads (which __syncthreads would also drain).
__device__ __forceinline__ void barrier_lds_only() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// acc[bm][bn] += A-tile * B-tile^T over K slices [0, ceil(k_total / 64)).  The operands
// clamp / meet zero padding so that reads past k_total contribute zero.
// `smem` must hold Cfg::kLdsBytes.  Ends with a workgroup barrier, after which the LDS may
// be reused by the caller.
//
// Software pipeline.  Global -> LDS runs STAGES - 1 K slices ahead (STAGES LDS stages; a
// slice of a 256 x 128 tile lasts only ~0.5 us, less than a trip to L2 / HBM, hence three
// stages there).  LDS -> registers runs one k16 step ahead (two fragment sets): while the
// MFMAs of step kk run, the fragments of step kk + 1 are already being read.  The one
// workgroup barrier per slice sits before the MFMAs of a wavefront's last step: by then every
// wavefront has issued (and waited for) all its LDS reads of the current stage, so after
// the barrier (a) the next slice's data, whose loads each wavefront has waited for, is
// visible to all and its first fragments can be read under those last MFMAs, and (b)
// the current stage may be overwritten by the loads issued at the top of the next
// iteration.
template <class Cfg, bool A_KMAJOR, bool B_KMAJOR, bool PEEL = false, class OpA, class OpB>
__device__ __forceinline__ void gemm_mainloop(f32x16 (&acc)[Cfg::TM][Cfg::TN], const OpA& A, const OpB& B,
                                               int k_total, CCE_LDS char* smem) {
    constexpr int S = Cfg::STAGES, BK = Cfg::BK;
    constexpr int kAhead = (S - 2) * Cfg::kLoadsPerSlice;    // loads that may stay in flight
    constexpr int SPS = Cfg::kSteps;
    FragAddr<A_KMAJOR, Cfg::BM, Cfg::TM, SPS, Cfg::KG, Cfg::BK> fa;
    FragAddr<B_KMAJOR, Cfg::BN, Cfg::TN, SPS, Cfg::KG, Cfg::BK> fb;
    fa.init(wave_m<Cfg>() * (Cfg::TM * 32), wave_kg<Cfg>());
    fb.init(wave_n<Cfg>() * (Cfg::TN * 32), wave_kg<Cfg>());

    const int KT = (k_total + BK - 1) / BK;
#pragma unroll
    for (int s = 0; s < S - 1; ++s) {
        if (s < KT) {
            A.issue(smem + s * Cfg::kStage, s * BK);
            B.issue(smem + s * Cfg::kStage + Cfg::kAStage, s * BK);
        }
    }
    if (KT >= S - 1) barrier_pending_loads<kAhead>();
    else barrier_pending_loads<0>();

    bf16x8 af[2][Cfg::TM], bfr[2][Cfg::TN];
#pragma unroll
    for (int bm = 0; bm < Cfg::TM; ++bm) af[0][bm] = fa.load(smem, bm, 0);
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) bfr[0][bn] = fb.load(smem + Cfg::kAStage, bn, 0);

    int cur_s = 0;                       // stage holding slice kt
    // One K slice.  more: slice kt + S - 1 exists and is requested during this one (a bool, or a
    // std::true_type / std::false_type where the caller knows it at compile time).
    auto slice = [&](int kt, auto more_tag, auto full_tag) {
        const bool MORE = more_tag;
        constexpr bool FULL = decltype(full_tag)::value;      // the requested slice is a full one of both operands
        CCE_LDS char* cur = smem + cur_s * Cfg::kStage;
        const int nxt_s = (cur_s + 1 == S) ? 0 : cur_s + 1;
        CCE_LDS char* nxt = smem + nxt_s * Cfg::kStage;
        const int ld_s = (cur_s == 0) ? S - 1 : cur_s - 1;       // stage of slice kt - 1, free again
        if (MORE) {
            A.template issue<FULL>(smem + ld_s * Cfg::kStage, (kt + S - 1) * BK);
            B.template issue<FULL>(smem + ld_s * Cfg::kStage + Cfg::kAStage, (kt + S - 1) * BK);
        }
#pragma unroll
        for (int kk = 0; kk < SPS; ++kk) {
            const int c = kk & 1, n = c ^ 1;
            if (kk < SPS - 1) {
#pragma unroll
                for (int bm = 0; bm < Cfg::TM; ++bm) af[n][bm] = fa.load(cur, bm, kk + 1);
#pragma unroll
                for (int bn = 0; bn < Cfg::TN; ++bn) bfr[n][bn] = fb.load(cur + Cfg::kAStage, bn, kk + 1);
            } else {
                // slice kt + 1 must have landed; younger slices may still be in flight
                if (MORE) barrier_pending_loads<kAhead>();
                else barrier_pending_loads<0>();
#pragma unroll
                for (int bm = 0; bm < Cfg::TM; ++bm) af[n][bm] = fa.load(nxt, bm, 0);
#pragma unroll
                for (int bn = 0; bn < Cfg::TN; ++bn) bfr[n][bn] = fb.load(nxt + Cfg::kAStage, bn, 0);
            }
#pragma unroll
            for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
                for (int bn = 0; bn < Cfg::TN; ++bn)
                    acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[c][bm], bfr[c][bn], acc[bm][bn], 0, 0, 0);
            // issue order for the scheduler: the LDS reads of the next step are spread
            // one (or two) at a time behind the first MFMAs of this step
            constexpr int kReads = Cfg::TM * (A_KMAJOR ? 1 : 2) + Cfg::TN * (B_KMAJOR ? 1 : 2);
            constexpr int kMfma = Cfg::TM * Cfg::TN;
            constexpr int kPer = (kReads + kMfma - 1) / kMfma;
            SchedInterleave<0, kMfma, kReads, kPer>::run();
        }
        cur_s = nxt_s;
    };
    if constexpr (PEEL) {
        // The last S - 1 slices request nothing: peeled off, so that neither loop body branches on it.
        // Pays in the contraction kernels (2.0 - 2.6 % per launch); the forward and the gradient-tile
        // kernel were 0.5 - 1 % faster with the one loop below.
        // Likewise the slices whose request is a full slice of both operands (all but a ragged last one)
        // run a body whose loads need no clamping of k-rows, hence no branch.
        const int n_more = KT - (S - 1) > 0 ? KT - (S - 1) : 0;
        const int fa_n = A.full_slices(), fb_n = B.full_slices();
        int n_full = (fa_n < fb_n ? fa_n : fb_n) - (S - 1);          // request kt + S - 1 < full slices
        n_full = n_full < 0 ? 0 : (n_full < n_more ? n_full : n_more);
        for (int kt = 0; kt < n_full; ++kt) slice(kt, std::true_type{}, std::true_type{});
        for (int kt = n_full; kt < n_more; ++kt) slice(kt, std::true_type{}, std::false_type{});
        for (int kt = n_more; kt < KT; ++kt) slice(kt, std::false_type{}, std::false_type{});
    } else {
        for (int kt = 0; kt < KT; ++kt) slice(kt, kt + S - 1 < KT, std::false_type{});
    }
    barrier_pending_loads<0>();
}

// ------------------------------------------------------------------------------------------
// FP8 (E4M3) variant of the main loop for two K-major operands with block scales: one
// power-of-two scale (a biased exponent byte, as the block-scaled MFMA takes it) per row and
// 128 consecutive K elements.  v_mfma_scale_f32_32x32x64_f8f6f4 multiplies 64 K values per
// instruction and applies both operands' scales itself, at twice the bf16 rate for the same
// LDS and global traffic per instruction: a 128-byte row of a stage now holds 128 K values,
// so the stage geometry, the global->LDS loads and the swizzle are those of the bf16 loop
// (the operands are handed in as bf16 matrices of half the width), and a K slice is 128.
//
// A lane's 32 operand bytes are the two 16-byte fragments the bf16 loop would read for two
// consecutive k16 steps.  Which K positions the hardware assigns to them does not matter:
// A and B use the same assignment, a dot product does not depend on the order of its terms,
// and all 64 K values of an instruction lie in one 128-block, i.e. share one scale per row.
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;

// Block scales of a quantised matrix, in the order the block-scaled MFMA consumes them:
// [D / 128 blocks][ceil(rows / 128) groups][32][4] bytes -- byte j of dword i of a group is the
// exponent byte of row 128 g + 32 j + i.  A wavefront whose 32-row blocks start at a multiple
// of 128 rows then gets the scales of four blocks with ONE dword load per lane and 128-block,
// and picks block j with the instruction's byte selector.
struct ScaleGroup {
    const uint32_t* p;      // this lane's dword of K block 0
    uint32_t step;          // dwords from one K block to the next
    __device__ __forceinline__ void init(const void* scales, int groups, int group) {
        group = group < groups ? group : groups - 1;            // rows past the matrix are masked by the caller
        p = (const uint32_t*)scales + (size_t)group * 32 + (threadIdx.x & 31);
        step = (uint32_t)groups * 32u;
    }
    __device__ __forceinline__ uint32_t load(int kb) const { return p[(size_t)kb * step]; }
};

// One block-scaled FP8 MFMA; OA / OB select the scale byte of each operand (compile time).
template <int OA, int OB>
__device__ __forceinline__ f32x16 mfma_fp8(const i32x8 a, const i32x8 b, const f32x16 c, int sa, int sb) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, OA, sa, OB, sb);
}
__device__ __forceinline__ f32x16 mfma_fp8_sel(int oa, int ob, const i32x8 a, const i32x8 b, const f32x16 c, int sa, int sb) {
    switch (oa * 2 + ob) {          // folded after unrolling
        case 0: return mfma_fp8<0, 0>(a, b, c, sa, sb);
        case 1: return mfma_fp8<0, 1>(a, b, c, sa, sb);
        case 2: return mfma_fp8<1, 0>(a, b, c, sa, sb);
        case 3: return mfma_fp8<1, 1>(a, b, c, sa, sb);
        case 4: return mfma_fp8<2, 0>(a, b, c, sa, sb);
        case 5: return mfma_fp8<2, 1>(a, b, c, sa, sb);
        case 6: return mfma_fp8<3, 0>(a, b, c, sa, sb);
        default: return mfma_fp8<3, 1>(a, b, c, sa, sb);
    }
}

// SA: scale group of the wavefront's TM = 4 A blocks (128 rows); SB: scale group that
// contains its TN = 2 B blocks, b_half = which half of that group (0: rows 0..63).
template <class Cfg>
__device__ __forceinline__ void gemm_mainloop_fp8(f32x16 (&acc)[Cfg::TM][Cfg::TN],
                                                   const OperandTile<true, Cfg::BM>& A,
                                                   const OperandTile<true, Cfg::BN>& B,
                                                   const ScaleGroup& SA, const ScaleGroup& SB, int b_half,
                                                   int k_total, CCE_LDS char* smem) {
    static_assert(Cfg::STAGES == 2 && Cfg::KG == 1 && Cfg::TM == 4 && Cfg::TN == 2, "256 x 256 tile, two stages");
    FragAddr<true, Cfg::BM, Cfg::TM, 4, 1> fa;
    FragAddr<true, Cfg::BN, Cfg::TN, 4, 1> fb;
    fa.init(wave_m<Cfg>() * (Cfg::TM * 32), 0);
    fb.init(wave_n<Cfg>() * (Cfg::TN * 32), 0);
    auto frag = [](const CCE_LDS char* op, uint32_t a, int b) {
        return *(const CCE_LDS i32x4*)(op + a + b * (32 * 128));
    };

    const int KT = (k_total + 127) / 128;
    const int b_shift = 16 * b_half;
    uint32_t sa_next = SA.load(0), sb_next = SB.load(0);

    A.issue(smem, 0);
    B.issue(smem + Cfg::kAStage, 0);
    barrier_pending_loads<0>();

    // A fragments are refreshed in place, block by block, behind the MFMAs that used them; B
    // fragments (needed by every block of a step) are double buffered.
    i32x4 af[Cfg::TM][2], bfr[2][Cfg::TN][2];
#pragma unroll
    for (int bm = 0; bm < Cfg::TM; ++bm) { af[bm][0] = frag(smem, fa.a[0], bm); af[bm][1] = frag(smem, fa.a[1], bm); }
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) {
        bfr[0][bn][0] = frag(smem + Cfg::kAStage, fb.a[0], bn);
        bfr[0][bn][1] = frag(smem + Cfg::kAStage, fb.a[1], bn);
    }

    int cur_s = 0;
    for (int kt = 0; kt < KT; ++kt) {
        CCE_LDS char* cur = smem + cur_s * Cfg::kStage;
        CCE_LDS char* nxt = smem + (cur_s ^ 1) * Cfg::kStage;
        const bool more = kt + 1 < KT;
        // scales of this slice (requested one slice ago, complete since the last barrier) and
        // request of the next slice's, ahead of the operand loads
        const int sa = (int)sa_next, sb = (int)(sb_next >> b_shift);
        // Consume the two scale words HERE, before this iteration's operand loads are issued:
        // the compiler places its wait for them at their first use and cannot see the
        // inline-assembly loads, so a first use after those would make it wait for them too.
        asm volatile("" :: "v"(sa), "v"(sb));
        const int kn = more ? kt + 1 : kt;
        sa_next = SA.load(kn);
        sb_next = SB.load(kn);
        if (more) {
            A.issue(nxt, (kt + 1) * kBK);
            B.issue(nxt + Cfg::kAStage, (kt + 1) * kBK);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int c = t, n = t ^ 1;
            const CCE_LDS char* src = cur;
            int j0 = 2;
            if (t == 1) {
                // slice kt + 1 must have landed before its fragments are read
                barrier_pending_loads<0>();
                src = nxt;
                j0 = 0;
            }
#pragma unroll
            for (int bn = 0; bn < Cfg::TN; ++bn) {
                bfr[n][bn][0] = frag(src + Cfg::kAStage, fb.a[j0], bn);
                bfr[n][bn][1] = frag(src + Cfg::kAStage, fb.a[j0 + 1], bn);
            }
#pragma unroll
            for (int bm = 0; bm < Cfg::TM; ++bm) {
                const i32x8 a8 = __builtin_shufflevector(af[bm][0], af[bm][1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int bn = 0; bn < Cfg::TN; ++bn) {
                    const i32x8 b8 = __builtin_shufflevector(bfr[c][bn][0], bfr[c][bn][1], 0, 1, 2, 3, 4, 5, 6, 7);
                    acc[bm][bn] = mfma_fp8_sel(bm, bn, a8, b8, acc[bm][bn], sa, sb);
                }
                af[bm][0] = frag(src, fa.a[j0], bm);
                af[bm][1] = frag(src, fa.a[j0 + 1], bm);
            }
            // issue order for the scheduler: the four B reads behind the first two MFMAs, then
            // each A block's two reads behind the MFMA that follows the last use of the block
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0); __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0); __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        cur_s ^= 1;
    }
    barrier_pending_loads<0>();
}

// ------------------------------------------------------------------------------------------
// Tiles of eight wavefronts in two groups of four, one of each group to a SIMD, that take turns: while one group
// multiplies, the other reads its next fragments from LDS and requests the next slice, a barrier at every turn.  A
// wavefront owns NA x NB blocks of 16 x 16 (v_mfma_f32_16x16x32_bf16: lane l holds column l % 16, rows 4 (l / 16) + 0 .. 3),
// 4 x 2 wavefronts a tile of 64 NA x 32 NB.  Fragments need no second buffer (the other group's products hide their
// latency), which leaves the registers for 384 x 256 outputs (gradient tiles 252; the forward all 256 and 13 values of a lane in
// scratch, 17 with label smoothing, of which it fetches ten and writes one to three a tile, none in a slice): a sixth fewer operand bytes per product than 256 x 256 from
// L2, a fifth fewer from LDS, and the 16 x 16 form draws less power than the 32 x 32 one, whose smaller number of
// instructions the turns make up for.  What bounds it is power: 18432 x 8192 x 4096 in one launch after the other, random /
// constant operands, TFLOP/s: TileBig's loop 1 400 / 1 920; these turns with 32 x 32 x 16 at 256 x 256 1 425 / 2 015, at
// 384 x 256 1 475 / 2 195; with 16 x 16 x 32 at 256 x 256 1 530 / 1 930, at 384 x 256 1 645 / 2 155 (K = 896: TileBig's
// 1 350 / 1 755, 384 x 256 1 540 / 1 915).
template <int NA_, int NB_>
struct PingTile {
    static constexpr int NA = NA_, NB = NB_, WM = 4, WN = 2;
    static constexpr int kThreads = 512, BK = 64;
    static constexpr int TMR = 16 * NA, TNR = 16 * NB;          // rows and columns of a wavefront
    static constexpr int BM = WM * TMR, BN = WN * TNR;
    static constexpr int kAStage = BM * BK * 2, kStage = (BM + BN) * BK * 2;
    static constexpr int kLdsBytes = 2 * kStage;
    static constexpr int kALoads = BM / 64, kBLoads = BN / 64;  // 16-byte loads per thread and slice
    static constexpr int kParts = 2, QA = NA / kParts;          // a step's products in two turns, over half of the A blocks each
    static_assert(NA % kParts == 0 && BN % 64 == 0 && kLdsBytes <= 160 * 1024, "whole parts and loads; two stages");
};
typedef PingTile<6, 8> TileTall;        // 384 x 256, wave tile 96 x 128
typedef PingTile<4, 8> TileSquare;      // 256 x 256, wave tile 64 x 128: where the taller tiles leave compute units idle

// Rows of the A stage that a wavefront's blocks stand for.  Halves: block i of part p covers rows p BM / 2 + 16 (QA wave + i),
// so that a tile of BM / 2 rows is its first part alone.  Pairs: blocks 2 j and 2 j + 1 share rows 32 j ... 32 j + 31 of the
// wavefront, lane group g holding rows 8 g .. 8 g + 7 of them, four in each block: 16 bytes of bf16 results in a row.
enum class ARows { kHalves, kPairs };

template <class Cfg, ARows ROWS>
struct PingPong {
    CCE_LDS char* smem;
    int group, wm, wn;           // wave-uniform
    uint32_t fa, fb;             // fragment addresses of the first step; the second is 64 bytes away, either side
    int cur;                     // stage of the current slice

    static __device__ __forceinline__ int a_swizzle(int row) {
        // a lane's 16 bytes go to physical chunk c ^ swizzle of its 128-byte row: the 16 rows of a fragment differ in it
        return ROWS == ARows::kHalves ? (row >> 1) & 7 : ((row >> 1) & 1) | (((row >> 3) & 3) << 1);
    }
    __device__ __forceinline__ void init(CCE_LDS char* smem_) {
        smem = smem_;
        cur = 0;
        const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        group = wave >> 2;
        wm = wave / Cfg::WN;
        wn = wave % Cfg::WN;
        const int r = l & 15, h = l >> 4;
        const int arow = ROWS == ARows::kHalves ? wm * (16 * Cfg::QA) + r : wm * Cfg::TMR + 8 * (r >> 2) + (r & 3);
        const int brow = wn * Cfg::TNR + r;
        fa = (uint32_t)(arow * 128 + ((h ^ a_swizzle(arow)) << 4));
        fb = (uint32_t)(Cfg::kAStage + brow * 128 + ((h ^ ((brow >> 1) & 7)) << 4));
    }
    static constexpr int a_offset(int i) {
        return ROWS == ARows::kHalves ? (i / Cfg::QA * (Cfg::BM / 2) + i % Cfg::QA * 16) * 128 : (i / 2 * 32 + i % 2 * 4) * 128;
    }
    // Row of the tile of accumulator element r of block i, and column of block j, of the calling lane.
    __device__ __forceinline__ int row(int i, int r) const {
        const int g = (threadIdx.x & 63) >> 4;
        return ROWS == ARows::kHalves ? i / Cfg::QA * (Cfg::BM / 2) + (wm * Cfg::QA + i % Cfg::QA) * 16 + 4 * g + r
                                      : wm * Cfg::TMR + i / 2 * 32 + 8 * g + i % 2 * 4 + r;
    }
    __device__ __forceinline__ int col(int j) const { return wn * Cfg::TNR + j * 16 + (int)(threadIdx.x & 15); }

    static __device__ __forceinline__ void barrier() { asm volatile("s_barrier" ::: "memory"); }
    // In front of the first slice, whose loads have been requested into stage 0.
    __device__ __forceinline__ void start() {
        asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        if (group) barrier();
    }
    // Behind the last slice of a tile and behind its epilogue: group 1 passes its barrier there, so that the groups' epilogues run
    // beside each other.
    __device__ __forceinline__ void tile_done() {
        if (!group) barrier();
    }
    __device__ __forceinline__ void tile_end() {
        if (group) barrier();
    }
    // Behind the last tile: both groups have passed the same barriers.
    __device__ __forceinline__ void finish() {
        if (!group) barrier();
    }

    // One slice of 64, a barrier() to follow (or tile_done()).  PARTS: 1 leaves out the second half of the A rows.  request(stage, half): issues one half of the loads of the slice behind this one, where there is one.
    //
    // Turns: group 0 reads in turn 2 i and multiplies in 2 i + 1, group 1 one turn later.  The loads of slice t + 1 are issued in the
    // first reading turns of slice t, when every wavefront has its fragments of slice t - 1 (lgkmcnt(0) in front of the barriers), and
    // each wavefront waits for its own (vmcnt(0)) in its last reading turn of slice t, which is in front of the barrier that precedes
    // group 0's first reading turn of slice t + 1.
    template <class Request>
    __device__ __forceinline__ void slice(f32x4 (&acc)[Cfg::NA][Cfg::NB], int parts, Request request) {
        CCE_LDS char* const st = smem + cur * Cfg::kStage;
        const int next = cur ^ 1;
        bf16x8 a[Cfg::QA], b[Cfg::NB];
        auto turn = [&](auto step, auto part) {
            constexpr int s = decltype(step)::value, p = decltype(part)::value;
            __builtin_amdgcn_sched_barrier(0);
            if (p == 0) {
#pragma unroll
                for (int j = 0; j < Cfg::NB; ++j) b[j] = *(const CCE_LDS bf16x8*)(st + (fb ^ (uint32_t)(s * 64)) + j * 2048);
            }
#pragma unroll
            for (int i = 0; i < Cfg::QA; ++i) a[i] = *(const CCE_LDS bf16x8*)(st + (fa ^ (uint32_t)(s * 64)) + a_offset(p * Cfg::QA + i));
            if (s == 0) {
                request(next, p);
                if (p == 0 && parts == 1) request(next, 1);
            }
            if (s == 1 && p == 0 && parts == 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (s == 1 && p == 1) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < Cfg::QA; ++i)
#pragma unroll
                for (int jj = 0; jj < Cfg::NB; ++jj) {
                    const int j = i & 1 ? Cfg::NB - 1 - jj : jj;          // (back and forth: the B operand of the last product stays: 1 %)
                    f32x4& c = acc[p * Cfg::QA + i][j];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], c, 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        };
        using Zero = std::integral_constant<int, 0>;
        using One = std::integral_constant<int, 1>;
        turn(Zero{}, Zero{});
        barrier();
        if (parts == 2) {
            turn(Zero{}, One{});
            barrier();
        }
        turn(One{}, Zero{});
        if (parts == 2) {
            barrier();
            turn(One{}, One{});
        }
        cur = next;
    }
};

// Global -> LDS loads of two K-major operands for these tiles.  Load i of a thread brings 16 bytes of row 64 i + 8 wave +
// lane / 8 of the stage, A rows in front of B rows.  A rows are relative to the tile's first one, those behind the last valid
// one read that again; B rows lie at any offsets (a row map).
template <class Cfg, ARows ROWS>
struct PingLoads {
    const char* a;               // next slice: A's first row of the tile and B, both at the slice's K offset (uniform)
    const char* b;
    uint32_t a_off, a_last, a_step;
    uint32_t b_off[Cfg::kBLoads];
    uint32_t chunk, lds0;
    bool on;
    __device__ __forceinline__ int row(int i) const { return 64 * i + 8 * (int)(threadIdx.x >> 6) + (int)((threadIdx.x & 63) >> 3); }
    __device__ __forceinline__ void init(CCE_LDS char* smem, uint32_t ld_bytes) {
        chunk = (uint32_t)((threadIdx.x & 7) ^ PingPong<Cfg, ROWS>::a_swizzle(row(0))) * 16u;
        a_off = (uint32_t)row(0) * ld_bytes + chunk;
        a_step = 64u * ld_bytes;
        lds0 = (uint32_t)(uintptr_t)smem + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * 1024u;
    }
    // B row i of this thread is row `r` of its matrix.
    __device__ __forceinline__ void set_b_row(int i, int r, uint32_t ld_bytes) {
        b_off[i] = (uint32_t)r * ld_bytes + (uint32_t)((threadIdx.x & 7) ^ ((row(0) >> 1) & 7)) * 16u;
    }
    __device__ __forceinline__ void tile(const char* a_tile, int a_rows, const char* b_matrix, uint32_t ld_bytes) {
        a = a_tile;
        b = b_matrix;
        a_last = (uint32_t)(a_rows - 1) * ld_bytes + chunk;
    }
    __device__ __forceinline__ void issue(int stage, int half) const {
        constexpr int NL = Cfg::kALoads + Cfg::kBLoads;
        const uint32_t to = lds0 + (uint32_t)stage * Cfg::kStage;
        uint32_t first = a_off;
        asm volatile("" : "+v"(first));                 // (the sums below stay here: kept over the loop they cost registers)
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if ((i < NL / 2) != (half == 0)) continue;
            if (i < Cfg::kALoads) {
                const uint32_t o = first + (uint32_t)i * a_step;
                load16_to_lds_sbase(a, o < a_last ? o : a_last, to + (uint32_t)i * 8192u);
            } else {
                load16_to_lds_sbase(b, b_off[i - Cfg::kALoads], to + (uint32_t)i * 8192u);
            }
        }
    }
};

// ------------------------------------------------------------------------------------------
// Contractions on 256 x 256 tiles of two groups of wavefronts that take turns (see PingTile), X K-slow, the chunk in either way.
// X, a matrix row per k (hidden or weight rows), gives 256 of its D columns, the gradient chunk G 256 of its rows or columns:
// C[g, x] with X as the A operand, so that a lane holds four consecutive columns of a result row.  2 x 4 wavefronts of 128 x 64,
// group = wavefront row: where the tile's second 128 columns lie behind the matrix, that group only loads (the other one's turns
// then follow each other: 0.66 of the time).  One turn per slice of 32: every fragment of a slice is read at once, 32 products to
// 24 transpose reads of 8 bytes a lane, the loads of a later slice among the products.
//
// LDS layout, a lane's 16 bytes at lane * 16 of a wavefront's 1 KB: X in blocks of 64 columns, [block][32 k][128 B], the 32-byte
// unit u of a row at u ^ (bit 1 of k + 2 bit 3 of k); G K-slow in blocks of 32 columns (a panel's width), [block][32 k][64 B], at
// u ^ bit 3 of k: the 8 k-rows x 32 bytes that two lane groups of a transpose read touch per clock cover all 64 banks (measured
// 229 of 256 B/clk, and 64 with the units in place; a seventh of the LDS's busy cycles count as conflicts).  G K-major: [row][64 B],
// chunk c at c ^ bits 2, 3 of the row.
//
// What bounds it is power.  4096 x 24576 x 4096 in one launch after the other, TFLOP/s on random / constant operands: 256 x 256 by
// gemm_mainloop 1 436 / 1 892, 256 x 128 1 292 / 1 786, these 1 583 / 2 158 (with the loads in the reading turns, three stages
// 1 436 / 1 898; 256 x 384 outputs, which have the registers for that form alone, 1 655 / 2 209 and in place no faster: items half as
// long again, a launch's last round emptier).
struct TurnTile {
    static constexpr int NA = 8, NB = 4, BM = 256, BN = 256, BK = 32, STAGES = 4;        // BM: columns of X, BN: rows / columns of G
    static constexpr int kThreads = 512;
    static constexpr int kXStage = BM * BK * 2, kStage = (BM + BN) * BK * 2, kLdsBytes = STAGES * kStage;
    static constexpr int kXLoads = 2, kLoads = 4;               // 16-byte loads per thread and slice
};

// The calling lane's number, without the thread id.
__device__ __forceinline__ int wave_lane() { return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// MAP: the k-rows of X are reached through a table in LDS, as in OperandTile.
template <bool G_KMAJOR, int MAP>
struct TurnLoop {
    typedef TurnTile Cfg;
    CCE_LDS char* smem;
    const char* x;               // uniform: the next slice's first row (MAP: row 0 of the matrix), columns of load 0
    const char* g;               // uniform: the next slice
    uint32_t x_step;             // from load 0's columns to load 1's
    uint32_t x_off, g_off;       // this thread's place in a slice (MAP: in the next slice)
    uint32_t ld, panel, lds0;
    int rows;                    // valid k-rows of X from the next slice on
    int k;                       // MAP: first table entry of the next slice
    const CCE_LDS uint32_t* kmap;
    const CCE_LDS uint16_t* kmap16;
    uint32_t xa, ga;             // fragment addresses in a stage, of unit 0 (the others by xor)
    int wave, group;

    // (from the lane number at each use: kept over the loop they would take registers that the accumulators need)
    __device__ __forceinline__ int x_row() const { return 8 * (wave & 3) + (wave_lane() >> 3); }
    __device__ __forceinline__ uint32_t x_chunk() const {
        const int row = x_row();
        return (uint32_t)(((wave_lane() & 7) ^ (2 * (((row >> 1) & 1) | (((row >> 3) & 1) << 1)))) * 16);
    }

    // X: matrix with rows of ld_bytes and n_cols columns, from the reduction's first row on (MAP: from its first row on), of which
    // k_rows are valid (at least one); the tile's columns from col0 on.  G: the chunk, its rows (K-major) or columns from free0 on,
    // from k0 on; panels of 32 columns.
    __device__ __forceinline__ void init(CCE_LDS char* smem_, int wave_, const void* X, uint32_t ld_bytes, int col0, int n_cols, int k_rows,
                                         const uint16_t* G, uint32_t panel_elements, int free0, int k0) {
        smem = smem_;
        ld = ld_bytes;
        panel = panel_elements * 2u;
        rows = k_rows;
        const int l = wave_lane();
        wave = wave_;
        group = wave >> 2;
        lds0 = (uint32_t)(uintptr_t)smem + (uint32_t)wave * 1024u;
        // load i of X: block 2 i + wave / 4 of 64 columns (blocks behind the matrix: its last one)
        const int last = (n_cols - 1 - col0) >> 6;
        const int b0 = group < last ? group : last, b1 = 2 + group < last ? 2 + group : last;
        x = (const char*)X + (size_t)(col0 + b0 * 64) * 2;
        x_step = (uint32_t)(b1 - b0) * 128u;
        x_off = (uint32_t)x_row() * ld + x_chunk();
        k = 0;
        kmap = nullptr;
        kmap16 = nullptr;
        if (G_KMAJOR) {
            g = (const char*)G + (size_t)(k0 / 32) * panel + (size_t)free0 * 64;
            const int row = wave * 16 + (l >> 2);
            g_off = (uint32_t)(row * 64 + (((l & 3) ^ ((row >> 2) & 3)) << 4));
        } else {
            g = (const char*)G + (size_t)(free0 / 32) * panel + (size_t)k0 * 64;
            const int row = 16 * (wave & 1) + (l >> 2);
            g_off = (uint32_t)(wave >> 1) * panel + (uint32_t)(row * 64 + (((l & 3) ^ (2 * ((row >> 3) & 1))) << 4));
        }
        const int wn = wave & 3, h = l >> 4, jj = l & 15;
        const int kr = 8 * h + (jj >> 2), q = jj & 3;           // transpose reads: this lane's k-row (and the one 4 on), its 8 bytes
        xa = (uint32_t)(group * (2 * 32 * 128) + kr * 128 + (((kr >> 1) & 1) | (((kr >> 3) & 1) << 1)) * 32 + q * 8);
        const int row = wn * 16 * Cfg::NB + jj;
        ga = (uint32_t)Cfg::kXStage + (G_KMAJOR ? (uint32_t)(row * 64 + ((h ^ ((row >> 2) & 3)) << 4))
                                                : (uint32_t)(wn * (Cfg::NB / 2) * (32 * 64) + kr * 64 + ((kr >> 3) & 1) * 32 + q * 8));
    }
    // MAP: x_off of the slice whose first table entry is k.
    __device__ __forceinline__ void look_up() {
        x_off = (MAP == 1 ? kmap[k + x_row()] : __umul24((uint32_t)kmap16[k + x_row()], ld)) + x_chunk();
    }
    // A slice of `rows` valid rows: behind the last one that one again, whose products meet the chunk's zeros.
    __device__ __forceinline__ void ragged() {
        if (MAP == 0) x_off = (uint32_t)(x_row() < rows ? x_row() : rows - 1) * ld + x_chunk();
    }
    __device__ __forceinline__ void load(int stage, int i) const {
        const uint32_t to = lds0 + (uint32_t)stage * Cfg::kStage + (uint32_t)i * 8192u;
        if (i < Cfg::kXLoads) load16_to_lds_sbase(x + i * x_step, x_off, to);
        else load16_to_lds_sbase(g + (size_t)((uint32_t)(i - Cfg::kXLoads) * (G_KMAJOR ? 8192u : 4u * panel)), g_off, to);
    }
    static __device__ __forceinline__ void barrier() { asm volatile("s_barrier" ::: "memory"); }
    static __device__ __forceinline__ bf16x8 transposed(const CCE_LDS char* p, int four_rows) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CCE_LDS s16x4*)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CCE_LDS s16x4*)(p + four_rows));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }

    // Slices that hold k_rows rows; MAP: the table has entries for as many whole slices and one more (any that may be read).
    static __device__ __forceinline__ int slices(int k_rows) {
        const int n = (k_rows + 31) / 32;
        return n < Cfg::STAGES ? Cfg::STAGES : n;
    }

    // KT slices of 32 (at least STAGES).  Without ON (columns behind the matrix) loads and barriers only.  Group 0 reads in turn 2 t and multiplies
    // in 2 t + 1, group 1 one turn later, a barrier behind every turn.  Slice t + STAGES - 1 is requested in the multiplying turns of
    // slice t, into the stage of slice t - 1, whose fragments every wavefront has by then (lgkmcnt(0) in front of the barriers); slice t + 1 has landed when a wavefront leaves its reading turn of slice t (its own loads, vmcnt), which is in
    // front of the barrier that precedes group 0's reading turn of t + 1.
    template <bool ON>
    __device__ __forceinline__ void turns(f32x4 (&acc)[Cfg::NA][Cfg::NB], int KT) {
        constexpr int S = Cfg::STAGES, NL = Cfg::kLoads;
        for (int s = 0; s < S - 1; ++s) {
            if (MAP) look_up();
            else if (rows < 32) ragged();
#pragma unroll
            for (int i = 0; i < NL; ++i) load(s, i);
            g += G_KMAJOR ? (size_t)panel : (size_t)2048;
            k += 32;
            if (rows > 32) {
                rows -= 32;
                if (MAP == 0) x += (size_t)(32u * ld);
            }
        }
        if (MAP) look_up();
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((S - 2) * NL) : "memory");
        if (group) barrier();
        int cur = 0;
        auto slice = [&](auto more_tag) {
            constexpr bool MORE = decltype(more_tag)::value;    // another slice is requested
            const CCE_LDS char* const st = smem + cur * Cfg::kStage;
            const int to = cur == 0 ? S - 1 : cur - 1;
            bf16x8 a[Cfg::NA], b[Cfg::NB];
            __builtin_amdgcn_sched_barrier(0);
            if (ON) {
#pragma unroll
                for (int i = 0; i < Cfg::NA; ++i) a[i] = transposed(st + (xa ^ (uint32_t)((i & 3) * 32)) + (i >> 2) * (32 * 128), 4 * 128);
#pragma unroll
                for (int j = 0; j < Cfg::NB; ++j) {
                    if (G_KMAJOR) b[j] = *(const CCE_LDS bf16x8*)(st + ga + j * 1024);
                    else b[j] = transposed(st + (ga ^ (uint32_t)((j & 1) * 32)) + (j >> 1) * (32 * 64), 4 * 64);
                }
            }
            if (MORE) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(NL) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            constexpr int NM = Cfg::NA * Cfg::NB, GAP = NM / (NL + 1);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int j = m / Cfg::NA, i = j & 1 ? Cfg::NA - 1 - m % Cfg::NA : m % Cfg::NA;
                if (ON) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
                if (MORE && m % GAP == GAP - 1 && m / GAP < NL) {
                    __builtin_amdgcn_sched_barrier(0);
                    load(to, m / GAP);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (MORE) {
                g += G_KMAJOR ? (size_t)panel : (size_t)2048;
                if (MAP == 0) {
                    x += (size_t)(32u * ld);
                } else {
                    k += 32;
                    look_up();
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            cur = cur == S - 1 ? 0 : cur + 1;
        };
        rows -= 32 * (KT - S);                                  // of the last slice, the only ragged one beyond the first STAGES - 1
        // (both loops rolled: slices in a row, without a loop, cost some 40 registers)
#pragma nounroll
        for (int t = S - KT; t <= 0; ++t) {
            if (t == 0 && rows < 32) ragged();
            slice(std::true_type{});
            barrier();
        }
#pragma nounroll
        for (int t = S - 1;;) {
            slice(std::false_type{});
            if (--t == 0) break;
            barrier();
        }
        if (!group) barrier();
        barrier();
    }

    __device__ __forceinline__ void run(f32x4 (&acc)[Cfg::NA][Cfg::NB], int KT) { turns<true>(acc, KT); }
    __device__ __forceinline__ void idle(int KT) {
        f32x4 none[Cfg::NA][Cfg::NB];
        turns<false>(none, KT);
    }
};

// Tile coordinates of accumulator element acc[bm][bn][r] of the calling lane.
template <class Cfg>
__device__ __forceinline__ int acc_row(int bm, int r) {
    const int l = threadIdx.x & 63;
    return wave_m<Cfg>() * (Cfg::TM * 32) + bm * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
}
template <class Cfg>
__device__ __forceinline__ int acc_col(int bn) {
    const int l = threadIdx.x & 63;
    return wave_n<Cfg>() * (Cfg::TN * 32) + bn * 32 + (l & 31);
}

}  // namespace cce
