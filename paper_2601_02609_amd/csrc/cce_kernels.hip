// libcce: fused LM-head projection + token-level cross-entropy for gfx950 (MI355X).
// Device kernels and the C ABI declared in include/cce.h.
//
// Forward (chunked cross-entropy forward algorithm of the Cut Cross-Entropy section):
//   lse_partial_kernel   logit tile (MFMA) -> online (max, sum-exp) per token, carried in
//                        registers across the vocabulary tiles of one split (online-softmax
//                        definition); one (m, d) pair per token and split is written out
//   finalize_kernel      merges the pairs of all splits (block form of the same recurrence),
//                        lse = m + ln d, label logit by an fp32 dot product, loss = lse - z_y,
//                        ignore_index rows -> 0
// Backward (CCE backward theorem and chunk-level backward algorithm), for each
// [row block x vocabulary chunk]:
//   grad_tile_kernel     recomputes the logit tile, forms dloss * (exp(z - lse) - onehot),
//                        rounds to bf16 and stores it in a scratch chunk G[rows][chunk]
//   grad_gemm_kernel     dH_block += G * W_chunk   and   dW_chunk (+)= G^T * H_block
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <math.h>
#include <mutex>
#include <vector>

#include "../../include/cce.h"
#include "../../include/cce_shard.h"
#include "../../include/cce_fp8.h"
#include "../../include/cce_compact.h"
#include "fused_backward.h"
#include "gemm_core.h"
#include "host_util.h"
#include "plan.h"
#include "wg_map.h"

namespace cce {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
template <class Cfg> constexpr int kGRowBytes = Cfg::BM * 2 + 16;     // LDS staging row of a G tile (bf16 + pad)

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Merge two (max, sum) pairs kept in the log2 domain; safe for empty pairs (m = -inf, d = 0).
__device__ __forceinline__ void md_merge(float& m, float& d, float m2, float d2) {
    const float mn = fmaxf(m, m2);
    const float ms = (mn == -INFINITY) ? 0.f : mn;
    d = d * fast_exp2(m - ms) + d2 * fast_exp2(m2 - ms);
    m = mn;
}

// ------------------------------------------------------------------------------------------
// Forward: per (token tile, vocabulary split) online log-sum-exp.
// Tile orientation: M = vocabulary (A = W, K-major), N = tokens (B = H, K-major), so that in
// the 32x32 accumulator layout a lane owns ONE token column and 16 vocabulary rows of each
// block: the running max / sum of a token is lane-local until the very end.
// partials[token * S + split] = (m, d) with m in the log2 domain (m = max_v z * log2 e).
// ------------------------------------------------------------------------------------------
// SUMZ (label smoothing only): the sum of a token's logits over the vocabulary split is carried
// along as well, partial_sumz[token * S + split]; the smoothed loss needs their mean.
// FP8: H and W are E4M3 bytes (row length D) with one scale-exponent byte per row and 128
// columns in hscale / wscale (grouped layout, see ScaleGroup); the logit tile is then formed by the
// block-scaled FP8 MFMA loop and everything after it is unchanged.
struct Fp8Scales {
    const void* hscale;
    const void* wscale;
    int hgroups, wgroups;       // ceil(rows / 128) of each matrix
};

// Exponent byte of (row, 128-block kb) in the grouped scale layout (see ScaleGroup).
__device__ __forceinline__ int scale_byte(const void* scales, int groups, int row, int kb) {
    const uint8_t* s = (const uint8_t*)scales;
    return s[(((size_t)kb * groups + (row >> 7)) * 32 + (row & 31)) * 4 + ((row >> 5) & 3)];
}

template <bool SUMZ, bool FP8, class Cfg = TileBig>
__global__ __launch_bounds__(Cfg::kThreads, 2) void lse_partial_kernel(
        const void* __restrict__ H, const void* __restrict__ W,
        int N, int D, int V, int TT, int VT, int S, float2* __restrict__ partials,
        float* __restrict__ partial_sumz, const Fp8Scales fp8, const int32_t* __restrict__ perm,
        int32_t* __restrict__ status, const int32_t* __restrict__ rows_splits) {
    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    CCE_LDS char* smem = (CCE_LDS char*)smem_generic;

    // The status word starts at zero (status: null where the label scan has written it).  The first
    // launch behind this one that sets bits in it is finalize_kernel: no clearing launch is needed
    // (it took 1.4 us and a launch boundary of about 2 at the smallest shapes).
    if (status && blockIdx.x == 0 && threadIdx.x == 0) status[0] = 0;

    // The rows that take part and the splits that fit them, where only the device knows (see row_scan_kernel); the
    // workgroups beyond are not needed.
    if (rows_splits) {
        N = rows_splits[0];
        S = rows_splits[1];
        TT = (N + Cfg::BN - 1) / Cfg::BN;
        if (rows_splits[3]) perm = nullptr;           // every row takes part
    }
    const int n_work = rows_splits ? TT * S : (int)gridDim.x;
    if ((int)blockIdx.x >= n_work) return;

    // Work index -> (token tile, vocabulary split).  The 32 workgroups that share an XCD (and
    // its 4 MB L2) take a panel of 4 token tiles x all splits: per K slice they touch 4 H
    // tiles + S W tiles instead of 32 + 1, which is what keeps most operand fetches in L2.
    const int lin = xcd_round_id(blockIdx.x, n_work, 2048 / Cfg::NW);
    int tt, s;
    group_map(lin, TT, S, 32 / Cfg::NW, tt, s);
    const int vt0 = (int)((int64_t)s * VT / S), vt1 = (int)((int64_t)(s + 1) * VT / S);
    const int l = threadIdx.x & 63;
    const int wm = wave_m<Cfg>();

    const int ld = FP8 ? D / 2 : D;               // row length in 2-byte units
    OperandTile<true, Cfg::BN, false, Cfg::NW, Cfg::BK> Bop;
    Bop.init(H, ld, tt * Cfg::BN, N, ld, perm);       // perm: token t of the tile space is row perm[t] of H
    ScaleGroup SB;
    const int b_row0 = tt * Cfg::BN + wave_n<Cfg>() * (Cfg::TN * 32);      // this wavefront's first token
    if (FP8) SB.init(fp8.hscale, fp8.hgroups, b_row0 >> 7);

    float run_m[Cfg::TN], run_d[Cfg::TN], run_z[Cfg::TN];
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) { run_m[bn] = -INFINITY; run_d[bn] = 0.f; run_z[bn] = 0.f; }

    for (int vt = vt0; vt < vt1; ++vt) {
        f32x16 acc[Cfg::TM][Cfg::TN];
#pragma unroll
        for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
            for (int bn = 0; bn < Cfg::TN; ++bn)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[bm][bn][r] = 0.f;

        OperandTile<true, Cfg::BM, false, Cfg::NW, Cfg::BK> Aop;
        Aop.init(W, ld, vt * Cfg::BM, V, ld);
        if constexpr (FP8) {
            ScaleGroup SA;
            SA.init(fp8.wscale, fp8.wgroups, (vt * Cfg::BM + wm * (Cfg::TM * 32)) >> 7);
            gemm_mainloop_fp8<Cfg>(acc, Aop, Bop, SA, SB, (b_row0 >> 6) & 1, D, smem);
        } else {
            gemm_mainloop<Cfg, true, true>(acc, Aop, Bop, D, smem);
        }

        if ((vt + 1) * Cfg::BM > V) {       // ragged last vocabulary tile: mask rows >= V
#pragma unroll
            for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const bool dead = vt * Cfg::BM + acc_row<Cfg>(bm, r) >= V;
#pragma unroll
                    for (int bn = 0; bn < Cfg::TN; ++bn)
                        acc[bm][bn][r] = dead ? -INFINITY : acc[bm][bn][r];
                }
        }
#pragma unroll
        for (int bn = 0; bn < Cfg::TN; ++bn) {
            float tmax = -INFINITY;
#pragma unroll
            for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
                for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, acc[bm][bn][r]);
            const float mn = fmaxf(run_m[bn], tmax * kLog2e);
            const float ms = (mn == -INFINITY) ? 0.f : mn;
            float sum = 0.f;
#pragma unroll
            for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
                for (int r = 0; r < 16; ++r) sum += fast_exp2(fmaf(acc[bm][bn][r], kLog2e, -ms));
            run_d[bn] = run_d[bn] * fast_exp2(run_m[bn] - ms) + sum;
            run_m[bn] = mn;
            if (SUMZ) {
                float sz = 0.f;
#pragma unroll
                for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
                    for (int r = 0; r < 16; ++r) sz += (acc[bm][bn][r] == -INFINITY) ? 0.f : acc[bm][bn][r];   // masked tail rows
                run_z[bn] += sz;
            }
        }
    }

    // lanes l and l ^ 32 hold the same token column (different vocabulary rows)
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) {
        const float om = __shfl_xor(run_m[bn], 32), od = __shfl_xor(run_d[bn], 32);
        md_merge(run_m[bn], run_d[bn], om, od);
        if (SUMZ) run_z[bn] += __shfl_xor(run_z[bn], 32);
    }
    // the WM waves stacked along the vocabulary dimension share token columns: merge via LDS
    CCE_LDS f32x2* red = (CCE_LDS f32x2*)smem;        // [WM][BN]
    CCE_LDS float* redz = (CCE_LDS float*)(smem + Cfg::WM * Cfg::BN * 8);   // [WM][BN]
    if (l < 32) {
#pragma unroll
        for (int bn = 0; bn < Cfg::TN; ++bn) {
            red[wm * Cfg::BN + acc_col<Cfg>(bn)] = f32x2{run_m[bn], run_d[bn]};
            if (SUMZ) redz[wm * Cfg::BN + acc_col<Cfg>(bn)] = run_z[bn];
        }
    }
    __syncthreads();
    if (threadIdx.x < Cfg::BN) {
        const int tok = tt * Cfg::BN + threadIdx.x;
        float m = -INFINITY, d = 0.f, z = 0.f;
#pragma unroll
        for (int w = 0; w < Cfg::WM; ++w) {
            const f32x2 p = red[w * Cfg::BN + threadIdx.x];
            md_merge(m, d, p.x, p.y);
            if (SUMZ) z += redz[w * Cfg::BN + threadIdx.x];
        }
        if (tok < N) {
            partials[(size_t)tok * S + s] = make_float2(m, d);
            if (SUMZ) partial_sumz[(size_t)tok * S + s] = z;
        }
    }
}

// Lanes 32 ... 63 of a and lanes 0 ... 31 of b change places; the same of the odd rows of 16 lanes of a and the even ones of b.
__device__ __forceinline__ void swap_halves(float& a, float& b) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float((uint32_t)s[0]);
    b = __uint_as_float((uint32_t)s[1]);
}
__device__ __forceinline__ void swap_rows(float& a, float& b) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float((uint32_t)s[0]);
    b = __uint_as_float((uint32_t)s[1]);
}

// The same on tiles of two groups of wavefronts (see PingTile), bf16 operands, where that is faster (forward_tile).  The vocabulary
// split is cut at multiples of half a tile's rows (a last half tile saves a third of its slices' time: half of the products and of A's
// fragments, none of the loads nor of the epilogue), and a workgroup's slices follow each other without a gap: the first slice of a
// vocabulary tile is requested in front of the last products of the one before.  A token column lies in four lane groups: each
// keeps the (max, sum) of a quarter of the columns.  A tile's parts are formed in each lane by itself and get to those groups by
// lanes that change places, 12 instructions a tile without LDS: a common maximum by 32 shuffles through LDS in front of the
// exponentials made forwards of few slices slower than lse_partial_kernel's (256 x 256 tiles, us, that one / shuffles / this:
// 29040 x 64 x 32290 239 / 291 / 257, 8883 x 128 x 97046 290 / 323 / 290, 23189 x 256 x 84156 992 / 1048 / 969).
template <bool SUMZ, class Cfg>
__global__ __launch_bounds__(Cfg::kThreads, 2) void lse_partial_ping_kernel(
        const void* __restrict__ H, const void* __restrict__ W,
        int N, int D, int V, int TT, int S, float2* __restrict__ partials, float* __restrict__ partial_sumz,
        const int32_t* __restrict__ perm, int32_t* __restrict__ status, const int32_t* __restrict__ rows_splits) {
    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    CCE_LDS char* smem = (CCE_LDS char*)smem_generic;
    if (status && blockIdx.x == 0 && threadIdx.x == 0) status[0] = 0;        // (see lse_partial_kernel)
    if (rows_splits) {
        N = rows_splits[0];
        S = rows_splits[1];
        TT = (N + Cfg::BN - 1) / Cfg::BN;
        if (rows_splits[3]) perm = nullptr;           // every row takes part
    }
    const int n_work = rows_splits ? TT * S : (int)gridDim.x;
    if ((int)blockIdx.x >= n_work) return;
    const int lin = xcd_round_id(blockIdx.x, n_work, 256);
    int tt, s;
    group_map(lin, TT, S, 4, tt, s);                  // (an XCD's workgroups: 4 token tiles x all splits, see lse_partial_kernel)
    constexpr int kUnit = Cfg::BM / 2;
    const int units = (V + kUnit - 1) / kUnit;
    const int v_begin = (int)((int64_t)s * units / S) * kUnit;
    int v_end = (int)((int64_t)(s + 1) * units / S) * kUnit;
    v_end = v_end < V ? v_end : V;

    const uint32_t ld = (uint32_t)D * 2u;
    const int KT = D / Cfg::BK;
    PingPong<Cfg, ARows::kHalves> pp;
    PingLoads<Cfg, ARows::kHalves> loads;
    pp.init(smem);
    loads.init(smem, ld);
#pragma unroll
    for (int i = 0; i < Cfg::kBLoads; ++i) {
        int row = tt * Cfg::BN + loads.row(i);
        row = row < N ? row : N - 1;
        if (perm) {
            const int mapped = perm[row];             // token t of the tile space is row perm[t] of H
            row = mapped < 0 ? 0 : mapped;
        }
        loads.set_b_row(i, row, ld);
    }
    auto request = [&](int stage, int half) {
        if (loads.on) loads.issue(stage, half);
    };
    auto tile_rows = [&](int v) { return v_end - v < Cfg::BM ? v_end - v : Cfg::BM; };

    float run_m[Cfg::NB / 4], run_d[Cfg::NB / 4], run_z[Cfg::NB / 4];        // of column 4 q + lane group
#pragma unroll
    for (int q = 0; q < Cfg::NB / 4; ++q) { run_m[q] = -INFINITY; run_d[q] = 0.f; run_z[q] = 0.f; }
    const int g = (threadIdx.x & 63) >> 4;

    loads.on = true;
    loads.tile((const char*)W + (size_t)v_begin * ld, tile_rows(v_begin), (const char*)H, ld);
    // (what the compiler has loaded so far has to be there: it cannot see the loads of the slices)
    __builtin_amdgcn_s_waitcnt(0x0f70);               // vmcnt(0)
    loads.issue(0, 0);
    loads.issue(0, 1);
    pp.start();
    for (int v = v_begin; v < v_end; v += Cfg::BM) {
        f32x4 acc[Cfg::NA][Cfg::NB];
        const int rows = tile_rows(v), parts = rows > kUnit ? 2 : 1;
        auto next_slice = [&](int kt) {               // what slice kt's turns request
            if (kt + 1 < KT) {
                loads.a += 2 * Cfg::BK;
                loads.b += 2 * Cfg::BK;
            } else if (v + Cfg::BM < v_end) {
                loads.tile((const char*)W + (size_t)(v + Cfg::BM) * ld, tile_rows(v + Cfg::BM), (const char*)H, ld);
            } else {
                loads.on = false;
            }
        };
#pragma unroll
        for (int i = 0; i < Cfg::NA; ++i)
#pragma unroll
            for (int j = 0; j < Cfg::NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma nounroll
        for (int kt = 0;;) {
            next_slice(kt);
            pp.slice(acc, parts, request);
            if (++kt == KT) break;
            pp.barrier();
        }
        pp.tile_done();
        if (rows < Cfg::BM) {                         // rows that are not this split's
#pragma unroll
            for (int i = 0; i < Cfg::NA; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool dead = pp.row(i, r) >= rows;
#pragma unroll
                    for (int j = 0; j < Cfg::NB; ++j) acc[i][j][r] = dead ? -INFINITY : acc[i][j][r];
                }
        }
#pragma unroll
        for (int q = 0; q < Cfg::NB / 4; ++q) {
            float m[4], d[4], z[4];                   // of columns 4 q ... 4 q + 3, this lane's rows
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = 4 * q + e;
                float tmax = -INFINITY;
#pragma unroll
                for (int i = 0; i < Cfg::NA; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) tmax = fmaxf(tmax, acc[i][j][r]);
                m[e] = tmax * kLog2e;
                const float ms = (m[e] == -INFINITY) ? 0.f : m[e];
                d[e] = 0.f;
                z[e] = 0.f;
#pragma unroll
                for (int i = 0; i < Cfg::NA; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) d[e] += fast_exp2(fmaf(acc[i][j][r], kLog2e, -ms));
                if (SUMZ) {
#pragma unroll
                    for (int i = 0; i < Cfg::NA; ++i)
#pragma unroll
                        for (int r = 0; r < 4; ++r) z[e] += (acc[i][j][r] == -INFINITY) ? 0.f : acc[i][j][r];
                }
            }
            // the lane groups' parts of four columns become one column each: 32 lanes, then 16 lanes change places
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                swap_halves(m[e], m[e + 2]);
                swap_halves(d[e], d[e + 2]);
                md_merge(m[e], d[e], m[e + 2], d[e + 2]);
                if (SUMZ) { swap_halves(z[e], z[e + 2]); z[e] += z[e + 2]; }
            }
            swap_rows(m[0], m[1]);
            swap_rows(d[0], d[1]);
            md_merge(m[0], d[0], m[1], d[1]);
            md_merge(run_m[q], run_d[q], m[0], d[0]);
            if (SUMZ) { swap_rows(z[0], z[1]); run_z[q] += z[0] + z[1]; }
        }
        pp.tile_end();
    }
    pp.finish();

    // the WM wavefronts stacked along the vocabulary share token columns: merge via LDS
    CCE_LDS f32x2* red = (CCE_LDS f32x2*)smem;        // [WM][BN]
    CCE_LDS float* redz = (CCE_LDS float*)(smem + Cfg::WM * Cfg::BN * 8);   // [WM][BN]
#pragma unroll
    for (int q = 0; q < Cfg::NB / 4; ++q) {
        const int col = pp.wn * Cfg::TNR + (4 * q + g) * 16 + (int)(threadIdx.x & 15);
        red[pp.wm * Cfg::BN + col] = f32x2{run_m[q], run_d[q]};
        if (SUMZ) redz[pp.wm * Cfg::BN + col] = run_z[q];
    }
    __syncthreads();
    if (threadIdx.x < Cfg::BN) {
        const int tok = tt * Cfg::BN + threadIdx.x;
        float m = -INFINITY, d = 0.f, z = 0.f;
#pragma unroll
        for (int w = 0; w < Cfg::WM; ++w) {
            const f32x2 p = red[w * Cfg::BN + threadIdx.x];
            md_merge(m, d, p.x, p.y);
            if (SUMZ) z += redz[w * Cfg::BN + threadIdx.x];
        }
        if (tok < N) {
            partials[(size_t)tok * S + s] = make_float2(m, d);
            if (SUMZ) partial_sumz[(size_t)tok * S + s] = z;
        }
    }
}

// ------------------------------------------------------------------------------------------
// Forward finalisation: one wavefront per token.
// ------------------------------------------------------------------------------------------
// With `stats` (vocabulary-parallel share): W holds the rows [v_off, v_off + V) of the full
// matrix; instead of a loss the kernel writes, for EVERY token, the shard's statistics
// stats[tok] = (max logit, sum exp(z - max), label logit or 0 when the label lies in another
// shard, sum of logits or 0) in natural units; labels are not judged here.
__global__ __launch_bounds__(256) void finalize_kernel(
        const uint16_t* __restrict__ H, const uint16_t* __restrict__ W, const int32_t* __restrict__ labels,
        const float2* __restrict__ partials, const float* __restrict__ partial_sumz,
        int N, int D, int V, int S, int32_t ignore_index, float label_smoothing, float z_loss,
        float* __restrict__ loss, float* __restrict__ lse, int32_t* __restrict__ status,
        int v_off, float4* __restrict__ stats, const Fp8Scales fp8, const int32_t* __restrict__ perm,
        const int32_t* __restrict__ rows_splits) {
    if (rows_splits) S = rows_splits[1];
    const int l = threadIdx.x & 63;
    const int ctok = blockIdx.x * 4 + (threadIdx.x >> 6);     // token of the (compact) tile space
    if (ctok >= N) return;
    // row skipping: partials are indexed by the compact token, everything else by the original row
    const int tok = perm ? perm[ctok] : ctok;
    if (tok < 0) return;
    const int64_t y_local = (int64_t)labels[tok] - v_off;
    const int32_t y = (y_local >= 0 && y_local < V) ? (int32_t)y_local : -1;     // row of W, or none
    const bool in_range = y >= 0;
    if (!stats && (labels[tok] == ignore_index || !in_range)) {
        if (l == 0) {
            loss[tok] = 0.f;
            lse[tok] = 0.f;
            if (labels[tok] != ignore_index) atomicOr(status, CCE_STATUS_BAD_LABEL);
        }
        return;
    }
    float m = -INFINITY, d = 0.f, sumz = 0.f;
    for (int i = l; i < S; i += 64) {
        const float2 p = partials[(size_t)ctok * S + i];
        md_merge(m, d, p.x, p.y);
        if (partial_sumz) sumz += partial_sumz[(size_t)ctok * S + i];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const float om = __shfl_xor(m, o), od = __shfl_xor(d, o);
        md_merge(m, d, om, od);
        sumz += __shfl_xor(sumz, o);
    }
    // label logit: fp32 dot product of the two bf16 rows
    const uint16_t* h = H + (size_t)tok * D;
    const uint16_t* w = W + (size_t)(in_range ? y : 0) * D;
    float zy = 0.f;
    if (fp8.hscale) {
        // E4M3 rows: four codes per lane and step, decoded by the hardware conversion, the
        // 128-block's two scale exponents applied exactly with ldexp
        const uint8_t* h8 = (const uint8_t*)H + (size_t)tok * D;
        const uint8_t* w8 = (const uint8_t*)W + (size_t)(in_range ? y : 0) * D;
        for (int k = l * 4; in_range && k < D; k += 256) {
            const int hv = *(const int*)(h8 + k), wv = *(const int*)(w8 + k);
            const f32x2 h01 = __builtin_amdgcn_cvt_pk_f32_fp8(hv, false), h23 = __builtin_amdgcn_cvt_pk_f32_fp8(hv, true);
            const f32x2 w01 = __builtin_amdgcn_cvt_pk_f32_fp8(wv, false), w23 = __builtin_amdgcn_cvt_pk_f32_fp8(wv, true);
            const float p = fmaf(h01.x, w01.x, fmaf(h01.y, w01.y, fmaf(h23.x, w23.x, h23.y * w23.y)));
            zy += ldexpf(p, scale_byte(fp8.hscale, fp8.hgroups, tok, k >> 7) + scale_byte(fp8.wscale, fp8.wgroups, y, k >> 7) - 254);
        }
    } else
    for (int k = l * 2; in_range && k < D; k += 128) {
        const uint32_t hv = *(const uint32_t*)(h + k), wv = *(const uint32_t*)(w + k);
        zy = fmaf(__uint_as_float(hv << 16), __uint_as_float(wv << 16), zy);
        zy = fmaf(__uint_as_float(hv & 0xffff0000u), __uint_as_float(wv & 0xffff0000u), zy);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) zy += __shfl_xor(zy, o);
    if (l == 0 && stats) {
        stats[tok] = make_float4(m * kLn2, d, zy, sumz);
    } else if (l == 0) {
        const float out = (m + fast_log2(d)) * kLn2;
        lse[tok] = out;
        // (1 - eps) (lse - z_y) + eps (lse - mean_v z_v) + lambda lse^2   (smoothed cross-entropy
        // and z-loss definitions); eps = lambda = 0 leaves lse - z_y
        float t = out - zy;
        if (label_smoothing != 0.f) t = (1.f - label_smoothing) * t + label_smoothing * (out - sumz / (float)V);
        if (z_loss != 0.f) t = fmaf(z_loss * out, out, t);
        loss[tok] = t;
    }
}

// Vocabulary-parallel merge: one thread per token folds the P shard statistics
// stats[p * N + tok] = (m, d, z_y, sum z) in shard order with the online-softmax merge and
// writes the same loss / lse as finalize_kernel does for the undivided vocabulary.
__global__ __launch_bounds__(256) void shard_merge_kernel(
        const float4* __restrict__ stats, int P, const int32_t* __restrict__ labels, int N, int V,
        int32_t ignore_index, float label_smoothing, float z_loss,
        float* __restrict__ loss, float* __restrict__ lse, int32_t* __restrict__ status) {
    const int tok = blockIdx.x * 256 + threadIdx.x;
    if (tok >= N) return;
    const int32_t y = labels[tok];
    if (y == ignore_index || y < 0 || y >= V) {
        loss[tok] = 0.f;
        lse[tok] = 0.f;
        if (y != ignore_index && status) atomicOr(status, CCE_STATUS_BAD_LABEL);
        return;
    }
    float m = -INFINITY, d = 0.f, zy = 0.f, sumz = 0.f;
    for (int p = 0; p < P; ++p) {
        const float4 st = stats[(size_t)p * N + tok];
        md_merge(m, d, st.x * kLog2e, st.y);
        zy += st.z;
        sumz += st.w;
    }
    const float out = (m + fast_log2(d)) * kLn2;
    lse[tok] = out;
    float t = out - zy;
    if (label_smoothing != 0.f) t = (1.f - label_smoothing) * t + label_smoothing * (out - sumz / (float)V);
    if (z_loss != 0.f) t = fmaf(z_loss * out, out, t);
    loss[tok] = t;
}

// Number of rows that take part in the loss (label in range and not ignore_index), counted by
// one workgroup.  Integer counting: the result does not depend on the order.
__device__ __forceinline__ int count_valid_rows(const int32_t* labels, int N, int V, int32_t ignore_index, int* scratch) {
    constexpr int U = 8;            // loads in flight per thread: one workgroup, bound by their latency
    int c = 0;
    for (int i = threadIdx.x; i < N; i += U * blockDim.x) {
        int32_t y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) y[u] = i + u * (int)blockDim.x < N ? labels[i + u * (int)blockDim.x] : ignore_index;
#pragma unroll
        for (int u = 0; u < U; ++u) c += (y[u] != ignore_index && y[u] >= 0 && y[u] < V) ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o);
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = c;
    __syncthreads();
    int total = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) total += scratch[w];
    __syncthreads();
    return total;
}

// Mean reduction of the backward: every row's upstream gradient is grad_scale / n_valid
// (the materialising cross-entropy kernel of the paper divides the gradient by the number
// of non-ignored rows).  One workgroup of 1024 threads; out is a single float.
__global__ __launch_bounds__(1024) void mean_scale_kernel(const int32_t* __restrict__ labels, int N, int V,
                                                          int32_t ignore_index, float grad_scale, float* __restrict__ out) {
    __shared__ int scratch[16];
    const int n = count_valid_rows(labels, N, V, ignore_index, scratch);
    if (threadIdx.x == 0) out[0] = n > 0 ? grad_scale / (float)n : 0.f;
}

// Mean of the per-token losses over the non-ignored rows (0 when there are none).  One
// workgroup; each thread sums a strided subset in fp32, then a fixed tree: the result is
// reproducible run to run.  `kept` (optional, device): the number of rows that took part, where
// that is not the number of valid labels (row skipping with a bound that dropped rows).
__global__ __launch_bounds__(1024) void mean_loss_kernel(const float* __restrict__ loss, const int32_t* __restrict__ labels,
                                                         int N, int V, int32_t ignore_index, float* __restrict__ out,
                                                         const int32_t* __restrict__ kept) {
    __shared__ int scratch[16];
    __shared__ float fsum[16];
    const int n = kept ? kept[0] : count_valid_rows(labels, N, V, ignore_index, scratch);
    constexpr int U = 8;            // loads in flight per thread
    float a = 0.f;
    for (int i = threadIdx.x; i < N; i += U * blockDim.x) {              // ignored rows hold 0
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = i + u * (int)blockDim.x < N ? loss[i + u * (int)blockDim.x] : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) a += v[u];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) a += __shfl_xor(a, o);
    if ((threadIdx.x & 63) == 0) fsum[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int w = 0; w < 16; ++w) t += fsum[w];
        out[0] = n > 0 ? t / (float)n : 0.f;
    }
}

// ------------------------------------------------------------------------------------------
// Rows of `rows` planned ones that take part when the first is number `first` of those that do (count[0] in all).
__device__ __forceinline__ int rows_left(const int32_t* count, int first, int rows) {
    const int left = count[0] - first;
    return left < 0 ? 0 : (left < rows ? left : rows);
}

// ------------------------------------------------------------------------------------------
// Backward, step 1: recompute one logit tile and store the bf16 gradient tile
//   G[i, v] = dloss_i * ((1 + 2 lambda lse_i) exp(z_iv - lse_i) - (1 - eps) [v == y_i] - eps / V),
//   0 where the row is ignored / beyond N or the column is beyond V.  eps = lambda = 0 is the
//   plain softmax - onehot of the CCE backward theorem; eps is the label-smoothing weight
//   (smoothed cross-entropy definition), lambda the z-loss weight (z-loss gradient
//   proposition).  dloss == nullptr selects mean reduction: dloss_i = *mean_scale for all i.
// W may be a vocabulary shard: its V rows are the rows [v_off, v_off + V) of a V_total-row
// matrix, labels index the full one (v_off = 0, V_total = V without sharding).
// Same orientation as the forward (lane owns a token column).  The tile is staged in LDS as
// [token][vocab] and written to the scratch chunk G in panels of 1 << panel_shift vocabulary columns (see PanelTile).
// Grid: one workgroup per tile of the [row block x chunk]; tile index -> (ti, vi).
// ------------------------------------------------------------------------------------------
template <bool FP8, class Cfg = TileBig>
__global__ __launch_bounds__(Cfg::kThreads, 2) void grad_tile_kernel(
        const void* __restrict__ H, const void* __restrict__ W, const int32_t* __restrict__ labels,
        const float* __restrict__ lse, const float* __restrict__ dloss, const float* __restrict__ mean_scale,
        int N, int D, int V, int32_t ignore_index, float label_smoothing, float z_loss,
        int row0, int n_row_tiles, int v0, int n_v_tiles,
        uint16_t* __restrict__ G, uint32_t panel, int panel_shift, int v_off, int V_total, const Fp8Scales fp8,
        const int32_t* __restrict__ perm, const int32_t* __restrict__ count, int first_row) {
    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    CCE_LDS char* smem = (CCE_LDS char*)smem_generic;
    const int l = threadIdx.x & 63;
    const int wm = wave_m<Cfg>();

    // (count: the rows that take part, where only the device knows; this launch's begin at first_row of them)
    if (count) {
        N = rows_left(count, first_row, N);
        n_row_tiles = (N + 255) / 256 * (256 / Cfg::BN);        // whole 256-row tiles: the contractions read them
        if (count[1]) {                               // every row takes part: no lookup in front of the first slice
            H = (const char*)H + (size_t)first_row * (size_t)D * (FP8 ? 1 : 2);
            perm = nullptr;
        }
    }
    if ((int)blockIdx.x >= n_row_tiles * n_v_tiles) return;
    const int lin = xcd_round_id(blockIdx.x, n_row_tiles * n_v_tiles, 2048 / Cfg::NW);
    int ti, vi;
    group_map(lin, n_row_tiles, n_v_tiles, 32 / Cfg::NW, ti, vi);          // an XCD works on ~4 x 8 tiles
    const int tok0 = row0 + ti * Cfg::BN;        // first token of the tile (global index)
    const int vt0 = v0 + vi * Cfg::BM;           // first vocabulary row of the tile (global index)

    f32x16 acc[Cfg::TM][Cfg::TN];
#pragma unroll
    for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
        for (int bn = 0; bn < Cfg::TN; ++bn)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[bm][bn][r] = 0.f;

    // Per-token scalars of this lane's columns, and the label of the row this thread will flag:
    // only the raw loads are issued here -- unconditional, from clamped indices, so that there is
    // no branch the compiler would have to wait behind -- and everything derived from them is
    // computed after the main loop, under which their latency hides.
    int32_t raw_y[Cfg::TN], raw_row_y;
    float raw_dl[Cfg::TN], raw_ls[Cfg::TN];
    const float uniform_dl = dloss ? 0.f : mean_scale[0];
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) {
        const int tok = tok0 + acc_col<Cfg>(bn);
        const int t = tok < N ? tok : N - 1;
        raw_y[bn] = labels[t];
        raw_dl[bn] = dloss ? dloss[t] : uniform_dl;
        raw_ls[bn] = lse[t];
    }
    {
        const int tok = tok0 + (int)(threadIdx.x & (Cfg::BN - 1));
        raw_row_y = labels[tok < N ? tok : N - 1];
    }

    OperandTile<true, Cfg::BM, false, Cfg::NW, Cfg::BK> Aop;
    OperandTile<true, Cfg::BN, false, Cfg::NW, Cfg::BK> Bop;
    const int ld = FP8 ? D / 2 : D;               // row length in 2-byte units
    Aop.init(W, ld, vt0, V, ld);
    Bop.init(H, ld, tok0, N, ld, perm);           // perm (row skipping): token t is row perm[t] of H
    if constexpr (FP8) {
        ScaleGroup SA, SB;
        const int b_row0 = first_row + tok0 + wave_n<Cfg>() * (Cfg::TN * 32);       // (counted rows: scales in their order)
        SA.init(fp8.wscale, fp8.wgroups, (vt0 + wm * (Cfg::TM * 32)) >> 7);
        SB.init(fp8.hscale, fp8.hgroups, b_row0 >> 7);
        gemm_mainloop_fp8<Cfg>(acc, Aop, Bop, SA, SB, (b_row0 >> 6) & 1, D, smem);
    } else {
        gemm_mainloop<Cfg, true, true>(acc, Aop, Bop, D, smem);
    }

    int32_t col_y[Cfg::TN];
    float col_sp[Cfg::TN], col_ch[Cfg::TN], col_ncs[Cfg::TN], col_nl2[Cfg::TN];
    const float eps_over_v = label_smoothing / (float)V_total;
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) {
        const bool tok_ok = tok0 + acc_col<Cfg>(bn) < N;
        // label as a row of W (W holds the rows [v_off, v_off + V) of a V_total-row matrix)
        const int64_t y_local = tok_ok ? (int64_t)raw_y[bn] - v_off : -1;
        col_y[bn] = (y_local >= 0 && y_local < V) ? (int32_t)y_local : -1;
        const float dl = tok_ok ? raw_dl[bn] : 0.f;
        const float ls = tok_ok ? raw_ls[bn] : 0.f;
        col_sp[bn] = dl * fmaf(2.f * z_loss, ls, 1.f);      // factor of the softmax term
        col_ch[bn] = dl * (1.f - label_smoothing);          // subtracted at the label
        col_ncs[bn] = -dl * eps_over_v;                     // added everywhere
        col_nl2[bn] = -ls * kLog2e;
    }
    const bool row_live = threadIdx.x < Cfg::BN && tok0 + (int)threadIdx.x < N &&
                          raw_row_y != ignore_index && raw_row_y >= 0 && raw_row_y < V_total;

    CCE_LDS unsigned char* live_flags = (CCE_LDS unsigned char*)(smem + Cfg::BN * kGRowBytes<Cfg>);
    if (threadIdx.x < Cfg::BN) live_flags[threadIdx.x] = row_live ? 1 : 0;

    // Epilogue: softmax gradient, bf16, staged in LDS as [token][vocab] and stored with
    // whole 128-byte lines of the panels.  Done in TN phases (the 32 token columns per wavefront of block
    // bn): the global stores of one phase drain while the next phase is computed, and the
    // barriers wait for LDS traffic only.
    const bool ragged = vt0 + Cfg::BM > V;                  // only the last vocabulary tile needs column masking
    constexpr int kChunks = Cfg::BM / 8, kRowsPerPass = Cfg::kThreads / kChunks;       // 16-byte chunks of a row
    const int chunk = threadIdx.x % kChunks;
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) {
        const int col = acc_col<Cfg>(bn);
        const int32_t y = col_y[bn];
        const float sp = col_sp[bn], ch = col_ch[bn], ncs = col_ncs[bn];
        const float nl2 = col_nl2[bn];
        const int yrel = y - (vt0 + wm * (Cfg::TM * 32));     // label relative to this wave's rows
        const bool hit = (yrel >= 0) && (yrel < Cfg::TM * 32);
#pragma unroll
        for (int bm = 0; bm < Cfg::TM; ++bm) {
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                float g[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] = fmaf(fast_exp2(fmaf(acc[bm][bn][r4 * 4 + e], kLog2e, nl2)), sp, ncs);
                const int rrel = bm * 32 + 8 * r4 + 4 * (l >> 5);      // first of 4 consecutive rows
                if (hit) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) g[e] -= (rrel + e == yrel) ? ch : 0.f;
                }
                const int vrow = wm * (Cfg::TM * 32) + rrel;            // row inside the tile
                if (ragged) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) g[e] = (vt0 + vrow + e < V) ? g[e] : 0.f;
                }
                union { __bf16 h[4]; u32x2 u; } pk;
#pragma unroll
                for (int e = 0; e < 4; ++e) pk.h[e] = (__bf16)g[e];
                // (token rows with bit 3 set keep the two 8-byte halves of every 16-byte chunk swapped:
                // with a row pitch that is a multiple of 16 bytes, rows c and c + 8 of the 16 lanes
                // an 8-byte write serves per cycle would otherwise hit the same LDS banks)
                *(CCE_LDS u32x2*)(smem + col * kGRowBytes<Cfg> + ((vrow * 2) ^ (col & 8))) = pk.u;
            }
        }
        barrier_lds_only();
        // rows of this phase: tokens 64 * wn + 32 * bn + (0..31) for the WN wavefront columns;
        // thread -> (row index t / kChunks + kRowsPerPass j, 16-byte chunk t % kChunks)
#pragma unroll
        for (int j = 0; j < (Cfg::WN * 32) / kRowsPerPass; ++j) {
            const int idx = (int)threadIdx.x / kChunks + kRowsPerPass * j;
            const int row = (idx >> 5) * (Cfg::TN * 32) + bn * 32 + (idx & 31);
            const bool live = live_flags[row] != 0;
            u32x4 v = {0u, 0u, 0u, 0u};
            if (live) {
                v = *(const CCE_LDS u32x4*)(smem + row * kGRowBytes<Cfg> + chunk * 16);
                if (row & 8) v = u32x4{v.z, v.w, v.x, v.y};           // undo the half swap of the staging writes
            }
            *(u32x4*)(G + (size_t)((vi * Cfg::BM + chunk * 8) >> panel_shift) * panel + ((size_t)(ti * Cfg::BN + row) << panel_shift) +
              ((chunk * 8) & ((1 << panel_shift) - 1))) = v;
        }
    }
}

// The same on tiles of two groups of wavefronts (see PingTile), bf16 operands; n_v_tiles of them cover the chunk's v_cols
// columns.  A lane holds eight consecutive columns of a token: the bf16 results go from the registers to the chunk, 16 bytes per
// lane and whole 64-byte pieces of a panel's rows, without staging or barriers.  The tokens' labels, lse and upstream gradients are
// brought into the LDS stage that the last slice leaves free.
template <class Cfg>
__device__ __forceinline__ void grad_tile_ping(
        const void* __restrict__ H, const void* __restrict__ W, const int32_t* __restrict__ labels,
        const float* __restrict__ lse, const float* __restrict__ dloss, const float* __restrict__ mean_scale,
        int N, int D, int V, int32_t ignore_index, float label_smoothing, float z_loss,
        int row0, int n_row_tiles, int v0, int v_cols, int n_v_tiles,
        uint16_t* __restrict__ G, uint32_t panel, int panel_shift, int v_off, int V_total,
        const int32_t* __restrict__ perm) {
    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    CCE_LDS char* smem = (CCE_LDS char*)smem_generic;
    const uint32_t ld = (uint32_t)D * 2u;
    if ((int)blockIdx.x >= n_row_tiles * n_v_tiles) return;
    const int lin = xcd_round_id(blockIdx.x, n_row_tiles * n_v_tiles, 256);
    int ti, vi;
    group_map(lin, n_row_tiles, n_v_tiles, 4, ti, vi);
    const int tok0 = row0 + ti * Cfg::BN;             // first token of the tile (global index)
    const int vt0 = v0 + vi * Cfg::BM;                // first vocabulary row of the tile (global index)
    const float uniform_dl = dloss ? 0.f : mean_scale[0];

    PingPong<Cfg, ARows::kPairs> pp;
    PingLoads<Cfg, ARows::kPairs> loads;
    pp.init(smem);
    loads.init(smem, ld);
#pragma unroll
    for (int i = 0; i < Cfg::kBLoads; ++i) {
        int row = tok0 + loads.row(i);
        row = row < N ? row : N - 1;
        if (perm) {
            const int mapped = perm[row];             // (row skipping: token t is row perm[t] of H)
            row = mapped < 0 ? 0 : mapped;
        }
        loads.set_b_row(i, row, ld);
    }
    const int w_row = vt0 < V ? vt0 : V - 1;          // (the last tile of a chunk may lie behind the matrix: zeros)
    loads.tile((const char*)W + (size_t)w_row * ld, V - w_row < Cfg::BM ? V - w_row : Cfg::BM, (const char*)H, ld);
    __builtin_amdgcn_s_waitcnt(0x0f70);               // vmcnt(0): see lse_partial_ping_kernel
    loads.issue(0, 0);
    loads.issue(0, 1);

    const int KT = D / Cfg::BK;
    f32x4 acc[Cfg::NA][Cfg::NB];
#pragma unroll
    for (int i = 0; i < Cfg::NA; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    loads.on = true;
    auto request = [&](int stage, int half) {
        if (loads.on) {
            loads.issue(stage, half);
        } else if (half == 0) {
            // the last slice: the tokens' scalars, 256 of each, labels and lse by the wavefronts of group 0, dloss by those of group 1
            const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), part = wave & 3;
            int tok = tok0 + part * 64 + (int)(threadIdx.x & 63);
            tok = tok < N ? tok : N - 1;
            const uint32_t to = (uint32_t)(uintptr_t)smem + (uint32_t)stage * Cfg::kStage + (uint32_t)part * 256u;
            if (wave < 4) {
                load4_to_lds_sbase(labels, (uint32_t)tok * 4u, to);
                load4_to_lds_sbase(lse, (uint32_t)tok * 4u, to + 1024u);
            } else if (dloss) {
                load4_to_lds_sbase(dloss, (uint32_t)tok * 4u, to + 2048u);
            }
        }
    };
    static_assert(Cfg::BN == 256, "four wavefronts of tokens");
    pp.start();
#pragma nounroll
    for (int kt = 0;;) {
        loads.a += 2 * Cfg::BK;
        loads.b += 2 * Cfg::BK;
        loads.on = kt + 1 < KT;
        pp.slice(acc, 2, request);
        if (++kt == KT) break;
        pp.barrier();
    }
    pp.tile_done();
    const CCE_LDS int32_t* const raw_y = (const CCE_LDS int32_t*)(smem + pp.cur * Cfg::kStage);
    const CCE_LDS float* const raw_ls = (const CCE_LDS float*)(raw_y + 256);
    const CCE_LDS float* const raw_dl = raw_ls + 256;

    const float eps_over_v = label_smoothing / (float)V_total;
    const bool ragged = vt0 + Cfg::BM > V;            // only the last vocabulary tile needs column masking
    const int g = (threadIdx.x & 63) >> 4;
    const int wave_col = vi * Cfg::BM + pp.wm * Cfg::TMR;         // first column of this wavefront in the chunk
#pragma unroll
    for (int j = 0; j < Cfg::NB; ++j) {
        const int t = pp.col(j);
        const int32_t label = raw_y[t];
        const bool live = tok0 + t < N && label != ignore_index && label >= 0 && label < V_total;
        const float ls = raw_ls[t], dl = dloss ? raw_dl[t] : uniform_dl;
        const float sp = dl * fmaf(2.f * z_loss, ls, 1.f);        // factor of the softmax term
        const float ch = dl * (1.f - label_smoothing);            // subtracted at the label
        const float ncs = -dl * eps_over_v;                       // added everywhere
        const float nl2 = -ls * kLog2e;
        // label as a column relative to this lane's first one (W holds the rows [v_off, v_off + V) of V_total)
        const int64_t y_local = (int64_t)label - v_off;
        const int yrel = y_local >= 0 && y_local < V ? (int)y_local - v0 - wave_col - 8 * g : -1;
#pragma unroll
        for (int q = 0; q < Cfg::NA / 2; ++q) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = fmaf(fast_exp2(fmaf(acc[2 * q + e / 4][j][e % 4], kLog2e, nl2)), sp, ncs);
            const int hit = yrel - 32 * q;
            if (hit >= 0 && hit < 8) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] -= e == hit ? ch : 0.f;
            }
            const int c = wave_col + 32 * q + 8 * g;              // column in the chunk
            if (ragged) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = v0 + c + e < V ? x[e] : 0.f;
            }
            union { __bf16 h[8]; u32x4 u; } pk;
#pragma unroll
            for (int e = 0; e < 8; ++e) pk.h[e] = (__bf16)x[e];
            if (!live) pk.u = u32x4{0u, 0u, 0u, 0u};
            if (wave_col + 32 * q < v_cols)
                *(u32x4*)(G + (size_t)(c >> panel_shift) * panel + ((size_t)(ti * Cfg::BN + t) << panel_shift) + (c & ((1 << panel_shift) - 1))) = pk.u;
        }
    }
    pp.tile_end();
    pp.finish();
}

template <class Cfg>
__global__ __launch_bounds__(Cfg::kThreads, 2) void grad_tile_ping_kernel(
        const void* __restrict__ H, const void* __restrict__ W, const int32_t* __restrict__ labels,
        const float* __restrict__ lse, const float* __restrict__ dloss, const float* __restrict__ mean_scale,
        int N, int D, int V, int32_t ignore_index, float label_smoothing, float z_loss,
        int row0, int n_row_tiles, int v0, int v_cols, int n_v_tiles,
        uint16_t* __restrict__ G, uint32_t panel, int panel_shift, int v_off, int V_total, const int32_t* __restrict__ perm) {
    grad_tile_ping<Cfg>(H, W, labels, lse, dloss, mean_scale, N, D, V, ignore_index, label_smoothing, z_loss, row0, n_row_tiles, v0, v_cols,
                        n_v_tiles, G, panel, panel_shift, v_off, V_total, perm);
}

// Counted rows (see grad_tile_kernel): the taller or the square tiles, whichever take less time for the row tiles that are left
// (tall_grad_tiles).  28 of 32 row tiles x 40 at D = 896: 1120 square ones are five rounds of 256 compute units, 756 tall ones three:
// 139 -> 120 us (both forms in one kernel: the registers of the taller one, 252, and all of the LDS, as that one has by itself).
__global__ __launch_bounds__(TileTall::kThreads, 2) void grad_tile_counted_kernel(
        const void* __restrict__ H, const void* __restrict__ W, const int32_t* __restrict__ labels,
        const float* __restrict__ lse, const float* __restrict__ dloss, const float* __restrict__ mean_scale,
        int N, int D, int V, int32_t ignore_index, float label_smoothing, float z_loss, int v0, int n_v_tiles,
        uint16_t* __restrict__ G, uint32_t panel, int panel_shift, int v_off, int V_total,
        const int32_t* __restrict__ perm, const int32_t* __restrict__ count, int first_row, int cus) {
    N = rows_left(count, first_row, N);
    if (N <= 0) return;
    const int n_row_tiles = (N + 255) / 256;
    if (count[1]) {                                   // every row takes part: no lookup in front of the first slice
        H = (const char*)H + (size_t)first_row * ((size_t)D * 2);
        perm = nullptr;
    }
    const int n_tall = (n_v_tiles * 256 + TileTall::BM - 1) / TileTall::BM;
    if (tall_grad_tiles(n_row_tiles, n_v_tiles, D, cus))
        grad_tile_ping<TileTall>(H, W, labels, lse, dloss, mean_scale, N, D, V, ignore_index, label_smoothing, z_loss, 0, n_row_tiles, v0,
                                 n_v_tiles * 256, n_tall, G, panel, panel_shift, v_off, V_total, perm);
    else
        grad_tile_ping<TileSquare>(H, W, labels, lse, dloss, mean_scale, N, D, V, ignore_index, label_smoothing, z_loss, 0, n_row_tiles, v0,
                                   n_v_tiles * 256, n_v_tiles, G, panel, panel_shift, v_off, V_total, perm);
}

// ------------------------------------------------------------------------------------------
// Backward, step 2: the two gradient contractions of one [row block x chunk], in ONE launch
// so that their tiles fill the GPU together.  Both have N = hidden dimension:
//   dH job (A K-major): C[token, d] = sum_v G[token, v] * W[v, d]
//   dW job (A K-slow ): C[vocab, d] = sum_i G[i, vocab] * H[i, d]
// A is the scratch chunk G (zero padded to tile multiples in both directions), B is a slice
// of an input tensor in K-slow layout.  The result is added to / stored in the job's output
// (see GemmJob for its two forms).  Rows >= m_valid and columns >= n_valid are
// dropped.  The host puts the job with the longer reduction first; xcd_two_job_map deals the items
// of both jobs to the workgroup ids so that every XCD starts with its share of the long ones.
// ------------------------------------------------------------------------------------------
// LDS of grad_gemm_kernel: the main loop's stages (the exchange between K groups fits them).
constexpr int kGemmLdsBig = TileBig::kLdsBytes, kGemmLdsNarrow = TileNarrow::kLdsBytes, kGemmLdsSmall = TileSmall::kLdsBytes;
constexpr int kGemmLdsDuo = TileDuo::kLdsBytes;
// Counted rows (mode 9): bytes of the row map's 16-bit entries, whole or as many as leave room for two workgroups to a unit.
template <class Cfg> constexpr int counted_table_bytes() { return Cfg::NW == 4 ? 80 * 1024 - Cfg::kLdsBytes : kRowTableBytes; }
static_assert(counted_table_bytes<TileDuo>() % 512 == 0 && counted_table_bytes<TileDuo>() > 0, "whole row tiles");
// Row skipping: the LDS table of one row block's row map (kRowTableBytes, plan.h) sits behind these.
static_assert(kGemmLdsNarrow + kRowTableBytes <= 160 * 1024 && kGemmLdsBig + kRowTableBytes <= 160 * 1024 && kGemmLdsSmall + kRowTableBytes <= 160 * 1024, "row table must fit the LDS");

// Tiles of two wavefront groups: the row table has room for the entries that a loop looks up behind its last slice, without use.
constexpr int kTurnTableBytes = kRowTableBytes + 128;
static_assert(TurnTile::kLdsBytes + kTurnTableBytes <= 160 * 1024, "row table must fit the LDS");

// Output of a job, one of three forms:
//   fp32 (the dW job): out_f32 (+)= C when `beta`.
//   fp32 running sum + bf16 result (the dH job): out_f32 is a workspace accumulator over the
//   vocabulary chunks; on the `final` chunk the sum is rounded to bf16 into out_hi (dHidden).
//   split running sum (the dH job, out_lo given): the fp32 sum is kept as two 16-bit planes --
//   the upper halves of the fp32 words in the bf16 output tensor itself (out_hi, whose final
//   content is written by the last chunk), the lower halves in the workspace (out_lo) -- so
//   that the accumulator costs 2 instead of 4 workspace bytes per element; the split is exact.
//   It costs ~2 us per launch (8-byte instead of 16-byte accesses) and is used only where the
//   smaller accumulator buys a better tiling.
//
// K split: a job with few output tiles and a long reduction is cut into n_split parts of split_k
// (a multiple of 256; the last part may be shorter), each a set of work items of its own.  Part 0
// goes to out_f32, part s >= 1 to the fp32 plane part + (s - 1) * part_stride; part s adds to what
// its output holds when s < beta_n.  The planes are summed by a later launch in a fixed order.
// What it is for: at N = 509, D = 896, V = 151936 the dH job is 14 tiles whose reduction of 2376
// slices lasted 1.7 ms while 242 compute units had nothing to do; in 6 parts (84 items beside the
// dW job's) the whole step went from 1825 to 778 us.  Where the reductions of both jobs fill the
// GPU anyway a split only adds plane traffic: the planner (plan.h) prices both.
struct GemmJob {
    int a_kmajor;               // 1: A is K-major (the dH job), 0: A is K-slow (the dW job)
    const uint16_t* A; uint32_t panel;           // the gradient chunk, see PanelTile
    const void* B; int ldb; int b_k_n; int k_total;
    int n_tiles; int n_work; int m_valid; int n_valid;
    int n_split; int split_k; float* part; int64_t part_stride;
    float* out_f32; int64_t ld_out; int beta_n;
    uint16_t* out_hi; uint16_t* out_lo; int final;
    const int32_t* row_map;     // row skipping: out_hi row of tile row r is row_map[r] (-1: none); else nullptr
    const char* zero_row;       // row skipping: a row of zeros, read by the dW job where no row takes part
    int first_row;              // row_map's first entry is that of this compact row
    const int32_t* count; int rows;             // counted rows (MODE 9): see rows_left
};

// Result of a work item, straight from the accumulators.  A lane holds one column of a 32 x 32 block and, per
// register, two rows of it lie in a wavefront: a dword store is two full 128-byte segments, so nothing is staged
// through LDS and only the K groups' exchange needs a barrier.  The 16-bit forms exchange values between neighbouring
// lanes first (even lanes keep the first of two rows, odd lanes the second), so that a lane again moves one dword:
// two neighbouring columns of a row.  Bound by the burst of stores and old values that all work items of a round make
// at once (256 of 256 x 128: 33 MB, 6 us at the rate of HBM) and by the latency of the first of them.  Measured against
// the tile staged through LDS for 16-byte row accesses, us per launch: 16 x 16 tiles at D = 896 60.2 -> 57.0, at
// D = 1024 64.2 -> 61.9, 12 x 20 at D = 1024 70.4 -> 65.8, 256 x 256 tiles of 16 x 16 at D = 1024 87.9 -> 85.2; only the
// planes of the split running sum lose (64-byte segments: items of 96 slices 101.1 -> 101.8).
template <class Cfg, bool A_KMAJOR, int MODE>
__device__ __forceinline__ void store_result(f32x16 (&acc)[Cfg::TM][Cfg::TN], const GemmJob& j, float* out, bool beta, int mi, int ni,
                                             int m_valid, CCE_LDS char* smem) {
    constexpr bool SPLIT = A_KMAJOR && (MODE & 1) != 0, ROWMAP = A_KMAJOR && (MODE & 6) != 0;
    constexpr int KG = Cfg::KG, NB = Cfg::TM / KG;              // 32-row bands that a wavefront stores
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), l = threadIdx.x & 63;
    const int kg = wave / (Cfg::WM * Cfg::WN), wm = wave % (Cfg::WM * Cfg::WN) / Cfg::WN, wn = wave % Cfg::WN;
    const int row0 = mi * Cfg::BM + wm * (Cfg::TM * 32), col0 = ni * Cfg::BN + wn * (Cfg::TN * 32);
    const bool inside = col0 < j.n_valid;                       // all columns of a wavefront or none (n_valid is a multiple of 64)
    const uint32_t ld = (uint32_t)j.ld_out;
    // fp32 form: this lane's column, its four-row half; 16-bit forms: its pair of columns, its row of the pair
    const uint32_t lane_off = (uint32_t)(4 * (l >> 5)) * ld + (uint32_t)(l & 31);
    const int pair_row = 4 * (l >> 5) + (l & 1), pair_col = l & 30;
    auto block_row = [](int r) { return 8 * (r >> 2) + (r & 3); };         // of register r, without the lane's half

    auto run = [&](auto first, auto full) {
        constexpr int B0 = decltype(first)::value;
        constexpr bool FULL = decltype(full)::value;
        float old[2][Cfg::TN][16];                              // split form: 8 words of upper halves, 8 of lower halves
        int orow[2][8];                                         // split form: out_hi row of each register pair
        auto fetch = [&](int set, int bm) {
            const int brow = row0 + bm * 32;
            if constexpr (SPLIT) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int row = brow + block_row(2 * i) + pair_row;
                    orow[set][i] = row < m_valid ? (ROWMAP ? j.row_map[row] : row) : -1;
                }
            }
#pragma unroll
            for (int i = 0; i < (SPLIT ? 8 : 16) * Cfg::TN; ++i) {
                const int r = SPLIT ? i % 8 : i / Cfg::TN, bn = SPLIT ? i / 8 : i % Cfg::TN;
                if constexpr (SPLIT) {
                    const int row = brow + block_row(2 * r) + pair_row, col = col0 + bn * 32 + pair_col;
                    const bool ok = row < m_valid && beta;
                    old[set][bn][r] = ok && orow[set][r] >= 0 ? *(const float*)(j.out_hi + (size_t)orow[set][r] * ld + col) : 0.f;
                    old[set][bn][8 + r] = ok ? *(const float*)(j.out_lo + (size_t)row * ld + col) : 0.f;
                } else {
                    const float* p = out + (size_t)(brow + block_row(r)) * ld + col0 + bn * 32;
                    old[set][bn][r] = FULL || brow + block_row(r) + 4 * (l >> 5) < m_valid ? p[lane_off] : 0.f;
                }
            }
        };
        if (inside && (beta || SPLIT)) fetch(0, B0);
        if constexpr (KG == 2) {
            // the two K groups hold partial sums of the same positions: each hands the blocks that it does not store to
            // its partner, a lane's registers to the same lane
            constexpr int O0 = B0 == 0 ? NB : 0;
            CCE_LDS char* mine = smem + (size_t)(wave * 16384 + l * 16);
#pragma unroll
            for (int b = 0; b < NB * Cfg::TN; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x16& v = acc[O0 + b / Cfg::TN][b % Cfg::TN];
                    *(CCE_LDS f32x4*)(mine + (b * 4 + q) * 1024) = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
                }
            if (inside && (beta || SPLIT)) fetch(1, B0 + 1);                // (NB = 2; the blocks handed over are free)
            barrier_lds_only();
        }
        if (!inside) return;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int bm = B0 + b, brow = row0 + bm * 32;
            __builtin_amdgcn_sched_barrier(0);                  // keeps the next band's registers out of this one
            if (KG == 1 && (beta || SPLIT) && b + 1 < NB) fetch((b + 1) & 1, bm + 1);
            // the blocks beside each other at once: a longer run of every row (one by one with the planes, whose old values
            // take the registers)
            constexpr int STEP = SPLIT ? 1 : Cfg::TN;
#pragma unroll
            for (int bn0 = 0; bn0 < Cfg::TN; bn0 += STEP) {
                float v[Cfg::TN][16];
#pragma unroll
                for (int bn = bn0; bn < bn0 + STEP; ++bn) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[bn][r] = acc[bm][bn][r];
                    if constexpr (KG == 2) {
                        const CCE_LDS char* theirs = smem + (size_t)((wave ^ (Cfg::WM * Cfg::WN)) * 16384 + l * 16);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x4 t = *(const CCE_LDS f32x4*)(theirs + ((b * Cfg::TN + bn) * 4 + q) * 1024);
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[bn][4 * q + e] += t[e];
                        }
                    }
                    if (!SPLIT && beta) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) v[bn][r] += old[b & 1][bn][r];
                    }
                }
                if (!SPLIT && !(A_KMAJOR && j.final)) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
#pragma unroll
                        for (int bn = bn0; bn < bn0 + STEP; ++bn) {
                            float* p = out + (size_t)(brow + block_row(r)) * ld + col0 + bn * 32;
                            if (FULL || brow + block_row(r) + 4 * (l >> 5) < m_valid) p[lane_off] = v[bn][r];
                        }
                    continue;
                }
                if constexpr (A_KMAJOR) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int row = brow + block_row(2 * i) + pair_row;
                        int to;
                        if constexpr (SPLIT) to = orow[b & 1][i];
                        else to = row < m_valid ? (ROWMAP ? j.row_map[row] : row) : -1;
#pragma unroll
                        for (int bn = bn0; bn < bn0 + STEP; ++bn) {
                            const int col = col0 + bn * 32 + pair_col;
                            // even lanes: (own, neighbour's) of register 2i; odd lanes: (neighbour's, own) of register 2i + 1
                            const float give = (l & 1) ? v[bn][2 * i] : v[bn][2 * i + 1];
                            const float got = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, give), 0xB1, 0xF, 0xF, true));
                            float x = (l & 1) ? got : v[bn][2 * i], y = (l & 1) ? v[bn][2 * i + 1] : got;
                            if constexpr (SPLIT) {
                                const uint32_t hi = __builtin_bit_cast(uint32_t, old[b & 1][bn][i]), lo = __builtin_bit_cast(uint32_t, old[b & 1][bn][8 + i]);
                                x += __builtin_bit_cast(float, (hi << 16) | (lo & 0xffffu));
                                y += __builtin_bit_cast(float, (hi & 0xffff0000u) | (lo >> 16));
                            }
                            if (j.final) {
                                union { __bf16 h[2]; uint32_t u; } cv;
                                cv.h[0] = (__bf16)x;
                                cv.h[1] = (__bf16)y;
                                uint16_t* const result = MODE == 9 ? j.out_lo : j.out_hi;
                                if (to >= 0) *(uint32_t*)(result + (size_t)to * ld + col) = cv.u;
                            } else {
                                const uint32_t bx = __builtin_bit_cast(uint32_t, x), by = __builtin_bit_cast(uint32_t, y);
                                if (to >= 0) *(uint32_t*)(j.out_hi + (size_t)to * ld + col) = (by & 0xffff0000u) | (bx >> 16);
                                if (row < m_valid) *(uint32_t*)(j.out_lo + (size_t)row * ld + col) = (by << 16) | (bx & 0xffffu);
                            }
                        }
                    }
                }
            }
        }
    };
    const bool full = row0 + Cfg::TM * 32 <= m_valid;
    auto with_rows = [&](auto first) {
        if (full) run(first, std::true_type{});
        else run(first, std::false_type{});
    };
    if (KG == 1 || kg == 0) with_rows(std::integral_constant<int, 0>{});
    else with_rows(std::integral_constant<int, Cfg::TM / 2>{});
}

// MODE bit 0: the launch's dH job uses the split running sum; bit 1: its bf16 rows go through
// row_map and the dW job reads hidden rows through it (row skipping in the caller's tensors);
// MODE 4: only the bf16 rows go through row_map (row skipping on a gathered copy of the hidden
// rows); MODE 9: the number of rows that take part is found on the device (count), the dW job reads hidden rows through
// row_map as 16-bit entries, the dH job's planes lie in compact rows and its bf16 result replaces the lower halves, from
// where scatter_rows_kernel takes it.  Launch-wide constants, compiled as separate kernels so that the plain form carries none
// of their code.  K split exists in modes 0 and 4.
template <class Cfg, bool A_KMAJOR, int MODE>
__device__ __forceinline__ void run_gemm_job(const GemmJob& j, int item, int rows, CCE_LDS char* smem) {
    constexpr bool COUNTED = (MODE & 8) != 0, KSPLIT = (MODE & 3) == 0 && !COUNTED;
    int part = 0;
    if (KSPLIT && j.n_split > 1) {
        const int per = j.n_work / j.n_split;
        part = item / per;
        item -= part * per;
    }
    const int k0 = KSPLIT ? part * j.split_k : 0;
    const int k_len = COUNTED && !A_KMAJOR ? (rows + 255) / 256 * 256 : !KSPLIT ? j.k_total : (j.k_total - k0 < j.split_k ? j.k_total - k0 : j.split_k);
    float* const out_f32 = part == 0 ? j.out_f32 : j.part + (size_t)(part - 1) * j.part_stride;
    const bool beta = part < j.beta_n;
    const int mi = item / j.n_tiles, ni = item % j.n_tiles;    // consecutive items share the A band

    f32x16 acc[Cfg::TM][Cfg::TN];
#pragma unroll
    for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
        for (int bn = 0; bn < Cfg::TN; ++bn)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[bm][bn][r] = 0.f;

    constexpr int kMapB = A_KMAJOR ? 0 : COUNTED ? 2 : (MODE & 2) != 0 ? 1 : 0;        // row skipping, dW job
    PanelTile<A_KMAJOR, Cfg::BM, Cfg::NW, Cfg::BK> Aop;
    OperandTile<false, Cfg::BN, kMapB, Cfg::NW, Cfg::BK> Bop;
    Aop.init(j.A, j.panel, mi * Cfg::BM, k0);
    Bop.init((const uint16_t*)j.B + (size_t)k0 * j.ldb, j.ldb, ni * Cfg::BN, j.n_valid, j.b_k_n - k0);
    if constexpr (kMapB == 1) {
        // row skipping, dW job: the reduction runs over the compact rows of the block, whose hidden rows are scattered over
        // the original tensor.  Their byte offsets are put into LDS, behind everything the kernel otherwise uses.
        // Compact rows that stand for none take the first valid row, whose products meet the chunk's zero rows;
        // where there is no valid row at all, a row of zeros (whatever a skipped row holds -- NaN included -- would
        // meet the other operand's zero in the MFMA).
        CCE_LDS uint32_t* tab = (CCE_LDS uint32_t*)(smem + Cfg::kLdsBytes);
        const int32_t some = __builtin_amdgcn_readfirstlane(j.row_map[-j.first_row]);
        for (int i = threadIdx.x; i < j.k_total; i += Cfg::kThreads) {
            const int32_t row = i < j.b_k_n ? j.row_map[i] : -1;
            tab[i] = some < 0 ? 0u : (uint32_t)(row < 0 ? some : row) * (uint32_t)(j.ldb * 2);
        }
        __syncthreads();
        Bop.kmap = tab;
        if (some < 0) Bop.base = j.zero_row;
    }
    constexpr int kMapRows = counted_table_bytes<Cfg>() / 2;
    constexpr bool kPieces = kMapB == 2 && kMapRows < kRowTableBytes / 2;
    for (int k1 = 0;;) {                                         // one pass, but for counted rows that exceed the table
        const int k_now = kPieces && k_len - k1 > kMapRows ? kMapRows : k_len - k1;
        if constexpr (kMapB == 2) {
            // the rows that take part, in 16 bits (at most 65536 rows); behind the last one (-1) that row again, whose products
            // meet the chunk's zero rows.  All loads at once (an entry per thread after the other: backward of
            // 8192 x 896 x 151936 with 15 % ignored 5.98 -> 5.96 ms, without 6.50 -> 6.47; FP8 logits 5.37 -> 5.35, 5.91 -> 5.87)
            CCE_LDS uint16_t* tab = (CCE_LDS uint16_t*)(smem + Cfg::kLdsBytes);
            constexpr int kQuads = kMapRows / (4 * Cfg::kThreads);
            const int32_t last = j.row_map[rows > 0 ? rows - 1 : 0];
            i32x4 m[kQuads];
#pragma unroll
            for (int u = 0; u < kQuads; ++u) {
                const int i = 4 * (u * Cfg::kThreads + (int)threadIdx.x);
                if (i < k_now) m[u] = *(const i32x4*)(j.row_map + k1 + i);
            }
#pragma unroll
            for (int u = 0; u < kQuads; ++u) {
                const int i = 4 * (u * Cfg::kThreads + (int)threadIdx.x);
                if (i < k_now) {
                    const i32x4 v = m[u];
                    *(CCE_LDS u32x2*)(tab + i) = u32x2{(uint32_t)(v.x < 0 ? last : v.x) | (uint32_t)(v.y < 0 ? last : v.y) << 16,
                                                       (uint32_t)(v.z < 0 ? last : v.z) | (uint32_t)(v.w < 0 ? last : v.w) << 16};
                }
            }
            __syncthreads();
            Bop.kmap16 = tab;
        }
        // Whatever the compiler loaded so far has to be there: it cannot see the main loop's loads, and a register still
        // waited for inside the loop (a field of the job, say) becomes a wait for all of them in every slice.
        __builtin_amdgcn_s_waitcnt(0x0f70);                      // vmcnt(0)
        gemm_mainloop<Cfg, A_KMAJOR, false, true>(acc, Aop, Bop, k_now, smem);           // ends with a barrier
        k1 += k_now;
        if (!kPieces || k1 >= k_len) break;
        Aop.init(j.A, j.panel, mi * Cfg::BM, k1);
    }

    store_result<Cfg, A_KMAJOR, MODE>(acc, j, out_f32, beta, mi, ni, COUNTED && A_KMAJOR ? rows : j.m_valid, smem);
}

// Result of a work item on tiles of two wavefront groups (TurnTile), straight from the accumulators.  A lane holds four columns of
// a result row in every block: fp32 results and what they are added to move 16 bytes at a time, two blocks to a 128-byte line.  In
// the 16-bit forms lanes of neighbouring 16 change places first, so that a lane has eight columns of one of two blocks: 16 bytes of
// either plane, 64 in a row.  Old values are fetched half a block column ahead.
template <bool A_KMAJOR, int MODE>
__device__ __forceinline__ void store_turn_result(f32x4 (&acc)[TurnTile::NA][TurnTile::NB], const GemmJob& j, float* out, bool beta, int row0, int col0, int m_valid, int wave) {
    constexpr bool SPLIT = A_KMAJOR && (MODE & 1) != 0, ROWMAP = A_KMAJOR && (MODE & 6) != 0;
    const int l = wave_lane(), lg = l >> 4;                     // (not from threadIdx: a register less over the loop)
    const int col = col0 + (wave >> 2) * 128;                   // this wavefront's first column
    row0 += (wave & 3) * 64 + (l & 15);             // this lane's row in block 0
    const uint32_t ld = (uint32_t)j.ld_out;
    const int pair_col = 16 * (lg & 1) + 4 * (lg & 2);          // 16-bit forms: this lane's eight columns of a pair of blocks
    auto run = [&](auto pairs_tag) {
        constexpr bool PAIRS = decltype(pairs_tag)::value;
        // step (block column jb, half h): blocks 4 h ... 4 h + 3, 64 columns
        f32x4 old[2][4];
        int to[2] = {-1, -1};                                   // 16-bit forms: result row, by the block column's parity
        auto fetch = [&](int set, int jb, int h) {
            const int row = row0 + 16 * jb, c0 = col + 64 * h;
            const bool ok = row < m_valid;
            if (PAIRS && h == 0) to[jb & 1] = !ok ? -1 : ROWMAP ? j.row_map[row] : row;
            if (!SPLIT && !beta) return;
#pragma unroll
            for (int i = 0; i < 4; ++i) old[set][i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (c0 >= j.n_valid) return;
            if constexpr (SPLIT) {
                // upper halves of pair i / 2 (old[0], old[2]), lower halves
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int c = c0 + 32 * (i >> 1) + pair_col;
                    const uint16_t* p = (i & 1) ? j.out_lo + (size_t)row * ld + c : j.out_hi + (size_t)to[jb & 1] * ld + c;
                    if (beta && to[jb & 1] >= 0) old[set][i] = *(const f32x4*)p;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int c = PAIRS ? c0 + 32 * (i >> 1) + pair_col + 4 * (i & 1) : c0 + 16 * i + 4 * lg;
                    if (ok) old[set][i] = *(const f32x4*)(out + (size_t)row * ld + c);
                }
            }
        };
        fetch(0, 0, 0);
#pragma unroll
        for (int s = 0; s < 2 * TurnTile::NB; ++s) {
            const int jb = s >> 1, h = s & 1, set = s & 1;
            __builtin_amdgcn_sched_barrier(0);
            if (s + 1 < 2 * TurnTile::NB) fetch(set ^ 1, (s + 1) >> 1, (s + 1) & 1);
            const int row = row0 + 16 * jb, c0 = col + 64 * h;
            const bool ok = row < m_valid;
            if (c0 >= j.n_valid) continue;
            if constexpr (!PAIRS) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    f32x4 v = acc[4 * h + i][jb];
                    if (beta) v += old[set][i];
                    if (ok) *(f32x4*)(out + (size_t)row * ld + c0 + 16 * i + 4 * lg) = v;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    float x[8];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        x[r] = acc[4 * h + 2 * i][jb][r];
                        x[4 + r] = acc[4 * h + 2 * i + 1][jb][r];
                        swap_rows(x[r], x[4 + r]);
                    }
                    const int c = c0 + 32 * i + pair_col, t = to[jb & 1];
                    if constexpr (SPLIT) {
                        const u32x4 hi = __builtin_bit_cast(u32x4, old[set][2 * i]), lo = __builtin_bit_cast(u32x4, old[set][2 * i + 1]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            x[2 * e] += __builtin_bit_cast(float, (hi[e] << 16) | (lo[e] & 0xffffu));
                            x[2 * e + 1] += __builtin_bit_cast(float, (hi[e] & 0xffff0000u) | (lo[e] >> 16));
                        }
                    } else if (beta) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) x[e] += old[set][2 * i + (e >> 2)][e & 3];
                    }
                    if (!SPLIT || j.final) {
                        union { __bf16 h[8]; u32x4 u; } cv;
#pragma unroll
                        for (int e = 0; e < 8; ++e) cv.h[e] = (__bf16)x[e];
                        uint16_t* const result = MODE == 9 ? j.out_lo : j.out_hi;
                        if (t >= 0) *(u32x4*)(result + (size_t)t * ld + c) = cv.u;
                    } else {
                        u32x4 hi, lo;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const uint32_t bx = __builtin_bit_cast(uint32_t, x[2 * e]), by = __builtin_bit_cast(uint32_t, x[2 * e + 1]);
                            hi[e] = (by & 0xffff0000u) | (bx >> 16);
                            lo[e] = (by << 16) | (bx & 0xffffu);
                        }
                        if (t >= 0) *(u32x4*)(j.out_hi + (size_t)t * ld + c) = hi;
                        if (ok) *(u32x4*)(j.out_lo + (size_t)row * ld + c) = lo;
                    }
                }
            }
        }
    };
    if (col >= j.n_valid) return;
    if (A_KMAJOR && (SPLIT || j.final)) run(std::true_type{});
    else if constexpr (!SPLIT) run(std::false_type{});
}

// One work item on such tiles (modes as for run_gemm_job).
template <bool A_KMAJOR, int MODE>
__device__ __forceinline__ void run_turn_item(const GemmJob& j, int item, int rows, CCE_LDS char* smem) {
    typedef TurnTile Cfg;
    constexpr bool COUNTED = (MODE & 8) != 0, KSPLIT = (MODE & 3) == 0 && !COUNTED;
    int part = 0;
    if (KSPLIT && j.n_split > 1) {
        const int per = j.n_work / j.n_split;
        part = item / per;
        item -= part * per;
    }
    const int row0 = item / j.n_tiles * Cfg::BN, col0 = item % j.n_tiles * Cfg::BM;       // consecutive items share rows of the chunk
    const int k0 = KSPLIT ? part * j.split_k : 0;
    int k_rows = j.b_k_n - k0;                                  // rows of X that take part
    if (KSPLIT && k_rows > j.split_k) k_rows = j.split_k;
    if (COUNTED && !A_KMAJOR) k_rows = rows;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    float* const out_f32 = part == 0 ? j.out_f32 : j.part + (size_t)(part - 1) * j.part_stride;
    const bool beta = part < j.beta_n;

    constexpr int MAP = A_KMAJOR ? 0 : COUNTED ? 2 : (MODE & 2) != 0 ? 1 : 0;
    const char* X = (const char*)j.B + (size_t)k0 * (size_t)(j.ldb * 2);
    if constexpr (MAP == 1) {                                   // (see run_gemm_job)
        CCE_LDS uint32_t* tab = (CCE_LDS uint32_t*)(smem + Cfg::kLdsBytes);
        const int32_t some = __builtin_amdgcn_readfirstlane(j.row_map[-j.first_row]);
        for (int i = threadIdx.x; i < j.k_total; i += kThreads) {
            const int32_t row = i < j.b_k_n ? j.row_map[i] : -1;
            tab[i] = some < 0 ? 0u : (uint32_t)(row < 0 ? some : row) * (uint32_t)(j.ldb * 2);
        }
        if (some < 0) X = j.zero_row;
        __syncthreads();
    }
    if constexpr (MAP == 2) {                                   // (see run_gemm_job)
        if (rows == 0) {                                        // none takes part: there is no chunk
            if (!beta)
                for (int i = threadIdx.x; i < Cfg::BN * 64; i += kThreads) {
                    const int row = row0 + i / 64, col = col0 + i % 64 * 4;
                    if (row < j.m_valid && col < j.n_valid) *(f32x4*)(out_f32 + (size_t)row * (uint32_t)j.ld_out + col) = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            return;
        }
        CCE_LDS uint16_t* tab = (CCE_LDS uint16_t*)(smem + Cfg::kLdsBytes);
        constexpr int kQuads = kRowTableBytes / 2 / (4 * kThreads);
        const int32_t last = j.row_map[rows > 0 ? rows - 1 : 0];
        const int n = (rows + 255) / 256 * 256;
        i32x4 m[kQuads];
#pragma unroll
        for (int u = 0; u < kQuads; ++u) {
            const int i = 4 * (u * kThreads + (int)threadIdx.x);
            if (i < n) m[u] = *(const i32x4*)(j.row_map + i);
        }
#pragma unroll
        for (int u = 0; u < kQuads; ++u) {
            const int i = 4 * (u * kThreads + (int)threadIdx.x);
            if (i < n) {
                const i32x4 v = m[u];
                *(CCE_LDS u32x2*)(tab + i) = u32x2{(uint32_t)(v.x < 0 ? last : v.x) | (uint32_t)(v.y < 0 ? last : v.y) << 16,
                                                   (uint32_t)(v.z < 0 ? last : v.z) | (uint32_t)(v.w < 0 ? last : v.w) << 16};
            }
        }
        __syncthreads();
    }
    TurnLoop<A_KMAJOR, MAP> loop;
    loop.init(smem, wave, X, (uint32_t)(j.ldb * 2), col0, j.n_valid, k_rows, j.A, j.panel, row0, k0);
    if (MAP == 1) loop.kmap = (const CCE_LDS uint32_t*)(smem + Cfg::kLdsBytes);
    if (MAP == 2) loop.kmap16 = (const CCE_LDS uint16_t*)(smem + Cfg::kLdsBytes);
    __builtin_amdgcn_s_waitcnt(0x0f70);                         // vmcnt(0): see run_gemm_job
    const int KT = loop.slices(k_rows);
    if (col0 + 128 * loop.group >= j.n_valid) {                 // (its columns lie behind the matrix: loads and barriers only)
        loop.idle(KT);
        return;
    }
    f32x4 acc[Cfg::NA][Cfg::NB];
#pragma unroll
    for (int a = 0; a < Cfg::NA; ++a)
#pragma unroll
        for (int b = 0; b < Cfg::NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    loop.run(acc, KT);
    store_turn_result<A_KMAJOR, MODE>(acc, j, out_f32, beta, row0, col0, COUNTED && A_KMAJOR ? rows : j.m_valid, wave);
}

template <class Cfg, int MODE>
__global__ __launch_bounds__(Cfg::kThreads, 2) void grad_gemm_kernel(const GemmJob first, const GemmJob second) {
    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    CCE_LDS char* smem = (CCE_LDS char*)smem_generic;
    constexpr bool COUNTED = (MODE & 8) != 0;
    constexpr int kRows = std::is_same<Cfg, TurnTile>::value ? 256 : Cfg::BM;        // result rows of an item
    int rows = 0, n1 = first.n_work, n2 = second.n_work;
    bool swapped = false;
    if constexpr (COUNTED) {
        // Items and reductions of the rows that take part: the dH job's items follow them, the dW job's reduction.
        rows = rows_left(first.count, first.first_row, first.rows);
        const int tiles = (rows + 255) / 256;
        auto items = [&](const GemmJob& j) { return j.a_kmajor ? tiles * (256 / kRows) * j.n_tiles : (tiles == 0 && j.beta_n ? 0 : j.n_work); };
        auto length = [&](const GemmJob& j) { return j.a_kmajor ? j.k_total : tiles * 256; };
        swapped = length(first) < length(second);               // longer reduction first
        n1 = items(swapped ? second : first);
        n2 = items(swapped ? first : second);
        if ((int)blockIdx.x >= n1 + n2) return;
    }
    bool in_first;
    int item;
    if (n1 >= 8 && n2 >= 8) {
        xcd_two_job_map(blockIdx.x, n1, n2, in_first, item);
    } else {
        const int lin = xcd_round_id(blockIdx.x, n1 + n2, 131072 / Cfg::kThreads);
        in_first = lin < n1;
        item = in_first ? lin : lin - n1;
    }
    const GemmJob& j = in_first != swapped ? first : second;
    if constexpr (std::is_same<Cfg, TurnTile>::value) {
        if (j.a_kmajor) run_turn_item<true, MODE>(j, item, rows, smem);
        else run_turn_item<false, (MODE & 10)>(j, item, rows, smem);
    } else {
        if (j.a_kmajor) run_gemm_job<Cfg, true, MODE>(j, item, rows, smem);
        else run_gemm_job<Cfg, false, (MODE & 10)>(j, item, rows, smem);
    }
}

// E4M3 scale bytes of the rows that take part, in their order and the grouped layout (see ScaleGroup); one dword, i.e.
// four rows of one 128-column block, per thread.  Rows that stand for none get scale 1.
__global__ __launch_bounds__(256) void compact_scales_kernel(const void* __restrict__ scales, int groups, const int32_t* __restrict__ perm,
                                                             int groups_c, int blocks, uint32_t* __restrict__ out) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= blocks * groups_c * 32) return;
    const int kb = i / (groups_c * 32), g = (i >> 5) % groups_c;
    uint32_t word = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = perm[g * 128 + q * 32 + (i & 31)];
        word |= (uint32_t)(row < 0 ? 127 : scale_byte(scales, groups, row, kb)) << (8 * q);
    }
    out[i] = word;
}

// Split running sum of counted rows: dHidden row perm[r] = compact row r of the result; zero rows where the label takes
// no part.  One wavefront per row of either kind.
__global__ __launch_bounds__(256) void scatter_rows_kernel(const uint16_t* __restrict__ rows, const int32_t* __restrict__ perm,
                                                           const int32_t* __restrict__ count, const int32_t* __restrict__ labels, int N, int V,
                                                           int32_t ignore_index, int D, uint16_t* __restrict__ dhidden) {
    const int l = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= N) return;
    const int32_t y = labels[r];
    if (y == ignore_index || y < 0 || y >= V) {
        u32x4* zero = (u32x4*)(dhidden + (size_t)r * D);
        for (int c = l; c < (D >> 3); c += 64) zero[c] = u32x4{0u, 0u, 0u, 0u};
    }
    if (r < count[0]) {
        const u32x4* from = (const u32x4*)(rows + (size_t)r * D);
        u32x4* to = (u32x4*)(dhidden + (size_t)perm[r] * D);
        for (int c = l; c < (D >> 3); c += 64) to[c] = from[c];
    }
}

// ------------------------------------------------------------------------------------------
// Sums of the K-split planes (fixed order: reproducible).  One 16-byte group per thread; a few
// megabytes that the contraction has just written, i.e. cache traffic bound by the launch itself.
// ------------------------------------------------------------------------------------------
// dHidden row row_map[r] (or r) = bf16(sum of the planes' row r); D4 = D / 4 groups per row.
__global__ __launch_bounds__(256) void dh_planes_kernel(const float* __restrict__ planes, int n_planes, int64_t stride,
                                                        int64_t groups, int D4, uint16_t* __restrict__ dhidden,
                                                        const int32_t* __restrict__ row_map) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= groups) return;
    f32x4 s = *(const f32x4*)(planes + i * 4);
    for (int p = 1; p < n_planes; ++p) s += *(const f32x4*)(planes + (size_t)p * stride + i * 4);
    union { __bf16 h[4]; u32x2 u; } cv;
#pragma unroll
    for (int e = 0; e < 4; ++e) cv.h[e] = (__bf16)s[e];
    const int64_t row = i / D4;
    const int64_t to = row_map ? (int64_t)row_map[row] : row;
    if (to >= 0) *(u32x2*)(dhidden + (to * D4 + (i - row * D4)) * 4) = cv.u;
}

// dW += sum of the planes.
__global__ __launch_bounds__(256) void dw_planes_kernel(float* __restrict__ dw, const float* __restrict__ planes,
                                                        int n_planes, int64_t stride, int64_t groups) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= groups) return;
    f32x4 s = *(const f32x4*)(dw + i * 4);
    for (int p = 0; p < n_planes; ++p) s += *(const f32x4*)(planes + (size_t)p * stride + i * 4);
    *(f32x4*)(dw + i * 4) = s;
}

// ------------------------------------------------------------------------------------------
// Row skipping (label scan of the path's first step: rows whose label is ignore_index take no
// part in any product, so they need not be computed at all).  The valid rows are gathered, in
// order, into a compact row space in which the unchanged kernels run; results are scattered
// back.  perm[r] = original row of compact row r, -1 for the padding behind the last valid one.
// ------------------------------------------------------------------------------------------
// rows_splits (optional): the forward of a call that does not know its number of valid rows takes it from here,
// rows_splits[0], and with it the vocabulary splits that fit so many rows, rows_splits[1]: the rule of make_plan over the
// s <= s_max whose workgroups the launch has.  One thread per s.
struct SplitRule { int32_t* rows_splits; int vocab_tiles, cus, s_max, workgroups; };

// One workgroup of 1024 threads: stable compaction of the valid rows (label in [0, V) and not
// ignore_index).  At most max_rows are kept (more: CCE_STATUS_ROW_BOUND, the rest is dropped).
// loss / lse of the rows that are not valid, and of valid rows that were dropped, are set to zero
// when the pointers are given (a caller that does not poll the status word then sees a zero
// contribution from a dropped row, not stale memory).  zero_row (optional): zero_row_len bf16 zeros
// are written there.  The status word (optional) is WRITTEN here (bad label / bound bits or 0): the scan is
// the first launch of a forward or row-skipping call and needs no clearing launch in front of it.  A
// backward over all rows gives none: it says nothing about its labels, whichever way it runs.
// Each wavefront owns a contiguous run of rows and takes 64 at a time, coalesced, positions from the
// ballot; the sixteen wavefront totals go through LDS: one barrier.  Eight label loads are in flight per
// lane.  One workgroup against the latency of its loads is all that bounds it: with a run of rows per
// THREAD (uncoalesced, one load after another) it took 28.7 us for 16384 rows, now 9.8.
__global__ __launch_bounds__(1024) void row_scan_kernel(
        const int32_t* __restrict__ labels, int N, int V, int32_t ignore_index, int max_rows, int rows_pad,
        int32_t* __restrict__ perm, int32_t* __restrict__ count_out, int32_t* __restrict__ status,
        float* __restrict__ loss, float* __restrict__ lse, uint16_t* __restrict__ zero_row, int zero_row_len, const SplitRule rule) {
    __shared__ unsigned long long wave_best[16];
    __shared__ int wave_total[16];
    __shared__ int wave_bad[16];
    constexpr int U = 8;                              // 64-row groups a wavefront has in flight
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = ((N + 1023) / 1024) * 64;         // rows per wavefront
    const int i0 = wave * per < N ? wave * per : N, i1 = i0 + per < N ? i0 + per : N;
    auto is_valid = [&](int32_t y) { return y != ignore_index && y >= 0 && y < V; };
    int c = 0;
    bool bad = false;
    int32_t y0[U];                                    // the first labels are kept: 8192 rows are not read twice
    for (int i = i0; i < i1; i += 64 * U) {
        int32_t y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) y[u] = i + 64 * u + lane < i1 ? labels[i + 64 * u + lane] : ignore_index;
        if (i == i0) {
#pragma unroll
            for (int u = 0; u < U; ++u) y0[u] = y[u];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c += __popcll(__ballot(is_valid(y[u])));  // the same in every lane
            bad = bad || (y[u] != ignore_index && !is_valid(y[u]));
        }
    }
    const bool wave_has_bad = __ballot(bad) != 0;
    if (lane == 0) { wave_total[wave] = c; wave_bad[wave] = wave_has_bad ? 1 : 0; }
    __syncthreads();
    int before = 0, total = 0, any_bad = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        const int t = wave_total[w];
        before += w < wave ? t : 0;
        total += t;
        any_bad |= wave_bad[w];
    }
    int pos = before;                                 // valid rows in front of the group
    for (int i = i0; i < i1; i += 64 * U) {
        int32_t y[U];
        if (i == i0) {
#pragma unroll
            for (int u = 0; u < U; ++u) y[u] = y0[u];
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) y[u] = i + 64 * u + lane < i1 ? labels[i + 64 * u + lane] : ignore_index;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = i + 64 * u + lane;
            const bool valid = is_valid(y[u]);
            const unsigned long long set = __ballot(valid);
            const int mine = pos + (int)__popcll(set & ((1ull << lane) - 1ull));
            const bool keep = valid && mine < max_rows;
            if (keep) perm[mine] = row;
            if (!keep && loss && row < i1) {
                loss[row] = 0.f;
                lse[row] = 0.f;
            }
            pos += (int)__popcll(set);
        }
    }
    if (zero_row)
        for (int c = tid; c < zero_row_len; c += 1024) zero_row[c] = 0;
    const int kept = total < max_rows ? total : max_rows;
    for (int r = kept + tid; r < rows_pad; r += 1024) perm[r] = -1;
    if (tid == 0) {
        count_out[0] = kept;
        count_out[1] = kept == N ? 1 : 0;             // the row map is the identity
        if (status) status[0] = (any_bad ? CCE_STATUS_BAD_LABEL : 0) | (total > max_rows ? CCE_STATUS_ROW_BOUND : 0);
    }
    if (rule.rows_splits) {
        const int tiles = (kept + 255) / 256, s = tid + 1;
        unsigned long long best = ~0ull;
        if (s <= rule.s_max && (s == 1 || tiles * s <= rule.workgroups)) {
            const unsigned rounds = (unsigned)(tiles * s + rule.cus - 1) / (unsigned)rule.cus;
            const unsigned per = (unsigned)(rule.vocab_tiles + s - 1) / (unsigned)s;
            best = ((unsigned long long)rounds * (4ull * per + 1ull) << 10) | (unsigned long long)tid;      // the smallest s of equal ones
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const unsigned long long other = __shfl_xor(best, o);
            best = other < best ? other : best;
        }
        if (lane == 0) wave_best[wave] = best;
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int w = 0; w < 16; ++w) best = wave_best[w] < best ? wave_best[w] : best;
            rule.rows_splits[0] = kept;
            rule.rows_splits[1] = (int)(best & 1023ull) + 1;
        }
    }
}

// Backward of the row-skipping calls, after the scan, in one launch:
// (a) per-row scalars into the compact row space: labels (ignore_index for padding) and up to two
//     fp32 vectors (0 for padding) -- thread r of the grid handles compact row r;
// (b) zero rows of dHidden for every row that takes no part: label not valid, or a valid row that
//     the compaction dropped because the caller's bound was too small (the compaction is stable, so
//     those are the valid rows behind the last kept one) -- one wavefront per original row.
// Grid: enough workgroups of 256 for both, i.e. max(ceil(rows_pad / 256), ceil(N / 4)).  rows_pad = 0
// leaves (a) out, dhidden = nullptr (b).
__global__ __launch_bounds__(256) void compact_prepare_backward_kernel(
        const int32_t* __restrict__ perm, const int32_t* __restrict__ count, int rows_pad,
        const int32_t* __restrict__ labels, int N, int V, int32_t ignore_index, int32_t* __restrict__ labels_c,
        const float* __restrict__ a, float* __restrict__ a_c, const float* __restrict__ b, float* __restrict__ b_c,
        int D, uint16_t* __restrict__ dhidden) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r < rows_pad) {
        const int from = perm[r];
        labels_c[r] = from >= 0 ? labels[from] : ignore_index;
        if (a) a_c[r] = from >= 0 ? a[from] : 0.f;
        if (b) b_c[r] = from >= 0 ? b[from] : 0.f;
    }
    const int l = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (!dhidden || row >= N) return;
    const int32_t y = labels[row];
    const int kept = count[0];
    const int last_kept = kept > 0 ? perm[kept - 1] : -1;
    if (y != ignore_index && y >= 0 && y < V && row <= last_kept) return;
    u32x4* dr = (u32x4*)(dhidden + (size_t)row * D);
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (int c = l; c < (D >> 3); c += 64) dr[c] = z;
}

// Copy of the hidden rows that take part, in compact order; rows that stand for none become zeros
// (their gradient is zero, but whatever a skipped row holds -- NaN included -- would meet that zero
// in the dW product).  One wavefront per row.
__global__ __launch_bounds__(256) void compact_gather_kernel(const uint16_t* __restrict__ hidden, const int32_t* __restrict__ perm,
                                                             int rows, int D, uint16_t* __restrict__ out) {
    const int l = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int from = perm[r];
    const u32x4* src = (const u32x4*)(hidden + (size_t)(from < 0 ? 0 : from) * D);
    u32x4* dst = (u32x4*)(out + (size_t)r * D);
    for (int c = l; c < (D >> 3); c += 64) dst[c] = from < 0 ? u32x4{0u, 0u, 0u, 0u} : src[c];
}

// ------------------------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------------------------
thread_local int g_last_hip_error = 0;

// Optional per-kernel-family timing with HIP events (cce_profile_begin / cce_profile_end).
// Off by default; when on, every launch of a timed family is bracketed by two events on the
// caller's stream.  Not thread safe: profile from one host thread at a time.
struct ProfState {
    bool on = false;
    std::vector<hipEvent_t> pool;
    size_t used = 0;
    struct Span { int fam; size_t e0, e1; };
    std::vector<Span> spans;
    size_t take() {
        if (used == pool.size()) {
            hipEvent_t e;
            if (!hip_ok(hipEventCreate(&e))) return (size_t)-1;
            pool.push_back(e);
        }
        return used++;
    }
};
static ProfState g_prof;
static std::mutex g_prof_mu;            // guards g_prof (spans of concurrent callers interleave but stay consistent)
static std::atomic<bool> g_prof_on{false};

struct ProfSpan {
    int fam; hipStream_t s; size_t e0 = (size_t)-1;
    ProfSpan(int fam_, hipStream_t s_) : fam(fam_), s(s_) {
        if (!g_prof_on.load(std::memory_order_relaxed)) return;
        std::lock_guard<std::mutex> lock(g_prof_mu);
        if (!g_prof.on) return;
        e0 = g_prof.take();
        if (e0 != (size_t)-1) (void)hipEventRecord(g_prof.pool[e0], s);
    }
    ~ProfSpan() {
        if (e0 == (size_t)-1) return;
        std::lock_guard<std::mutex> lock(g_prof_mu);
        if (!g_prof.on) return;
        const size_t e1 = g_prof.take();
        if (e1 == (size_t)-1) return;
        (void)hipEventRecord(g_prof.pool[e1], s);
        g_prof.spans.push_back({fam, e0, e1});
    }
};

static int check_common(const void* hidden, const void* weight, const int32_t* labels,
                        int64_t N, int64_t D, int64_t V, void* workspace, size_t workspace_bytes, Plan* plan) {
    if (!hidden || !weight || !labels || !workspace) return CCE_ERR_INVALID;
    if (N <= 0 || D <= 0 || V <= 0) return CCE_ERR_INVALID;
    if (D % 64 != 0) return CCE_ERR_UNSUPPORTED;
    if (N > (1 << 30) || V > (1 << 30) || V * D * 2 >= ((int64_t)1 << 32) || N * D * 2 >= ((int64_t)1 << 32))
        return CCE_ERR_UNSUPPORTED;
    if (((uintptr_t)hidden | (uintptr_t)weight | (uintptr_t)labels) & 15) return CCE_ERR_INVALID;
    if ((uintptr_t)workspace & 255) return CCE_ERR_INVALID;
    if (!make_plan(N, D, V, plan)) return CCE_ERR_INVALID;
    if (workspace_bytes < plan->total) return CCE_ERR_INVALID;
    return CCE_OK;
}

// An error left behind by an earlier, unrelated HIP call of this thread must not be reported as
// this call's: it is dropped before the first launch, so that the check after the last launch
// sees this call's launches only.
static inline void drop_stale_hip_error() { (void)hipGetLastError(); }

template <class K>
static bool allow_big_lds(K kernel, int bytes) {
    return hip_ok(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
}

template <class Cfg> constexpr int grad_tile_lds() {
    const int staging = Cfg::BN * kGRowBytes<Cfg> + Cfg::BN;
    return staging > Cfg::kLdsBytes ? staging : Cfg::kLdsBytes;
}
constexpr int kGradTileLds = grad_tile_lds<TileBig>();       // (FP8 logits)

template <int D, bool SHARED>
static bool allow_fused_lds() {
    return allow_big_lds(fused_backward_kernel<D, SHARED, false>, FusedTile<D, SHARED>::kLdsBytes) &&
           allow_big_lds(fused_backward_kernel<D, SHARED, true>, FusedTile<D, SHARED>::kLdsBytes);
}

// The MFMA kernels use more dynamic LDS than the default limit: raise it once per device
// (not per call, so that the compute calls consist of kernel launches only).
static bool ensure_kernel_attributes() {
    static std::mutex mu;
    static bool done[64] = {};
    int dev = 0;
    if (!hip_ok(hipGetDevice(&dev))) return false;
    if (dev < 0 || dev >= 64) return false;
    std::lock_guard<std::mutex> lock(mu);
    if (done[dev]) return true;
    if (!allow_big_lds(lse_partial_ping_kernel<false, TileTall>, TileTall::kLdsBytes)) return false;
    if (!allow_big_lds(lse_partial_ping_kernel<true, TileTall>, TileTall::kLdsBytes)) return false;
    if (!allow_big_lds(lse_partial_ping_kernel<false, TileSquare>, TileSquare::kLdsBytes)) return false;
    if (!allow_big_lds(lse_partial_ping_kernel<true, TileSquare>, TileSquare::kLdsBytes)) return false;
    if (!allow_big_lds(grad_tile_ping_kernel<TileTall>, TileTall::kLdsBytes)) return false;
    if (!allow_big_lds(grad_tile_ping_kernel<TileSquare>, TileSquare::kLdsBytes)) return false;
    if (!allow_big_lds(grad_tile_counted_kernel, TileTall::kLdsBytes)) return false;
    if (!allow_big_lds(lse_partial_kernel<false, false>, TileBig::kLdsBytes)) return false;
    if (!allow_big_lds(lse_partial_kernel<true, false>, TileBig::kLdsBytes)) return false;
    if (!allow_big_lds(lse_partial_kernel<false, true>, TileBig::kLdsBytes)) return false;
    if (!allow_big_lds(lse_partial_kernel<false, false, TileSmall>, TileSmall::kLdsBytes)) return false;
    if (!allow_big_lds(lse_partial_kernel<true, false, TileSmall>, TileSmall::kLdsBytes)) return false;
    if (!allow_big_lds(grad_tile_kernel<false, TileSmall>, grad_tile_lds<TileSmall>())) return false;
    if (!allow_big_lds(grad_tile_kernel<true>, kGradTileLds)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileBig, 0>, kGemmLdsBig)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileNarrow, 0>, kGemmLdsNarrow)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileSmall, 0>, kGemmLdsSmall)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileSmall, 1>, kGemmLdsSmall)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileSmall, 2>, kGemmLdsSmall + kRowTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileSmall, 3>, kGemmLdsSmall + kRowTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileSmall, 4>, kGemmLdsSmall)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileBig, 4>, kGemmLdsBig)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileNarrow, 4>, kGemmLdsNarrow)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileBig, 1>, kGemmLdsBig)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileNarrow, 1>, kGemmLdsNarrow)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileBig, 2>, kGemmLdsBig + kRowTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileNarrow, 2>, kGemmLdsNarrow + kRowTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileBig, 3>, kGemmLdsBig + kRowTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileNarrow, 3>, kGemmLdsNarrow + kRowTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileDuo, 0>, kGemmLdsDuo)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileDuo, 1>, kGemmLdsDuo)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileDuo, 4>, kGemmLdsDuo)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileNarrow, 9>, kGemmLdsNarrow + kRowTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileSmall, 9>, kGemmLdsSmall + kRowTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TileDuo, 9>, kGemmLdsDuo + counted_table_bytes<TileDuo>())) return false;
    if (!allow_big_lds(grad_gemm_kernel<TurnTile, 0>, TurnTile::kLdsBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TurnTile, 1>, TurnTile::kLdsBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TurnTile, 2>, TurnTile::kLdsBytes + kTurnTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TurnTile, 3>, TurnTile::kLdsBytes + kTurnTableBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TurnTile, 4>, TurnTile::kLdsBytes)) return false;
    if (!allow_big_lds(grad_gemm_kernel<TurnTile, 9>, TurnTile::kLdsBytes + kTurnTableBytes)) return false;
    if (!allow_fused_lds<64, false>()) return false;
    if (!allow_fused_lds<64, true>()) return false;
    if (!allow_fused_lds<128, false>()) return false;
    if (!allow_fused_lds<128, true>()) return false;
    done[dev] = true;
    return true;
}

// The bf16 gradient tiles of n_row_tiles x n_v_tiles tiles of 256 x 256.
static void launch_grad_tiles(const void* H, const void* W, const int32_t* labels, const float* lse, const float* dloss,
                              const float* mean_scale, int N, int D, int V, int32_t ignore_index, float label_smoothing, float z_loss,
                              int row0, int n_row_tiles, int v0, int n_v_tiles, uint16_t* G, uint32_t panel, int panel_shift, int v_off, int V_total,
                              const int32_t* perm, hipStream_t stream, const int32_t* count = nullptr, int first_row = 0) {
    const Fp8Scales none = {nullptr, nullptr, 0, 0};
    if (use_small_tiles(n_row_tiles, n_v_tiles))
        hipLaunchKernelGGL((grad_tile_kernel<false, TileSmall>), dim3(4 * n_row_tiles * n_v_tiles), dim3(kThreads), grad_tile_lds<TileSmall>(),
                           stream, H, W, labels, lse, dloss, mean_scale, N, D, V, ignore_index, label_smoothing, z_loss, row0,
                           2 * n_row_tiles, v0, 2 * n_v_tiles, G, panel, panel_shift, v_off, V_total, none, perm, count, first_row);
    else if (count)                                   // (row0 is 0: rows and scalars of the step itself)
        hipLaunchKernelGGL(grad_tile_counted_kernel, dim3(n_row_tiles * n_v_tiles), dim3(kThreads), TileTall::kLdsBytes, stream,
                           H, W, labels, lse, dloss, mean_scale, N, D, V, ignore_index, label_smoothing, z_loss, v0, n_v_tiles,
                           G, panel, panel_shift, v_off, V_total, perm, count, first_row, device_cu_count());
    else if (tall_grad_tiles(n_row_tiles, n_v_tiles, (int)D, device_cu_count())) {
        const int tiles = (n_v_tiles * 256 + TileTall::BM - 1) / TileTall::BM;
        hipLaunchKernelGGL(grad_tile_ping_kernel<TileTall>, dim3(n_row_tiles * tiles), dim3(kThreads), TileTall::kLdsBytes, stream,
                           H, W, labels, lse, dloss, mean_scale, N, D, V, ignore_index, label_smoothing, z_loss, row0,
                           n_row_tiles, v0, n_v_tiles * 256, tiles, G, panel, panel_shift, v_off, V_total, perm);
    } else
        hipLaunchKernelGGL(grad_tile_ping_kernel<TileSquare>, dim3(n_row_tiles * n_v_tiles), dim3(kThreads), TileSquare::kLdsBytes, stream,
                           H, W, labels, lse, dloss, mean_scale, N, D, V, ignore_index, label_smoothing, z_loss, row0,
                           n_row_tiles, v0, n_v_tiles * 256, n_v_tiles, G, panel, panel_shift, v_off, V_total, perm);
}

// A launch on tiles of two wavefront groups: the jobs' items in those tiles.
template <int MODE>
static void launch_turn_contractions(GemmJob first, GemmJob second, hipStream_t stream) {
    auto items = [&](GemmJob& j) {
        j.n_tiles = (j.n_valid + TurnTile::BM - 1) / TurnTile::BM;
        if (j.n_work > 0) j.n_work = (j.m_valid + TurnTile::BN - 1) / TurnTile::BN * j.n_tiles * j.n_split;
    };
    items(first);
    items(second);
    ProfSpan span(CCE_KERNEL_GRAD_GEMM, stream);
    hipLaunchKernelGGL((grad_gemm_kernel<TurnTile, MODE>), dim3(first.n_work + second.n_work), dim3(kThreads),
                       TurnTile::kLdsBytes + ((MODE & 10) ? kTurnTableBytes : 0), stream, first, second);
}

// Both contractions of counted rows (mode 9), the row table behind the stages; tile: counted_contraction_kind.  (All of them
// 256 x 128 one to a unit, backwards without ignored rows were 2.3 % behind those that do not look for them at
// 5200 x 2048 x 65001, 4.5 % at 8192 x 512 x 140000, 5.8 % at 2527 x 3584 x 68330: 0.9, 0.8 and 0.4 so.)
static void launch_counted_contractions(int kind, bool turn, const GemmJob& first, const GemmJob& second, hipStream_t stream) {
    if (turn) {
        launch_turn_contractions<9>(first, second, stream);
        return;
    }
    const int work = first.n_work + second.n_work;
    ProfSpan span(CCE_KERNEL_GRAD_GEMM, stream);
    if (kind == 3)
        hipLaunchKernelGGL((grad_gemm_kernel<TileDuo, 9>), dim3(work), dim3(TileDuo::kThreads), kGemmLdsDuo + counted_table_bytes<TileDuo>(), stream,
                           first, second);
    else if (kind == 2)
        hipLaunchKernelGGL((grad_gemm_kernel<TileSmall, 9>), dim3(work), dim3(kThreads), kGemmLdsSmall + kRowTableBytes, stream, first, second);
    else
        hipLaunchKernelGGL((grad_gemm_kernel<TileNarrow, 9>), dim3(work), dim3(kThreads), kGemmLdsNarrow + kRowTableBytes, stream, first, second);
}

template <int D, bool SHARED>
static void launch_fused(const FusedArgs& a, int dh_first, hipStream_t stream) {
    const dim3 grid((unsigned)(a.n_h + a.n_w));
    if (a.label_smoothing == 0.f) hipLaunchKernelGGL((fused_backward_kernel<D, SHARED, false>), grid, dim3(256), (FusedTile<D, SHARED>::kLdsBytes), stream, a, dh_first);
    else hipLaunchKernelGGL((fused_backward_kernel<D, SHARED, true>), grid, dim3(256), (FusedTile<D, SHARED>::kLdsBytes), stream, a, dh_first);
}

// A launch of one or both contractions (modes 0, 1 and 4 of grad_gemm_kernel).
template <int MODE>
static void launch_contractions(int kind, bool turn, const GemmJob& first, const GemmJob& second, hipStream_t stream) {
    if (turn) {
        launch_turn_contractions<MODE>(first, second, stream);
        return;
    }
    const int work = first.n_work + second.n_work;
    ProfSpan span(CCE_KERNEL_GRAD_GEMM, stream);
    if (kind == 3)
        hipLaunchKernelGGL((grad_gemm_kernel<TileDuo, MODE>), dim3(work), dim3(256), kGemmLdsDuo, stream, first, second);
    else if (kind == 0)
        hipLaunchKernelGGL((grad_gemm_kernel<TileBig, MODE>), dim3(work), dim3(kThreads), kGemmLdsBig, stream, first, second);
    else if (kind == 2)
        hipLaunchKernelGGL((grad_gemm_kernel<TileSmall, MODE>), dim3(work), dim3(kThreads), kGemmLdsSmall, stream, first, second);
    else
        hipLaunchKernelGGL((grad_gemm_kernel<TileNarrow, MODE>), dim3(work), dim3(kThreads), kGemmLdsNarrow, stream, first, second);
}

}  // namespace cce

using namespace cce;

extern "C" {

const char* cce_version(void) { return "0.1.0"; }

const char* cce_strerror(int code) {
    switch (code) {
        case CCE_OK: return "ok";
        case CCE_ERR_INVALID: return "invalid argument (null or misaligned pointer, non-positive size, workspace too small)";
        case CCE_ERR_UNSUPPORTED: return "unsupported shape (D must be a multiple of 64; tensors must stay below 4 GiB of bf16)";
        case CCE_ERR_HIP: return "HIP runtime error (see cce_last_hip_error)";
        case CCE_ERR_TOO_LARGE: return "problem needs more scratch than the static buffer of cce_forward_static holds (use cce_forward with a workspace)";
        default: return "unknown error code";
    }
}

int cce_last_hip_error(void) { return g_last_hip_error; }

size_t cce_workspace_bytes(int64_t N, int64_t D, int64_t V) {
    Plan p;
    if (N <= 0 || D <= 0 || V <= 0 || D % 64 != 0) return 0;
    if (!make_plan(N, D, V, &p)) return 0;
    return workspace_to_ask_for(p, N, D, V, false);
}

size_t cce_materialised_logit_bytes(int64_t N, int64_t V) {
    if (N <= 0 || V <= 0) return 0;
    return (size_t)N * (size_t)V * 4u;
}

static bool variant_ok(float label_smoothing, float z_loss) {
    return label_smoothing >= 0.f && label_smoothing < 1.f && z_loss >= 0.f && isfinite(z_loss);
}

// Row skipping: what the two implementation functions need to run in the compact row space.
struct CompactCtx {
    Plan plan;                  // made for the compact rows
    const int32_t* perm;        // device: original row of each compact row, -1 for padding
    const char* zero_row = nullptr;   // device: D bf16 zeros (backward only)
    // backward only: the order, and the caller's rows and labels for the zero rows of dHidden
    Schedule order;
    int64_t all_rows = 0;
    const int32_t* all_labels = nullptr;
    const int32_t* count = nullptr;
    int D = 0, V = 0;
    int32_t ignore_index = 0;
    void zero_skipped(hipStream_t stream, void* dHidden) const {
        hipLaunchKernelGGL(compact_prepare_backward_kernel, dim3((unsigned)((all_rows + 3) / 4)), dim3(256), 0, stream,
                           perm, count, 0, all_labels, (int)all_rows, V, ignore_index, (int32_t*)nullptr,
                           (const float*)nullptr, (float*)nullptr, (const float*)nullptr, (float*)nullptr, D, (uint16_t*)dHidden);
    }
};

// A backward over all rows that leaves the ignored ones out by a count found on the device.
struct CountedRows { const int32_t* perm; const int32_t* count; };

// Forward over the V rows of `weight`, which are the rows [v_off, v_off + V) of the full
// matrix.  With `stats` the per-token shard statistics are written instead of loss / lse
// (`smooth` then says whether the logit sums are wanted).
static int forward_impl(const void* hidden, const void* weight, const int32_t* labels,
                        int64_t N, int64_t D, int64_t V, int32_t ignore_index,
                        float label_smoothing, float z_loss,
                        float* loss, float* lse, float* mean_loss,
                        int64_t v_off, float* stats, bool want_sumz, const Fp8Scales* fp8_in,
                        void* workspace, size_t workspace_bytes, void* stream_, const CompactCtx* cc = nullptr,
                        int32_t* status_word = nullptr) {
    Plan p;
    Fp8Scales fp8 = {nullptr, nullptr, 0, 0};
    if (fp8_in) {
        fp8 = *fp8_in;
        if (!fp8.hscale || !fp8.wscale || D % 128 != 0) return fp8.hscale && fp8.wscale ? CCE_ERR_UNSUPPORTED : CCE_ERR_INVALID;
        if (((uintptr_t)fp8.hscale | (uintptr_t)fp8.wscale) & 3) return CCE_ERR_INVALID;
    }
    if (!stats && (!loss || !lse)) return CCE_ERR_INVALID;
    if (((uintptr_t)loss | (uintptr_t)lse | (uintptr_t)mean_loss) & 3) return CCE_ERR_INVALID;
    if ((uintptr_t)stats & 15) return CCE_ERR_INVALID;
    if (!variant_ok(label_smoothing, z_loss)) return CCE_ERR_INVALID;
    if (v_off < 0 || v_off > (1 << 30)) return CCE_ERR_INVALID;
    if (cc) {
        p = cc->plan;           // arguments were checked, the status word written (by the label scan), by the caller
    } else {
        int rc = check_common(hidden, weight, labels, N, D, V, workspace, workspace_bytes, &p);
        if (rc != CCE_OK) return rc;
    }
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)workspace;
    int32_t* status = status_word ? status_word : (int32_t*)(ws + p.off_status);
    float2* partials = (float2*)(ws + p.off_partials);
    const bool smooth = stats ? want_sumz : label_smoothing != 0.f;
    float* sumz = smooth ? (float*)(ws + p.off_sumz) : (float*)nullptr;

    const int32_t* fwd_perm = cc ? cc->perm : (const int32_t*)nullptr;
    if (!ensure_kernel_attributes()) return CCE_ERR_HIP;
    if (!cc) drop_stale_hip_error();
    int32_t* clear = cc ? (int32_t*)nullptr : status;
    const int32_t* rows_splits = nullptr;
    int grid = p.TT * p.S;
    // All rows, ignored ones among them perhaps: large forwards leave those out without being told how many there are.
    const ForwardSkip skip = cc || stats ? ForwardSkip{} : forward_skip(p, D, fp8_in != nullptr);
    Fp8Scales tile_fp8 = fp8;                                   // (the label logit keeps the caller's scales)
    if (skip.use) {
        int32_t* const perm = (int32_t*)(ws + skip.off_perm);
        int32_t* const found = (int32_t*)(ws + skip.off_found);
        partials = (float2*)(ws + skip.off_partials);
        if (smooth) sumz = (float*)(ws + skip.off_sumz);
        grid = skip.workgroups;
        hipLaunchKernelGGL(row_scan_kernel, dim3(1), dim3(1024), 0, stream, labels, (int)N, (int)V, ignore_index, (int)N, p.TT * 256,
                           perm, found + 2, status, loss, lse, (uint16_t*)nullptr, 0,
                           SplitRule{found, p.VT, device_cu_count(), skip.s_max, skip.workgroups});
        if (fp8_in) {
            const int groups = p.TT * 2, words = (int)(D / 128) * groups * 32;
            hipLaunchKernelGGL(compact_scales_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream, fp8.hscale, fp8.hgroups,
                               (const int32_t*)perm, groups, (int)(D / 128), (uint32_t*)(ws + skip.off_scales));
            tile_fp8.hscale = ws + skip.off_scales;
            tile_fp8.hgroups = groups;
        }
        fwd_perm = perm;
        rows_splits = found;
        clear = nullptr;                                         // the scan writes the status word
    }
    const int S = p.small_tiles && !fp8_in ? p.fwd_vt() : p.S;         // vocabulary splits of this forward
    {
        ProfSpan span(CCE_KERNEL_LSE_PARTIAL, stream);
        if (fp8_in)
            hipLaunchKernelGGL((lse_partial_kernel<false, true>), dim3(grid), dim3(kThreads), TileBig::kLdsBytes, stream,
                               hidden, weight, (int)N, (int)D, (int)V, p.TT, p.VT, p.S, partials, sumz, tile_fp8, fwd_perm, clear, rows_splits);
        else {
#define CCE_LAUNCH_FORWARD(CFG, WORK, TOKEN_TILES, VOCAB_TILES) \
    do { \
        if (smooth) hipLaunchKernelGGL((lse_partial_kernel<true, false, CFG>), dim3(WORK), dim3(kThreads), CFG::kLdsBytes, stream, \
                                       hidden, weight, (int)N, (int)D, (int)V, TOKEN_TILES, VOCAB_TILES, S, partials, sumz, fp8, fwd_perm, clear, rows_splits); \
        else hipLaunchKernelGGL((lse_partial_kernel<false, false, CFG>), dim3(WORK), dim3(kThreads), CFG::kLdsBytes, stream, \
                                hidden, weight, (int)N, (int)D, (int)V, TOKEN_TILES, VOCAB_TILES, S, partials, sumz, fp8, fwd_perm, clear, rows_splits); \
    } while (0)
#define CCE_LAUNCH_PING_FORWARD(CFG) \
    do { \
        if (smooth) hipLaunchKernelGGL((lse_partial_ping_kernel<true, CFG>), dim3(grid), dim3(kThreads), CFG::kLdsBytes, stream, \
                                       hidden, weight, (int)N, (int)D, (int)V, p.TT, S, partials, sumz, fwd_perm, clear, rows_splits); \
        else hipLaunchKernelGGL((lse_partial_ping_kernel<false, CFG>), dim3(grid), dim3(kThreads), CFG::kLdsBytes, stream, \
                                hidden, weight, (int)N, (int)D, (int)V, p.TT, S, partials, sumz, fwd_perm, clear, rows_splits); \
    } while (0)
            switch (forward_tile(p, D)) {
                case kForwardSmall: CCE_LAUNCH_FORWARD(TileSmall, p.fwd_tt() * S, p.fwd_tt(), p.fwd_vt()); break;
                case kForwardBig: CCE_LAUNCH_FORWARD(TileBig, grid, p.TT, p.VT); break;
                case kForwardSquare: CCE_LAUNCH_PING_FORWARD(TileSquare); break;
                case kForwardTall: CCE_LAUNCH_PING_FORWARD(TileTall); break;
            }
#undef CCE_LAUNCH_FORWARD
#undef CCE_LAUNCH_PING_FORWARD
        }
    }
    hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)((N + 3) / 4)), dim3(256), 0, stream,
                       (const uint16_t*)hidden, (const uint16_t*)weight, labels, partials, (const float*)sumz,
                       (int)N, (int)D, (int)V, S, ignore_index, label_smoothing, z_loss, loss, lse, status,
                       (int)v_off, (float4*)stats, fp8, fwd_perm, rows_splits);
    if (mean_loss && !stats)
        hipLaunchKernelGGL(mean_loss_kernel, dim3(1), dim3(1024), 0, stream,
                           (const float*)loss, labels, (int)N, (int)V, ignore_index, mean_loss, rows_splits);
    if (!hip_ok(hipGetLastError())) return CCE_ERR_HIP;
    return CCE_OK;
}

int cce_forward_ex(const void* hidden, const void* weight, const int32_t* labels,
                   int64_t N, int64_t D, int64_t V, int32_t ignore_index,
                   float label_smoothing, float z_loss,
                   float* loss, float* lse, float* mean_loss,
                   void* workspace, size_t workspace_bytes, void* stream_) {
    return forward_impl(hidden, weight, labels, N, D, V, ignore_index, label_smoothing, z_loss,
                        loss, lse, mean_loss, 0, nullptr, false, nullptr, workspace, workspace_bytes, stream_);
}

int cce_shard_forward(const void* hidden, const void* weight_shard, const int32_t* labels,
                      int64_t N, int64_t D, int64_t Vs, int64_t vocab_offset, int want_sumz,
                      float* stats, void* workspace, size_t workspace_bytes, void* stream_) {
    if (!stats) return CCE_ERR_INVALID;
    return forward_impl(hidden, weight_shard, labels, N, D, Vs, -1, 0.f, 0.f, nullptr, nullptr, nullptr,
                        vocab_offset, stats, want_sumz != 0, nullptr, workspace, workspace_bytes, stream_);
}

int cce_shard_merge(const float* stats, int P, const int32_t* labels, int64_t N, int64_t V_total,
                    int32_t ignore_index, float label_smoothing, float z_loss,
                    float* loss, float* lse, float* mean_loss, int32_t* status, void* stream_) {
    if (!stats || !labels || !loss || !lse) return CCE_ERR_INVALID;
    if (P <= 0 || P > 4096 || N <= 0 || N > (1 << 30) || V_total <= 0 || V_total > (1 << 30)) return CCE_ERR_INVALID;
    if (((uintptr_t)stats & 15) || (((uintptr_t)loss | (uintptr_t)lse | (uintptr_t)mean_loss | (uintptr_t)status | (uintptr_t)labels) & 3))
        return CCE_ERR_INVALID;
    if (!variant_ok(label_smoothing, z_loss)) return CCE_ERR_INVALID;
    hipStream_t stream = (hipStream_t)stream_;
    drop_stale_hip_error();
    hipLaunchKernelGGL(shard_merge_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, stream,
                       (const float4*)stats, P, labels, (int)N, (int)V_total, ignore_index, label_smoothing, z_loss,
                       loss, lse, status);
    if (mean_loss)
        hipLaunchKernelGGL(mean_loss_kernel, dim3(1), dim3(1024), 0, stream,
                           (const float*)loss, labels, (int)N, (int)V_total, ignore_index, mean_loss, (const int32_t*)nullptr);
    if (!hip_ok(hipGetLastError())) return CCE_ERR_HIP;
    return CCE_OK;
}

int cce_forward(const void* hidden, const void* weight, const int32_t* labels,
                int64_t N, int64_t D, int64_t V, int32_t ignore_index,
                float* loss, float* lse, void* workspace, size_t workspace_bytes, void* stream_) {
    return cce_forward_ex(hidden, weight, labels, N, D, V, ignore_index, 0.f, 0.f, loss, lse, nullptr,
                          workspace, workspace_bytes, stream_);
}

// ------------------------------------------------------------------------------------------
// cce_forward for callers that cannot allocate or bring a workspace: the forward's scratch (status
// word, per-split (max, sum-exp) pairs) lives in a file-scope device array.  In host code the
// array's name is only a handle: its device address is looked up once per device with
// hipGetSymbolAddress and that address, never the name, is what kernels and plans are given.
// ------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[CCE_STATIC_SCRATCH_BYTES];

// Device address of this device's copy of `scratch` (each GPU holds its own), or nullptr.
static void* static_scratch_address() {
    static std::mutex mu;
    static void* address[64] = {};
    int dev = 0;
    if (!hip_ok(hipGetDevice(&dev)) || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!address[dev]) {
        void* ptr = nullptr;
        if (!hip_ok(hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch))) || !ptr) return nullptr;
        address[dev] = ptr;
    }
    return address[dev];
}

int cce_forward_static(const void* hidden, const void* weight, const int32_t* labels,
                       int64_t N, int64_t D, int64_t V, int32_t ignore_index,
                       float* loss, float* lse, int32_t* status, void* stream_) {
    if (!hidden || !weight || !labels || !loss || !lse) return CCE_ERR_INVALID;
    if (N <= 0 || D <= 0 || V <= 0 || ((uintptr_t)status & 3)) return CCE_ERR_INVALID;
    if (D % 64 != 0) return CCE_ERR_UNSUPPORTED;
    Plan p;
    if (!make_plan(N, D, V, &p)) return CCE_ERR_INVALID;
    // the forward touches the workspace up to the end of the partial results only, or to the end of forward_skip's
    // layout, which is taken where it fits the array
    if (p.off_dhacc > (size_t)CCE_STATIC_SCRATCH_BYTES) return CCE_ERR_TOO_LARGE;
    void* ws = static_scratch_address();
    if (!ws) return CCE_ERR_HIP;
    // forward_impl checks a workspace against the whole plan (forward + backward); only the array's
    // bytes exist here and only those are addressed by the forward kernels
    return forward_impl(hidden, weight, labels, N, D, V, ignore_index, 0.f, 0.f, loss, lse, nullptr,
                        0, nullptr, false, nullptr, ws, p.total, stream_, nullptr, status);
}

// The backward in the order of a Schedule (plan.h); arguments as in backward_impl, checked there.
// Row skipping: the hidden rows that take part are gathered first -- for one row block into dHidden,
// which is as large and is not written before the last contraction; per row block into the workspace.
static void run_schedule(const Schedule& sc, const void* hidden, const void* weight, const int32_t* labels,
                        const float* lse, const float* dloss, const float* mean_scale,
                        int64_t N, int64_t D, int64_t V, int64_t v_off, int64_t V_total, int32_t ignore_index,
                        float label_smoothing, float z_loss, void* dHidden, float* dW, int accumulate_dW,
                        const void* logit_hidden, const void* logit_weight, const Fp8Scales* fp8,
                        char* ws, hipStream_t stream, const CompactCtx* cc, const CountedRows* counted) {
    const Fp8Scales scales = fp8 ? *fp8 : Fp8Scales{nullptr, nullptr, 0, 0};
    const int d_tiles = (int)((D + gemm_tile_of_kind(sc.kind).bn - 1) / gemm_tile_of_kind(sc.kind).bn);
    const Knobs knobs = Knobs::read();
    const int64_t block = (int64_t)sc.a * 256;
    float* planes = (float*)(ws + sc.off_acc);
    float* part_w = (float*)(ws + sc.off_part_w);
    const bool one_block = block >= N;
    for (int64_t r0 = 0; r0 < N; r0 += block) {
        const int64_t rows = N - r0 < block ? N - r0 : block;
        // hidden rows of this block, densely
        const uint16_t* h_rows = (const uint16_t*)hidden + (size_t)r0 * D;
        if (cc) {
            uint16_t* hc = one_block ? (uint16_t*)dHidden : (uint16_t*)(ws + sc.off_hc);
            hipLaunchKernelGGL(compact_gather_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, stream,
                               (const uint16_t*)hidden, cc->perm + r0, (int)rows, (int)D, hc);
            h_rows = hc;
        }
        int planes_written = 0;
        bool summed = false;                                     // dHidden written by the contractions themselves
        for (int64_t v0 = 0; v0 < V; ) {
            const ScheduleChunk ch = schedule_chunk(sc, D, V - v0);
            const int v_tiles = (int)ch.b;
            const int64_t cols = V - v0 < (int64_t)v_tiles * 256 ? V - v0 : (int64_t)v_tiles * 256;
            const bool last = v0 + cols >= V;
            const int ldg = v_tiles * 256;
            int n_split_h = 1;
            // Steps over ch.rows row tiles each, all of the block's rows where the chunk is wide enough.
            for (int64_t s0 = 0; s0 < rows; s0 += (int64_t)ch.rows * 256) {
                const int64_t srows = rows - s0 < (int64_t)ch.rows * 256 ? rows - s0 : (int64_t)ch.rows * 256;
                const int row_tiles = (int)((srows + 255) / 256);
                const int64_t row0 = r0 + s0;
                const uint16_t* h_step = h_rows + (size_t)s0 * D;
                const size_t g_bytes = (size_t)row_tiles * 256 * (size_t)ldg * 2;
                // parts of the two reductions, in whole tiles of 256
                const LaunchShape shape = launch_shape(row_tiles, v_tiles, sc.split_h, sc.split_w, planes_written > 0, row0 > 0 || accumulate_dW);
                const int kh = shape.kh, kw = shape.kw, n_split_w = shape.parts_w;
                const bool dw_beta = shape.dw_beta;
                n_split_h = shape.parts_h;
                const LaunchTiles tiles = launch_tiles(shape, D, sc.kind, sc.split_acc != 0, false, counted != nullptr, knobs);
                const int kind = tiles.kind;
                const bool turn = tiles.turn;
                const int panel_shift = turn || kind == 3 ? 5 : 6;    // log2 of the K slice of the contractions' tiles
                const uint32_t panel = (uint32_t)(row_tiles * 256) << panel_shift;
                uint16_t* G = ch.in_tail ? (uint16_t*)((char*)dW + (((size_t)V * (size_t)D * 4 - g_bytes) & ~(size_t)255))
                                         : (uint16_t*)(ws + sc.off_g);
                {
                    // tokens are counted inside the step: its rows and per-row scalars are contiguous
                    ProfSpan span(CCE_KERNEL_GRAD_TILE, stream);
                    const dim3 grid((unsigned)(row_tiles * v_tiles));
                    if (fp8 && counted)
                        hipLaunchKernelGGL(grad_tile_kernel<true>, grid, dim3(kThreads), kGradTileLds, stream,
                                           logit_hidden, logit_weight, labels + row0, lse + row0, dloss ? dloss + row0 : dloss, mean_scale,
                                           (int)srows, (int)D, (int)V, ignore_index, label_smoothing, z_loss, 0, row_tiles, (int)v0, v_tiles,
                                           G, panel, panel_shift, (int)v_off, (int)V_total, scales, counted->perm + row0, counted->count, (int)row0);
                    else if (fp8)
                        hipLaunchKernelGGL(grad_tile_kernel<true>, grid, dim3(kThreads), kGradTileLds, stream,
                                           logit_hidden, logit_weight, labels, lse, dloss, mean_scale, (int)N, (int)D, (int)V,
                                           ignore_index, label_smoothing, z_loss, (int)row0, row_tiles, (int)v0, v_tiles, G, panel, panel_shift,
                                           (int)v_off, (int)V_total, scales, (const int32_t*)nullptr, (const int32_t*)nullptr, 0);
                    else if (counted)
                        launch_grad_tiles(hidden, weight, labels + row0, lse + row0, dloss ? dloss + row0 : dloss, mean_scale,
                                          (int)srows, (int)D, (int)V, ignore_index, label_smoothing, z_loss, 0, row_tiles, (int)v0,
                                          v_tiles, G, panel, panel_shift, (int)v_off, (int)V_total, counted->perm + row0, stream,
                                          counted->count, (int)row0);
                    else
                        launch_grad_tiles((const void*)h_step, weight, labels + row0, lse + row0, dloss ? dloss + row0 : dloss, mean_scale,
                                          (int)srows, (int)D, (int)V, ignore_index, label_smoothing, z_loss, 0, row_tiles, (int)v0,
                                          v_tiles, G, panel, panel_shift, (int)v_off, (int)V_total, (const int32_t*)nullptr, stream);
                }
                const int per256 = 256 / gemm_tile_of_kind(kind).bm;
                GemmJob dh;
                dh.a_kmajor = 1;
                dh.A = G; dh.panel = panel;
                dh.B = (const void*)((const uint16_t*)weight + (size_t)v0 * D); dh.ldb = (int)D; dh.b_k_n = (int)cols;
                dh.k_total = ldg; dh.n_tiles = d_tiles; dh.split_k = kh * 256; dh.n_split = n_split_h;
                dh.n_work = row_tiles * per256 * d_tiles * dh.n_split;
                dh.m_valid = (int)srows; dh.n_valid = (int)D; dh.ld_out = D;
                dh.out_f32 = sc.split_acc ? (float*)nullptr : planes + (size_t)s0 * D;
                dh.part = planes + sc.plane_h + (size_t)s0 * D; dh.part_stride = sc.plane_h;
                dh.beta_n = planes_written;
                // (gathered rows in dHidden: it is written by the contraction only where that is the one step)
                dh.final = last && sc.split_h == 1 && !(cc && one_block && (v0 > 0 || row_tiles < sc.a)) ? 1 : 0;
                summed = dh.final != 0;
                dh.out_hi = (uint16_t*)dHidden + (cc ? (size_t)0 : (size_t)row0 * D);
                dh.out_lo = sc.split_acc ? (uint16_t*)planes + (size_t)s0 * D : (uint16_t*)nullptr;
                dh.row_map = cc ? cc->perm + row0 : (const int32_t*)nullptr;
                dh.zero_row = nullptr;
                GemmJob dw;
                dw.a_kmajor = 0;
                dw.A = G; dw.panel = panel;
                dw.B = (const void*)h_step; dw.ldb = (int)D; dw.b_k_n = (int)srows;
                dw.k_total = row_tiles * 256; dw.n_tiles = d_tiles; dw.split_k = kw * 256; dw.n_split = n_split_w;
                dw.n_work = v_tiles * per256 * d_tiles * dw.n_split;
                dw.m_valid = (int)cols; dw.n_valid = (int)D;
                dw.out_f32 = dW + (size_t)v0 * D; dw.part = part_w; dw.part_stride = sc.plane_w; dw.ld_out = D;
                dw.beta_n = dw_beta ? 1 : 0;
                dw.final = 0; dw.out_hi = nullptr; dw.out_lo = nullptr; dw.row_map = nullptr; dw.zero_row = nullptr;

                dh.count = dw.count = nullptr;
                dh.first_row = dw.first_row = 0;
                dh.rows = dw.rows = (int)srows;
                if (counted) {
                    dh.count = dw.count = counted->count;
                    dh.first_row = dw.first_row = (int)row0;
                    dw.B = hidden;
                    dh.row_map = dw.row_map = counted->perm + row0;
                    launch_counted_contractions(kind, turn, dh, dw, stream);
                    continue;
                }
                const bool dh_first = kh >= kw;                          // longer items first
                const GemmJob& first = dh_first ? dh : dw;
                const GemmJob& second = dh_first ? dw : dh;
                if (dh.final && cc && one_block) {
                    // this dH job writes dHidden, which still holds the rows the dW job reads
                    GemmJob none = dh;
                    none.n_work = 0;
                    launch_contractions<0>(kind, turn, dw, none, stream);
                    launch_contractions<4>(kind, turn, dh, none, stream);
                } else if (dh.final && cc) {
                    launch_contractions<4>(kind, turn, first, second, stream);
                } else if (sc.split_acc) {
                    launch_contractions<1>(kind, turn, first, second, stream);
                } else {
                    launch_contractions<0>(kind, turn, first, second, stream);
                }
                if (dw.n_split > 1) {
                    const int64_t groups = cols * (D / 4);
                    hipLaunchKernelGGL(dw_planes_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, stream,
                                       dW + (size_t)v0 * D, (const float*)part_w, dw.n_split - 1, sc.plane_w, groups);
                }
            }
            planes_written = planes_written > n_split_h ? planes_written : n_split_h;
            v0 += cols;
        }
        if (!summed) {
            const int64_t groups = rows * (D / 4);
            hipLaunchKernelGGL(dh_planes_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, stream,
                               (const float*)planes, planes_written, sc.plane_h, groups, (int)(D / 4),
                               (uint16_t*)dHidden + (cc ? (size_t)0 : (size_t)r0 * D), cc ? cc->perm + r0 : (const int32_t*)nullptr);
        }
    }
}

// The backward of all rows without a gradient chunk, see fused_backward.h.
static void run_fused(const FusedChoice& f, const Plan& p, const void* hidden, const void* weight, const int32_t* labels, const float* lse,
                      const float* dloss, const float* mean_scale, int64_t N, int64_t D, int64_t V, int64_t v_off, int64_t V_total,
                      int32_t ignore_index, float label_smoothing, float z_loss, void* dHidden, float* dW, int accumulate_dW, char* ws,
                      hipStream_t stream) {
    FusedArgs a;
    a.H = (const uint16_t*)hidden; a.W = (const uint16_t*)weight;
    a.labels = labels; a.lse = lse; a.dloss = dloss; a.mean_scale = mean_scale;
    a.N = (int)N; a.V = (int)V; a.V_total = (int)V_total; a.v_off = (int)v_off; a.ignore_index = ignore_index;
    a.label_smoothing = label_smoothing; a.z_loss = z_loss;
    a.dHidden = (uint16_t*)dHidden; a.dW = dW; a.beta = accumulate_dW ? 1 : 0;
    a.stride_h = N * D; a.stride_w = V * D;
    a.planes_h = (float*)(ws + p.off_dhacc);
    a.planes_w = a.planes_h + (f.parts_h > 1 ? (size_t)f.parts_h * (size_t)a.stride_h : (size_t)0);
    a.parts_h = f.parts_h; a.parts_w = f.parts_w; a.len_h = f.len_h; a.len_w = f.len_w; a.n_h = f.n_h; a.n_w = f.n_w;
    const int dh_first = f.len_h >= f.len_w ? 1 : 0;
    {
        ProfSpan span(CCE_KERNEL_GRAD_GEMM, stream);
        if (D == 64 && f.shared) launch_fused<64, true>(a, dh_first, stream);
        else if (D == 64) launch_fused<64, false>(a, dh_first, stream);
        else if (f.shared) launch_fused<128, true>(a, dh_first, stream);
        else launch_fused<128, false>(a, dh_first, stream);
    }
    if (f.parts_h > 1) {
        const int64_t groups = N * (D / 4);
        hipLaunchKernelGGL(dh_planes_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, stream, (const float*)a.planes_h, f.parts_h,
                           a.stride_h, groups, (int)(D / 4), (uint16_t*)dHidden, (const int32_t*)nullptr);
    }
    if (f.parts_w > 1) {
        const int64_t groups = V * (D / 4);
        hipLaunchKernelGGL(dw_planes_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, stream, dW, (const float*)a.planes_w,
                           f.parts_w - 1, a.stride_w, groups);
    }
}

// Backward over the V rows of `weight`, which are the rows [v_off, v_off + V) of a matrix of
// V_total rows that `labels`, label smoothing and the validity of a row refer to.
static int backward_impl(const void* hidden, const void* weight, const int32_t* labels,
                         const float* lse, const float* dloss, float grad_scale,
                         int64_t N, int64_t D, int64_t V, int64_t v_off, int64_t V_total, int32_t ignore_index,
                         float label_smoothing, float z_loss,
                         void* dHidden, float* dW, int accumulate_dW,
                         const void* logit_hidden, const void* logit_weight, const Fp8Scales* fp8_in,
                         void* workspace, size_t workspace_bytes, void* stream_, const CompactCtx* cc = nullptr) {
    Plan p;
    // The logit tiles are recomputed from logit_hidden / logit_weight (the bf16 operands, or
    // their E4M3 copies with fp8_in); the two gradient contractions always use the bf16 ones.
    Fp8Scales fp8 = {nullptr, nullptr, 0, 0};
    if (fp8_in) {
        fp8 = *fp8_in;
        if (!fp8.hscale || !fp8.wscale || !logit_hidden || !logit_weight) return CCE_ERR_INVALID;
        if (D % 128 != 0) return CCE_ERR_UNSUPPORTED;
        if (((uintptr_t)fp8.hscale | (uintptr_t)fp8.wscale) & 3) return CCE_ERR_INVALID;
        if (((uintptr_t)logit_hidden | (uintptr_t)logit_weight) & 15) return CCE_ERR_INVALID;
    }
    if (!lse || !dHidden || !dW) return CCE_ERR_INVALID;
    if (((uintptr_t)dHidden | (uintptr_t)dW) & 15) return CCE_ERR_INVALID;
    if (!variant_ok(label_smoothing, z_loss)) return CCE_ERR_INVALID;
    if (v_off < 0 || V_total > (1 << 30) || v_off + V > V_total) return CCE_ERR_INVALID;
    Schedule sc;
    FusedChoice fused = {};
    if (cc) {
        p = cc->plan;
        sc = cc->order;
    } else {
        int rc = check_common(hidden, weight, labels, N, D, V, workspace, workspace_bytes, &p);
        if (rc != CCE_OK) return rc;
        if (!fp8_in) fused = fused_backward_choice(p, N, D, V);
        if (!fused.use) plan_backward(&p, N, D, V, false, !accumulate_dW, workspace_bytes, &sc);
    }
    if (!ensure_kernel_attributes()) return CCE_ERR_HIP;
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)workspace;
    // mean reduction: the common upstream gradient grad_scale / n_valid lives in the status block
    float* mean_scale = (float*)(ws + p.off_status + 64);
    if (!cc) drop_stale_hip_error();
    if (!dloss)
        hipLaunchKernelGGL(mean_scale_kernel, dim3(1), dim3(1024), 0, stream,
                           labels, (int)N, (int)V_total, ignore_index, grad_scale, mean_scale);
    if (fused.use) {
        run_fused(fused, p, hidden, weight, labels, lse, dloss, mean_scale, N, D, V, v_off, V_total, ignore_index, label_smoothing, z_loss,
                  dHidden, dW, accumulate_dW, ws, stream);
        if (!hip_ok(hipGetLastError())) return CCE_ERR_HIP;
        return CCE_OK;
    }
    const int grad_lds = kGradTileLds;

    const BackwardSkip skip = cc || V_total != V ? BackwardSkip{} : backward_skip(p, sc, D, fp8_in != nullptr);
    if (skip.use) {
        int32_t* const perm = (int32_t*)(ws + skip.off_perm);
        int32_t* const labels_c = (int32_t*)(ws + skip.off_labels);
        float* const lse_c = (float*)(ws + skip.off_lse);
        float* const dloss_c = (float*)(ws + skip.off_dloss);
        int32_t* const count = (int32_t*)(ws + skip.off_count);
        const int rows_pad = p.TT * 256;
        hipLaunchKernelGGL(row_scan_kernel, dim3(1), dim3(1024), 0, stream, labels, (int)N, (int)V, ignore_index, (int)N, rows_pad, perm, count,
                           (int32_t*)nullptr, (float*)nullptr, (float*)nullptr, (uint16_t*)nullptr, 0, SplitRule{});
        hipLaunchKernelGGL(compact_prepare_backward_kernel, dim3((unsigned)(rows_pad / 256)), dim3(256), 0, stream,
                           (const int32_t*)perm, (const int32_t*)count, rows_pad, labels, (int)N, (int)V, ignore_index, labels_c,
                           lse, lse_c, dloss, dloss_c, (int)D, (uint16_t*)nullptr);
        if (fp8_in) {
            const int groups = p.TT * 2, words = (int)(D / 128) * groups * 32;
            hipLaunchKernelGGL(compact_scales_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream, fp8.hscale, fp8.hgroups,
                               (const int32_t*)perm, groups, (int)(D / 128), (uint32_t*)(ws + skip.off_scales));
            fp8.hscale = ws + skip.off_scales;
            fp8.hgroups = groups;
        }
        const CountedRows counted = {perm, count};
        run_schedule(sc, hidden, weight, labels_c, lse_c, dloss ? dloss_c : (const float*)nullptr, mean_scale, N, D, V, v_off, V_total, ignore_index,
                     label_smoothing, z_loss, dHidden, dW, accumulate_dW, logit_hidden, logit_weight, fp8_in ? &fp8 : nullptr,
                     ws, stream, nullptr, &counted);
        hipLaunchKernelGGL(scatter_rows_kernel, dim3((unsigned)((N + 3) / 4)), dim3(256), 0, stream, (const uint16_t*)(ws + sc.off_acc),
                           (const int32_t*)perm, (const int32_t*)count, labels, (int)N, (int)V, ignore_index, (int)D, (uint16_t*)dHidden);
        if (!hip_ok(hipGetLastError())) return CCE_ERR_HIP;
        return CCE_OK;
    }
    if (sc.use) {
        run_schedule(sc, hidden, weight, labels, lse, dloss, mean_scale, N, D, V, v_off, V_total, ignore_index,
                     label_smoothing, z_loss, dHidden, dW, accumulate_dW, logit_hidden, logit_weight, fp8_in ? &fp8 : nullptr,
                     ws, stream, cc, nullptr);
        if (cc && order_uses_dhidden(p, sc)) cc->zero_skipped(stream, dHidden);
        if (!hip_ok(hipGetLastError())) return CCE_ERR_HIP;
        return CCE_OK;
    }

    // The [row block x vocabulary chunk] steps in execution order: the Plan's blocks from the first to
    // the last, or those of a schedule that keeps sums or chunks in dHidden, from the last to the first.
    struct Step { int64_t r0, rows, v0, cols; int row_tiles, v_tiles; bool first_chunk, last_chunk, first_block; const RowBlock* block; };
    std::vector<RowBlock> blocks;
    if (sc.n_blocks) blocks.assign(sc.blocks, sc.blocks + sc.n_blocks);
    else
        for (int r = 0; r < p.TT; r += (int)(p.Nb / 256))
            blocks.push_back({r, (int)(p.Nb / 256), (int)(p.Vc / 256), p.gemm_kind, p.split_acc, false, false, p.off_dhacc, p.off_g});
    std::vector<Step> steps;
    for (const RowBlock& k : blocks) {
        const int64_t r0 = (int64_t)k.r0 * 256, block = (int64_t)k.a * 256, chunk = (int64_t)k.b * 256;
        const int64_t rows = (N - r0 < block) ? (N - r0) : block;
        for (int64_t v0 = 0; v0 < V; v0 += chunk) {
            const int64_t cols = (V - v0 < chunk) ? (V - v0) : chunk;
            steps.push_back({r0, rows, v0, cols, (int)((rows + 255) / 256), (int)((cols + 255) / 256), v0 == 0, v0 + cols >= V,
                             &k == &blocks[0], &k});
        }
    }
    const int K = (int)steps.size();
    const Knobs knobs = Knobs::read();

    for (int k = 0; k < K; ++k) {
        const Step& st = steps[k];
        const RowBlock& blk = *st.block;
        const int d_tiles = (int)((D + gemm_tile_of_kind(blk.kind).bn - 1) / gemm_tile_of_kind(blk.kind).bn);
        const LaunchTiles tiles = launch_tiles(launch_shape(st.row_tiles, st.v_tiles, 1, 1, !st.first_chunk, !st.first_block || accumulate_dW), D,
                                               blk.kind, blk.split_acc != 0, cc != nullptr, false, knobs);
        const GemmTile gt = gemm_tile_of_kind(tiles.kind);
        const bool turn = tiles.turn;
        const int per256 = 256 / gt.bm;                           // contraction row tiles per 256 rows
        uint16_t* G = (uint16_t*)((blk.g_in_dh ? (char*)dHidden : ws) + blk.off_g);
        char* acc = (blk.acc_in_dh ? (char*)dHidden : ws) + blk.off_acc;     // fp32 dH sums, or their lower halves (see GemmJob)
        const int ldg = st.v_tiles * 256;                       // the chunk is stored densely padded
        const int panel_shift = turn || gt.kind == 3 ? 5 : 6;            // log2 of the K slice of the contractions' tiles
        const uint32_t panel = (uint32_t)(st.row_tiles * 256) << panel_shift;
        const int n_rows_h = (int)N;
        // 1. gradient tiles of this [row block x chunk]
        {
            ProfSpan span(CCE_KERNEL_GRAD_TILE, stream);
            if (fp8_in)
                hipLaunchKernelGGL(grad_tile_kernel<true>, dim3(st.row_tiles * st.v_tiles), dim3(kThreads), grad_lds, stream,
                                   logit_hidden, logit_weight, labels, lse, dloss, (const float*)mean_scale,
                                   (int)N, (int)D, (int)V, ignore_index, label_smoothing, z_loss,
                                   (int)st.r0, st.row_tiles, (int)st.v0, st.v_tiles, G, panel, panel_shift, (int)v_off, (int)V_total, fp8,
                                   cc ? cc->perm : (const int32_t*)nullptr, (const int32_t*)nullptr, 0);
            else
                launch_grad_tiles(hidden, weight, labels, lse, dloss, (const float*)mean_scale, n_rows_h, (int)D, (int)V, ignore_index,
                                  label_smoothing, z_loss, (int)st.r0, st.row_tiles, (int)st.v0, st.v_tiles, G, panel, panel_shift, (int)v_off,
                                  (int)V_total, cc ? cc->perm : (const int32_t*)nullptr, stream);
        }
        // 2. both contractions in one launch
        // dH block += G * W_chunk      (M = tokens, K = chunk columns, N = D)
        GemmJob dh;
        dh.a_kmajor = 1;
        dh.A = G; dh.panel = panel;
        dh.B = (const void*)((const uint16_t*)weight + (size_t)st.v0 * D); dh.ldb = (int)D; dh.b_k_n = (int)st.cols;
        dh.k_total = ldg; dh.n_tiles = d_tiles; dh.n_work = st.row_tiles * per256 * d_tiles;
        dh.m_valid = (int)st.rows; dh.n_valid = (int)D;
        dh.out_f32 = blk.split_acc ? (float*)nullptr : (float*)acc; dh.ld_out = D; dh.beta_n = st.first_chunk ? 0 : 1;
        dh.out_hi = (uint16_t*)dHidden + (cc ? (size_t)0 : (size_t)st.r0 * D); dh.out_lo = blk.split_acc ? (uint16_t*)acc : (uint16_t*)nullptr;
        dh.final = st.last_chunk ? 1 : 0;
        dh.row_map = cc ? cc->perm + st.r0 : (const int32_t*)nullptr;
        dh.zero_row = nullptr;
        dh.n_split = 1; dh.split_k = dh.k_total; dh.part = nullptr; dh.part_stride = 0;
        // dW chunk (+)= G^T * H_block   (M = chunk columns, K = rows, N = D)
        GemmJob dw;
        dw.a_kmajor = 0;
        dw.A = G; dw.panel = panel;
        // (row skipping: hidden is the caller's tensor and the block's rows are reached through the row map)
        dw.B = cc ? hidden : (const void*)((const uint16_t*)hidden + (size_t)st.r0 * D); dw.ldb = (int)D; dw.b_k_n = (int)st.rows;
        dw.k_total = st.row_tiles * 256; dw.n_tiles = d_tiles; dw.n_work = st.v_tiles * per256 * d_tiles;
        dw.m_valid = (int)st.cols; dw.n_valid = (int)D;
        dw.out_f32 = dW + (size_t)st.v0 * D; dw.ld_out = D; dw.beta_n = (!st.first_block || accumulate_dW) ? 1 : 0;
        dw.out_hi = nullptr; dw.out_lo = nullptr; dw.final = 0;
        dw.row_map = cc ? cc->perm + st.r0 : (const int32_t*)nullptr;
        dw.zero_row = cc ? cc->zero_row : (const char*)nullptr;
        dw.n_split = 1; dw.split_k = dw.k_total; dw.part = nullptr; dw.part_stride = 0;
        dh.count = dw.count = nullptr; dh.first_row = dw.first_row = (int)st.r0; dh.rows = dw.rows = (int)st.rows;
        const bool dh_first = dh.k_total >= dw.k_total;          // longer reduction first
        const GemmJob& first = dh_first ? dh : dw;
        const GemmJob& second = dh_first ? dw : dh;
        const int work = dh.n_work + dw.n_work;

        const int mode = (blk.split_acc ? 1 : 0) | (cc ? 2 : 0);
        if (turn) {
            if (mode == 0) launch_turn_contractions<0>(first, second, stream);
            else if (mode == 1) launch_turn_contractions<1>(first, second, stream);
            else if (mode == 2) launch_turn_contractions<2>(first, second, stream);
            else launch_turn_contractions<3>(first, second, stream);
        } else {
            ProfSpan span(CCE_KERNEL_GRAD_GEMM, stream);
#define CCE_LAUNCH_GEMM(CFG, MODE, LDS) \
    hipLaunchKernelGGL((grad_gemm_kernel<CFG, MODE>), dim3(work), dim3(kThreads), (LDS) + ((MODE) >= 2 ? kRowTableBytes : 0), stream, first, second)
            if (gt.kind == 3) {
                if (mode == 0) hipLaunchKernelGGL((grad_gemm_kernel<TileDuo, 0>), dim3(work), dim3(TileDuo::kThreads), kGemmLdsDuo, stream, first, second);
                else hipLaunchKernelGGL((grad_gemm_kernel<TileDuo, 1>), dim3(work), dim3(TileDuo::kThreads), kGemmLdsDuo, stream, first, second);
            } else if (gt.kind == 0) {
                if (mode == 0) CCE_LAUNCH_GEMM(TileBig, 0, kGemmLdsBig); else if (mode == 1) CCE_LAUNCH_GEMM(TileBig, 1, kGemmLdsBig);
                else if (mode == 2) CCE_LAUNCH_GEMM(TileBig, 2, kGemmLdsBig); else CCE_LAUNCH_GEMM(TileBig, 3, kGemmLdsBig);
            } else if (gt.kind == 2) {
                if (mode == 0) CCE_LAUNCH_GEMM(TileSmall, 0, kGemmLdsSmall); else if (mode == 1) CCE_LAUNCH_GEMM(TileSmall, 1, kGemmLdsSmall);
                else if (mode == 2) CCE_LAUNCH_GEMM(TileSmall, 2, kGemmLdsSmall); else CCE_LAUNCH_GEMM(TileSmall, 3, kGemmLdsSmall);
            } else {
                if (mode == 0) CCE_LAUNCH_GEMM(TileNarrow, 0, kGemmLdsNarrow); else if (mode == 1) CCE_LAUNCH_GEMM(TileNarrow, 1, kGemmLdsNarrow);
                else if (mode == 2) CCE_LAUNCH_GEMM(TileNarrow, 2, kGemmLdsNarrow); else CCE_LAUNCH_GEMM(TileNarrow, 3, kGemmLdsNarrow);
            }
#undef CCE_LAUNCH_GEMM
        }
    }
    if (cc && order_uses_dhidden(p, sc)) cc->zero_skipped(stream, dHidden);
    if (!hip_ok(hipGetLastError())) return CCE_ERR_HIP;
    return CCE_OK;
}

int cce_backward_ex(const void* hidden, const void* weight, const int32_t* labels,
                    const float* lse, const float* dloss, float grad_scale,
                    int64_t N, int64_t D, int64_t V, int32_t ignore_index,
                    float label_smoothing, float z_loss,
                    void* dHidden, float* dW, int accumulate_dW,
                    void* workspace, size_t workspace_bytes, void* stream_) {
    return backward_impl(hidden, weight, labels, lse, dloss, grad_scale, N, D, V, 0, V, ignore_index,
                         label_smoothing, z_loss, dHidden, dW, accumulate_dW, nullptr, nullptr, nullptr,
                         workspace, workspace_bytes, stream_);
}

static bool choose_compact_plan(int64_t N, int64_t D, int64_t V, int64_t max_valid_rows, Plan* p, bool* use_compact) {
    return plan_row_skipping(N, D, V, max_valid_rows, g_force_row_skipping.load(std::memory_order_relaxed), p, use_compact);
}

// Row skipping: shared argument checks and plan.
static int compact_plan(const void* hidden, const void* weight, const int32_t* labels, int64_t N, int64_t D, int64_t V,
                        int64_t max_valid_rows, void* workspace, size_t workspace_bytes, Plan* p, bool* compact_out) {
    if (!hidden || !weight || !labels || !workspace) return CCE_ERR_INVALID;
    if (N <= 0 || D <= 0 || V <= 0 || max_valid_rows < 0) return CCE_ERR_INVALID;
    if (D % 64 != 0) return CCE_ERR_UNSUPPORTED;
    if (N > (1 << 30) || V > (1 << 30) || V * D * 2 >= ((int64_t)1 << 32) || N * D * 2 >= ((int64_t)1 << 32))
        return CCE_ERR_UNSUPPORTED;
    if (((uintptr_t)hidden | (uintptr_t)weight | (uintptr_t)labels) & 15) return CCE_ERR_INVALID;
    if ((uintptr_t)workspace & 255) return CCE_ERR_INVALID;
    bool use_compact = false;
    if (!choose_compact_plan(N, D, V, max_valid_rows, p, &use_compact)) return CCE_ERR_INVALID;
    if (workspace_bytes < p->total) return CCE_ERR_INVALID;
    *compact_out = use_compact;
    return CCE_OK;
}

int cce_set_row_skipping(int mode) {
    if (mode < 0 || mode > 2) return CCE_ERR_INVALID;
    g_force_row_skipping.store(mode, std::memory_order_relaxed);
    return CCE_OK;
}

int cce_get_row_skipping(int64_t N, int64_t D, int64_t V, int64_t max_valid_rows, int* skipping) {
    Plan p;
    bool use_compact = false;
    if (!skipping || N <= 0 || D <= 0 || V <= 0 || max_valid_rows < 0) return CCE_ERR_INVALID;
    if (D % 64 != 0) return CCE_ERR_UNSUPPORTED;
    if (!choose_compact_plan(N, D, V, max_valid_rows, &p, &use_compact)) return CCE_ERR_INVALID;
    *skipping = use_compact ? 1 : 0;
    return CCE_OK;
}

int cce_get_compact_tiling(int64_t N, int64_t D, int64_t V, int64_t max_valid_rows,
                           int* row_tiles, int* vocab_tiles) {
    Plan p;
    bool use_compact = false;
    if (!row_tiles || !vocab_tiles || N <= 0 || D <= 0 || V <= 0 || max_valid_rows < 0) return CCE_ERR_INVALID;
    if (D % 64 != 0) return CCE_ERR_UNSUPPORTED;
    if (!choose_compact_plan(N, D, V, max_valid_rows, &p, &use_compact)) return CCE_ERR_INVALID;
    *row_tiles = (int)(p.Nb / 256);
    *vocab_tiles = (int)(p.Vc / 256);
    return CCE_OK;
}

size_t cce_compact_workspace_bytes(int64_t N, int64_t D, int64_t V, int64_t max_valid_rows) {
    Plan p;
    bool use_compact = false;
    if (N <= 0 || D <= 0 || V <= 0 || D % 64 != 0 || max_valid_rows < 0) return 0;
    if (!choose_compact_plan(N, D, V, max_valid_rows, &p, &use_compact)) return 0;
    return workspace_to_ask_for(p, N, D, V, true);
}

int cce_forward_compact_ex(const void* hidden, const void* weight, const int32_t* labels,
                           int64_t N, int64_t D, int64_t V, int32_t ignore_index, int64_t max_valid_rows,
                           float label_smoothing, float z_loss,
                           float* loss, float* lse, float* mean_loss,
                           void* workspace, size_t workspace_bytes, void* stream_) {
    CompactCtx cc;
    if (!loss || !lse || (((uintptr_t)loss | (uintptr_t)lse | (uintptr_t)mean_loss) & 3)) return CCE_ERR_INVALID;
    if (!variant_ok(label_smoothing, z_loss)) return CCE_ERR_INVALID;
    bool use_compact = false;
    int rc = compact_plan(hidden, weight, labels, N, D, V, max_valid_rows, workspace, workspace_bytes, &cc.plan, &use_compact);
    if (rc != CCE_OK) return rc;
    if (!use_compact)
        return forward_impl(hidden, weight, labels, N, D, V, ignore_index, label_smoothing, z_loss, loss, lse, mean_loss,
                            0, nullptr, false, nullptr, workspace, workspace_bytes, stream_);
    if (!ensure_kernel_attributes()) return CCE_ERR_HIP;
    const Plan& p = cc.plan;
    const int64_t M = max_valid_rows < 1 ? 1 : (max_valid_rows < N ? max_valid_rows : N);
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)workspace;
    int32_t* status = (int32_t*)(ws + p.off_status);
    int32_t* perm = (int32_t*)(ws + p.off_perm);
    const int rows_pad = (int)p.rows_pad;
    drop_stale_hip_error();
    // (the scan writes the status word: no clearing launch)
    hipLaunchKernelGGL(row_scan_kernel, dim3(1), dim3(1024), 0, stream, labels, (int)N, (int)V, ignore_index,
                       (int)(max_valid_rows < N ? max_valid_rows : N), rows_pad, perm, (int32_t*)(ws + p.off_count), status, loss, lse,
                       (uint16_t*)nullptr, 0, SplitRule{});
    // the kernels fetch hidden rows through perm and write loss / lse to the original rows
    cc.perm = perm;
    rc = forward_impl(hidden, weight, labels, M, D, V, ignore_index, label_smoothing, z_loss, loss, lse, nullptr,
                      0, nullptr, false, nullptr, workspace, workspace_bytes, stream_, &cc);
    if (rc != CCE_OK || !mean_loss) return rc;
    // mean over the rows that took part: the rows left out hold loss 0
    hipLaunchKernelGGL(mean_loss_kernel, dim3(1), dim3(1024), 0, stream,
                       (const float*)loss, labels, (int)N, (int)V, ignore_index, mean_loss, (const int32_t*)(ws + p.off_count));
    if (!hip_ok(hipGetLastError())) return CCE_ERR_HIP;
    return CCE_OK;
}

int cce_forward_compact(const void* hidden, const void* weight, const int32_t* labels,
                        int64_t N, int64_t D, int64_t V, int32_t ignore_index, int64_t max_valid_rows,
                        float* loss, float* lse, void* workspace, size_t workspace_bytes, void* stream_) {
    return cce_forward_compact_ex(hidden, weight, labels, N, D, V, ignore_index, max_valid_rows, 0.f, 0.f,
                                  loss, lse, nullptr, workspace, workspace_bytes, stream_);
}

int cce_backward_compact_ex(const void* hidden, const void* weight, const int32_t* labels,
                            const float* lse, const float* dloss, float grad_scale,
                            int64_t N, int64_t D, int64_t V, int32_t ignore_index, int64_t max_valid_rows,
                            float label_smoothing, float z_loss,
                            void* dHidden, float* dW, int accumulate_dW,
                            void* workspace, size_t workspace_bytes, void* stream_) {
    CompactCtx cc;
    if (!lse || !dHidden || !dW) return CCE_ERR_INVALID;
    if (((uintptr_t)dHidden | (uintptr_t)dW) & 15) return CCE_ERR_INVALID;
    if (!variant_ok(label_smoothing, z_loss)) return CCE_ERR_INVALID;
    bool use_compact = false;
    int rc = compact_plan(hidden, weight, labels, N, D, V, max_valid_rows, workspace, workspace_bytes, &cc.plan, &use_compact);
    if (rc != CCE_OK) return rc;
    if (!use_compact)
        return backward_impl(hidden, weight, labels, lse, dloss, grad_scale, N, D, V, 0, V, ignore_index, label_smoothing, z_loss,
                             dHidden, dW, accumulate_dW, nullptr, nullptr, nullptr, workspace, workspace_bytes, stream_);
    if (!ensure_kernel_attributes()) return CCE_ERR_HIP;
    const int64_t M = max_valid_rows < 1 ? 1 : (max_valid_rows < N ? max_valid_rows : N);
    plan_backward(&cc.plan, M, D, V, true, !accumulate_dW, workspace_bytes, &cc.order);
    const Plan& p = cc.plan;
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)workspace;
    int32_t* status = (int32_t*)(ws + p.off_status);
    int32_t* perm = (int32_t*)(ws + p.off_perm);
    int32_t* labels_c = (int32_t*)(ws + p.off_labels_c);
    float* lse_c = (float*)(ws + p.off_fa_c);
    float* dloss_c = (float*)(ws + p.off_fb_c);
    const int rows_pad = (int)p.rows_pad;
    drop_stale_hip_error();
    hipLaunchKernelGGL(row_scan_kernel, dim3(1), dim3(1024), 0, stream, labels, (int)N, (int)V, ignore_index,
                       (int)(max_valid_rows < N ? max_valid_rows : N), rows_pad, perm, (int32_t*)(ws + p.off_count), status,
                       (float*)nullptr, (float*)nullptr, (uint16_t*)(ws + p.off_zero_row), (int)D, SplitRule{});
    {
        // (dHidden's rows that take no part become zeros here, or behind an order that uses dHidden)
        uint16_t* zero = order_uses_dhidden(p, cc.order) ? (uint16_t*)nullptr : (uint16_t*)dHidden;
        const unsigned g_gather = (unsigned)((rows_pad + 255) / 256), g_zero = zero ? (unsigned)((N + 3) / 4) : 0u;
        hipLaunchKernelGGL(compact_prepare_backward_kernel, dim3(g_gather > g_zero ? g_gather : g_zero), dim3(256), 0, stream,
                           (const int32_t*)perm, (const int32_t*)(ws + p.off_count), rows_pad,
                           labels, (int)N, (int)V, ignore_index, labels_c, lse, lse_c, dloss, dloss_c,
                           (int)D, zero);
    }
    cc.perm = perm;
    cc.zero_row = ws + p.off_zero_row;
    cc.all_rows = N; cc.all_labels = labels; cc.count = (const int32_t*)(ws + p.off_count);
    cc.D = (int)D; cc.V = (int)V; cc.ignore_index = ignore_index;
    // mean reduction (dloss == NULL) counts the compact labels: the rows that take part
    return backward_impl(hidden, weight, labels_c, lse_c, dloss ? dloss_c : (const float*)nullptr, grad_scale, M, D, V, 0, V,
                         ignore_index, label_smoothing, z_loss,
                         dHidden, dW, accumulate_dW, nullptr, nullptr, nullptr, workspace, workspace_bytes, stream_, &cc);
}

int cce_backward_compact(const void* hidden, const void* weight, const int32_t* labels,
                         const float* lse, const float* dloss,
                         int64_t N, int64_t D, int64_t V, int32_t ignore_index, int64_t max_valid_rows,
                         void* dHidden, float* dW, int accumulate_dW,
                         void* workspace, size_t workspace_bytes, void* stream_) {
    if (!dloss) return CCE_ERR_INVALID;
    return cce_backward_compact_ex(hidden, weight, labels, lse, dloss, 1.f, N, D, V, ignore_index, max_valid_rows, 0.f, 0.f,
                                   dHidden, dW, accumulate_dW, workspace, workspace_bytes, stream_);
}

int cce_fp8_forward(const void* hidden_q, const void* hidden_scales, const void* weight_q, const void* weight_scales,
                    const int32_t* labels, int64_t N, int64_t D, int64_t V, int32_t ignore_index,
                    float* loss, float* lse, void* workspace, size_t workspace_bytes, void* stream_) {
    const Fp8Scales fp8 = {hidden_scales, weight_scales, (int)((N + 127) / 128), (int)((V + 127) / 128)};
    return forward_impl(hidden_q, weight_q, labels, N, D, V, ignore_index, 0.f, 0.f, loss, lse, nullptr,
                        0, nullptr, false, &fp8, workspace, workspace_bytes, stream_);
}

int cce_fp8_backward(const void* hidden_q, const void* hidden_scales, const void* weight_q, const void* weight_scales,
                     const void* hidden, const void* weight, const int32_t* labels,
                     const float* lse, const float* dloss,
                     int64_t N, int64_t D, int64_t V, int32_t ignore_index,
                     void* dHidden, float* dW, int accumulate_dW,
                     void* workspace, size_t workspace_bytes, void* stream_) {
    if (!dloss) return CCE_ERR_INVALID;
    const Fp8Scales fp8 = {hidden_scales, weight_scales, (int)((N + 127) / 128), (int)((V + 127) / 128)};
    return backward_impl(hidden, weight, labels, lse, dloss, 1.f, N, D, V, 0, V, ignore_index, 0.f, 0.f,
                         dHidden, dW, accumulate_dW, hidden_q, weight_q, &fp8, workspace, workspace_bytes, stream_);
}

int cce_shard_backward(const void* hidden, const void* weight_shard, const int32_t* labels,
                       const float* lse, const float* dloss, float grad_scale,
                       int64_t N, int64_t D, int64_t Vs, int64_t vocab_offset, int64_t V_total,
                       int32_t ignore_index, float label_smoothing, float z_loss,
                       void* dHidden_partial, float* dW_shard, int accumulate_dW,
                       void* workspace, size_t workspace_bytes, void* stream_) {
    return backward_impl(hidden, weight_shard, labels, lse, dloss, grad_scale, N, D, Vs, vocab_offset, V_total,
                         ignore_index, label_smoothing, z_loss, dHidden_partial, dW_shard, accumulate_dW,
                         nullptr, nullptr, nullptr, workspace, workspace_bytes, stream_);
}

int cce_backward(const void* hidden, const void* weight, const int32_t* labels,
                 const float* lse, const float* dloss,
                 int64_t N, int64_t D, int64_t V, int32_t ignore_index,
                 void* dHidden, float* dW, int accumulate_dW,
                 void* workspace, size_t workspace_bytes, void* stream_) {
    if (!dloss) return CCE_ERR_INVALID;
    return cce_backward_ex(hidden, weight, labels, lse, dloss, 1.f, N, D, V, ignore_index, 0.f, 0.f,
                           dHidden, dW, accumulate_dW, workspace, workspace_bytes, stream_);
}

int cce_set_backward_tiling(int row_tiles, int vocab_tiles) {
    if (row_tiles < 0 || vocab_tiles < 0 || (row_tiles == 0) != (vocab_tiles == 0)) return CCE_ERR_INVALID;
    if (row_tiles > 0x7fff || vocab_tiles > 0xffff) return CCE_ERR_INVALID;
    g_force_tiling.store((row_tiles << 16) | vocab_tiles, std::memory_order_relaxed);
    return CCE_OK;
}

int cce_get_backward_tiling(int64_t N, int64_t D, int64_t V, int* row_tiles, int* vocab_tiles) {
    Plan p;
    if (!row_tiles || !vocab_tiles) return CCE_ERR_INVALID;
    if (N <= 0 || D <= 0 || V <= 0) return CCE_ERR_INVALID;
    if (D % 64 != 0) return CCE_ERR_UNSUPPORTED;
    if (!make_plan(N, D, V, &p)) return CCE_ERR_INVALID;
    *row_tiles = (int)(p.Nb / 256);
    *vocab_tiles = (int)(p.Vc / 256);
    return CCE_OK;
}

int cce_set_backward_gemm_tile(int tile_cols) {
    if (tile_cols != 0 && tile_cols != 128 && tile_cols != 256) return CCE_ERR_INVALID;
    g_force_gemm_cols.store(tile_cols, std::memory_order_relaxed);
    return CCE_OK;
}

int cce_set_backward_accumulator(int mode) {
    if (mode < 0 || mode > 2) return CCE_ERR_INVALID;
    g_force_split_acc.store(mode, std::memory_order_relaxed);
    return CCE_OK;
}

int cce_get_backward_accumulator(int64_t N, int64_t D, int64_t V, int* mode) {
    Plan p;
    if (!mode || N <= 0 || D <= 0 || V <= 0) return CCE_ERR_INVALID;
    if (D % 64 != 0) return CCE_ERR_UNSUPPORTED;
    if (!make_plan(N, D, V, &p)) return CCE_ERR_INVALID;
    *mode = p.split_acc ? 2 : 1;
    return CCE_OK;
}

int cce_get_backward_gemm_tile(int64_t N, int64_t D, int64_t V, int* tile_rows, int* tile_cols) {
    Plan p;
    if (!tile_rows || !tile_cols) return CCE_ERR_INVALID;
    if (N <= 0 || D <= 0 || V <= 0) return CCE_ERR_INVALID;
    if (D % 64 != 0) return CCE_ERR_UNSUPPORTED;
    if (!make_plan(N, D, V, &p)) return CCE_ERR_INVALID;
    const GemmTile gt = gemm_tile_of_kind(p.gemm_kind);
    *tile_rows = gt.bm;
    *tile_cols = gt.bn;
    return CCE_OK;
}

int cce_profile_begin(void) {
    std::lock_guard<std::mutex> lock(g_prof_mu);
    g_prof.on = true;
    g_prof.used = 0;
    g_prof.spans.clear();
    g_prof_on.store(true, std::memory_order_relaxed);
    return CCE_OK;
}

int cce_profile_end(double* ms_out, int64_t* launches_out) {
    if (!ms_out || !launches_out) return CCE_ERR_INVALID;
    std::lock_guard<std::mutex> lock(g_prof_mu);
    g_prof_on.store(false, std::memory_order_relaxed);
    g_prof.on = false;
    for (int i = 0; i < CCE_KERNEL_FAMILIES; ++i) { ms_out[i] = 0.0; launches_out[i] = 0; }
    for (const ProfState::Span& sp : g_prof.spans) {
        float ms = 0.f;
        if (!hip_ok(hipEventSynchronize(g_prof.pool[sp.e1]))) return CCE_ERR_HIP;
        if (!hip_ok(hipEventElapsedTime(&ms, g_prof.pool[sp.e0], g_prof.pool[sp.e1]))) return CCE_ERR_HIP;
        ms_out[sp.fam] += ms;
        launches_out[sp.fam] += 1;
    }
    g_prof.spans.clear();
    g_prof.used = 0;
    return CCE_OK;
}

int cce_read_status(const void* workspace, void* stream_, int32_t* status_out) {
    if (!workspace || !status_out) return CCE_ERR_INVALID;
    hipStream_t stream = (hipStream_t)stream_;
    if (!hip_ok(hipMemcpyAsync(status_out, workspace, sizeof(int32_t), hipMemcpyDeviceToHost, stream))) return CCE_ERR_HIP;
    if (!hip_ok(hipStreamSynchronize(stream))) return CCE_ERR_HIP;
    return CCE_OK;
}

}  // extern "C"
