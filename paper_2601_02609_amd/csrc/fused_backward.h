// Backward for a hidden size of 64 or 128, without a gradient chunk in memory (CCE backward theorem and chunk-level backward algorithm,
// with the chunk in registers).  Where D is that small, a gradient chunk costs more to write and to read twice than to form twice: 6
// bytes of memory traffic per logit against 4 D flops.  One launch holds two jobs:
//
//   dW: a tile of vocabulary rows stays in registers, the tokens stream past it;    dH: a tile of tokens stays, the vocabulary streams.
//
// Each streamed tile of 128 rows is brought into LDS once (global_load_lds), read K-major for the logits and with the transpose read for
// the contraction.  Logits are formed as z[c, r] (c streamed, r stationary), so that a lane holds column r and, of two blocks of 16
// streamed rows, rows 4 g ... 4 g + 3 of each (g = lane / 16): rounded to bf16 these eight are the lane's fragment of the contraction
// out[d, r] += T[c, d] z'[c, r], with the streamed rows of its 32 k-slots in that order on both sides.  Nothing passes through LDS.
//
// Bound by the vector ALU: per logit and lane two multiply-adds, an exponential (16 clocks of a wavefront) and half a conversion, 26
// clocks for 16 (D = 64) or 32 (D = 128) of products; what is reached is about their sum, 44 clocks a logit at D = 64.  Wavefronts of 64
// stationary rows at D = 64, of 32 at D = 128, where twice the columns take the registers.  28457 x 64 x 48721: 3.32 ms in launches over
// a gradient chunk (66 of them, 8.3 GB of chunk traffic), 0.74 ms; 22053 x 128 x 77882 4.12 and 1.81; 256 x 64 x 1000 15.2 us and 10.2.
#pragma once

#include "gemm_core.h"

namespace cce {

// SHARED: the four wavefronts share a tile's stationary rows and stream a quarter of the rows each, so that a streamed range of few
// rows, or a part of one, is walked by four (256 x 64 x 1000: 14.5 us without, 7.1).  At D = 64 its wavefronts have half of the rows, and
// four workgroups fit a compute unit (the same throughput, 835 us for 816 at 28457 x 64 x 48721, but less latency: 7.1 us for 8.8).
template <int D_, bool SHARED_>
struct FusedTile {
    static constexpr bool SHARED = SHARED_;
    static constexpr int D = D_, RB = D_ == 64 && !SHARED_ ? 4 : 2;      // blocks of 16 stationary rows of a wavefront
    static constexpr int kToUnit = D_ == 64 && SHARED_ ? 4 : 2; // workgroups to a compute unit, wavefronts to a SIMD
    static constexpr int KS = D / 32, DB = D / 16, C = 128, kThreads = 256;
    static constexpr int kStage = C * D * 2, kScalars = 6 * C * 4;       // streamed rows; streamed tokens' scalars (dW job)
    static constexpr int kReduce = SHARED ? 4 * DB * RB * 1024 : 0;      // the wavefronts' sums
    static constexpr int kLdsBytes = 2 * (kStage + kScalars) > kReduce ? 2 * (kStage + kScalars) : kReduce;
    static constexpr int kRows = 16 * RB, kTileRows = SHARED ? kRows : 4 * kRows;       // of a wavefront, of a work item
    static_assert(D == 64 || D == 128, "whole k16 x 2 steps, registers");
    static_assert(kToUnit * kLdsBytes <= 160 * 1024, "the stages of all workgroups of a compute unit");
};

struct FusedArgs {
    const uint16_t* H; const uint16_t* W;
    const int32_t* labels; const float* lse; const float* dloss; const float* mean_scale;
    int N, V, V_total, v_off; int32_t ignore_index; float label_smoothing, z_loss;
    uint16_t* dHidden; float* dW; int beta;
    float* planes_h; float* planes_w; int64_t stride_h, stride_w;        // parts of the streamed range: dH all, dW from the second on
    int parts_h, parts_w, len_h, len_w;                         // parts, streamed tiles per part
    int n_h, n_w;                                               // work items
};

// A token's scalars: nl2 = -lse log2 e, factor of the softmax term, subtracted at the label, added everywhere; label as a row of W (or
// none).  Rows that take no part (!live) have zeros whatever lse and dloss hold.  As fp32 products those do not make their gradients zero:
// a logit of such a row may overflow, its hidden row is any finite one.  In the dH job its row is cleared; the dW job multiplies by the
// factor with 0 * x = 0 for every x, or, where label smoothing fuses another term with that product, clears the rounded gradients of
// streamed rows among which one takes no part.  (Clearing without smoothing too: 28457 x 64 x 48721 with 15 % ignored 727 -> 805 us;
// the multiplication takes no longer than one that lets infinities through, 741 and 734.)
struct FusedToken { float nl2, sp, ch, ncs; int label; bool live; };
__device__ __forceinline__ FusedToken fused_token(const FusedArgs& a, int token) {
    const int t = token < a.N ? token : a.N - 1;
    const int32_t y = a.labels[t];
    const float ls = a.lse[t], dl = a.dloss ? a.dloss[t] : a.mean_scale[0];
    const bool live = token < a.N && y != a.ignore_index && y >= 0 && y < a.V_total;
    FusedToken r;
    r.live = live;
    r.nl2 = live ? -ls * 1.4426950408889634f : 0.f;
    r.sp = live ? dl * fmaf(2.f * a.z_loss, ls, 1.f) : 0.f;
    r.ch = live ? dl * (1.f - a.label_smoothing) : 0.f;
    r.ncs = live ? -dl * (a.label_smoothing / (float)a.V_total) : 0.f;
    const int64_t local = (int64_t)y - a.v_off;
    r.label = live && local >= 0 && local < a.V ? (int)local : -(1 << 30);
    return r;
}

// a * b, and zero where either is zero, whatever the other is (v_mul_legacy_f32).
__device__ float mul_zero(float a, float b) __asm("llvm.amdgcn.fmul.legacy");

// SMOOTH (dW job): with label smoothing.
template <int D, bool SHARED, bool DW, bool SMOOTH>
__device__ __forceinline__ void fused_item(const FusedArgs& a, int item, CCE_LDS char* smem) {
    typedef FusedTile<D, SHARED> F;
    constexpr int RB = F::RB, KS = F::KS, DB = F::DB, PITCH = 2 * D;
    const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = l & 15, g = l >> 4;
    const int rows = DW ? a.V : a.N, stream = DW ? a.N : a.V;
    const uint16_t* const S = DW ? a.W : a.H;
    const char* const T = (const char*)(DW ? a.H : a.W);
    const int parts = DW ? a.parts_w : a.parts_h, len = DW ? a.len_w : a.len_h;
    const int part = item % parts, wg_row0 = item / parts * F::kTileRows;
    const int row0 = wg_row0 + (SHARED ? 0 : wave * F::kRows);  // this wavefront's first stationary row
    const int all = (stream + F::C - 1) / F::C, t_begin = part * len, t_end = t_begin + len < all ? t_begin + len : all;

    bf16x8 s[RB][KS];                                           // stationary rows: B operand of the logits
    float nl2[RB], sp[RB], ncs[RB], ch[RB];                     // dH job: their scalars
    int label[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const int row = row0 + 16 * b + n, from = row < rows ? row : rows - 1;
#pragma unroll
        for (int k = 0; k < KS; ++k) s[b][k] = *(const bf16x8*)(S + (size_t)from * D + 32 * k + 8 * g);
        if (!DW) {
            const FusedToken t = fused_token(a, row);
            nl2[b] = t.nl2; sp[b] = t.sp; ncs[b] = t.ncs; ch[b] = t.ch; label[b] = t.label;
            if (!t.live) {                                      // takes no part: logits of zero, 1 * 0 + 0
#pragma unroll
                for (int k = 0; k < KS; ++k) s[b][k] = __builtin_bit_cast(bf16x8, i32x4{0, 0, 0, 0});
            }
        }
    }
    f32x4 out[DB][RB];
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int b = 0; b < RB; ++b) out[d][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // 16-byte chunk c of row r of a streamed tile lies at c ^ swizzle(r): the 16 rows of a K-major fragment meet every bank once, and so
    // do the 8 rows x 32 bytes that two lane groups of a transpose read touch.  (Over a quarter of the LDS's busy cycles count as conflicts all
    // the same: 27 % at D = 64, 30 % at D = 128.)
    auto swizzle = [](int r) { return D == 64 ? (((r >> 1) & 3) << 1) | ((r >> 3) & 1) : ((r & 7) << 1) | ((r >> 3) & 1); };
    constexpr int CPR = D / 8, RPL = 64 / CPR;                  // chunks of a row, rows of a wavefront's load
    const int load_row = RPL * wave + l / CPR;
    const uint32_t load_chunk = (uint32_t)(((l % CPR) ^ swizzle(load_row)) * 16), load_off = (uint32_t)load_row * PITCH + load_chunk;
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem + (uint32_t)wave * 1024u;
    auto issue = [&](int t, int stage) {
        const char* const base = T + (size_t)t * F::kStage;
        const uint32_t to = lds0 + (uint32_t)stage * F::kStage;
        if ((t + 1) * F::C <= stream) {
#pragma unroll
            for (int i = 0; i < F::kStage / 4096; ++i) load16_to_lds_sbase(base + i * 4096, load_off, to + (uint32_t)i * 4096u);
        } else {                                                // rows behind the last one: that one again
#pragma unroll
            for (int i = 0; i < F::kStage / 4096; ++i) {
                int r = load_row + 4 * RPL * i;
                r = r < stream - t * F::C ? r : stream - t * F::C - 1;
                load16_to_lds_sbase(base, (uint32_t)r * PITCH + load_chunk, to + (uint32_t)i * 4096u);
            }
        }
    };
    // dW job: the streamed tokens' scalars and, per 32 of them, whether one has its label among this workgroup's rows (1) and whether one
    // takes no part (2, with smoothing); behind those, 16 bits per token that clear the gradients of the ones that take none
    CCE_LDS char* const scalars = smem + 2 * F::kStage;
    auto put_scalars = [&](const FusedToken& t, int stage) {
        CCE_LDS float* const v = (CCE_LDS float*)(scalars + stage * F::kScalars);
        const int i = (int)threadIdx.x;
        v[i] = t.nl2; v[F::C + i] = t.sp; v[3 * F::C + i] = t.ch;
        ((CCE_LDS int*)v)[4 * F::C + i] = t.label;
        if (SMOOTH) v[2 * F::C + i] = t.ncs;
        const uint64_t hit = __ballot((unsigned)(t.label - wg_row0) < (unsigned)F::kTileRows);
        int flags = (uint32_t)(hit >> (l & 32)) != 0 ? 1 : 0;
        if (SMOOTH) {
            flags |= (uint32_t)(__ballot(!t.live) >> (l & 32)) != 0 ? 2 : 0;
            ((CCE_LDS uint16_t*)v)[2 * (5 * F::C + 4) + i] = t.live ? 0xffffu : 0u;
        }
        if ((l & 31) == 0) ((CCE_LDS int*)v)[5 * F::C + i / 32] = flags;
    };

    if (t_begin < t_end) {
        if (DW && wave < 2) put_scalars(fused_token(a, t_begin * F::C + (int)threadIdx.x), 0);
        __builtin_amdgcn_s_waitcnt(0x0f70);                     // vmcnt(0): the compiler cannot see the loads below
        issue(t_begin, 0);
    }
    const uint32_t frag = (uint32_t)(n * PITCH + ((g ^ swizzle(n)) << 4));                     // logits: row n, chunk g
    const int tr_row = 4 * g + (n >> 2);                                                       // contraction: rows 4 g + e, e = n / 4
    const uint32_t tr = (uint32_t)(tr_row * PITCH + ((((n >> 1) & 1) ^ swizzle(tr_row)) << 4) + (n & 1) * 8);
    for (int t = t_begin; t < t_end; ++t) {
        const int stage = (t - t_begin) & 1;
        barrier_pending_loads<0>();                             // tile t has landed, nobody reads the other stage any more
        FusedToken next;
        const bool more = t + 1 < t_end;
        if (DW && more && wave < 2) next = fused_token(a, (t + 1) * F::C + (int)threadIdx.x);
        if (more) issue(t + 1, stage ^ 1);
        const CCE_LDS char* const tile = smem + stage * F::kStage;
        const CCE_LDS char* const sc = scalars + stage * F::kScalars;
        const bool ragged = !DW && (t + 1) * F::C > stream;
        bool hits = false;                                      // dH job: a label of these rows lies in the tile
        if (!DW) {
            bool mine = false;
#pragma unroll
            for (int b = 0; b < RB; ++b) mine = mine || (unsigned)(label[b] - t * F::C) < (unsigned)F::C;
            hits = __ballot(mine) != 0;
        }
#pragma unroll 1
        for (int q = SHARED ? wave : 0; q < 4; q += SHARED ? 4 : 1) {
            const CCE_LDS char* const rows32 = tile + q * 32 * PITCH;
            f32x4 z[2][RB], vn[2], vs[2], va[2];
            if (DW) {
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const CCE_LDS char* const at = sc + (q * 32 + 16 * m + 4 * g) * 4;
                    vn[m] = *(const CCE_LDS f32x4*)at;
                    vs[m] = *(const CCE_LDS f32x4*)(at + 4 * F::C);
                    if (SMOOTH) va[m] = *(const CCE_LDS f32x4*)(at + 8 * F::C);
                }
            }
#pragma unroll
            for (int m = 0; m < 2; ++m) {
#pragma unroll
                for (int b = 0; b < RB; ++b) z[m][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    const bf16x8 x = *(const CCE_LDS bf16x8*)(rows32 + m * 16 * PITCH + (frag ^ (uint32_t)(k * 64)));
#pragma unroll
                    for (int b = 0; b < RB; ++b) z[m][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, s[b][k], z[m][b], 0, 0, 0);
                }
            }
            const int c0 = t * F::C + q * 32 + 4 * g;           // this lane's streamed rows: c0 + 16 m + e
            bf16x8 p[RB];
            int flags = 0;
            if (DW) {
#pragma unroll
                for (int b = 0; b < RB; ++b)
#pragma unroll
                    for (int m = 0; m < 2; ++m)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float x = __builtin_amdgcn_exp2f(fmaf(z[m][b][e], 1.4426950408889634f, vn[m][e]));
                            z[m][b][e] = SMOOTH ? fmaf(x, vs[m][e], va[m][e]) : mul_zero(x, vs[m][e]);
                        }
                flags = ((const CCE_LDS int*)sc)[5 * F::C + q];
                if (SMOOTH ? (flags & 1) != 0 : flags != 0) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        const CCE_LDS char* const at = sc + (q * 32 + 16 * m + 4 * g) * 4;
                        const f32x4 vc = *(const CCE_LDS f32x4*)(at + 12 * F::C);
                        const i32x4 vy = *(const CCE_LDS i32x4*)(at + 16 * F::C);
#pragma unroll
                        for (int b = 0; b < RB; ++b)
#pragma unroll
                            for (int e = 0; e < 4; ++e) z[m][b][e] -= vy[e] == row0 + 16 * b + n ? vc[e] : 0.f;
                    }
                }
            } else {
#pragma unroll
                for (int b = 0; b < RB; ++b)
#pragma unroll
                    for (int m = 0; m < 2; ++m)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            z[m][b][e] = fmaf(__builtin_amdgcn_exp2f(fmaf(z[m][b][e], 1.4426950408889634f, nl2[b])), sp[b], ncs[b]);
                bool here = false;                              // a label among these 32 rows
                if (hits) {
#pragma unroll
                    for (int b = 0; b < RB; ++b) here = here || (unsigned)(label[b] - (c0 - 4 * g)) < 32u;
                }
                if (__ballot(here) != 0) {
#pragma unroll
                    for (int b = 0; b < RB; ++b)
#pragma unroll
                        for (int m = 0; m < 2; ++m)
#pragma unroll
                            for (int e = 0; e < 4; ++e) z[m][b][e] -= label[b] == c0 + 16 * m + e ? ch[b] : 0.f;
                }
                if (ragged) {                                   // vocabulary rows behind the last one
#pragma unroll
                    for (int b = 0; b < RB; ++b)
#pragma unroll
                        for (int m = 0; m < 2; ++m)
#pragma unroll
                            for (int e = 0; e < 4; ++e) z[m][b][e] = c0 + 16 * m + e < stream ? z[m][b][e] : 0.f;
                }
            }
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e) p[b][4 * m + e] = (__bf16)z[m][b][e];
            if (DW && SMOOTH && (flags & 2)) {
                const CCE_LDS char* const at = sc + (5 * F::C + 4) * 4 + (q * 32 + 4 * g) * 2;
                const u32x2 lo = *(const CCE_LDS u32x2*)at, hi = *(const CCE_LDS u32x2*)(at + 32);
#pragma unroll
                for (int b = 0; b < RB; ++b)
                    p[b] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, p[b]) & u32x4{lo.x, lo.y, hi.x, hi.y});
            }
#pragma unroll
            for (int d = 0; d < DB; ++d) {
                const CCE_LDS char* const at = rows32 + (tr ^ (uint32_t)(d * 32));
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CCE_LDS s16x4*)at);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CCE_LDS s16x4*)(at + 16 * PITCH));
                const bf16x8 x = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int b = 0; b < RB; ++b) out[d][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, p[b], out[d][b], 0, 0, 0);
            }
        }
        if (DW && more && wave < 2) put_scalars(next, stage ^ 1);
    }
    barrier_pending_loads<0>();

    // results: lane (n, g) holds columns 16 d + 4 g ... + 3 of row row0 + 16 b + n
    auto store = [&](int d, int b, f32x4 v) {
        const int row = row0 + 16 * b + n, col = 16 * d + 4 * g;
        if (row >= rows) return;
        const size_t at = (size_t)row * D + col;
        if (DW) {
            float* const to = part == 0 ? a.dW : a.planes_w + (size_t)(part - 1) * a.stride_w;
            if (part == 0 && a.beta) v += *(const f32x4*)(to + at);
            *(f32x4*)(to + at) = v;
        } else if (parts > 1) {
            *(f32x4*)(a.planes_h + (size_t)part * a.stride_h + at) = v;
        } else {
            union { __bf16 h[4]; u32x2 u; } cv;
#pragma unroll
            for (int e = 0; e < 4; ++e) cv.h[e] = (__bf16)v[e];
            *(u32x2*)(a.dHidden + at) = cv.u;
        }
    };
    if constexpr (SHARED) {
        CCE_LDS char* const mine = smem + wave * (DB * RB * 1024) + l * 16;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int b = 0; b < RB; ++b) *(CCE_LDS f32x4*)(mine + (d * RB + b) * 1024) = out[d][b];
        barrier_lds_only();
#pragma unroll 1
        for (int i = wave; i < DB * RB; i += 4) {
            f32x4 v = *(const CCE_LDS f32x4*)(smem + i * 1024 + l * 16);
#pragma unroll
            for (int w = 1; w < 4; ++w) v += *(const CCE_LDS f32x4*)(smem + (w * DB * RB + i) * 1024 + l * 16);
            store(i / RB, i % RB, v);
        }
    } else {
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int b = 0; b < RB; ++b) store(d, b, out[d][b]);
    }
}

template <int D, bool SHARED, bool SMOOTH>
__global__ __launch_bounds__(256, (FusedTile<D, SHARED>::kToUnit)) void fused_backward_kernel(const FusedArgs a, int dh_first) {
    extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
    CCE_LDS char* smem = (CCE_LDS char*)smem_generic;
    const int item = (int)blockIdx.x, first = dh_first ? a.n_h : a.n_w;          // the job of the longer items first
    const bool dh = (item < first) == (dh_first != 0);
    const int i = item < first ? item : item - first;
    if (dh) fused_item<D, SHARED, false, SMOOTH>(a, i, smem);
    else fused_item<D, SHARED, true, SMOOTH>(a, i, smem);
}

}  // namespace cce
