// State pass of the vector-decay kernels where few long sequences are cut into segments that different workgroups walk: what
// a segment alone adds to the state, and its total decay per key channel.
//   forward order (the state S):        U = sum_j (prod_{s > j} lambda_s . k_j) v_j^T      over the segment's tokens
//   reversed order (the adjoint G / q_scale, decayed to the state before the segment):
//                                       U = sum_i (prod_{s <= i} lambda_s . q_i) g_i^T
// with lambda 1 at a row boundary.  Both take their decays as running products <= 1 from the segment's end (its start) on:
// nothing to divide, no range to leave, and no accumulator to rescale.
//
// A wavefront needs no other: it walks a quarter of the segment's chunks of 32 tokens in a slot of its own, all 64 x 64
// of the state in its accumulators, without a barrier; the four states are put together at the end.  Rows are read as whole
// 128-byte lines (eight lanes of 16 bytes: 49 ns a 32-row tile and compute unit; the 8-byte pieces of 16 rows that the
// scan wants, straight from memory, take 230) and turned in the slot.
#pragma once

#include "lasad_gated_chunk.h"

namespace lasad {
namespace gchunk {

struct StatePass {
    const void *lam, *key, *val, *val_lo;      // key NULL: 1 - lambda.  val_lo: low-order part of val, or NULL
    lasad_layout_t in;
    int Hh, grid_w, start_pos, n_tokens, mode;
    SegPlan plan;
};

constexpr int kStateRow = 3 * D + 16;          // K^ hi, lo, V
constexpr int kStateSlot = SlotMap<kStateRow>::kHalfs;
constexpr int kStateLdsBytes = 4 * D * 4 + 4 * D * D * 4;      // at the end: the wavefronts' decays and states
static_assert(kStateLdsBytes >= 4 * kStateSlot * 2, "a slot for each wavefront");

// By a workgroup of four wavefronts; lds: kStateLdsBytes.  REV: the reversed order.  KEY: 0 the key is 1 - lambda, 1 given.
// FUSED: lambda holds gate logits (sigmoid), and a given key is a pre-activation (SiLU).  The 64 x 64 state goes to
// out.at(0 ..), the decays to decay.at(0 ..) (base NULL: nowhere).
template <int REV, int KEY, int FUSED, int LO>
__device__ __forceinline__ void state_pass(const StatePass &a, int bh, int seg, unsigned char *lds, const RowState &out, const RowState &decay)
{
    using Map = SlotMap<kStateRow>;
    constexpr int kKh = 0, kKl = D, kV = 2 * D;
    const int b = bh / a.Hh, h = bh - b * a.Hh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pr = lane & 15, g = lane >> 4, l16 = pr;
    const int first = a.plan.start(seg) / C;
    const int end_tok = seg == a.plan.n_seg - 1 ? a.n_tokens : a.plan.start(seg + 1);
    const int n_chunks = (end_tok + C - 1) / C - first;
    // this wavefront's run of chunks, walked towards the segment's start (REV: end)
    const int c_lo = first + n_chunks * wave / 4, c_hi = first + n_chunks * (wave + 1) / 4;
    uint16_t *const slot = (uint16_t *)lds + wave * kStateSlot;

    const int64_t base = (int64_t)b * a.in.stride_b + (int64_t)h * a.in.stride_h;
    const uint32_t row = (uint32_t)a.in.stride_n * 2;
    // rows r0 .. of a chunk: eight lanes a row, eight rows an instruction
    const int lr = lane >> 3, lc = lane & 7;
    u32x4 rl[4], rk[4], rv[4], ro[4];
    auto fetch = [&](int chunk) {
        const int last = min(C, end_tok - chunk * C) - 1;
        const int64_t at = base + (int64_t)chunk * C * a.in.stride_n;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t o = min(8 * i + lr, last) * row + lc * 16;
            rl[i] = *(const u32x4 *)((const char *)((const uint16_t *)a.lam + at) + o);
            if (KEY) rk[i] = *(const u32x4 *)((const char *)((const uint16_t *)a.key + at) + o);
            rv[i] = *(const u32x4 *)((const char *)((const uint16_t *)a.val + at) + o);
            if (LO) ro[i] = *(const u32x4 *)((const char *)((const uint16_t *)a.val_lo + at) + o);
        }
    };

    f32x4v acc[4][4];                              // [key tile][value tile]
    float R[2][8];                                 // decay of the chunks walked before, in lane pr = 0; else 1
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[t][u] = f32x4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) R[s][e] = 1.0f;

    if (c_lo < c_hi) fetch(REV ? c_lo : c_hi - 1);             // ahead of everything that does not need it
    __builtin_amdgcn_sched_barrier(0);
    SplitConst sc;
    sc.init();
    RowBoundaries bounds;
    bounds.init(a.start_pos + (REV ? c_lo : c_hi - 1) * C, a.grid_w, a.mode, C);
    const SlotPtr<kStateRow> sp(slot, lane);
    // the token of this lane's step 0 / 1 (in walking order of the running products)
    const int m0 = REV ? 2 * pr : C - 1 - 2 * pr, m1 = REV ? m0 + 1 : m0 - 1;
    for (int i = 0; i < c_hi - c_lo; ++i) {
        const int chunk = REV ? c_lo + i : c_hi - 1 - i;
        const int left = end_tok - chunk * C;
        // raw rows into the slot: the decay where K^ hi will be, a given key where K^ lo will be
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 8 * j + lr;
            const bool live = r < left;
            uint16_t *const p = slot + Map::row(r) + Map::piece(r, lc);
            *(u32x4 *)(p + kKh) = rl[j];
            if (KEY) *(u32x4 *)(p + kKl) = rk[j];
            *(u32x4 *)(p + kV) = live ? rv[j] : u32x4{0u, 0u, 0u, 0u};
        }
        u32x4 lo_now[4];
        if (LO) {
#pragma unroll
            for (int j = 0; j < 4; ++j) { lo_now[j] = 8 * j + lr < left ? ro[j] : u32x4{0u, 0u, 0u, 0u}; asm volatile("" : "+v"(lo_now[j])); }
        }
        if (i + 1 < c_hi - c_lo) fetch(REV ? chunk + 1 : chunk - 1);
        const uint32_t bmask = bounds.mask();      // tokens at a row boundary
        if (REV) bounds.advance();
        else bounds.retreat();
        const bool one0 = ((bmask >> m0) & 1u) || m0 >= left, one1 = ((bmask >> m1) & 1u) || m1 >= left;
#pragma unroll
        for (int s = 0; s < 2; ++s) {              // channels 32 s + 8 g .. + 7
            float x[2][8], k[2][8];
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int m = it ? m1 : m0;
                const uint16_t *const p = slot + Map::row(m) + Map::piece(m, 4 * s + g);
                const uint4 w = *(const uint4 *)(p + kKh);
                float f[4];
                unpack4(make_uint2(w.x, w.y), f);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[it][e] = f[e];
                unpack4(make_uint2(w.z, w.w), f);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[it][4 + e] = f[e];
                if (KEY) {
                    const uint4 y = *(const uint4 *)(p + kKl);
                    unpack4(make_uint2(y.x, y.y), f);
#pragma unroll
                    for (int e = 0; e < 4; ++e) k[it][e] = f[e];
                    unpack4(make_uint2(y.z, y.w), f);
#pragma unroll
                    for (int e = 0; e < 4; ++e) k[it][4 + e] = f[e];
                }
                const bool one = it ? one1 : one0, live = m < left;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (FUSED) {
                        const float ez = exp_neg(x[it][e]);
                        x[it][e] = __builtin_amdgcn_rcpf(1.0f + ez);
                        if (!KEY) k[it][e] = ez >= 1e30f ? 1.0f : ez * x[it][e];        // 1 - lambda (NaN stays)
                        else k[it][e] *= __builtin_amdgcn_rcpf(1.0f + exp_neg(k[it][e]));
                    } else if (!KEY) {
                        k[it][e] = 1.0f - x[it][e];
                    }
                    x[it][e] = one ? 1.0f : x[it][e];
                    k[it][e] = live ? k[it][e] : 0.f;
                }
            }
            uint4 hi[2], lo[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {          // four channels at a time
                float tot[4], exc[4], kt[2][4];
#pragma unroll
                for (int e = 0; e < 4; ++e) tot[e] = (R[s][4 * q + e] * x[0][4 * q + e]) * x[1][4 * q + e];
                row_scan_mul4(tot, exc);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int c = 4 * q + e;
                    const float before = pr == 0 ? R[s][c] : exc[e];
                    const float mid = before * x[0][c];
                    kt[0][e] = k[0][c] * (REV ? mid : before);
                    kt[1][e] = k[1][c] * (REV ? tot[e] : mid);
                    const float all = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(tot[e]), 0x15F, 0xf, 0xf, true));    // of lane 15
                    R[s][c] = pr == 0 ? all : 1.0f;
                }
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    uint2 h2, l2;
                    split2(kt[it][0], kt[it][1], h2.x, l2.x, sc);
                    split2(kt[it][2], kt[it][3], h2.y, l2.y, sc);
                    if (q == 0) { hi[it].x = h2.x; hi[it].y = h2.y; lo[it].x = l2.x; lo[it].y = l2.y; }
                    else { hi[it].z = h2.x; hi[it].w = h2.y; lo[it].z = l2.x; lo[it].w = l2.y; }
                }
            }
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int m = it ? m1 : m0;
                uint16_t *const p = slot + Map::row(m) + Map::piece(m, 4 * s + g);
                *(uint4 *)(p + kKh) = hi[it];
                *(uint4 *)(p + kKl) = lo[it];
            }
        }
        Frag fv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) fv[u] = sp.tokens(kV + 16 * u);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const Frag kh = sp.state_rows(kKh, t), kl = sp.state_rows(kKl, t);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[t][u] = mfma16(kh, fv[u], acc[t][u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[t][u] = mfma16(kl, fv[u], acc[t][u]);
        }
        if (LO) {                                  // the low-order part of v in the place of v
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 8 * j + lr;
                *(u32x4 *)(slot + Map::row(r) + Map::piece(r, lc) + kV) = lo_now[j];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) fv[u] = sp.tokens(kV + 16 * u);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const Frag kh = sp.state_rows(kKh, t);
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[t][u] = mfma16(kh, fv[u], acc[t][u]);
            }
        }
    }

    // Together: S = U_3 + D_3 U_2 + D_3 D_2 U_1 + ... (REV: U_0 + D_0 U_1 + ...).  Every wavefront scales its state by the decays
    // of the runs between it and the segment's end (start); then all 256 threads add the four up through LDS (in a fixed order; pair
    // by pair, a wavefront at a time, the pass took 1 us more).
    float *const sD = (float *)lds;                // [wave][64]
    float *const sAcc = sD + 4 * D;                // [wave][64][64]
    __syncthreads();
    if (pr == 0) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) sD[wave * D + 32 * s + 8 * g + e] = R[s][e];
    }
    __syncthreads();
    if (decay.base && threadIdx.x < D) {
        const int c = threadIdx.x;
        *decay.at(c) = (sD[c] * sD[D + c]) * (sD[2 * D + c] * sD[3 * D + c]);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = state_channel(t, g) + r;
            float f = 1.0f;
            for (int w = 0; w < 4; ++w)
                if (REV ? w < wave : w > wave) f *= sD[w * D + c];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[t][u][r] *= f;
        }
    float *const mine = sAcc + wave * D * D;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[(state_channel(t, g) + r) * D + 16 * u + l16] = acc[t][u][r];
    __syncthreads();
    for (int i = threadIdx.x * 4; i < D * D; i += 1024) {
        const f32x4v *const p = (const f32x4v *)(sAcc + i);
        *(f32x4v *)out.at(i) = (p[0] + p[D * D / 4]) + (p[2 * (D * D / 4)] + p[3 * (D * D / 4)]);
    }
}

}  // namespace gchunk
}  // namespace lasad
