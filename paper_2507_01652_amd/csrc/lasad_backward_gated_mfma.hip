// Chunked matrix-core passes of the vector-decay backward for few or short sequences (bf16 inputs, head dim 64; the rule is at
// chunk_plan in lasad_backward_gated.hip): all three side by side, each with a compute unit of its own, on the building blocks of the
// forward (lasad_gated_chunk.h: chunks of 32 tokens, loader wavefronts one chunk ahead, compute wavefronts that own 16
// columns of the state).  lasad_backward_gated.hip has the derivation.  Two kinds of pass:
//
// ROW pass (dv): the forward itself over the reversed sequence, query := the key of the token
//   (1 - lambda if tied), key := q, value := d_o, decay of step m := lambda of step m - 1.
//
// COL pass (dq; dk over the reversed sequence): with A_i the chunk-local running product of the
//   decay and Z~_j = z_j / A_j (z the key for dq, q for dk),
//       out_i = A_i (.) [ S x_i + sum_{j<=i} (x_i . y_j) Z~_j ],   S <- diag(A_end) (S + Z~^T Y)
//   (x, y: d_o and v for dq, v and d_o for dk), times q_scale.  Here a compute wavefront owns 16 KEY channels c: its
//   accumulators hold S^T, a tile's rows being value channels e and its columns c, so that S x contracts over the rows,
//   the row scaling by A_end is one factor per lane, and x and y enter as the plain bf16 tensors they are (one MFMA per
//   score step instead of three).  The loaders leave A itself as an fp32 tile.
//
// A chunk that leaves the range of the factorisation sends the workgroup to the token-serial walk
// of the same pass (lasad_scan.h with operand roles).
#include "lasad_gated_chunk.h"
#include "lasad_scan.h"

namespace lasad {

namespace {

using namespace gchunk;

constexpr int kThreads = 256;                  // of one role: compute, loaders
constexpr int64_t kMaxStride = 1 << 25;        // 32 rows of it, two bytes an element, stay below 2^32

enum { DQ = 0, DV = 1, DK = 2 };

// A token's row of a chunk slot (bf16 elements): Z~ hi, lo, then COL: x, y, the low-order part of one of them;
// ROW: Q~ hi, lo, V, low-order part of V.
template <int PASS>
struct Slot {
    static constexpr bool COL = PASS != DV;
    static constexpr int ROW = (COL ? 5 : 6) * D + 16;
    static constexpr int Zh = 0, Zl = D;
    static constexpr int X = 2 * D;                            // COL
    static constexpr int Qh = 2 * D, Ql = 3 * D;               // ROW
    static constexpr int Y = COL ? 3 * D : 4 * D;              // y; ROW: V
    static constexpr int Lo = COL ? 4 * D : 5 * D;             // low-order part of d_o: x (dq), y (dk), V (dv)
    using Map = SlotMap<ROW>;
    static constexpr int kHalfs = Map::kHalfs;
    // two slots, the output tiles, COL: the tiles of A
    static constexpr int kBytes = 2 * kHalfs * 2 + 2 * C * OS * 4 + (COL ? 2 * C * OS * 4 : 0);
};
constexpr int kLdsBytes = Slot<DQ>::kBytes > Slot<DV>::kBytes ? Slot<DQ>::kBytes : Slot<DV>::kBytes;

// The token-serial walk of a pass, out of line.  It is handed the arguments where the launch put
// them (the kernel-argument segment): references to the kernel's by-value parameter, or copies,
// would make every thread of every launch write them to its stack first.
template <int OUT_BF16, int COL>
__device__ __noinline__ void redo_roles(const ForwardArgs *a, const scan::ScanRoles *r, int bh, LdsFloat *lds)
{
    if (COL) scan::scan_sequence<1, 0, scan::ROLES_COL, 64>(*a, bh, 0, (float *)lds, r);
    else scan::scan_sequence<1, OUT_BF16, scan::ROLES_ROW, 64>(*a, bh, 0, (float *)lds, r);
}

// A loader thread's share of a chunk: tokens 2 pr, 2 pr + 1 and channels pcol .. + 3 of the decay, z and (ROW) query
// tensors, and one 16-byte piece of a row of x, y and the low-order part of d_o.  Uniform bases, advanced chunk by chunk
// on the scalar unit, plus 32-bit byte offsets; the reversed passes (negative token stride) keep their bases at the
// chunk's last token, the lowest address.  Rows past the end re-read the last token.
// A reversed pass starts with the chunk that the forward one ends with: its first `lead` rows are no tokens (they re-read
// the first one), so that both have their chunks' ends at the same tokens, where the finishing kernel wants their states.
template <int PASS, int OWNKEY, int LO, int NG>
struct PassStage {
    static constexpr bool REV = PASS != DQ, COL = PASS != DV, ZLOAD = PASS != DQ || OWNKEY;
    const char *l, *z, *q, *x, *y, *lo;
    uint32_t row;                      // bytes from token to token
    int left;                          // rows from the chunk's first one on, > 0
    int lead;                          // REV: rows of the chunk before the walk's first token
    bool start;                        // REV: the walk's first chunk: its first step has no decay to read
    struct Regs {
        uint2 rl[2], rz[2], rq[2];
        u32x4 rx, ry, rlo;
    };

    // from the walk's row `first` on, n rows; its first `pad` rows (REV) are no tokens
    __device__ __forceinline__ void init(const ForwardArgs &a, int64_t base, int first, int n, int pad)
    {
        left = n;
        start = first == 0;
        lead = start ? pad : 0;
        const int64_t s = a.in.stride_n;
        row = (uint32_t)(REV ? -s : s) * 2;
        const int64_t b = base + (first + (REV ? C - 1 - pad : 0)) * s;
        l = (const char *)((const uint16_t *)a.lam + b);
        z = ZLOAD ? (const char *)((const uint16_t *)a.k + b) : nullptr;
        q = COL ? nullptr : (const char *)((const uint16_t *)a.q + b);
        x = COL ? (const char *)((const uint16_t *)a.q + b) : nullptr;
        y = (const char *)((const uint16_t *)a.v + b);
        lo = LO ? (const char *)((const uint16_t *)(PASS == DQ ? a.q_lo : a.v_lo) + b) : nullptr;
    }
    __device__ __forceinline__ void fetch(Regs &f, int pr, int pcol, int st) const
    {
        const int last = REV ? C - 1 : min(C, left) - 1;
        const int m0 = REV ? max(2 * pr, lead) : min(2 * pr, last), m1 = REV ? max(2 * pr + 1, lead) : min(2 * pr + 1, last);
        const int mv = REV ? max(st >> 3, lead) : min(st >> 3, last);
        const uint32_t o0 = (REV ? last - m0 : m0) * row + pcol * 2, o1 = (REV ? last - m1 : m1) * row + pcol * 2;
        const uint32_t ov = (REV ? last - mv : mv) * row + (st & 7) * 16;
        if (REV) {                     // step m applies the decay of the token walked before it
            f.rl[0] = *(const uint2 *)(l + (start && m0 == lead ? o0 : o0 + row));
            f.rl[1] = *(const uint2 *)(l + (start && m1 == lead ? o1 : o1 + row));
        } else {
            f.rl[0] = *(const uint2 *)(l + o0);
            f.rl[1] = *(const uint2 *)(l + o1);
        }
        if (ZLOAD) { f.rz[0] = *(const uint2 *)(z + o0); f.rz[1] = *(const uint2 *)(z + o1); }
        if (!COL) { f.rq[0] = *(const uint2 *)(q + o0); f.rq[1] = *(const uint2 *)(q + o1); }
        if (COL) f.rx = *(const u32x4 *)(x + ov);
        f.ry = *(const u32x4 *)(y + ov);
        if (LO) f.rlo = *(const u32x4 *)(lo + ov);
    }
    // on to the group's next chunk; past the end the last one is read again
    __device__ __forceinline__ void next(int64_t stride_n)
    {
        if (left <= NG * C) return;
        left -= NG * C;
        lead = 0;
        start = false;
        const int64_t adv = NG * C * stride_n * 2;
        l += adv; y += adv;
        if (ZLOAD) z += adv;
        if (!COL) q += adv;
        if (COL) x += adv;
        if (LO) lo += adv;
    }
};

// One pass of sequence bh by the calling workgroup of four compute wavefronts and NG groups of four loaders; ka, kr: its
// arguments and operand roles in the kernel-argument segment (for the redo).
template <int PASS, int OUT_BF16, int OWNKEY, int FUSED, int LO, int NG>
__device__ __forceinline__ void pass_body(const ForwardArgs &a, const ForwardArgs *ka, const scan::ScanRoles *kr, int bh,
                                          unsigned char *smem, float (*sTot)[D], int (*sTrip)[4])
{
    using SL = Slot<PASS>;
    constexpr bool REV = PASS != DQ, COL = SL::COL;
    uint16_t *const slots = (uint16_t *)smem;
    float *const outs = (float *)(slots + 2 * SL::kHalfs);
    float *const decays = outs + 2 * C * OS;               // COL: A, laid out like an output tile
    const int b = bh / a.Hh, h = bh - b * a.Hh;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int pad = REV ? (C - 1) - (a.n_tokens - 1) % C : 0;      // rows before the walk's first token
    const int n = a.n_tokens + pad;                        // rows
    // (one loader group: the walk goes two chunks at a time; the second may be empty)
    const int n_chunks = NG == 1 ? (n + 2 * C - 1) / (2 * C) * 2 : (n + C - 1) / C;
    SplitConst sc;
    sc.init();
    auto redo = [&]() {
        if (tid < scan::kThreads) redo_roles<OUT_BF16, COL>(ka, kr, bh, (LdsFloat *)smem);
    };

    if (wave >= 4) {
        // ===================================== loader wavefronts =====================================
        const int grp = NG == 2 ? (wave >> 2) - 1 : 0, lw = wave & 3, st = tid & 255;
        const int first = grp * C < n ? grp * C : 0;           // (a group without a chunk reads the first one, for nobody)
        const int pr = lane & 15, pcol = 16 * lw + 4 * (lane >> 4);
        using Stage = PassStage<PASS, OWNKEY, LO, NG>;
        Stage sg;
        sg.init(a, (int64_t)b * a.in.stride_b + (int64_t)h * a.in.stride_h, first, n - first, pad);
        typename Stage::Regs r0, r1;               // (one loader group: two chunks of loads in flight)
        sg.fetch(r0, pr, pcol, st);                // ahead of everything that does not need it
        if (NG == 1) {
            sg.next(a.in.stride_n);
            sg.fetch(r1, pr, pcol, st);
        }
        __builtin_amdgcn_sched_barrier(0);
        RowBoundaries bounds;
        int col = a.start_pos;                     // of the walk's first row
        if (REV) {
            col = col % a.grid_w - pad % a.grid_w;
            if (col < 0) col += a.grid_w;
        }
        bounds.init(col + grp * C, a.grid_w, a.mode, NG * C);
        int left = n - grp * C;                    // rows from the next chunk to be prepared on
        const int put = SL::Map::at(2 * pr, pcol), put_piece = SL::Map::at(st >> 3, (st & 7) * 8);
        const int orow = st >> 3, ocol = (st & 7) * 8;
        const int64_t o_lane = orow * a.out.stride_n + ocol;
        int64_t o_chunk = (int64_t)b * a.out.stride_b + (int64_t)h * a.out.stride_h +
                          ((NG == 2 && grp == 0 ? C : 0) - pad) * a.out.stride_n;
        auto store_tile = [&](int chunk) {
            const float *tile = outs + (chunk & 1) * C * OS + orow * OS + ocol;
            float4 u = *(const float4 *)tile, w = *(const float4 *)(tile + 4);
            u = make_float4(u.x * a.q_scale, u.y * a.q_scale, u.z * a.q_scale, u.w * a.q_scale);
            w = make_float4(w.x * a.q_scale, w.y * a.q_scale, w.z * a.q_scale, w.w * a.q_scale);
            if (chunk * C + orow >= pad && chunk * C + orow < n) {
                const int64_t i = o_chunk + o_lane;
                if (OUT_BF16) {
                    gstore16<true>((uint16_t *)a.o + i, make_uint4(pack2(u.x, u.y), pack2(u.z, u.w), pack2(w.x, w.y), pack2(w.z, w.w)));
                } else {                           // (read again by the finishing kernel)
                    gstore16<false>((float *)a.o + i, u.x, u.y, u.z, u.w);
                    gstore16<false>((float *)a.o + i + 4, w.x, w.y, w.z, w.w);
                }
            }
            o_chunk += NG * C * a.out.stride_n;                // (of two groups, each stores every other tile)
        };

        // between the phases of a chunk's preparation
        uint2 pq[2];
        u32x4 px, py, plo;
        bool row_live;
        float z[2][4], x[2][4], tot[4], exc[4];

        // the plain rows into slot p (a row that is no token is a query that nobody stores, and zero as y)
        auto put_rows = [&](int p) {
            uint16_t *const piece = slots + p * SL::kHalfs + put_piece;
            if (COL) *(u32x4 *)&piece[SL::X] = px;
            *(u32x4 *)&piece[SL::Y] = row_live ? py : u32x4{0u, 0u, 0u, 0u};
            if (LO) *(u32x4 *)&piece[SL::Lo] = row_live ? plo : u32x4{0u, 0u, 0u, 0u};
        };
        // Phase A: everything that needs no slot; done: the finished chunk to be stored meanwhile, or -1.  One loader group
        // runs both phases in one period and puts the plain rows into slot p at once.  (Past the end the last chunk's data go
        // once more into a slot that nobody reads.)
        auto phase_a = [&](typename Stage::Regs &f, int p, int done, bool walk_start) {
            uint32_t bmask = bounds.mask();
            bounds.advance();
            const int lead = REV && walk_start ? pad : 0;
            if (REV && walk_start) bmask |= 1u << lead;        // (the walk's first step: no decay)
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                unpack4(f.rl[it], x[it]);
                if (sg.ZLOAD) unpack4(f.rz[it], z[it]);
                if (!COL) pq[it] = f.rq[it];
            }
            row_live = (st >> 3) >= lead && (st >> 3) < left;
            if (COL) px = f.rx;
            py = f.ry;
            if (LO) plo = f.rlo;
            if (NG == 1) {
                put_rows(p);
            } else {
                if (COL) asm volatile("" : "+v"(px));
                asm volatile("" : "+v"(py));
                if (LO) asm volatile("" : "+v"(plo));
            }
            // (the fetched registers are free from here on, and the compiler must see it so: lasad_forward_gated_chunk.hip)
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                asm volatile("" : "+v"(x[it][0]), "+v"(x[it][1]), "+v"(x[it][2]), "+v"(x[it][3]));
                if (sg.ZLOAD) asm volatile("" : "+v"(z[it][0]), "+v"(z[it][1]), "+v"(z[it][2]), "+v"(z[it][3]));
                if (!COL) asm volatile("" : "+v"(pq[it].x), "+v"(pq[it].y));
            }
            if (done >= 0) store_tile(done);
            __builtin_amdgcn_sched_barrier(0);
            sg.next(a.in.stride_n);
            sg.fetch(f, pr, pcol, st);
#pragma unroll
            for (int it = 0; it < 2; ++it) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (PASS == DQ && FUSED) {     // z = k = 1 - lambda = exp(-gate) lambda, and 1 / lambda = 1 + exp(-gate)
                        z[it][e] = exp_neg(x[it][e]);
                        x[it][e] = 1.0f + z[it][e];
                    } else if (FUSED) {
                        x[it][e] = 1.0f + exp_neg(x[it][e]);
                        z[it][e] *= __builtin_amdgcn_rcpf(1.0f + exp_neg(z[it][e]));
                    } else if (!sg.ZLOAD) {
                        z[it][e] = 1.0f - x[it][e];
                    }
                }
                if (bmask & (0x55555555u << it)) { // some token of this parity sits on a boundary: lambda 1
                    if ((bmask >> (2 * pr + it)) & 1u) {
                        asm volatile("");
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            // (the tied key keeps its own lambda, see the forward)
                            if (PASS == DQ && FUSED) z[it][e] = z[it][e] >= 1e30f ? 1.0f : z[it][e] * __builtin_amdgcn_rcpf(x[it][e]);
                            x[it][e] = 1.0f;
                        }
                    }
                }
            }
            if (left < C || (REV && lead > 0)) {   // rows that are no tokens get lambda 1, z = 0
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const bool live = 2 * pr + it >= lead && 2 * pr + it < left;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        x[it][e] = live ? x[it][e] : 1.0f;
                        z[it][e] = live ? z[it][e] : 0.f;
                    }
                }
            }
            left -= NG * C;
#pragma unroll
            for (int e = 0; e < 4; ++e) tot[e] = x[0][e] * x[1][e];
            row_scan_mul4(tot, exc);               // (FUSED: of the reciprocals throughout)
        };
        // Phase B: the chunk into slot p, and its range flag for the barrier that ends this period.
        auto phase_b = [&](int p) {
            if (NG == 2) put_rows(p);
            bool trip;
            if (FUSED) trip = !(fmaxf(fmaxf(tot[0], tot[1]), fmaxf(tot[2], tot[3])) <= kMaxInvDecay);
            else trip = !(fminf(fminf(tot[0], tot[1]), fminf(tot[2], tot[3])) >= 1.0f / kMaxInvDecay);
            if (pr == 15)
                *(float4 *)&sTot[p][pcol] = FUSED ? make_float4(__builtin_amdgcn_rcpf(tot[0]), __builtin_amdgcn_rcpf(tot[1]),
                                                                __builtin_amdgcn_rcpf(tot[2]), __builtin_amdgcn_rcpf(tot[3]))
                                                  : make_float4(tot[0], tot[1], tot[2], tot[3]);
            const bool any = __any(trip);
            if (lane == 0) sTrip[p][lw] = any ? 1 : 0;
            uint16_t *rows = slots + p * SL::kHalfs + put;
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                float zt[4], dec[4];               // Z~ and A of this token
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float before = it ? exc[e] * x[0][e] : exc[e];
                    const float after = it ? tot[e] : exc[e] * x[0][e];
                    if (PASS == DQ && FUSED) zt[e] = z[it][e] * before;
                    else if (FUSED) zt[e] = z[it][e] * after;
                    const float inv = __builtin_amdgcn_rcpf(after);
                    if (!FUSED) zt[e] = z[it][e] * inv;
                    dec[e] = FUSED && COL ? inv : after;
                }
                put_pair4(rows + it * SL::ROW + SL::Zh, rows + it * SL::ROW + SL::Zl, zt, sc);
                if (COL) {
                    *(float4 *)&decays[p * C * OS + (2 * pr + it) * OS + pcol] = make_float4(dec[0], dec[1], dec[2], dec[3]);
                } else {
                    float q[4];
                    unpack4(pq[it], q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (FUSED) q[e] = __builtin_amdgcn_rcpf((1.0f + exp_neg(-q[e])) * dec[e]);     // (1 - sigmoid(gate)) A
                        else q[e] = (OWNKEY ? q[e] : 1.0f - q[e]) * dec[e];
                    }
                    put_pair4(rows + it * SL::ROW + SL::Qh, rows + it * SL::ROW + SL::Ql, q, sc);
                }
            }
        };
        bool fine = true;
        if constexpr (NG == 1) {
            // Two chunks of loads in flight, in two sets of registers.  (A pair of chunks is always done as a whole, range
            // flags tested at its end: with a way out between its halves the compiler waits for both sets at the loop's top.)
            auto prepare = [&](typename Stage::Regs &f, int p, int done, bool walk_start) {
                phase_a(f, p, done, walk_start);
                phase_b(p);
            };
            prepare(r0, 0, -1, true);
            __syncthreads();
            for (int chunk = 0; fine && chunk < n_chunks; chunk += 2) {
                const int4 t0 = *(const int4 *)sTrip[0];
                prepare(r1, 1, chunk - 1, false);
                __syncthreads();
                const int4 t1 = *(const int4 *)sTrip[1];
                prepare(r0, 0, chunk, false);
                fine = (t0.x | t0.y | t0.z | t0.w | t1.x | t1.y | t1.z | t1.w) == 0;
                __syncthreads();
            }
        } else {
            // the groups take the chunks in turn, a period for each phase
            int4 f;                                // a chunk's range flags, read at the start of its period and tested at the end
            auto end_period = [&]() {
                fine = (f.x | f.y | f.z | f.w) == 0;
                __syncthreads();
            };
            phase_a(r0, 0, -1, grp == 0);
            if (grp == 0) phase_b(0);
            __syncthreads();
            if (grp == 1) {                        // period 0
                f = *(const int4 *)sTrip[0];
                phase_b(1);
                end_period();
            }
            for (int chunk = grp; fine && chunk < n_chunks; chunk += 2) {
                f = *(const int4 *)sTrip[chunk & 1];
                phase_a(r0, 0, chunk - 1, false);
                end_period();
                if (!fine || chunk + 1 == n_chunks) break;
                f = *(const int4 *)sTrip[(chunk + 1) & 1];
                phase_b(chunk & 1);
                end_period();
            }
        }
        if (!fine) redo();
        else if (NG == 1 || grp == (n_chunks & 1)) store_tile(n_chunks - 1);
        return;
    }

    // ===================================== compute wavefronts =====================================
    __builtin_amdgcn_s_setprio(2);                 // the chain from chunk to chunk; the loaders fill the gaps
    const int l16 = lane & 15, g = lane >> 4;
    const int col0 = 16 * wave;                    // value channels (ROW) / key channels (COL) of this wavefront
    // element (t, r) of the accumulators: ROW: S[state_channel(t, g) + r][col0 + l16]; COL: the same of S^T
    const int64_t s_off = (int64_t)bh * D * D + (COL ? (col0 + l16) * D : col0 + l16);
    f32x4v accS[4];
    const f32x4v zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) accS[t] = zero4;
    if (a.state_in) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) accS[t][r] = a.state_in[s_off + (state_channel(t, g) + r) * (COL ? 1 : D)];
    }

    // COL: the states at the segment bounds of the finishing kernel (seg_chunks chunks a segment, counted from the first
    // token; the reversed walk comes to them from the other end, its chunks' ends at the same tokens)
    const int n_bounds = COL && a.seg_states ? a.n_segments - 1 : 0;
    int bound = REV ? n_bounds - 1 : 0;                        // the next one
    int bound_at = REV ? (n + C - 1) / C - a.seg_chunks * n_bounds : a.seg_chunks;

    __syncthreads();
    bool fine = true;
    for (int chunk = 0; (fine || (NG == 1 && (chunk & 1))) && chunk < n_chunks; ++chunk) {
        const int4 f = *(const int4 *)sTrip[chunk & 1];
        const SlotPtr<SL::ROW> sp(slots + (chunk & 1) * SL::kHalfs, lane);
        f32x4v p00 = zero4, p01 = zero4, p11 = zero4;              // scores P^T[j][i]: (key tile, query tile)
        f32x4v o0 = zero4, o1 = zero4;                             // O^T[.][i] of the two query tiles
        if (COL) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const Frag x0 = sp.rows(0, SL::X, s), x1 = sp.rows(16, SL::X, s);
                const Frag y0 = sp.rows(0, SL::Y, s), y1 = sp.rows(16, SL::Y, s);
                Frag l0, l1;
                if (LO) { l0 = sp.rows(0, SL::Lo, s); l1 = sp.rows(16, SL::Lo, s); }
                Frag sh, sl;
                split_tiles(accS[2 * s], accS[2 * s + 1], sh, sl, sc);
                // ---- P^T[j][i] += sum_e Y[j][e] X[i][e],  O^T[c][i] += sum_e S[c][e] X[i][e] ----
                p00 = mfma16(y0, x0, p00);
                p01 = mfma16(y0, x1, p01);
                p11 = mfma16(y1, x1, p11);
                o0 = mfma16(sh, x0, o0);
                o1 = mfma16(sh, x1, o1);
                if (LO) {
                    p00 = PASS == DQ ? mfma16(y0, l0, p00) : mfma16(l0, x0, p00);
                    p01 = PASS == DQ ? mfma16(y0, l1, p01) : mfma16(l0, x1, p01);
                    p11 = PASS == DQ ? mfma16(y1, l1, p11) : mfma16(l1, x1, p11);
                }
                o0 = mfma16(sl, x0, o0);
                o1 = mfma16(sl, x1, o1);
                if (LO && PASS == DQ) {
                    o0 = mfma16(sh, l0, o0);
                    o1 = mfma16(sh, l1, o1);
                }
            }
        } else {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const Frag q0h = sp.rows(0, SL::Qh, s), q1h = sp.rows(16, SL::Qh, s);
                const Frag q0l = sp.rows(0, SL::Ql, s), q1l = sp.rows(16, SL::Ql, s);
                const Frag k0h = sp.rows(0, SL::Zh, s), k0l = sp.rows(0, SL::Zl, s);
                const Frag k1h = sp.rows(16, SL::Zh, s), k1l = sp.rows(16, SL::Zl, s);
                Frag sh, sl;
                split_tiles(accS[2 * s], accS[2 * s + 1], sh, sl, sc);
                p00 = mfma16(k0h, q0h, p00);
                p01 = mfma16(k0h, q1h, p01);
                p11 = mfma16(k1h, q1h, p11);
                o0 = mfma16(sh, q0h, o0);
                o1 = mfma16(sh, q1h, o1);
                p00 = mfma16(k0l, q0h, p00);
                p01 = mfma16(k0l, q1h, p01);
                p11 = mfma16(k1l, q1h, p11);
                o0 = mfma16(sl, q0h, o0);
                o1 = mfma16(sl, q1h, o1);
                p00 = mfma16(k0h, q0l, p00);
                p01 = mfma16(k0h, q1l, p01);
                p11 = mfma16(k1h, q1l, p11);
                o0 = mfma16(sh, q0l, o0);
                o1 = mfma16(sh, q1l, o1);
            }
        }
        causal_mask(p00, lane);
        causal_mask(p11, lane);
        Frag ph, pl;
        float *tile = outs + (chunk & 1) * C * OS + l16 * OS + col0 + 4 * g;
        if (COL) {
            const Frag zh = sp.tokens(SL::Zh + col0), zl = sp.tokens(SL::Zl + col0);
            // ---- S^T[e][c] += sum_j Y[j][e] Z~[j][c], O^T[c][i] += sum_j Z~[j][c] P^T[j][i] ----
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const Frag fy = sp.state_rows(SL::Y, t);
                accS[t] = mfma16(fy, zh, accS[t]);
                accS[t] = mfma16(fy, zl, accS[t]);
                if (LO && PASS == DK) accS[t] = mfma16(sp.state_rows(SL::Lo, t), zh, accS[t]);
            }
            split_tiles(p00, zero4, ph, pl, sc);                   // (keys 16 .. 31 come after queries 0 .. 15)
            o0 = mfma16(zh, ph, o0);
            o0 = mfma16(zl, ph, o0);
            o0 = mfma16(zh, pl, o0);
            split_tiles(p01, p11, ph, pl, sc);
            o1 = mfma16(zh, ph, o1);
            o1 = mfma16(zl, ph, o1);
            o1 = mfma16(zh, pl, o1);
            const float end = sTot[chunk & 1][col0 + l16];
#pragma unroll
            for (int t = 0; t < 4; ++t) accS[t] *= end;
            if (chunk + 1 == bound_at && (unsigned)bound < (unsigned)n_bounds) {
                float *p = a.seg_states + (((int64_t)bh * n_bounds + bound) * D + col0 + l16) * D;
#pragma unroll
                for (int t = 0; t < 4; ++t) *(f32x4v *)(p + state_channel(t, g)) = accS[t];
                bound += REV ? -1 : 1;
                bound_at += a.seg_chunks;
            }
            // O^T row 4 g + r is key channel col0 + 4 g + r of token l16 / 16 + l16: times its A
            const float *dec = decays + (chunk & 1) * C * OS + l16 * OS + col0 + 4 * g;
            const float4 d0 = *(const float4 *)dec, d1 = *(const float4 *)(dec + 16 * OS);
            *(float4 *)tile = make_float4(o0[0] * d0.x, o0[1] * d0.y, o0[2] * d0.z, o0[3] * d0.w);
            *(float4 *)(tile + 16 * OS) = make_float4(o1[0] * d1.x, o1[1] * d1.y, o1[2] * d1.z, o1[3] * d1.w);
        } else {
            const Frag fv = sp.tokens(SL::Y + col0);
            Frag fl;
            if (LO) fl = sp.tokens(SL::Lo + col0);
            // ---- S[c][n] += sum_j Z~[j][c] V[j][n], O^T[n][i] += sum_j V[j][n] P^T[j][i] ----
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const Frag zh = sp.state_rows(SL::Zh, t);
                accS[t] = mfma16(zh, fv, accS[t]);
                accS[t] = mfma16(sp.state_rows(SL::Zl, t), fv, accS[t]);
                if (LO) accS[t] = mfma16(zh, fl, accS[t]);
            }
            split_tiles(p00, zero4, ph, pl, sc);
            o0 = mfma16(fv, ph, o0);
            o0 = mfma16(fv, pl, o0);
            if (LO) o0 = mfma16(fl, ph, o0);
            split_tiles(p01, p11, ph, pl, sc);
            o1 = mfma16(fv, ph, o1);
            o1 = mfma16(fv, pl, o1);
            if (LO) o1 = mfma16(fl, ph, o1);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float4 t4 = *(const float4 *)&sTot[chunk & 1][state_channel(t, g)];
                accS[t][0] *= t4.x; accS[t][1] *= t4.y; accS[t][2] *= t4.z; accS[t][3] *= t4.w;
            }
            *(float4 *)tile = make_float4(o0[0], o0[1], o0[2], o0[3]);
            *(float4 *)(tile + 16 * OS) = make_float4(o1[0], o1[1], o1[2], o1[3]);
        }
        fine = fine && (f.x | f.y | f.z | f.w) == 0;
        __syncthreads();
    }
    if (n_bounds && tid == 0) ((int *)(a.seg_states + (int64_t)a.B * a.Hh * n_bounds * D * D))[bh] = fine;
    if (!fine) {
        redo();
        return;
    }
    if (a.state_out) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) a.state_out[s_off + (state_channel(t, g) + r) * (COL ? 1 : D)] = accS[t][r];
    }
}

struct PassSet {
    ForwardArgs a[3];              // dq, dv, dk: the pass's operands in the forward's fields
    scan::ScanRoles roles[3];      // the same passes for the token-serial walk (range fallback)
};

// The three passes of a call in one launch.  Workgroups come in groups of 8 sequences x 3 passes,
// a sequence's passes 8 workgroup ids apart: they start together on the same XCD (ids go round
// the 8 XCDs) and share what they both read through its L2 (dv and dk walk the same q, d_o and
// lambda rows in the same order).  TIED: the key is 1 - lambda.  FUSED (with TIED): the layer's
// backward: the q and lambda tensors hold Algorithm 1's pre-activation query and gate logits, and
// d_o comes as a bf16 pair hi + lo, both parts used in every pass (x of the dq pass, y of the dk pass, the value
// operand of the dv pass: one more MFMA per score or product step and per state term).  d_o is
// orthogonal to the recurrence output, which makes dq and dk small differences of larger terms
// early in a sequence; a single bf16 there costs up to 0.15 of the RMS in single elements, and in dv, which for
// the last tokens of a sequence is a multiple of a single d_o row, up to 0.02.
// NG = 2: a second loader group, for workgroups that have a compute unit to themselves (a lone workgroup is bound by what
// its loaders issue, as in the forward).
template <int OUT_BF16, int TIED, int FUSED, int NG>
__global__ void __launch_bounds__((1 + NG) * kThreads, NG == 1 ? 4 : 3)
backward_gated_passes_kernel(PassSet ps)
{
    constexpr int kScanFloats = scan::lds_floats<scan::ROLES_ROW>();
    static_assert(kLdsBytes >= kScanFloats * 4, "the redo needs the LDS block");
    __shared__ __attribute__((aligned(16))) unsigned char smem[kLdsBytes];
    __shared__ __attribute__((aligned(16))) float sTot[2][D];  // A_end per key channel, by chunk parity
    __shared__ __attribute__((aligned(16))) int sTrip[2][4];   // range flag of each loader wavefront, by barrier parity
    const int grp = blockIdx.x / 24, r = blockIdx.x - grp * 24;
    const int pass = r >> 3, bh = grp * 8 + (r & 7);
    if (bh >= ps.a[0].B * ps.a[0].Hh) return;                  // (the last group may be partly empty)
    const PassSet *kp = (const PassSet *)__builtin_amdgcn_kernarg_segment_ptr();
    if (pass == DQ) pass_body<DQ, 0, !TIED, FUSED, FUSED, NG>(ps.a[0], &kp->a[0], &kp->roles[0], bh, smem, sTot, sTrip);
    else if (pass == DV) pass_body<DV, OUT_BF16, !TIED, FUSED, FUSED, NG>(ps.a[1], &kp->a[1], &kp->roles[1], bh, smem, sTot, sTrip);
    else pass_body<DK, 0, !TIED, FUSED, FUSED, NG>(ps.a[2], &kp->a[2], &kp->roles[2], bh, smem, sTot, sTrip);
}

}  // namespace

bool backward_gated_passes_fit(int64_t stride_n) { return stride_n >= 0 && stride_n <= kMaxStride; }

// The three passes of the vector-decay backward with the matrix-core kernel, one launch.
// a[0..2], roles[0..2]: dq (column pass, forward order), dv (row pass, reversed; its query tensor
// is lambda itself when tied), dk (column pass, reversed), as lasad_backward_gated.hip sets them up.
hipError_t launch_backward_gated_passes(const ForwardArgs *a, const scan::ScanRoles *roles, bool tied, hipStream_t s)
{
    if (a[0].d != D || a[0].io_dtype != LASAD_BF16 || a[0].n_tokens < 1) return hipErrorInvalidValue;
    const int64_t n_seq = (int64_t)a[0].B * a[0].Hh;
    if ((n_seq + 7) / 8 * 24 > 0x7fffffff) return hipErrorInvalidValue;
    PassSet ps;
    for (int i = 0; i < 3; ++i) { ps.a[i] = a[i]; ps.roles[i] = roles[i]; }
    // Two loader groups where every workgroup has a compute unit: an XCD gets three workgroups of every eighth sequence and has
    // 32 units, so up to 80 sequences.  One -> two groups, us a
    // call: 80 of 576 44.1 -> 42.8, 88 -> 80 (fused layer); but 84 of 256 29.5 -> 32.7.  Two chunks
    // (one pair of one group) are bound by their first loads: 24 of 64 10.0 -> 10.4, of 96 13.4 -> 12.6.
    const bool pair = a[0].n_tokens > C && a[0].n_tokens <= 2 * C;
    const int ng = n_seq <= 80 && !pair ? 2 : 1;
    const dim3 grid((unsigned)((n_seq + 7) / 8 * 24)), block((1 + ng) * kThreads);
    const bool out16 = a[1].out_dtype == LASAD_BF16;
    if (a[0].fused_act && (!tied || !a[0].q_lo || !a[1].v_lo || !a[2].v_lo)) return hipErrorInvalidValue;
#define LASAD_LAUNCH1(O, T, F) do { \
        if (ng == 2) hipLaunchKernelGGL((backward_gated_passes_kernel<O, T, F, 2>), grid, block, 0, s, ps); \
        else hipLaunchKernelGGL((backward_gated_passes_kernel<O, T, F, 1>), grid, block, 0, s, ps); } while (0)
#define LASAD_LAUNCH(T, F) do { if (out16) LASAD_LAUNCH1(1, T, F); else LASAD_LAUNCH1(0, T, F); } while (0)
    if (a[0].fused_act) LASAD_LAUNCH(1, 1);
    else if (tied) LASAD_LAUNCH(1, 0);
    else LASAD_LAUNCH(0, 0);
#undef LASAD_LAUNCH
#undef LASAD_LAUNCH1
    return hipGetLastError();
}

}  // namespace lasad
