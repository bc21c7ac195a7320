// Chunked matrix-core kernels of the vector-decay backward (bf16 inputs, head dim 64), on the building blocks of the
// forward (lasad_gated_chunk.h: chunks of 32 tokens, loader wavefronts one chunk ahead, compute wavefronts that own 16
// columns of the state).  lasad_backward_gated.hip has the derivation.  Two walks, one launch each:
//
// Forward order (dq): with A_i the chunk-local running product of the decays and K~_j = k_j / A_j,
//       dq_i = q_scale A_i (.) [ S g_i + sum_{j<=i} (g_i . v_j) K~_j ],   S <- diag(A_end) (S + K~^T V).
//   A compute wavefront owns 16 KEY channels c: its accumulators hold S^T, a tile's rows being value channels e and its
//   columns c, so that S g contracts over the rows, the row scaling by A_end is one factor per lane, and g and v enter as
//   the plain bf16 tensors they are (one MFMA per score step instead of three).  dq goes to the workspace in fp32.
//
// Reversed order (dv, dk, and with the first walk's dq the decay gradient): A the running product in walking order, the
//   decay of a step that of the token walked before it, Q~_i = q_i / A_i, K^_j = k_j A_j:
//       dv_j = q_scale ( K^_j^T G + sum_{i walked before or at j} (K^_j . Q~_i) g_i ),
//       dk_j = q_scale A_j (.) [ G v_j + sum_i (v_j . g_i) Q~_i ],                  G <- diag(A_end) (G + Q~^T g).
//   Four compute wavefronts take dv (16 value channels of G each), four dk (16 key channels of G^T each), from one set of
//   prepared operands.  The running sum of r = q dq - k dk in walking order IS the suffix sum that the decay gradient
//   needs, so four finishing wavefronts end a chunk as soon as its dk tile is there: dq, dk and dlam leave in the caller's type.
//
// Against three independent passes and a finishing kernel, which read q, the decay, d_o up to four times and dk back from the
// workspace (us a call, graph replay, own key): 256 sequences of 256 tokens 56 -> 39, 512 of 24 x 24 234 -> 167, 96 of 64 x 64 in
// segments 410 -> 287; fused layer 384 of 256 131 -> 109.  Bound: dq by what it moves (96 of 64 x 64, behind a forward: 306 MB in 85
// us); the reversed walk by the longest wavefront of a period (2600 vector instructions a chunk in 5200 cycles of four SIMDs; 556 MB
// in 176 us).  Its address unit is as busy as its vector units, which is why rows are read and written as whole lines wherever LDS can
// turn them: finished rows stored straight from the lanes that make them took 400 us in the place of 314 (uncut).
//
// A chunk that leaves the range of the factorisation sends the sequence (segment) to the token-serial walks of the same passes
// (lasad_scan.h with operand roles).  The dq walk only says so and ends; the reversed kernel's workgroup then has a compute unit
// and sixteen wavefronts for all three, side by side, and the finishing step.  us a call whose gates all leave the range (own
// key), one after the other -> side by side: 96 x 256 tokens 288 -> 139, 96 x 1024 in segments 591 -> 284, 240 x 1024 1187 -> 528,
// 512 x 576 1206 -> 624.  (Three passes with a compute unit or half of one each: 119, 433, 764, 756.)
#include "lasad_gated_chunk.h"
#include "lasad_gated_finish.h"
#include "lasad_gated_backward.h"
#include "lasad_gated_state.h"
#include "lasad_scan.h"

namespace lasad {

namespace {

using namespace gchunk;

constexpr int kThreads = 256;                  // of one role: compute, loaders
constexpr int64_t kMaxStride = (1 << 25) - 1;  // 32 rows of it, four bytes an element, stay below 2^32

__device__ __forceinline__ const float *state_of(const float *states, int bh) { return states ? states + (int64_t)bh * D * D : nullptr; }

// Token-serial walk `w` (0 dq, 1 dv, 2 dk) of walking steps m0 .. m0 + n - 1 of sequence bh, from the state s_in (64 x 64, or NULL),
// by four wavefronts of the workgroup.
// Out of line, and handed the arguments where the launch put them (the kernel-argument segment): references to the
// kernel's by-value parameter, or copies, would make every thread of every launch write them to its stack first.
template <int OUT_BF16, int COL>
__device__ __noinline__ void redo_walk(const GatedChunkArgs *p, int w, int bh, int m0, int n, const float *s_in, float *s_out, LdsFloat *lds)
{
    ForwardArgs a = p->serial[w];
    scan::ScanRoles r = p->roles[w];
    for (int i = 0; i < 4; ++i) {
        if (r.ptr[i]) r.ptr[i] = (const uint16_t *)r.ptr[i] + m0 * a.in.stride_n;
        if (r.lo[i]) r.lo[i] = (const uint16_t *)r.lo[i] + m0 * a.in.stride_n;
    }
    a.o = (!COL && OUT_BF16) ? (void *)((uint16_t *)a.o + m0 * a.out.stride_n) : (void *)((float *)a.o + m0 * a.out.stride_n);
    a.start_pos += m0;
    a.n_tokens = n;
    a.state_in = s_in ? s_in - (int64_t)bh * D * D : nullptr;
    a.state_out = s_out;
    if (COL) scan::scan_sequence<1, 0, scan::ROLES_COL, 64, 1>(a, bh, 0, (float *)lds, &r);
    else scan::scan_sequence<1, OUT_BF16, scan::ROLES_ROW, 64, 1>(a, bh, 0, (float *)lds, &r);
}

// ============================================ dq, forward order ============================================

// A token's row of a chunk slot (bf16 elements): K~ hi, lo, g, v, the low-order part of g.
struct DqSlot {
    static constexpr int ROW = 5 * D + 16;
    static constexpr int Zh = 0, Zl = D, X = 2 * D, Y = 3 * D, Lo = 4 * D;
    using Map = SlotMap<ROW>;
    static constexpr int kHalfs = Map::kHalfs;
    // two slots, the output tiles, the tiles of A
    static constexpr int kBytes = 2 * kHalfs * 2 + 2 * C * OS * 4 + 2 * C * OS * 4;
};

// A loader thread's share of a chunk: tokens 2 pr, 2 pr + 1 and channels pcol .. + 3 of the decay and the key, and one
// 16-byte piece of a row of g, v and the low-order part of g.  Uniform bases, advanced chunk by chunk
// on the scalar unit, plus 32-bit byte offsets.  Rows past the end re-read the last token.
template <int OWNKEY, int LO, int NG>
struct DqStage {
    static constexpr bool TURN = NG == 1 && OWNKEY;        // decay and key: 16 bytes of one row, turned in the slot (as in the forward)
    const char *l, *z, *x, *y, *lo;
    uint32_t row;                      // bytes from token to token
    int left;                          // rows from the chunk's first one on, > 0
    struct Regs {
        uint2 rl[2], rz[2];
        u32x4 tl, tz;                  // (TURN)
        u32x4 rx, ry, rlo;
    };
    __device__ __forceinline__ void init(const GatedBackwardArgs &a, int64_t base, int n)
    {
        left = n;
        row = (uint32_t)a.in.stride_n * 2;
        l = (const char *)((const uint16_t *)a.lam + base);
        z = OWNKEY ? (const char *)((const uint16_t *)a.k + base) : nullptr;
        x = (const char *)((const uint16_t *)a.d_o + base);
        y = (const char *)((const uint16_t *)a.v + base);
        lo = LO ? (const char *)((const uint16_t *)a.d_o_lo + base) : nullptr;
    }
    __device__ __forceinline__ void fetch(Regs &f, int pr, int pcol, int st) const
    {
        const int last = min(C, left) - 1;
        const uint32_t o0 = min(2 * pr, last) * row + pcol * 2, o1 = min(2 * pr + 1, last) * row + pcol * 2;
        const uint32_t ov = min(st >> 3, last) * row + (st & 7) * 16;
        if (TURN) {
            const uint32_t o = min(Turn<DqSlot::ROW>::row(st & 63), last) * row + Turn<DqSlot::ROW>::byte(st >> 6, st & 63);
            f.tl = *(const u32x4 *)(l + o);
            if (OWNKEY) f.tz = *(const u32x4 *)(z + o);
        } else {
            f.rl[0] = *(const uint2 *)(l + o0);
            f.rl[1] = *(const uint2 *)(l + o1);
            if (OWNKEY) { f.rz[0] = *(const uint2 *)(z + o0); f.rz[1] = *(const uint2 *)(z + o1); }
        }
        f.rx = *(const u32x4 *)(x + ov);
        f.ry = *(const u32x4 *)(y + ov);
        if (LO) f.rlo = *(const u32x4 *)(lo + ov);
    }
    // on to the group's next chunk; past the end the last one is read again
    __device__ __forceinline__ void next(int64_t stride_n)
    {
        if (left <= NG * C) return;
        left -= NG * C;
        const int64_t adv = NG * C * stride_n * 2;
        l += adv; x += adv; y += adv;
        if (OWNKEY) z += adv;
        if (LO) lo += adv;
    }
};

// One workgroup per sequence or segment.  NG = 2: a second loader group, for workgroups that have a compute unit to
// themselves (a lone workgroup is bound by what its loaders issue, as in the forward).
// FUSED (tied key): the layer's backward: the decay tensor holds gate logits, and d_o comes as a bf16 pair hi + lo, both
// parts used.  d_o is orthogonal to the recurrence output, which makes dq and dk small differences of larger terms
// early in a sequence; a single bf16 there costs up to 0.15 of the RMS in single elements, and in dv, which for
// the last tokens of a sequence is a multiple of a single d_o row, up to 0.02.
template <int OWNKEY, int FUSED, int NG>
__global__ void __launch_bounds__((1 + NG) * kThreads, NG == 1 ? 4 : 3)
backward_gated_dq_kernel(GatedChunkArgs p)
{
    using SL = DqSlot;
    constexpr int LO = FUSED;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SL::kBytes];
    __shared__ __attribute__((aligned(16))) float sTot[2][D];  // A_end per key channel, by chunk parity
    __shared__ __attribute__((aligned(16))) int sTrip[2][4];   // range flag of each loader wavefront, by barrier parity
    const GatedBackwardArgs &a = p.b;
    uint16_t *const slots = (uint16_t *)smem;
    float *const outs = (float *)(slots + 2 * SL::kHalfs);
    float *const decays = outs + 2 * C * OS;               // A, laid out like an output tile
    const int bh = p.cut.n_seg == 1 ? blockIdx.x : blockIdx.x / p.cut.n_seg, seg = blockIdx.x - bh * p.cut.n_seg;
    const int b = bh / a.Hh, h = bh - b * a.Hh;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int t0 = p.cut.start(seg);
    const bool last_seg = seg == p.cut.n_seg - 1;
    const int n = (last_seg ? a.n_tokens : p.cut.start(seg + 1)) - t0;
    // (one loader group: the walk goes two chunks at a time; the second may be empty)
    const int n_chunks = NG == 1 ? (n + 2 * C - 1) / (2 * C) * 2 : (n + C - 1) / C;
    SplitConst sc;
    sc.init();

    if (wave >= 4) {
        // ===================================== loader wavefronts =====================================
        const int grp = NG == 2 ? (wave >> 2) - 1 : 0, lw = wave & 3, st = tid & 255;
        const int first = grp * C < n ? grp * C : 0;           // (a group without a chunk reads the first one, for nobody)
        const int pr = lane & 15, pcol = 16 * lw + 4 * (lane >> 4);
        using Stage = DqStage<OWNKEY, LO, NG>;
        const Turn<SL::ROW> turn(lw, lane);
        Stage sg;
        sg.init(a, (int64_t)b * a.in.stride_b + (int64_t)h * a.in.stride_h + (t0 + first) * a.in.stride_n, n - first);
        typename Stage::Regs r0, r1;               // (one loader group: two chunks of loads in flight)
        sg.fetch(r0, pr, pcol, st);                // ahead of everything that does not need it
        if (NG == 1) {
            sg.next(a.in.stride_n);
            sg.fetch(r1, pr, pcol, st);
        }
        __builtin_amdgcn_sched_barrier(0);
        RowBoundaries bounds;
        bounds.init(a.start_pos + t0 + grp * C, a.grid_w, a.mode, NG * C);
        int left = n - grp * C;                    // rows from the next chunk to be prepared on
        const int put = SL::Map::at(2 * pr, pcol), put_piece = SL::Map::at(st >> 3, (st & 7) * 8);
        const int orow = st >> 3, ocol = (st & 7) * 8;
        const int64_t w_stride = (int64_t)a.Hh * D;
        float *o_chunk = p.dq32 + ((int64_t)b * a.n_tokens + t0 + (NG == 2 && grp == 0 ? C : 0)) * w_stride + h * D;
        const int64_t o_lane = orow * w_stride + ocol;
        auto store_tile = [&](int chunk) {
            const float *tile = outs + (chunk & 1) * C * OS + orow * OS + ocol;
            float4 u = *(const float4 *)tile, w = *(const float4 *)(tile + 4);
            if (chunk * C + orow < n) {            // (read again by the reversed walk)
                gstore16<false>(o_chunk + o_lane, u.x * a.q_scale, u.y * a.q_scale, u.z * a.q_scale, u.w * a.q_scale);
                gstore16<false>(o_chunk + o_lane + 4, w.x * a.q_scale, w.y * a.q_scale, w.z * a.q_scale, w.w * a.q_scale);
            }
            o_chunk += NG * C * w_stride;          // (of two groups, each stores every other tile)
        };

        // between the phases of a chunk's preparation
        u32x4 px, py, plo;
        bool row_live;
        float z[2][4], x[2][4], tot[4], exc[4];

        // the plain rows into slot q (a row that is no token is a query that nobody stores, and zero as v)
        auto put_rows = [&](int q) {
            uint16_t *const piece = slots + q * SL::kHalfs + put_piece;
            *(u32x4 *)&piece[SL::X] = px;
            *(u32x4 *)&piece[SL::Y] = row_live ? py : u32x4{0u, 0u, 0u, 0u};
            if (LO) *(u32x4 *)&piece[SL::Lo] = row_live ? plo : u32x4{0u, 0u, 0u, 0u};
        };
        // Phase A: everything that needs no slot; done: the finished chunk to be stored meanwhile, or -1.  One loader group
        // runs both phases in one period and puts the plain rows into slot q at once.  (Past the end the last chunk's data go
        // once more into a slot that nobody reads.)
        auto phase_a = [&](typename Stage::Regs &f, int q, int done) {
            const uint32_t bmask = bounds.mask();
            bounds.advance();
            if (Stage::TURN) {
                turn.write(slots + q * SL::kHalfs, SL::Zh, f.tl);
                if (OWNKEY) turn.write(slots + q * SL::kHalfs, SL::Zl, f.tz);
            } else {
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    unpack4(f.rl[it], x[it]);
                    if (OWNKEY) unpack4(f.rz[it], z[it]);
                }
            }
            row_live = (st >> 3) < left;
            px = f.rx;
            py = f.ry;
            if (LO) plo = f.rlo;
            if (NG == 1) {
                put_rows(q);
            } else {
                asm volatile("" : "+v"(px));
                asm volatile("" : "+v"(py));
                if (LO) asm volatile("" : "+v"(plo));
            }
            // (the fetched registers are free from here on, and the compiler must see it so: lasad_forward_gated_chunk.hip)
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                if (Stage::TURN) break;
                asm volatile("" : "+v"(x[it][0]), "+v"(x[it][1]), "+v"(x[it][2]), "+v"(x[it][3]));
                if (OWNKEY) asm volatile("" : "+v"(z[it][0]), "+v"(z[it][1]), "+v"(z[it][2]), "+v"(z[it][3]));
            }
            if (done >= 0) store_tile(done);
            __builtin_amdgcn_sched_barrier(0);
            sg.next(a.in.stride_n);
            sg.fetch(f, pr, pcol, st);
            if (Stage::TURN) {
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    unpack4(turn.read(slots + q * SL::kHalfs, SL::Zh, it), x[it]);
                    if (OWNKEY) unpack4(turn.read(slots + q * SL::kHalfs, SL::Zl, it), z[it]);
                }
            }
#pragma unroll
            for (int it = 0; it < 2; ++it) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (FUSED) {                   // z = k = 1 - lambda = exp(-gate) lambda, and 1 / lambda = 1 + exp(-gate)
                        z[it][e] = exp_neg(x[it][e]);
                        x[it][e] = 1.0f + z[it][e];
                    } else if (!OWNKEY) {
                        z[it][e] = 1.0f - x[it][e];
                    }
                }
                if (bmask & (0x55555555u << it)) { // some token of this parity sits on a boundary: lambda 1
                    if ((bmask >> (2 * pr + it)) & 1u) {
                        asm volatile("");
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            // (the tied key keeps its own lambda, see the forward)
                            if (FUSED) z[it][e] = z[it][e] >= 1e30f ? 1.0f : z[it][e] * __builtin_amdgcn_rcpf(x[it][e]);
                            x[it][e] = 1.0f;
                        }
                    }
                }
            }
            if (left < C) {                        // rows that are no tokens get lambda 1, z = 0
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const bool live = 2 * pr + it < left;
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
        // Phase B: the chunk into slot q, and its range flag for the barrier that ends this period.
        auto phase_b = [&](int q) {
            if (NG == 2) put_rows(q);
            bool trip;
            if (FUSED) trip = !(fmaxf(fmaxf(tot[0], tot[1]), fmaxf(tot[2], tot[3])) <= kMaxInvDecay);
            else trip = !(fminf(fminf(tot[0], tot[1]), fminf(tot[2], tot[3])) >= 1.0f / kMaxInvDecay);
            if (pr == 15)
                *(float4 *)&sTot[q][pcol] = FUSED ? make_float4(__builtin_amdgcn_rcpf(tot[0]), __builtin_amdgcn_rcpf(tot[1]),
                                                                __builtin_amdgcn_rcpf(tot[2]), __builtin_amdgcn_rcpf(tot[3]))
                                                  : make_float4(tot[0], tot[1], tot[2], tot[3]);
            const bool any = __any(trip);
            if (lane == 0) sTrip[q][lw] = any ? 1 : 0;
            uint16_t *rows = slots + q * SL::kHalfs + put;
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                float zt[4], dec[4];               // K~ and A of this token
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float before = it ? exc[e] * x[0][e] : exc[e];
                    const float after = it ? tot[e] : exc[e] * x[0][e];
                    const float inv = __builtin_amdgcn_rcpf(after);
                    zt[e] = FUSED ? z[it][e] * before : z[it][e] * inv;
                    dec[e] = FUSED ? inv : after;
                }
                put_pair4(rows + it * SL::ROW + SL::Zh, rows + it * SL::ROW + SL::Zl, zt, sc);
                *(float4 *)&decays[q * C * OS + (2 * pr + it) * OS + pcol] = make_float4(dec[0], dec[1], dec[2], dec[3]);
            }
        };
        bool fine = true;
        if constexpr (NG == 1) {
            // Two chunks of loads in flight, in two sets of registers.  (A pair of chunks is always done as a whole, range
            // flags tested at its end: with a way out between its halves the compiler waits for both sets at the loop's top.)
            auto prepare = [&](typename Stage::Regs &f, int q, int done) {
                phase_a(f, q, done);
                phase_b(q);
            };
            prepare(r0, 0, -1);
            __syncthreads();
            for (int chunk = 0; fine && chunk < n_chunks; chunk += 2) {
                const int4 f0 = *(const int4 *)sTrip[0];
                prepare(r1, 1, chunk - 1);
                __syncthreads();
                const int4 f1 = *(const int4 *)sTrip[1];
                prepare(r0, 0, chunk);
                fine = (f0.x | f0.y | f0.z | f0.w | f1.x | f1.y | f1.z | f1.w) == 0;
                __syncthreads();
            }
        } else {
            // the groups take the chunks in turn, a period for each phase
            int4 f;                                // a chunk's range flags, read at the start of its period and tested at the end
            auto end_period = [&]() {
                fine = (f.x | f.y | f.z | f.w) == 0;
                __syncthreads();
            };
            phase_a(r0, 0, -1);
            if (grp == 0) phase_b(0);
            __syncthreads();
            if (grp == 1) {                        // period 0
                f = *(const int4 *)sTrip[0];
                phase_b(1);
                end_period();
            }
            for (int chunk = grp; fine && chunk < n_chunks; chunk += 2) {
                f = *(const int4 *)sTrip[chunk & 1];
                phase_a(r0, 0, chunk - 1);
                end_period();
                if (!fine || chunk + 1 == n_chunks) break;
                f = *(const int4 *)sTrip[(chunk + 1) & 1];
                phase_b(chunk & 1);
                end_period();
            }
        }
        if (fine && (NG == 1 || grp == (n_chunks & 1))) store_tile(n_chunks - 1);
        return;
    }

    // ===================================== compute wavefronts =====================================
    __builtin_amdgcn_s_setprio(2);                 // the chain from chunk to chunk; the loaders fill the gaps
    const int l16 = lane & 15, g = lane >> 4;
    const int col0 = 16 * wave;                    // key channels of this wavefront
    f32x4v accS[4];                                // S^T: element (t, r) is S[col0 + l16][state_channel(t, g) + r]
    const f32x4v zero4 = {0.f, 0.f, 0.f, 0.f};
    const int s_lane = (col0 + l16) * D;
#pragma unroll
    for (int t = 0; t < 4; ++t) accS[t] = zero4;
    if (const float *s_in = seg ? p.bound_s(bh, seg - 1) : state_of(a.state_in, bh)) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) accS[t][r] = s_in[s_lane + state_channel(t, g) + r];
    }
    // the states at the bounds of the parts
    const int real_chunks = (n + C - 1) / C;
    int part = 1, part_at = p.n_part > 1 ? real_chunks / p.n_part : 0;

    __syncthreads();
    bool fine = true;
    for (int chunk = 0; (fine || (NG == 1 && (chunk & 1))) && chunk < n_chunks; ++chunk) {
        const int4 f = *(const int4 *)sTrip[chunk & 1];
        const SlotPtr<SL::ROW> sp(slots + (chunk & 1) * SL::kHalfs, lane);
        f32x4v p00 = zero4, p01 = zero4, p11 = zero4;              // scores P^T[j][i]: (key tile, query tile)
        f32x4v o0 = zero4, o1 = zero4;                             // O^T[.][i] of the two query tiles
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const Frag x0 = sp.rows(0, SL::X, s), x1 = sp.rows(16, SL::X, s);
            const Frag y0 = sp.rows(0, SL::Y, s), y1 = sp.rows(16, SL::Y, s);
            Frag l0, l1;
            if (LO) { l0 = sp.rows(0, SL::Lo, s); l1 = sp.rows(16, SL::Lo, s); }
            Frag sh, sl;
            split_tiles(accS[2 * s], accS[2 * s + 1], sh, sl, sc);
            // ---- P^T[j][i] += sum_e V[j][e] g[i][e],  O^T[c][i] += sum_e S[c][e] g[i][e] ----
            p00 = mfma16(y0, x0, p00);
            p01 = mfma16(y0, x1, p01);
            p11 = mfma16(y1, x1, p11);
            o0 = mfma16(sh, x0, o0);
            o1 = mfma16(sh, x1, o1);
            if (LO) {
                p00 = mfma16(y0, l0, p00);
                p01 = mfma16(y0, l1, p01);
                p11 = mfma16(y1, l1, p11);
            }
            o0 = mfma16(sl, x0, o0);
            o1 = mfma16(sl, x1, o1);
            if (LO) {
                o0 = mfma16(sh, l0, o0);
                o1 = mfma16(sh, l1, o1);
            }
        }
        causal_mask(p00, lane);
        causal_mask(p11, lane);
        Frag ph, pl;
        const Frag zh = sp.tokens(SL::Zh + col0), zl = sp.tokens(SL::Zl + col0);
        // ---- S^T[e][c] += sum_j V[j][e] K~[j][c], O^T[c][i] += sum_j K~[j][c] P^T[j][i] ----
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const Frag fy = sp.state_rows(SL::Y, t);
            accS[t] = mfma16(fy, zh, accS[t]);
            accS[t] = mfma16(fy, zl, accS[t]);
        }
        split_tiles(p00, zero4, ph, pl, sc);                       // (keys 16 .. 31 come after queries 0 .. 15)
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
        if (chunk + 1 == part_at) {
            float *s = p.part_s(bh, seg, part - 1) + s_lane;
#pragma unroll
            for (int t = 0; t < 4; ++t) *(f32x4v *)(s + state_channel(t, g)) = accS[t];
            ++part;
            part_at = part < p.n_part ? part * real_chunks / p.n_part : 0;
        }
        // O^T row 4 g + r is key channel col0 + 4 g + r of token l16 / 16 + l16: times its A
        float *tile = outs + (chunk & 1) * C * OS + l16 * OS + col0 + 4 * g;
        const float *dec = decays + (chunk & 1) * C * OS + l16 * OS + col0 + 4 * g;
        const float4 d0 = *(const float4 *)dec, d1 = *(const float4 *)(dec + 16 * OS);
        *(float4 *)tile = make_float4(o0[0] * d0.x, o0[1] * d0.y, o0[2] * d0.z, o0[3] * d0.w);
        *(float4 *)(tile + 16 * OS) = make_float4(o1[0] * d1.x, o1[1] * d1.y, o1[2] * d1.z, o1[3] * d1.w);
        fine = fine && (f.x | f.y | f.z | f.w) == 0;
        __syncthreads();
    }
    if (tid == 0) p.kept[bh * p.cut.n_seg + seg] = fine;
    if (!fine) return;
    if (p.s_out && last_seg) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) p.s_out[(int64_t)bh * D * D + s_lane + state_channel(t, g) + r] = accS[t][r];
    }
}

// ============================================ dv, dk, dlam, reversed order ============================================

// A token's row of a chunk slot (bf16 elements): Q~ hi, lo, K^ hi, lo, v, g, the low-order part of g.
template <int OUT_BF16, int OWNKEY, int LO>
struct RevSlot {
    static constexpr int ROW = (LO ? 7 : 6) * D + 16;
    static constexpr int Zh = 0, Zl = D, Qh = 2 * D, Ql = 3 * D, X = 4 * D, Y = 5 * D, Lo = 6 * D;
    using Map = SlotMap<ROW>;
    static constexpr int kHalfs = Map::kHalfs;
    // What a loader thread hands to the same thread of the finishing wavefronts, in 16-byte pieces: A of its two rows; where
    // there is room (bf16 gradients) also q as read, lambda (FUSED: of the two rows; else as read) and the key as read.  (Read
    // from memory once more they took 55 of 350 us, 96 sequences of 4096 tokens.)
    static constexpr bool kHand = OUT_BF16;
    static constexpr int kHands = !kHand ? 2 : LO || OWNKEY ? 5 : 4, kHandFloats = 4 * kThreads;
    // a finished chunk's rows of dq, dlam, dk on their way out
    static constexpr int G = OUT_BF16 ? D : 2 * D, OUT_ROW = (OWNKEY ? 3 : 2) * G + 16;
    using OutMap = SlotMap<OUT_ROW>;
    // two each of slots, output tiles (dv, dk), the loaders' values, finished rows
    static constexpr int kBytes = 2 * (kHalfs * 2 + 2 * C * OS * 4 + kHands * kHandFloats * 4 + OutMap::kHalfs * 2);
};

// A loader or finishing thread's share of a chunk.  Row m of the walk's chunk is token (its last) - m: the bases stand at the
// chunk's first token, the lowest address.  The walk starts with the chunk that the forward one ends with, so its first `lead`
// rows may be no tokens (they re-read the last one).
struct RevRows {
    int lead;                          // rows of the chunk before the walk's first token
    int left;                          // chunks from this one on
    __device__ __forceinline__ int m(int i) const { return max(i, lead); }
    __device__ __forceinline__ bool next()     // to the next chunk; past the end the last one is read again
    {
        if (left == 1) return false;
        --left;
        lead = 0;
        return true;
    }
};

template <int CTRL>
__device__ __forceinline__ float dpp_shr(float x)          // 0 where there is no source
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float dpp_ror1(float x)         // rows of 16 lanes, turned by one
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x121, 0xf, 0xf, true));
}
__device__ __forceinline__ float dpp_last(float x)         // of the row's lane 15
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x15F, 0xf, 0xf, true));
}
// running sums of four values along the 16 lanes of a row (inclusive)
__device__ __forceinline__ void row_scan_add4(float (&x)[4])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] += dpp_shr<0x111>(x[e]);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] += dpp_shr<0x112>(x[e]);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] += dpp_shr<0x114>(x[e]);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] += dpp_shr<0x118>(x[e]);
}

// x / lambda to within 2^-24 of it and a last bit's rounding, for lambda from 2^-100 on (less sends the sequence to the token-serial
// walks): one step on the hardware's reciprocal, which alone is off by a bit.  Infinities and NaN stay what they are.  (The
// compiler's division, ten instructions: the call 2 to 4 % slower.)
__device__ __forceinline__ float quotient(float x, float lambda)
{
    const float r = __builtin_amdgcn_rcpf(lambda), q = x * r, t = fmaf(fmaf(-q, lambda, x), r, q);
    return t == t ? t : q;
}

// four values of a token's row, in the gradients' type
template <int OUT_BF16>
__device__ __forceinline__ void put_grad4(uint16_t *p, float a, float b, float c, float d)
{
    if (OUT_BF16) *(uint2 *)p = make_uint2(pack2(a, b), pack2(c, d));
    else *(float4 *)p = make_float4(a, b, c, d);
}

// The token-serial walks of a segment, by four wavefronts each, and the finishing step on what they leave, by all of them.
// dq only where its own walk did not hold: else it is there, and so is the sink.
constexpr int kRedoFloats = scan::lds_floats<scan::ROLES_ROW, 1>();
template <int OUT_BF16>
__device__ __noinline__ void redo_reversed(const GatedChunkArgs *p, int bh, int seg, LdsFloat *lds)
{
    const int t_lo = p->cut.start(seg);
    const bool last_seg = seg == p->cut.n_seg - 1;
    const int t_hi = last_seg ? p->b.n_tokens : p->cut.start(seg + 1);
    const float *sink = p->sink_of(bh, seg);
    const float *g_in = last_seg ? state_of(p->g_in, bh) : p->bound_g(bh, seg);
    const int m0 = p->b.n_tokens - t_hi, n = t_hi - t_lo;
    const bool no_dq = !p->kept[bh * p->cut.n_seg + seg];
    const int walk = __builtin_amdgcn_readfirstlane(threadIdx.x / scan::kThreads);
    LdsFloat *const mine = lds + walk * kRedoFloats;
    if (walk == 0 && no_dq) redo_walk<0, 1>(p, 0, bh, t_lo, n, seg ? p->bound_s(bh, seg - 1) : state_of(p->b.state_in, bh), last_seg ? p->s_out : nullptr, mine);
    else if (walk == 1) redo_walk<OUT_BF16, 0>(p, 1, bh, m0, n, g_in, seg == 0 ? p->g_out : nullptr, mine);
    else if (walk == 2) redo_walk<OUT_BF16, 1>(p, 2, bh, m0, n, g_in, nullptr, mine);
    else scan::barriers_only<1>(n);
    __syncthreads();                               // (dq32, dk32 and s_out of this sequence are this workgroup's own)
    const int c = threadIdx.x;
    float carry = 0.f;
    if (sink && c < D) {
        if (last_seg && no_dq) {                   // sum_n H[c][n] S_n[c][n], as gated_carried_finish_kernel adds it up
            float part[4] = {0.f, 0.f, 0.f, 0.f};
            const int64_t row = (int64_t)bh * D * D + c * D;
            for (int i = 0; i < D; ++i) part[i >> 4] = fmaf(p->b.d_state_out[row + i], p->s_out[row + i], part[i >> 4]);
            carry = (part[0] + part[1]) + (part[2] + part[3]);
        } else {
            carry = sink[c];
        }
    }
    const FinishWalk<1, OUT_BF16, D> f(p->b, p->dq32, p->dk32, bh, 0);
    f.walk(t_lo, t_hi, carry, (float *)lds);
}

// (The redo is called in one place, which all roles come to: three calls took 0.7 us of every launch, 81 sequences of 64 tokens.)
// One workgroup per sequence or segment, one barrier per chunk: in the period of chunk c four compute wavefronts take its dv
// and four its dk, four loaders prepare chunk c + 1, and four finishing wavefronts turn chunk c - 1 into dq, dk, dlam and dv.
template <int OUT_BF16, int OWNKEY, int FUSED>
__global__ void __launch_bounds__(4 * kThreads)
backward_gated_reversed_kernel(GatedChunkArgs p)
{
    constexpr int LO = FUSED;
    using SL = RevSlot<OUT_BF16, OWNKEY, LO>;
    constexpr int kRedoBytes = 3 * kRedoFloats * 4;
    static_assert(kRedoBytes >= finish_lds_floats<D>() * 4, "the finishing step needs the LDS block");
    __shared__ __attribute__((aligned(16))) unsigned char smem[SL::kBytes > kRedoBytes ? SL::kBytes : kRedoBytes];
    __shared__ __attribute__((aligned(16))) float sTot[2][D];      // A_end per key channel, by chunk parity
    __shared__ __attribute__((aligned(16))) float sSync[D];        // <G, S> at a part's bound
    __shared__ __attribute__((aligned(16))) int sTrip[2][4];       // range flag of each loader wavefront, by barrier parity
    const GatedBackwardArgs &a = p.b;
    uint16_t *const slots = (uint16_t *)smem;
    float *const outs = (float *)(slots + 2 * SL::kHalfs);         // [dv, dk][parity]
    float *const hands = outs + 4 * C * OS;                        // [parity][A, lambda]
    uint16_t *const done = (uint16_t *)(hands + 2 * SL::kHands * SL::kHandFloats);     // [parity]
    const int bh = p.cut.n_seg == 1 ? blockIdx.x : blockIdx.x / p.cut.n_seg, seg = blockIdx.x - bh * p.cut.n_seg;
    const int b = bh / a.Hh, h = bh - b * a.Hh;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int t_lo = p.cut.start(seg);
    const bool last_seg = seg == p.cut.n_seg - 1;
    const int t_hi = last_seg ? a.n_tokens : p.cut.start(seg + 1);
    const int pad = (C - 1) - (t_hi - t_lo - 1) % C;       // rows before the walk's first token
    const int n_chunks = (t_hi - t_lo + pad) / C;
    SplitConst sc;
    sc.init();
    const int lost = !p.kept[bh * p.cut.n_seg + seg];      // (tested with the first chunk's flags)
    bool fine = true;
    // the next bound between parts, from the segment's end on, and the chunks walked when it is reached
    int part = p.n_part - 1;
    auto part_chunks = [&]() { return part > 0 ? n_chunks - part * n_chunks / p.n_part : 0; };
    int part_at = part_chunks();

    // loaders and finishing wavefronts: this thread's rows 2 pr, 2 pr + 1, channels pcol .. + 3
    const int st = tid & 255;
    const int pr = lane & 15, pcol = 16 * (wave & 3) + 4 * (lane >> 4);
    const int64_t in_base = (int64_t)b * a.in.stride_b + (int64_t)h * a.in.stride_h + (t_hi + pad - C) * a.in.stride_n;
    const uint32_t row = (uint32_t)a.in.stride_n * 2;
    const int64_t adv = C * a.in.stride_n;

    if (wave >= 8 && wave < 12) {
        // ===================================== loader wavefronts =====================================
        const uint16_t *l = (const uint16_t *)a.lam + in_base, *z = (const uint16_t *)a.q + in_base;
        const uint16_t *k = OWNKEY ? (const uint16_t *)a.k + in_base : nullptr;
        const uint16_t *x_ = (const uint16_t *)a.v + in_base, *y = (const uint16_t *)a.d_o + in_base;
        const uint16_t *lo = LO ? (const uint16_t *)a.d_o_lo + in_base : nullptr;
        RevRows rows{pad, n_chunks};
        const int lw = wave & 3;
        u32x4 rl, rz, rk, rx, ry, rlo;
        auto fetch = [&]() {
            const uint32_t o = (C - 1 - rows.m(Turn<SL::ROW>::row(lane))) * row + Turn<SL::ROW>::byte(lw, lane);
            const uint32_t ov = (C - 1 - rows.m(st >> 3)) * row + (st & 7) * 16;
            rl = *(const u32x4 *)((const char *)l + o);
            rz = *(const u32x4 *)((const char *)z + o);
            if (OWNKEY) rk = *(const u32x4 *)((const char *)k + o);
            rx = *(const u32x4 *)((const char *)x_ + ov);
            ry = *(const u32x4 *)((const char *)y + ov);
            if (LO) rlo = *(const u32x4 *)((const char *)lo + ov);
        };
        fetch();                                   // ahead of everything that does not need it
        __builtin_amdgcn_sched_barrier(0);
        // the decay of a step is that of the token walked before it
        RowBoundaries bounds;
        {
            // (lasad_internal.h, reversed_start, of a walk from token t_hi - 1)
            const int W = a.grid_w, s = (a.start_pos % W + t_hi % W + (a.mode == LASAD_RESET_LAST_COL ? 2 : 0)) % W;
            int col = (s ? W - s : 0) - pad % W;
            if (col < 0) col += W;
            bounds.init(col, W, a.mode, C);
        }
        const Turn<SL::ROW> turn(lw, lane);
        const int put = turn.get, put_piece = SL::Map::at(st >> 3, (st & 7) * 8);
        float before[4] = {1.f, 1.f, 1.f, 1.f};    // (FUSED: the reciprocal of) lambda of the chunk before's rows 2 pr + 1
        // a chunk into slot q, and its range flag for the barrier that ends this period
        auto prepare = [&](int q, int lead) {
            uint32_t bmask = bounds.mask();
            bounds.advance();
            float x[2][4], own[2][4], qz[2][4], key[2][4];
            uint16_t *const slot = slots + q * SL::kHalfs;
            // (turned where the operands that come of them will be)
            turn.write(slot, SL::Zh, rl);
            turn.write(slot, SL::Zl, rz);
            if (OWNKEY) turn.write(slot, SL::Qh, rk);
            {
                const bool row_live = (st >> 3) >= lead;       // (a row that is no token is a query that nobody stores, and zero as y)
                uint16_t *const piece = slot + put_piece;
                *(u32x4 *)&piece[SL::X] = rx;
                *(u32x4 *)&piece[SL::Y] = row_live ? ry : u32x4{0u, 0u, 0u, 0u};
                if (LO) *(u32x4 *)&piece[SL::Lo] = row_live ? rlo : u32x4{0u, 0u, 0u, 0u};
            }
            // (the fetched registers are free from here on)
            __builtin_amdgcn_sched_barrier(0);
            if (rows.next()) {
                l -= adv; z -= adv; x_ -= adv; y -= adv;
                if (OWNKEY) k -= adv;
                if (LO) lo -= adv;
            }
            fetch();
            float *const h0 = hands + q * SL::kHands * SL::kHandFloats + st * 4;
            {
                uint2 wl[2], wz[2], wk[2];
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    wl[it] = turn.read(slot, SL::Zh, it);
                    wz[it] = turn.read(slot, SL::Zl, it);
                    if (OWNKEY) wk[it] = turn.read(slot, SL::Qh, it);
                    unpack4(wl[it], own[it]);
                    unpack4(wz[it], qz[it]);
                    if (OWNKEY) unpack4(wk[it], key[it]);
                }
                if (SL::kHand) {
                    *(uint4 *)(h0 + 2 * SL::kHandFloats) = make_uint4(wz[0].x, wz[0].y, wz[1].x, wz[1].y);
                    if (!FUSED) *(uint4 *)(h0 + 3 * SL::kHandFloats) = make_uint4(wl[0].x, wl[0].y, wl[1].x, wl[1].y);
                    if (OWNKEY) *(uint4 *)(h0 + 4 * SL::kHandFloats) = make_uint4(wk[0].x, wk[0].y, wk[1].x, wk[1].y);
                }
            }
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                float lam[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (FUSED) {
                        // 1 / lambda = 1 + exp(-gate), and the key 1 - lambda = exp(-gate) lambda (exp(-gate) up to infinity: 1; NaN stays)
                        const float ez = exp_neg(own[it][e]);
                        own[it][e] = 1.0f + ez;
                        lam[e] = __builtin_amdgcn_rcpf(own[it][e]);
                        key[it][e] = ez >= 1e30f ? 1.0f : ez * lam[e];
                        qz[it][e] *= __builtin_amdgcn_rcpf(1.0f + exp_neg(qz[it][e]));
                    } else if (!OWNKEY) {
                        key[it][e] = 1.0f - own[it][e];
                    }
                }
                if (SL::kHand && FUSED) *(float4 *)(h0 + (3 + it) * SL::kHandFloats) = make_float4(lam[0], lam[1], lam[2], lam[3]);
            }
            // the decay of row 2 pr is that of row 2 pr - 1, of the lane before; lane 0's of the chunk before
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float of = pr == 15 ? before[e] : own[1][e];
                before[e] = own[1][e];
                x[0][e] = dpp_ror1(of);
                x[1][e] = own[0][e];
            }
            if (lead >= 0) bmask |= 2u * (1u << lead) - 1u;    // the walk's start: rows that are no tokens, and its first step, have lambda 1
            if (bmask) {                           // and so have rows at a row boundary
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const bool one = (bmask >> (2 * pr + it)) & 1u;
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[it][e] = one ? 1.0f : x[it][e];
                }
            }
            float tot[4], exc[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) tot[e] = x[0][e] * x[1][e];
            row_scan_mul4(tot, exc);               // (FUSED: of the reciprocals throughout)
            bool trip;
            if (FUSED) trip = !(fmaxf(fmaxf(tot[0], tot[1]), fmaxf(tot[2], tot[3])) <= kMaxInvDecay);
            else trip = !(fminf(fminf(tot[0], tot[1]), fminf(tot[2], tot[3])) >= 1.0f / kMaxInvDecay);
            if (pr == 15)
                *(float4 *)&sTot[q][pcol] = FUSED ? make_float4(__builtin_amdgcn_rcpf(tot[0]), __builtin_amdgcn_rcpf(tot[1]),
                                                                __builtin_amdgcn_rcpf(tot[2]), __builtin_amdgcn_rcpf(tot[3]))
                                                  : make_float4(tot[0], tot[1], tot[2], tot[3]);
            const bool any = __any(trip);
            if (lane == 0) sTrip[q][wave & 3] = any ? 1 : 0;
            uint16_t *const dst = slot + put;
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                float zt[4], kt[4], A[4];
                const bool dead = lead > 0 && 2 * pr + it < lead;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float after = it ? tot[e] : exc[e] * x[0][e];
                    const float inv = __builtin_amdgcn_rcpf(after);
                    A[e] = FUSED ? inv : after;
                    zt[e] = dead ? 0.f : qz[it][e] * (FUSED ? after : inv);
                    kt[e] = key[it][e] * A[e];
                }
                put_pair4(dst + it * SL::ROW + SL::Zh, dst + it * SL::ROW + SL::Zl, zt, sc);
                put_pair4(dst + it * SL::ROW + SL::Qh, dst + it * SL::ROW + SL::Ql, kt, sc);
                *(float4 *)(h0 + it * SL::kHandFloats) = make_float4(A[0], A[1], A[2], A[3]);
            }
        };
        prepare(0, pad);
        __syncthreads();
        for (int chunk = 0; fine && chunk < n_chunks; ++chunk) {
            const int4 f = *(const int4 *)sTrip[chunk & 1];
            prepare((chunk + 1) & 1, -1);          // (past the end the last one goes once more into a slot that nobody reads)
            fine = (f.x | f.y | f.z | f.w | lost) == 0;
            __syncthreads();
        }
    } else if (wave >= 12) {
        // ===================================== finishing wavefronts =====================================
        const uint16_t *l = (const uint16_t *)a.lam + in_base, *z = (const uint16_t *)a.q + in_base;
        const uint16_t *k = OWNKEY ? (const uint16_t *)a.k + in_base : nullptr;
        const int64_t w_stride = (int64_t)a.Hh * D;
        const float *dq32 = p.dq32 + ((int64_t)b * a.n_tokens + (t_hi + pad - C)) * w_stride + h * D;
        RevRows rows{pad, n_chunks};
        uint2 rl[2], rz[2], rk[2];                 // (with kHand: from the loaders)
        float4 rdq[2];
        auto fetch = [&]() {
            const uint32_t m0 = C - 1 - rows.m(2 * pr), m1 = C - 1 - rows.m(2 * pr + 1);
            const uint32_t o0 = m0 * row + pcol * 2, o1 = m1 * row + pcol * 2;
            const uint32_t w0 = m0 * (uint32_t)w_stride * 4 + pcol * 4, w1 = m1 * (uint32_t)w_stride * 4 + pcol * 4;
            if (!SL::kHand) {
                rl[0] = *(const uint2 *)((const char *)l + o0);
                rl[1] = *(const uint2 *)((const char *)l + o1);
                rz[0] = *(const uint2 *)((const char *)z + o0);
                rz[1] = *(const uint2 *)((const char *)z + o1);
                if (OWNKEY) { rk[0] = *(const uint2 *)((const char *)k + o0); rk[1] = *(const uint2 *)((const char *)k + o1); }
            }
            rdq[0] = *(const float4 *)((const char *)dq32 + w0);
            rdq[1] = *(const float4 *)((const char *)dq32 + w1);
        };
        fetch();
        // a token whose decay is not applied: at a row boundary; from a zero state the first one's multiplies nothing
        RowBoundaries bounds;
        {
            // (as above, without the shift of one step)
            const int W = a.grid_w, s = (a.start_pos % W + t_hi % W + (a.mode == LASAD_RESET_LAST_COL ? 1 : W - 1)) % W;
            int col = (s ? W - s : 0) - pad % W;
            if (col < 0) col += W;
            bounds.init(col, W, a.mode, C);
        }
        float carry[4];                            // sum of r over the rows walked before
        {
            const float *sink = p.sink_of(bh, seg);
#pragma unroll
            for (int e = 0; e < 4; ++e) carry[e] = sink ? sink[pcol + e] : 0.f;
        }
        const int orow = st >> 3, ocol = (st & 7) * 8;
        int64_t at = (int64_t)b * a.grad.stride_b + (int64_t)h * a.grad.stride_h + (t_hi + pad - C) * a.grad.stride_n;     // the chunk's first token
        constexpr int E = OUT_BF16 ? 2 : 4;
        const uint32_t o_lane = (C - 1 - orow) * (uint32_t)a.grad.stride_n * E + ocol * E;
        const int put = SL::OutMap::at(2 * pr, pcol * (E / 2)), get = SL::OutMap::row(orow);
        // this thread's pieces of a chunk's rows, 128 bytes of a row by neighbouring lanes (a store instruction takes a compute
        // unit about 12 cycles a row that it touches): dq, dlam, dk as finished in the period before, and dv
        constexpr int kOut = OWNKEY ? 3 : 2, kPieces = OUT_BF16 ? 1 : 2;
        struct Leaving { u32x4 x[kOut * kPieces]; float4 v[2]; };
        auto read_done = [&](Leaving &r, int chunk) {
            const uint16_t *const src = done + (chunk & 1) * SL::OutMap::kHalfs;
#pragma unroll
            for (int i = 0; i < kOut; ++i)
#pragma unroll
                for (int j = 0; j < kPieces; ++j)
                    r.x[i * kPieces + j] = *(const u32x4 *)&src[get + SL::OutMap::piece(orow, i * (SL::G / 8) + ocol / 8 * (E / 2) + j)];
        };
        auto read_dv = [&](Leaving &r, int chunk) {
            const float *vt = outs + (chunk & 1) * C * OS + orow * OS + ocol;
            r.v[0] = *(const float4 *)vt;
            r.v[1] = *(const float4 *)(vt + 4);
        };
        auto store = [&](const Leaving &r, int chunk, int64_t first) {          // (its first token at `first`)
            if (chunk == 0 && orow < pad) return;
            char *const to[3] = {(char *)a.dq + first * E, (char *)a.dlam + first * E, OWNKEY ? (char *)a.dk + first * E : nullptr};
#pragma unroll
            for (int i = 0; i < kOut; ++i)
#pragma unroll
                for (int j = 0; j < kPieces; ++j) __builtin_nontemporal_store(r.x[i * kPieces + j], (u32x4 *)(to[i] + o_lane + 16 * j));
        };
        auto store_dv = [&](const Leaving &r, int chunk) {
            const float4 u = make_float4(r.v[0].x * a.q_scale, r.v[0].y * a.q_scale, r.v[0].z * a.q_scale, r.v[0].w * a.q_scale);
            const float4 w = make_float4(r.v[1].x * a.q_scale, r.v[1].y * a.q_scale, r.v[1].z * a.q_scale, r.v[1].w * a.q_scale);
            if (chunk == 0 && orow < pad) return;
            char *const v = (char *)a.dv + at * E + o_lane;
            if (OUT_BF16) {
                gstore16<true>(v, make_uint4(pack2(u.x, u.y), pack2(u.z, u.w), pack2(w.x, w.y), pack2(w.z, w.w)));
            } else {
                gstore16<true>((float *)v, u.x, u.y, u.z, u.w);
                gstore16<true>((float *)(v + 16), w.x, w.y, w.z, w.w);
            }
        };
        float4 A4[2], lam4[2];                     // the next chunk's, from the loaders
        auto take = [&](int chunk) {
            const float *const h0 = hands + (chunk & 1) * SL::kHands * SL::kHandFloats + st * 4;
            A4[0] = *(const float4 *)h0;
            A4[1] = *(const float4 *)(h0 + SL::kHandFloats);
            if (!SL::kHand) return;
            auto two = [&](int i, uint2 (&x)[2]) {
                const uint4 w = *(const uint4 *)(h0 + i * SL::kHandFloats);
                x[0] = make_uint2(w.x, w.y);
                x[1] = make_uint2(w.z, w.w);
            };
            two(2, rz);
            if (OWNKEY) two(4, rk);
            if (!FUSED) two(3, rl);
            else {
                lam4[0] = *(const float4 *)(h0 + 3 * SL::kHandFloats);
                lam4[1] = *(const float4 *)(h0 + 4 * SL::kHandFloats);
            }
        };
        // The rows finished in the period before leave at the start of this one, between the wait for this chunk's loads and the
        // issue of the next ones: no wait ever includes a store that is still on its way.
        auto finish = [&](int chunk) {
            const float *tile = outs + (2 + (chunk & 1)) * C * OS + 2 * pr * OS + pcol;
            const int lead = chunk == 0 ? pad : 0;
            uint32_t none = bounds.mask();
            bounds.advance();
            const bool bound_off = none >> (C - 1);
            if (chunk == n_chunks - 1 && t_lo == 0 && !a.state_in) none |= 1u << (C - 1);
            float q[4], k4[4], l4[2][4], dk[2][4], r[2][4], sum[4];
            // (everything that comes from LDS is asked for at once)
            Leaving out_rows;
            read_dv(out_rows, chunk);
            if (chunk > 0) read_done(out_rows, chunk - 1);
            const float4 tile4[2] = {*(const float4 *)tile, *(const float4 *)(tile + OS)};
            uint2 cz[2], ck[2], cl[2];             // (copies: the fetched registers are free from here on)
            float4 cdq[2];
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                cz[it] = rz[it];
                cl[it] = rl[it];
                ck[it] = rk[it];
                cdq[it] = rdq[it];
                asm volatile("" : "+v"(cdq[it].x), "+v"(cdq[it].y), "+v"(cdq[it].z), "+v"(cdq[it].w));
                if (!SL::kHand) {
                    asm volatile("" : "+v"(cz[it].x), "+v"(cz[it].y));
                    asm volatile("" : "+v"(cl[it].x), "+v"(cl[it].y));
                    if (OWNKEY) asm volatile("" : "+v"(ck[it].x), "+v"(ck[it].y));
                }
            }
            store_dv(out_rows, chunk);
            if (chunk > 0) store(out_rows, chunk - 1, at + C * a.grad.stride_n);
            __builtin_amdgcn_sched_barrier(0);
            if (rows.next()) {
                l -= adv; z -= adv; dq32 -= C * w_stride;
                if (OWNKEY) k -= adv;
            }
            fetch();
            uint16_t *const out = done + (chunk & 1) * SL::OutMap::kHalfs + put;
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const bool live = 2 * pr + it >= lead;
                const float4 t4 = tile4[it];
                dk[it][0] = t4.x * A4[it].x; dk[it][1] = t4.y * A4[it].y; dk[it][2] = t4.z * A4[it].z; dk[it][3] = t4.w * A4[it].w;
                const float dq[4] = {cdq[it].x, cdq[it].y, cdq[it].z, cdq[it].w};
                float dqo[4];
                unpack4(cz[it], q);
                if (!FUSED || !SL::kHand) unpack4(cl[it], l4[it]);
                else { l4[it][0] = lam4[it].x; l4[it][1] = lam4[it].y; l4[it][2] = lam4[it].z; l4[it][3] = lam4[it].w; }
                if (OWNKEY) unpack4(ck[it], k4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    dqo[e] = dq[e];
                    if (FUSED) {
                        const float s = __builtin_amdgcn_rcpf(1.0f + exp_neg(q[e]));
                        dqo[e] *= s * (1.0f + q[e] * (1.0f - s));            // SiLU'
                        q[e] *= s;
                        if (!SL::kHand) l4[it][e] = __builtin_amdgcn_rcpf(1.0f + exp_neg(l4[it][e]));
                    }
                    if (!OWNKEY) k4[e] = 1.0f - l4[it][e];
                    dk[it][e] *= a.q_scale;
                    r[it][e] = q[e] * dq[e] - k4[e] * dk[it][e];
                    if (lead) r[it][e] = live ? r[it][e] : 0.f;
                }
                put_grad4<OUT_BF16>(out + it * SL::OUT_ROW, dqo[0], dqo[1], dqo[2], dqo[3]);
                if (OWNKEY) put_grad4<OUT_BF16>(out + it * SL::OUT_ROW + 2 * SL::G, dk[it][0], dk[it][1], dk[it][2], dk[it][3]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = r[0][e] + r[1][e];
            row_scan_add4(sum);
            float suffix[2][4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                suffix[0][e] = carry[e] + (dpp_shr<0x111>(sum[e]) + r[0][e]);
                suffix[1][e] = carry[e] + sum[e];
                carry[e] = suffix[1][e];
            }
            if (chunk + 1 == part_at) {            // (lambda of the chunk's last row multiplies what its states give)
#pragma unroll
                for (int e = 0; e < 4; ++e) carry[e] = sSync[pcol + e] * a.q_scale * (bound_off ? 1.0f : l4[1][e]);
                --part;
                part_at = part_chunks();
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) carry[e] = dpp_last(carry[e]);       // the last row's, for every lane
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const bool off = (none >> (2 * pr + it)) & 1u;
                float dl[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (FUSED) dl[e] = ((off ? 0.f : suffix[it][e]) - dk[it][e] * l4[it][e]) * (1.0f - l4[it][e]);     // times sigmoid' = lambda (1 - lambda)
                    else dl[e] = (off ? 0.f : quotient(suffix[it][e], l4[it][e])) - (OWNKEY ? 0.f : dk[it][e]);
                }
                put_grad4<OUT_BF16>(out + it * SL::OUT_ROW + SL::G, dl[0], dl[1], dl[2], dl[3]);
            }
            at -= C * a.grad.stride_n;
        };
        __syncthreads();
        for (int chunk = 0; fine && chunk < n_chunks; ++chunk) {
            const int4 f = *(const int4 *)sTrip[chunk & 1];
            if (chunk > 0) finish(chunk - 1);
            take(chunk);
            fine = (f.x | f.y | f.z | f.w | lost) == 0;
            __syncthreads();
        }
        if (fine) {
            finish(n_chunks - 1);
            __syncthreads();                       // (the other wavefronts have left)
            Leaving rest;
            read_done(rest, n_chunks - 1);
            store(rest, n_chunks - 1, at + C * a.grad.stride_n);
        }
    } else {
        // ===================================== compute wavefronts =====================================
        __builtin_amdgcn_s_setprio(2);                 // the chain from chunk to chunk; the loaders fill the gaps
        const int l16 = lane & 15, g = lane >> 4;
        const bool is_dk = wave >= 4;
        const int col0 = 16 * (wave & 3);              // value channels (dv) / key channels (dk) of this wavefront
        // element (t, r) of the accumulators: dv: G[state_channel(t, g) + r][col0 + l16]; dk: the same of G^T
        const int s_lane = is_dk ? (col0 + l16) * D : col0 + l16, s_step = is_dk ? 1 : D;
        f32x4v accS[4];
        const f32x4v zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t) accS[t] = zero4;
        if (const float *g_in = last_seg ? state_of(p.g_in, bh) : p.bound_g(bh, seg)) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) accS[t][r] = g_in[s_lane + (state_channel(t, g) + r) * s_step];
        }
        __syncthreads();
        if (!is_dk) {
            for (int chunk = 0; fine && chunk < n_chunks; ++chunk) {
                const int4 f = *(const int4 *)sTrip[chunk & 1];
                const SlotPtr<SL::ROW> sp(slots + (chunk & 1) * SL::kHalfs, lane);
                f32x4v p00 = zero4, p01 = zero4, p11 = zero4;          // scores P^T[j][i]: (Q~ tile, K^ tile)
                f32x4v o0 = zero4, o1 = zero4;                         // O^T[n][i] of the two row tiles
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    if (s) __builtin_amdgcn_sched_barrier(0);
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
                causal_mask(p00, lane);
                causal_mask(p11, lane);
                Frag ph, pl;
                const Frag fv = sp.tokens(SL::Y + col0);
                Frag fl;
                if (LO) fl = sp.tokens(SL::Lo + col0);
                // ---- G[c][n] += sum_j Q~[j][c] g[j][n], O^T[n][i] += sum_j g[j][n] P^T[j][i] ----
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
                float *tile = outs + (chunk & 1) * C * OS + l16 * OS + col0 + 4 * g;
                *(float4 *)tile = make_float4(o0[0], o0[1], o0[2], o0[3]);
                *(float4 *)(tile + 16 * OS) = make_float4(o1[0], o1[1], o1[2], o1[3]);
                fine = (f.x | f.y | f.z | f.w | lost) == 0;
                __syncthreads();
            }
        } else {
            for (int chunk = 0; fine && chunk < n_chunks; ++chunk) {
                const int4 f = *(const int4 *)sTrip[chunk & 1];
                const SlotPtr<SL::ROW> sp(slots + (chunk & 1) * SL::kHalfs, lane);
                f32x4v p00 = zero4, p01 = zero4, p11 = zero4;          // scores P^T[j][i]: (g tile, v tile)
                f32x4v o0 = zero4, o1 = zero4;                         // O^T[c][i] / A of the two row tiles
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const Frag x0 = sp.rows(0, SL::X, s), x1 = sp.rows(16, SL::X, s);
                    const Frag y0 = sp.rows(0, SL::Y, s), y1 = sp.rows(16, SL::Y, s);
                    Frag l0, l1;
                    if (LO) { l0 = sp.rows(0, SL::Lo, s); l1 = sp.rows(16, SL::Lo, s); }
                    Frag sh, sl;
                    split_tiles(accS[2 * s], accS[2 * s + 1], sh, sl, sc);
                    p00 = mfma16(y0, x0, p00);
                    p01 = mfma16(y0, x1, p01);
                    p11 = mfma16(y1, x1, p11);
                    o0 = mfma16(sh, x0, o0);
                    o1 = mfma16(sh, x1, o1);
                    if (LO) {
                        p00 = mfma16(l0, x0, p00);
                        p01 = mfma16(l0, x1, p01);
                        p11 = mfma16(l1, x1, p11);
                    }
                    o0 = mfma16(sl, x0, o0);
                    o1 = mfma16(sl, x1, o1);
                }
                causal_mask(p00, lane);
                causal_mask(p11, lane);
                Frag ph, pl;
                const Frag zh = sp.tokens(SL::Zh + col0), zl = sp.tokens(SL::Zl + col0);
                // ---- G^T[e][c] += sum_j g[j][e] Q~[j][c], O^T[c][i] += sum_j Q~[j][c] P^T[j][i] ----
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const Frag fy = sp.state_rows(SL::Y, t);
                    accS[t] = mfma16(fy, zh, accS[t]);
                    accS[t] = mfma16(fy, zl, accS[t]);
                    if (LO) accS[t] = mfma16(sp.state_rows(SL::Lo, t), zh, accS[t]);
                }
                split_tiles(p00, zero4, ph, pl, sc);
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
                if (chunk + 1 == part_at) {
                    // sum over the value channels of G (at the chunk's last row) times S before it
                    const float *s = p.part_s(bh, seg, part - 1) + s_lane;
                    float acc = 0.f;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const f32x4v s4 = *(const f32x4v *)(s + state_channel(t, g));
                        acc += (s4[0] * accS[t][0] + s4[1] * accS[t][1]) + (s4[2] * accS[t][2] + s4[3] * accS[t][3]);
                    }
                    acc += __shfl_xor(acc, 16);
                    acc += __shfl_xor(acc, 32);
                    if (g == 0) sSync[col0 + l16] = acc;
                    --part;
                    part_at = part_chunks();
                }
                // O^T row 4 g + r is key channel col0 + 4 g + r of token l16 / 16 + l16 (its A: with the end of the chunk)
                float *tile = outs + (2 + (chunk & 1)) * C * OS + l16 * OS + col0 + 4 * g;
                *(float4 *)tile = make_float4(o0[0], o0[1], o0[2], o0[3]);
                *(float4 *)(tile + 16 * OS) = make_float4(o1[0], o1[1], o1[2], o1[3]);
                fine = (f.x | f.y | f.z | f.w | lost) == 0;
                __syncthreads();
            }
        }
        if (fine && p.g_out && seg == 0 && !is_dk) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) p.g_out[(int64_t)bh * D * D + s_lane + (state_channel(t, g) + r) * s_step] = accS[t][r];
        }
    }
    if (!fine)                                     // (every wavefront, after the barrier of the period that found a chunk out of range)
        redo_reversed<OUT_BF16>((const GatedChunkArgs *)__builtin_amdgcn_kernarg_segment_ptr(), bh, seg, (LdsFloat *)smem);
}

// ============================================ segments ============================================

// What every segment alone adds to the state (blockIdx.y 0: all segments but the last, into bounds_s) and to the adjoint
// state (1: all but the first, into bounds_g), and the segments' total decays (where the sinks will be).
template <int OWNKEY, int FUSED>
__global__ void __launch_bounds__(256, 2)
backward_gated_state_kernel(GatedChunkArgs p)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[kStateLdsBytes];
    const GatedBackwardArgs &a = p.b;
    const int nb = p.cut.n_seg - 1, bh = blockIdx.x / nb, i = blockIdx.x - bh * nb;
    float *const decays = p.sinks + (int64_t)bh * kMaxSegments * D;
    if (blockIdx.y == 0) {
        const StatePass sp{a.lam, a.k, a.v, nullptr, a.in, a.Hh, a.grid_w, a.start_pos, a.n_tokens, a.mode, p.cut};
        state_pass<0, OWNKEY, FUSED, 0>(sp, bh, i, lds, RowState{p.bound_s(bh, i), 0, 30}, RowState{decays + i * D, 0, 30});
    } else {
        const StatePass sp{a.lam, a.q, a.d_o, a.d_o_lo, a.in, a.Hh, a.grid_w, a.start_pos, a.n_tokens, a.mode, p.cut};
        const bool last = i + 2 == p.cut.n_seg;                // (the other decays come from the forward order)
        state_pass<1, 1, FUSED, FUSED>(sp, bh, i + 1, lds, RowState{p.bound_g(bh, i), 0, 30},
                                       RowState{last ? decays + (i + 1) * D : nullptr, 0, 30});
    }
}

// The states at the bounds from the segments' own, in place: P_{g+1} = diag(A_g) P_g + U_g from state_in on, and
// G_{g-1} = diag(A_g) G_g + U_g from g_in on; and at every bound what the suffix sums of the segment before it start from,
// q_scale sum_n P[c][n] G[c][n].  Four elements a thread, sixteen threads a row.
__global__ void __launch_bounds__(256)
backward_gated_fold_kernel(GatedChunkArgs p)
{
    const int bh = blockIdx.x >> 2, i = (blockIdx.x & 3) * 1024 + threadIdx.x * 4, c = i / D, nb = p.cut.n_seg - 1;
    float *const decays = p.sinks + (int64_t)bh * kMaxSegments * D + c;
    f32x4v u[kMaxSegments - 1], w[kMaxSegments - 1];
    float dec[kMaxSegments];
#pragma unroll
    for (int s = 0; s < kMaxSegments; ++s) dec[s] = decays[min(s, nb) * D];
#pragma unroll
    for (int s = 0; s < kMaxSegments - 1; ++s) {
        u[s] = *(const f32x4v *)(p.bound_s(bh, min(s, nb - 1)) + i);
        w[s] = *(const f32x4v *)(p.bound_g(bh, min(s, nb - 1)) + i);
    }
    f32x4v st = {0.f, 0.f, 0.f, 0.f}, g = st;
    if (p.b.state_in) st = *(const f32x4v *)(p.b.state_in + (int64_t)bh * D * D + i);
    if (p.g_in) g = *(const f32x4v *)(p.g_in + (int64_t)bh * D * D + i);
#pragma unroll
    for (int s = kMaxSegments - 2; s >= 0; --s) {
        if (s >= nb) continue;
        g = dec[s + 1] * g + w[s];
        w[s] = g;
        *(f32x4v *)(p.bound_g(bh, s) + i) = g;
    }
#pragma unroll
    for (int s = 0; s < kMaxSegments - 1; ++s) {
        if (s >= nb) continue;
        st = dec[s] * st + u[s];
        *(f32x4v *)(p.bound_s(bh, s) + i) = st;
        float acc = (st[0] * w[s][0] + st[1] * w[s][1]) + (st[2] * w[s][2] + st[3] * w[s][3]);
#pragma unroll
        for (int m = 8; m > 0; m >>= 1) acc += __shfl_xor(acc, m);
        if ((threadIdx.x & 15) == 0) decays[s * D] = acc * p.b.q_scale;      // (the row's threads are one wavefront's: all have read)
    }
}

}  // namespace

// (a lane's offsets in a chunk are 32 bits: 32 rows of four-byte elements)
bool backward_gated_chunk_fits(const GatedBackwardArgs &a)
{
    return a.in.stride_n >= 0 && a.in.stride_n <= kMaxStride && a.grad.stride_n >= 0 && a.grad.stride_n <= kMaxStride && a.Hh <= kMaxStride / D;
}

hipError_t launch_backward_gated_chunk_dq(const GatedChunkArgs &p, hipStream_t s)
{
    const GatedBackwardArgs &a = p.b;
    if (a.d != D || a.io_dtype != LASAD_BF16 || a.n_tokens < 1) return hipErrorInvalidValue;
    if (a.fused_act && (a.k || !a.d_o_lo)) return hipErrorInvalidValue;
    const int64_t n_wg = (int64_t)a.B * a.Hh * p.cut.n_seg;
    if (n_wg > 0x7fffffff) return hipErrorInvalidValue;
    const int ng = n_wg <= 256 ? 2 : 1;
    const dim3 grid((unsigned)n_wg), block((1 + ng) * kThreads);
#define LASAD_LAUNCH(K, F) do { \
        if (ng == 2) hipLaunchKernelGGL((backward_gated_dq_kernel<K, F, 2>), grid, block, 0, s, p); \
        else hipLaunchKernelGGL((backward_gated_dq_kernel<K, F, 1>), grid, block, 0, s, p); } while (0)
    if (a.fused_act) LASAD_LAUNCH(0, 1);
    else if (a.k) LASAD_LAUNCH(1, 0);
    else LASAD_LAUNCH(0, 0);
#undef LASAD_LAUNCH
    return hipGetLastError();
}

hipError_t launch_backward_gated_chunk_reversed(const GatedChunkArgs &p, hipStream_t s)
{
    const GatedBackwardArgs &a = p.b;
    if (a.d != D || a.io_dtype != LASAD_BF16 || a.n_tokens < 1) return hipErrorInvalidValue;
    if (a.fused_act && (a.k || !a.d_o_lo)) return hipErrorInvalidValue;
    const int64_t n_wg = (int64_t)a.B * a.Hh * p.cut.n_seg;
    if (n_wg > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)n_wg), block(4 * kThreads);
    const bool out16 = a.grad_dtype == LASAD_BF16;
#define LASAD_LAUNCH(K, F) do { \
        if (out16) hipLaunchKernelGGL((backward_gated_reversed_kernel<1, K, F>), grid, block, 0, s, p); \
        else hipLaunchKernelGGL((backward_gated_reversed_kernel<0, K, F>), grid, block, 0, s, p); } while (0)
    if (a.fused_act) LASAD_LAUNCH(0, 1);
    else if (a.k) LASAD_LAUNCH(1, 0);
    else LASAD_LAUNCH(0, 0);
#undef LASAD_LAUNCH
    return hipGetLastError();
}

hipError_t launch_backward_gated_chunk_states(const GatedChunkArgs &p, hipStream_t s)
{
    const GatedBackwardArgs &a = p.b;
    const int64_t n_seq = (int64_t)a.B * a.Hh;
    if (p.cut.n_seg < 2 || p.cut.n_seg > kMaxSegments || n_seq * 8 > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(n_seq * (p.cut.n_seg - 1)), 2);
    if (a.fused_act) hipLaunchKernelGGL((backward_gated_state_kernel<0, 1>), grid, dim3(256), 0, s, p);
    else if (a.k) hipLaunchKernelGGL((backward_gated_state_kernel<1, 0>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((backward_gated_state_kernel<0, 0>), grid, dim3(256), 0, s, p);
    hipLaunchKernelGGL(backward_gated_fold_kernel, dim3((unsigned)(n_seq * 4)), dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace lasad
