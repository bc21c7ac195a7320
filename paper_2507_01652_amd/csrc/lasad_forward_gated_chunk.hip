// Chunked forward for the vector, data-dependent decay of Section 3.4 / Algorithm 1 on the bf16 matrix
// cores (gfx950 MFMA), head dim 64, bf16 storage (lasad_gated_chunk.h has the chunk form, the tile
// layouts and the split of the work).
//
// A workgroup walks one sequence: four compute wavefronts (16 value channels each) and NG groups of four
// loader wavefronts.  While the compute wavefronts work on chunk c, the loaders
//   - finish chunk c - 1: the fp32 output tile is read from LDS, normalised (NORM), rounded and stored in
//     16-byte pieces;
//   - prepare chunk c + 1: phase A: gate activation (FUSED), running products of the decay along the tokens
//     (lane = token pair x 4 channels, a DPP scan over the 16 lanes of a row), and the loads of the next chunk as
//     soon as the registers are free; phase B: K~ and Q~, split into bf16 hi + lo, and the V rows, into LDS.
// Every LDS buffer is doubled; one barrier per chunk.
//
// NG = 1 (two workgroups of eight wavefronts per compute unit): both phases in one chunk period.  A lone
// workgroup is bound by that: a wavefront issues a vector instruction only every eight cycles or so, and the
// loaders' are the larger part.  With NG = 2 (twelve wavefronts, for workgroups that have a compute unit to
// themselves) the groups take the chunks in turn, a period for each phase.
//
// Bound by vector-instruction issue (about 1700 wave instructions per chunk, matrix instructions included, in
// 4000 cycles of four SIMDs at two workgroups per unit).  Measured against the kernels this one replaced (four wavefronts
// of 64-token chunks, or twelve with a workgroup per compute unit), bf16, us per call (graph replay): 512 sequences of
// 24 x 24 tokens, fused layer 54.6 -> 47.4, tied key 53.7 -> 42, own key 60.4 -> 44; 288 of 16 x 16 fused layer 26.4 -> 21.5;
// 96 of 64 x 64 132 -> 84 (segments); one workgroup per unit, 192 of 64 x 64 137 -> 125, own key 155 -> 151, 96 of 16 x 16
// 11.5 -> 11.0, own key 11.9 -> 12.0.  Slower: two chunks where the other had one, 24 x 64 tokens 5.1 -> 5.4, own key 5.3 -> 5.7.
//
// Precision: Q~, K~, P and S are computed operands and are each split into bf16 hi + lo (three MFMAs for
// a product of two split operands, two when one side is exact); v is exact bf16.
//
// Range.  K~ grows like 1 / A and Q~ shrinks like A.  Down to a chunk decay of 2^-100 per channel both stay
// normal numbers in fp32 and in their bf16 hi and lo parts for inputs of ordinary size (|k| 2^100 < 2^127;
// q_scale q 2^-100 and its low part, 2^-8 of it, > 2^-126), every valid score is a sum of products
// A_i / A_j <= 1, and a state row mixes only terms of its own channel.  A chunk whose total decay of some
// channel is below that (or zero) cannot be factored this way; the loaders see it one chunk ahead, and the
// workgroup redoes its whole sequence with the token-serial fp32 routine (lasad_scan.h).
#include "lasad_gated_chunk.h"
#include "lasad_gated_state.h"
#include "lasad_scan.h"

namespace lasad {

namespace {

using namespace gchunk;

constexpr int kThreads = 256;                  // of one role: compute, loader group
constexpr int64_t kMaxStride = 1 << 25;        // 32 rows of it, two bytes an element, stay below 2^32

// This thread's share of a chunk: tokens 2 pr, 2 pr + 1 (pr = lane & 15) and channels 16 lw + 4 (lane >> 4) .. + 3 of
// q, gate and key, and one 16-byte piece of a V row.  The addresses are a uniform base per tensor, advanced chunk by
// chunk on the scalar unit, plus 32-bit byte offsets of the lane; rows past the end re-read the last token.
// TURN (one loader group, own key): of q, gate and key 16 bytes of one row, turned to that share in the chunk's slot
// (gchunk::Turn).  us a call on rotating buffers: 512 sequences of 24 x 24 tokens 60.5 -> 51.5, 96 of 64 x 64 114 -> 110, 1000 of
// 16 x 16 59.6 -> 52.8.  With two tensors to turn in the place of three the address unit is not what the loaders wait for:
// tied key 512 of 24 x 24 46.6 -> 50, fused layer 48.2 -> 48.8.
template <int OWNKEY, int TURN>
struct Stage {
    const char *q, *l, *k, *v;
    uint32_t off, voff, row;           // bytes; row: one token on
    int left;                          // tokens from the base on, > 0
    uint2 rq[2], rl[2], rk[2];
    u32x4 tq, tl, tk;
    uint4 rv;

    __device__ __forceinline__ void init(const ForwardArgs &a, int64_t base, int n, int pr, int pcol, int st)
    {
        q = (const char *)((const uint16_t *)a.q + base);
        l = (const char *)((const uint16_t *)a.lam + base);
        k = OWNKEY ? (const char *)((const uint16_t *)a.k + base) : nullptr;
        v = (const char *)((const uint16_t *)a.v + base);
        left = n;
        row = (uint32_t)a.in.stride_n * 2;
        off = TURN ? 0 : 2 * pr * row + pcol * 2;
        voff = (st >> 3) * row + (st & 7) * 16;
    }
    // the chunk at the base.  (Always the same loads: a load under a condition would make the compiler wait for everything
    // outstanding wherever the paths meet.)
    __device__ __forceinline__ void fetch(int pr, int pcol, int st)
    {
        if (TURN) {
            const int last = min(left, C) - 1, lane = st & 63;
            const uint32_t o = min(Turn<kRow>::row(lane), last) * row + Turn<kRow>::byte(st >> 6, lane);
            tl = *(const u32x4 *)(l + o);
            tq = *(const u32x4 *)(q + o);
            if (OWNKEY) tk = *(const u32x4 *)(k + o);
            rv = *(const uint4 *)(v + (left < C ? min(st >> 3, last) * row + (st & 7) * 16 : voff));
            return;
        }
        uint32_t o0 = off, o1 = off + row, ov = voff;
        if (left < C) {
            o0 = min(2 * pr, left - 1) * row + pcol * 2;
            o1 = min(2 * pr + 1, left - 1) * row + pcol * 2;
            ov = min(st >> 3, left - 1) * row + (st & 7) * 16;
        }
        rl[0] = *(const uint2 *)(l + o0); rl[1] = *(const uint2 *)(l + o1);
        rq[0] = *(const uint2 *)(q + o0); rq[1] = *(const uint2 *)(q + o1);
        if (OWNKEY) { rk[0] = *(const uint2 *)(k + o0); rk[1] = *(const uint2 *)(k + o1); }
        rv = *(const uint4 *)(v + ov);
    }
    // moves the base `tokens` on; past the end of the sequence it stays (the last chunk is then read again)
    __device__ __forceinline__ void next(int tokens, int64_t stride_n)
    {
        if (left <= tokens) return;
        left -= tokens;
        const int64_t adv = tokens * stride_n * 2;
        q += adv; l += adv; v += adv;
        if (OWNKEY) k += adv;
    }
};

// rows of the output tensor that hold the state of the segment whose first token is t0
__device__ __forceinline__ RowState segment_state(const ForwardArgs &a, int b, int h, int t0)
{
    const int64_t row = (int64_t)b * a.out.stride_b + (int64_t)h * a.out.stride_h + (int64_t)t0 * a.out.stride_n;
    RowState r;
    if (a.out_dtype == LASAD_BF16) { r.base = (float *)((uint16_t *)a.o + row); r.stride = a.out.stride_n / 2; r.shift = 5; }
    else { r.base = (float *)a.o + row; r.stride = a.out.stride_n; r.shift = 6; }
    return r;
}

// The token-serial walk of tokens t0 .. t0 + n - 1 of a sequence, from the state s_in (or the call's state_in).
template <int OUT_BF16, int OWNKEY>
__device__ __noinline__ void redo_sequence(const ForwardArgs *args, int bh, int t0, int n, const float *s_in, LdsFloat *lds)
{
    ForwardArgs a = *args;
    a.q = (const uint16_t *)a.q + t0 * a.in.stride_n;
    a.lam = (const uint16_t *)a.lam + t0 * a.in.stride_n;
    if (OWNKEY) a.k = (const uint16_t *)a.k + t0 * a.in.stride_n;
    a.v = (const uint16_t *)a.v + t0 * a.in.stride_n;
    a.o = OUT_BF16 ? (void *)((uint16_t *)a.o + t0 * a.out.stride_n) : (void *)((float *)a.o + t0 * a.out.stride_n);
    a.start_pos += t0;
    if (t0 + n < a.n_tokens) a.state_out = nullptr;
    a.n_tokens = n;
    if (s_in) a.state_in = s_in - (int64_t)bh * D * D;
    scan::scan_sequence<1, OUT_BF16, OWNKEY ? scan::OWNKEY : scan::TIED, 64>(a, bh, 0, (float *)lds);
}

// What the normalisation's backward makes of an output row and the gradient of its normalised form, for a lane's eight of the
// row's channels (the row is eight lanes): d_o = rstd gw - o rstd^3 mean(gw o) with gw = d_out w, and d_out o rstd.
__device__ __forceinline__ void norm_backward8(const float (&o)[8], uint4 dout, const float (&w)[8], float eps, float (&res)[8], float (&dw)[8])
{
    float g[8];
    const uint32_t words[4] = {dout.x, dout.y, dout.z, dout.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        g[2 * e] = __uint_as_float(words[e] << 16);
        g[2 * e + 1] = __uint_as_float(words[e] & 0xffff0000u);
    }
    float ss = 0.f, go = 0.f, gw[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        gw[e] = g[e] * w[e];
        ss = fmaf(o[e], o[e], ss);
        go = fmaf(gw[e], o[e], go);
    }
    const float rstd = 1.0f / sqrtf(sum8(ss) * (1.0f / D) + eps);
    const float back = rstd * rstd * rstd * sum8(go) * (1.0f / D);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        res[e] = gw[e] * rstd - o[e] * back;
        dw[e] = g[e] * o[e] * rstd;
    }
}
// ... to memory
__device__ __forceinline__ void store_grad8(const NormBackwardArgs &nb, int64_t i, const float (&res)[8], const SplitConst &sc)
{
    if (nb.d_o_f32) {
        *(float4 *)((float *)nb.d_o + i) = make_float4(res[0], res[1], res[2], res[3]);
        *(float4 *)((float *)nb.d_o + i + 4) = make_float4(res[4], res[5], res[6], res[7]);
        return;
    }
    uint4 hi, lo;
    split2(res[0], res[1], hi.x, lo.x, sc);
    split2(res[2], res[3], hi.y, lo.y, sc);
    split2(res[4], res[5], hi.z, lo.z, sc);
    split2(res[6], res[7], hi.w, lo.w, sc);
    *(uint4 *)((uint16_t *)nb.d_o + i) = hi;
    if (nb.d_o_lo) *(uint4 *)((uint16_t *)nb.d_o_lo + i) = lo;
}
// The same from the fp32 rows that a token-serial walk of tokens t0 .. t0 + n - 1 has left in o, by its 256 threads, and their
// part of the weight's gradient.
__device__ __noinline__ void redo_norm_backward(const ForwardArgs *a, const NormBackwardArgs *nb, int bh, int t0, int n, float *wpart, float *lds)
{
    const int b = bh / a->Hh, h = bh - b * a->Hh;
    const int row = threadIdx.x >> 3, col = (threadIdx.x & 7) * 8;
    SplitConst sc;
    sc.init();
    float w[8], sum[8];
    for (int e = 0; e < 8; ++e) {
        w[e] = nb->norm_w ? nb->norm_w[h * D + col + e] : 1.0f;
        sum[e] = 0.f;
    }
    __syncthreads();                               // (o is this workgroup's own)
    for (int t = t0; t < t0 + n; t += 32) {
        const int tok = min(t + row, t0 + n - 1);  // (all eight lanes of a row take part in its sums)
        const float *o_row = (const float *)a->o + (int64_t)b * a->out.stride_b + (int64_t)tok * a->out.stride_n + (int64_t)h * a->out.stride_h + col;
        float o[8], res[8], dw[8];
        for (int e = 0; e < 8; ++e) o[e] = o_row[e];
        const uint4 g = *(const uint4 *)((const uint16_t *)nb->d_out + (int64_t)b * nb->dout.stride_b + (int64_t)tok * nb->dout.stride_n +
                                         (int64_t)h * nb->dout.stride_h + col);
        norm_backward8(o, g, w, nb->norm_eps, res, dw);
        if (t + row < t0 + n) {
            store_grad8(*nb, (int64_t)b * nb->dl.stride_b + (int64_t)tok * nb->dl.stride_n + (int64_t)h * nb->dl.stride_h + col, res, sc);
            for (int e = 0; e < 8; ++e) sum[e] += dw[e];
        }
    }
    for (int e = 0; e < 8; ++e) lds[row * D + col + e] = sum[e];
    __syncthreads();
    if (threadIdx.x < D) {
        float acc = 0.f;
        for (int r = 0; r < 32; ++r) acc += lds[r * D + threadIdx.x];
        wpart[threadIdx.x] = acc;
    }
}

// NORM: 1 the normalised output; 2 the output is not stored, but what the normalisation's backward makes of it, from the
// gradient's row that the loaders hold one tile ahead.  In a pass of its own that was another fp32 tensor written and read, bound
// by memory: 288 sequences of 16 x 16 tokens 23 + 16 us -> 29, a whole layer backward on rotating buffers 98 -> 90, 512 of 24 x 24
// 256 -> 222, 96 of 64 x 64 436 -> 388, 300 of 8 x 8 42 -> 38.  (Not for few sequences of middle length:
// forward_gated_norm_backward_pays.)
template <int OUT_BF16, int OWNKEY, int FUSED, int NORM, int NG>
__global__ void __launch_bounds__((1 + NG) * kThreads, NG == 1 ? 4 : 3)
forward_gated_chunk_kernel(ForwardArgs a, SegPlan plan, NormBackwardArgs nb)
{
    struct KernelArgs { ForwardArgs a; SegPlan plan; NormBackwardArgs nb; };       // as the launch lays them out
    // tiles, then the segment's incoming state (kept for a redo, which reads it before its own buffers reach that far)
    constexpr int kTileBytes = 2 * kSlot * 2 + 2 * C * OS * 4;
    constexpr int kScanBytes = scan::lds_floats<OWNKEY ? scan::OWNKEY : scan::TIED>() * 4;
    constexpr int kLdsBytes = kTileBytes + D * D * 4;
    static_assert(kLdsBytes >= kScanBytes && kTileBytes >= kScanBytes * 3 / 4, "the redo's buffers; its last quarter is written after a barrier");
    __shared__ __attribute__((aligned(16))) unsigned char smem[kLdsBytes];
    __shared__ __attribute__((aligned(16))) float sTot[2][D];              // A_end per key channel, by chunk parity
    __shared__ __attribute__((aligned(16))) int sTrip[2][4];               // range flag of each loader wavefront, by barrier parity
    __shared__ __attribute__((aligned(16))) float sW[NORM ? D : 1];        // norm weight (times q_scale)
    __shared__ __attribute__((aligned(16))) float sDw[NORM == 2 ? 4 * NG : 1][D];      // each loader wavefront's sums for the weight
    uint16_t *const slots = (uint16_t *)smem;
    float *const outs = (float *)(slots + 2 * kSlot);

    float *const seg_state = (float *)(smem + kTileBytes);
    const int bh = plan.n_seg == 1 ? blockIdx.x : blockIdx.x / plan.n_seg, seg = blockIdx.x - bh * plan.n_seg;
    const int b = bh / a.Hh, h = bh - b * a.Hh;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int seg_t0 = plan.start(seg);
    const bool last_seg = seg == plan.n_seg - 1;
    const int n = (last_seg ? a.n_tokens : plan.start(seg + 1)) - seg_t0;  // tokens of this workgroup
    const int n_chunks = (n + C - 1) / C;
    SplitConst sc;
    sc.init();

    // token-serial redo of the sequence by the first four wavefronts, out of line (inlined it would keep the argument
    // block in scratch memory); it reads the arguments where the launch put them
    auto redo = [&]() {
        if (tid >= scan::kThreads) return;
        const KernelArgs *ka = (const KernelArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        redo_sequence<OUT_BF16, OWNKEY>(&ka->a, bh, seg_t0, n, plan.n_seg > 1 ? seg_state : nullptr, (LdsFloat *)smem);
        if (NORM == 2)
            redo_norm_backward(&ka->a, &ka->nb, bh, seg_t0, n, ka->nb.wpart + ((int64_t)bh * plan.n_seg + seg) * D, (float *)smem);
    };

    if (wave >= 4) {
        // ===================================== loader wavefronts =====================================
        const int grp = NG == 2 ? (wave >> 2) - 1 : 0, lw = wave & 3, st = tid & 255;
        const int first = grp * C < n ? grp * C : 0;           // (a group without a chunk reads the first one, for nobody)
        const int pr = lane & 15, pcol = 16 * lw + 4 * (lane >> 4);
        const int64_t in_base = (int64_t)b * a.in.stride_b + (int64_t)h * a.in.stride_h + seg_t0 * a.in.stride_n;
        constexpr bool TURN = NG == 1 && OWNKEY;
        const Turn<kRow> turn(lw, lane);
        Stage<OWNKEY, TURN> sg;
        sg.init(a, in_base + first * a.in.stride_n, n - first, pr, pcol, st);
        sg.fetch(pr, pcol, st);                    // ahead of everything that does not need it (0.3 us a call)
        __builtin_amdgcn_sched_barrier(0);
        RowBoundaries bounds;
        bounds.init(a.start_pos + seg_t0 + grp * C, a.grid_w, a.mode, NG * C);
        int left = n - grp * C;                    // tokens from the next chunk to be prepared on
        const int put = SlotMap<kRow>::at(2 * pr, pcol), put_v = SlotMap<kRow>::at(st >> 3, (st & 7) * 8) + kColV;
        // the output tile of a finished chunk: thread = token st / 8, channels 8 (st & 7) .., times q_scale (NORM: and
        // the norm's factors: (q_scale o) / sqrt(mean((q_scale o)^2) + eps))
        const int orow = st >> 3, ocol = (st & 7) * 8;
        const float ms_scale = a.q_scale * a.q_scale * (1.0f / D);
        const int64_t o_lane = orow * a.out.stride_n + ocol;
        int64_t o_chunk = (int64_t)b * a.out.stride_b + (int64_t)h * a.out.stride_h +
                          (seg_t0 + (NG == 2 && grp == 0 ? C : 0)) * a.out.stride_n;
        // NORM 2: the gradient's row of the next tile to be stored, one period ahead
        uint4 rg = make_uint4(0u, 0u, 0u, 0u);
        float dw[8];
        int g_tok = NG == 2 && grp == 0 ? C : 0;               // that tile's first token (of two groups the second stores chunk 0)
        auto fetch_dout = [&]() {
            const int64_t tok = seg_t0 + min(g_tok + orow, n - 1);
            rg = *(const uint4 *)((const uint16_t *)nb.d_out + (int64_t)b * nb.dout.stride_b + (int64_t)h * nb.dout.stride_h +
                                  tok * nb.dout.stride_n + ocol);
            g_tok += NG * C;
        };
        if (NORM == 2) {
#pragma unroll
            for (int e = 0; e < 8; ++e) dw[e] = 0.f;
            fetch_dout();
        }
        auto store_tile = [&](int chunk) {
            const float *tile = outs + (chunk & 1) * C * OS + orow * OS + ocol;
            float4 u = *(const float4 *)tile, w = *(const float4 *)(tile + 4);
            if (NORM == 2) {
                const float4 w0 = *(const float4 *)&sW[ocol], w1 = *(const float4 *)&sW[ocol + 4];
                const float o[8] = {u.x * a.q_scale, u.y * a.q_scale, u.z * a.q_scale, u.w * a.q_scale,
                                    w.x * a.q_scale, w.y * a.q_scale, w.z * a.q_scale, w.w * a.q_scale};
                const float nw[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
                float res[8], dws[8];
                norm_backward8(o, rg, nw, nb.norm_eps, res, dws);
                if (chunk * C + orow < n) {
                    store_grad8(nb, (int64_t)b * nb.dl.stride_b + (int64_t)h * nb.dl.stride_h + (int64_t)(seg_t0 + chunk * C + orow) * nb.dl.stride_n + ocol, res, sc);
#pragma unroll
                    for (int e = 0; e < 8; ++e) dw[e] += dws[e];
                }
                return;
            }
            if (NORM) {
                const float ss = (u.x * u.x + u.y * u.y) + (u.z * u.z + u.w * u.w) + ((w.x * w.x + w.y * w.y) + (w.z * w.z + w.w * w.w));
                const float rstd = __builtin_amdgcn_rsqf(sum8(ss) * ms_scale + a.norm_eps);
                u = make_float4(u.x * rstd, u.y * rstd, u.z * rstd, u.w * rstd);
                w = make_float4(w.x * rstd, w.y * rstd, w.z * rstd, w.w * rstd);
            }
            float4 w0 = make_float4(a.q_scale, a.q_scale, a.q_scale, a.q_scale), w1 = w0;
            if (NORM) { w0 = *(const float4 *)&sW[ocol]; w1 = *(const float4 *)&sW[ocol + 4]; }
            u = make_float4(u.x * w0.x, u.y * w0.y, u.z * w0.z, u.w * w0.w);
            w = make_float4(w.x * w1.x, w.y * w1.y, w.z * w1.z, w.w * w1.w);
            if (chunk * C + orow < n) {
                const int64_t i = o_chunk + o_lane;
                if (OUT_BF16) {
                    gstore16<true>((uint16_t *)a.o + i, make_uint4(pack2(u.x, u.y), pack2(u.z, u.w), pack2(w.x, w.y), pack2(w.z, w.w)));
                } else {
                    gstore16<true>((float *)a.o + i, u.x, u.y, u.z, u.w);
                    gstore16<true>((float *)a.o + i + 4, w.x, w.y, w.z, w.w);
                }
            }
            o_chunk += NG * C * a.out.stride_n;                // (of two groups, each stores every other tile)
        };

        // between the phases: the query and V as read, the key (FUSED: exp(-z)), the decay (FUSED: its reciprocal), and the
        // running products over the token pairs up to and before this one
        uint2 pq[2];
        uint4 pv;
        bool v_live;
        float key[2][4], x[2][4], tot[4], exc[4];

        // done: the finished chunk to be stored meanwhile, or -1.  Past the end of the sequence (the last periods) the last
        // chunk's data go once more into a slot that nobody reads.
        auto phase_a = [&](int done, int p) {      // (p: the slot to come, TURN)
            const uint32_t bmask = bounds.mask();
            bounds.advance();
            if (TURN) {                            // where the operands that come of them will be
                uint16_t *const slot = slots + p * kSlot;
                turn.write(slot, kColKh, sg.tl);
                turn.write(slot, kColQh, sg.tq);
                if (OWNKEY) turn.write(slot, kColKl, sg.tk);
            }
            if (!TURN) {
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    pq[it] = sg.rq[it];
                    unpack4(sg.rl[it], x[it]);
                    if (OWNKEY) unpack4(sg.rk[it], key[it]);
                }
            }
            pv = sg.rv;
            v_live = (st >> 3) < left;
            asm volatile("" : "+v"(pv.x), "+v"(pv.y), "+v"(pv.z), "+v"(pv.w));
            // The fetched registers are free from here on (and the compiler must see it so, or it carries the loads around the
            // loop in other registers and waits for them at its end): the loads of the next chunk fly during the rest of
            // this one.
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                if (TURN) break;
                asm volatile("" : "+v"(pq[it].x), "+v"(pq[it].y));
                asm volatile("" : "+v"(x[it][0]), "+v"(x[it][1]), "+v"(x[it][2]), "+v"(x[it][3]));
                if (OWNKEY) asm volatile("" : "+v"(key[it][0]), "+v"(key[it][1]), "+v"(key[it][2]), "+v"(key[it][3]));
            }
            // (the store between the waits for these loads and the issue of the next ones: no wait ever includes a new store)
            if (done >= 0) store_tile(done);
            __builtin_amdgcn_sched_barrier(0);
            if (NORM == 2 && done >= 0) fetch_dout();
            sg.next(NG * C, a.in.stride_n);
            sg.fetch(pr, pcol, st);
            if (TURN) {
                const uint16_t *const slot = slots + p * kSlot;
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    pq[it] = turn.read(slot, kColQh, it);
                    unpack4(turn.read(slot, kColKh, it), x[it]);
                    if (OWNKEY) unpack4(turn.read(slot, kColKl, it), key[it]);
                }
            }
#pragma unroll
            for (int it = 0; it < 2; ++it) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (FUSED) {                   // 1 / lambda = 1 + exp(-z)
                        key[it][e] = exp_neg(x[it][e]);
                        x[it][e] = 1.0f + key[it][e];
                    } else if (!OWNKEY) {
                        key[it][e] = 1.0f - x[it][e];
                    }
                }
                if (bmask & (0x55555555u << it)) { // some token of this parity sits on a boundary: lambda 1
                    if ((bmask >> (2 * pr + it)) & 1u) {
                        asm volatile("");          // (a branch: few lanes, and the reciprocals are not for everybody)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            // FUSED: k = 1 - lambda = exp(-z) lambda, and K~ = k / A = exp(-z) / (A of the token before); at a
                            // boundary A does not change, and the key needs its own lambda (exp(-z) up to infinity: 1; NaN stays)
                            if (FUSED) key[it][e] = key[it][e] >= 1e30f ? 1.0f : key[it][e] * __builtin_amdgcn_rcpf(x[it][e]);
                            x[it][e] = 1.0f;
                        }
                    }
                }
            }
            if (left < C) {                        // tail chunk: rows past the end get lambda 1, q = k = v = 0
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const bool live = 2 * pr + it < left;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        x[it][e] = live ? x[it][e] : 1.0f;
                        key[it][e] = live ? key[it][e] : 0.f;
                    }
                    pq[it].x = live ? pq[it].x : 0u;
                    pq[it].y = live ? pq[it].y : 0u;
                }
            }
            left -= NG * C;
#pragma unroll
            for (int e = 0; e < 4; ++e) tot[e] = x[0][e] * x[1][e];
            row_scan_mul4(tot, exc);
        };
        // the chunk's operands into slot p; leaves the range flag for the barrier that ends this period
        auto phase_b = [&](int p) {
            *(uint4 *)&slots[p * kSlot + put_v] =
                make_uint4(v_live ? pv.x : 0u, v_live ? pv.y : 0u, v_live ? pv.z : 0u, v_live ? pv.w : 0u);
            bool trip;
            if (FUSED) trip = !(fmaxf(fmaxf(tot[0], tot[1]), fmaxf(tot[2], tot[3])) <= kMaxInvDecay);
            else trip = !(fminf(fminf(tot[0], tot[1]), fminf(tot[2], tot[3])) >= 1.0f / kMaxInvDecay);
            if (pr == 15)
                *(float4 *)&sTot[p][pcol] = FUSED ? make_float4(__builtin_amdgcn_rcpf(tot[0]), __builtin_amdgcn_rcpf(tot[1]),
                                                                __builtin_amdgcn_rcpf(tot[2]), __builtin_amdgcn_rcpf(tot[3]))
                                                  : make_float4(tot[0], tot[1], tot[2], tot[3]);
            const bool any = __any(trip);
            if (lane == 0) sTrip[p][lw] = any ? 1 : 0;
            uint16_t *rows = slots + p * kSlot + put;
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                float q[4], kt[4], qt[4];
                unpack4(pq[it], q);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float before = it ? exc[e] * x[0][e] : exc[e];       // A (FUSED: 1 / A) before this token
                    const float after = it ? tot[e] : exc[e] * x[0][e];        // ... and after it
                    if (FUSED) {                   // SiLU(q) A = q / ((1 + exp(-q)) (1 / A)); q_scale: with the output
                        kt[e] = key[it][e] * before;
                        qt[e] = q[e] * __builtin_amdgcn_rcpf((1.0f + exp_neg(q[e])) * after);
                    } else {
                        kt[e] = key[it][e] * __builtin_amdgcn_rcpf(after);
                        qt[e] = q[e] * after;
                    }
                }
                put_pair4(rows + it * kRow + kColKh, rows + it * kRow + kColKl, kt, sc);
                put_pair4(rows + it * kRow + kColQh, rows + it * kRow + kColQl, qt, sc);
            }
        };
        if (NORM == 1 && grp == 0 && st < D) sW[st] = a.q_scale * (a.norm_w ? a.norm_w[h * D + st] : 1.0f);
        if (NORM == 2 && grp == 0 && st < D) sW[st] = nb.norm_w ? nb.norm_w[h * D + st] : 1.0f;
        bool fine = true;
        int4 f;                                    // a chunk's range flags, read at the start of its period and tested at the end
        auto end_period = [&]() {
            fine = (f.x | f.y | f.z | f.w) == 0;
            __syncthreads();
        };
        if (NG == 2 && !FUSED) {
            // From the period before chunk 0 on, in which there are no flags to test, with one copy of each phase: at the start
            // of a call the code itself comes from memory (24 x 64 tokens 5.8 -> 5.5 us).  (The fused layer is 2 % slower so.)
            for (int chunk = -1;; ++chunk) {
                f = chunk < 0 ? make_int4(0, 0, 0, 0) : *(const int4 *)sTrip[chunk & 1];
                phase_a(chunk - 1, 0);
                if (grp == 1 || chunk >= 0) {      // (the first group runs both phases for chunk 0 at once)
                    end_period();
                    if (!fine || ++chunk == n_chunks) break;
                    f = *(const int4 *)sTrip[chunk & 1];
                }
                phase_b((chunk + 1) & 1);
                end_period();
                if (!fine || chunk + 1 == n_chunks) break;
            }
        } else {
            phase_a(-1, 0);
            if (grp == 0) phase_b(0);
            __syncthreads();
            if (NG == 2 && grp == 1) {             // period 0
                f = *(const int4 *)sTrip[0];
                phase_b(1);
                end_period();
            }
            for (int chunk = grp; fine && chunk < n_chunks; chunk += NG) {
                f = *(const int4 *)sTrip[chunk & 1];
                phase_a(chunk - 1, (chunk + NG) & 1);
                if (NG == 2) {
                    end_period();
                    if (!fine || chunk + 1 == n_chunks) break;
                    f = *(const int4 *)sTrip[(chunk + 1) & 1];
                }
                phase_b((chunk + NG) & 1);         // (one group: chunk + 1, prepared in one period; two: chunk + 2)
                end_period();
            }
        }
        if (!fine) redo();
        else if (NG == 1 || grp == (n_chunks & 1)) store_tile(n_chunks - 1);
        if (NORM == 2 && fine) {                   // the weight's gradient: eight rows a wavefront, then the wavefronts
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int m = 8; m <= 32; m <<= 1) dw[e] += __shfl_xor(dw[e], m);
            if (lane < 8) {
                *(float4 *)&sDw[wave - 4][8 * lane] = make_float4(dw[0], dw[1], dw[2], dw[3]);
                *(float4 *)&sDw[wave - 4][8 * lane + 4] = make_float4(dw[4], dw[5], dw[6], dw[7]);
            }
            __syncthreads();                       // (the compute wavefronts have left)
            if (grp == 0 && st < D) {
                float acc = 0.f;
#pragma unroll
                for (int w = 0; w < 4 * NG; ++w) acc += sDw[w][st];
                nb.wpart[((int64_t)bh * plan.n_seg + seg) * D + st] = acc;
            }
        }
        return;
    }

    // ===================================== compute wavefronts =====================================
    __builtin_amdgcn_s_setprio(2);                 // the chain from chunk to chunk; the loaders fill the gaps (1-3 % at 192 and at 480 workgroups)
    const int l16 = lane & 15, g = lane >> 4;
    const int col0 = 16 * wave;                    // value channels of this wavefront
    const int64_t s_off = (int64_t)bh * D * D + col0 + l16;
    f32x4v accS[4];                                // S[state_channel(t, g) + r][col0 + l16]
    const f32x4v zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) accS[t] = zero4;
    if (plan.n_seg > 1) {
        const RowState ps = segment_state(a, b, h, seg_t0);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) accS[t][r] = *ps.at((state_channel(t, g) + r) * D + col0 + l16);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) seg_state[(state_channel(t, g) + r) * D + col0 + l16] = accS[t][r];
    } else if (a.state_in) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) accS[t][r] = a.state_in[s_off + (state_channel(t, g) + r) * D];
    }

    const SlotPtr<> sp0(slots, lane);
    __syncthreads();
    bool fine = true;
    for (int chunk = 0; fine && chunk < n_chunks; ++chunk) {
        const int4 f = *(const int4 *)sTrip[chunk & 1];
        const SlotPtr<> sp(sp0, (chunk & 1) * kSlot);
        f32x4v p00 = zero4, p01 = zero4, p11 = zero4;              // scores P^T[j][i]: (key tile, query tile)
        f32x4v o0 = zero4, o1 = zero4;                             // O^T[n][i] of the two query tiles
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const Frag q0h = sp.rows(0, kColQh, s), q1h = sp.rows(16, kColQh, s);
            const Frag q0l = sp.rows(0, kColQl, s), q1l = sp.rows(16, kColQl, s);
            // ---- P^T[j][i] += sum_c K~[j][c] Q~[i][c],  O^T[n][i] += sum_c S^T[n][c] Q~[i][c] ----
            const Frag k0h = sp.rows(0, kColKh, s), k0l = sp.rows(0, kColKl, s);
            const Frag k1h = sp.rows(16, kColKh, s), k1l = sp.rows(16, kColKl, s);
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
        // ---- S[c][n] += sum_j K~[j][c] V[j][n] ----
        const Frag fv = sp.tokens(kColV + col0);
#pragma unroll
        for (int t = 0; t < 4; ++t) accS[t] = mfma16(sp.state_rows(kColKh, t), fv, accS[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) accS[t] = mfma16(sp.state_rows(kColKl, t), fv, accS[t]);
        // ---- O^T[n][i] += sum_j V[j][n] P^T[j][i] ----
        causal_mask(p00, lane);
        causal_mask(p11, lane);
        {
            Frag ph, pl;
            split_tiles(p00, zero4, ph, pl, sc);                   // (keys 16 .. 31 come after queries 0 .. 15)
            o0 = mfma16(fv, ph, o0);
            o0 = mfma16(fv, pl, o0);
            split_tiles(p01, p11, ph, pl, sc);
            o1 = mfma16(fv, ph, o1);
            o1 = mfma16(fv, pl, o1);
        }
        // ---- S row c times A_end[c] ----
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float4 t4 = *(const float4 *)&sTot[chunk & 1][state_channel(t, g)];
            accS[t][0] *= t4.x; accS[t][1] *= t4.y; accS[t][2] *= t4.z; accS[t][3] *= t4.w;
        }
        // O^T row 4 g + r is channel col0 + 4 g + r of token l16 / 16 + l16
        float *tile = outs + (chunk & 1) * C * OS + l16 * OS + col0 + 4 * g;
        *(float4 *)tile = make_float4(o0[0], o0[1], o0[2], o0[3]);
        *(float4 *)(tile + 16 * OS) = make_float4(o1[0], o1[1], o1[2], o1[3]);
        fine = (f.x | f.y | f.z | f.w) == 0;
        __syncthreads();
    }
    if (!fine) {
        redo();
        return;
    }
    if (a.state_out && last_seg) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) a.state_out[s_off + (state_channel(t, g) + r) * D] = accS[t][r];
    }
}

// State pass of the segment plan: what a segment (all but the last) adds to the state, and its total decay per key
// channel, into the rows of the segment after it (lasad_gated_state.h).
template <int OWNKEY, int FUSED>
__global__ void __launch_bounds__(256, 2)
gated_segment_state_kernel(ForwardArgs a, SegPlan plan)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[kStateLdsBytes];
    const int bh = blockIdx.x / (plan.n_seg - 1), seg = blockIdx.x - bh * (plan.n_seg - 1);
    const int b = bh / a.Hh, h = bh - b * a.Hh;
    const StatePass p{a.lam, OWNKEY ? a.k : nullptr, a.v, nullptr, a.in, a.Hh, a.grid_w, a.start_pos, a.n_tokens, a.mode, plan};
    const RowState out = segment_state(a, b, h, plan.start(seg + 1));
    RowState decay = out;                          // after the state: from row 4096 / (floats a row) on
    decay.base = out.at(D * D);
    state_pass<0, OWNKEY, FUSED, 0>(p, bh, seg, lds, out, decay);
}

// Fold: every segment's incoming state, P_0 = state_in, P_{g+1} = diag(A_g) P_g + U_g, in place (each element by one
// thread, the segments in order; all their loads are issued together).
constexpr int kMaxSegments = 16;
__global__ void __launch_bounds__(256)
gated_segment_fold_kernel(ForwardArgs a, SegPlan plan)
{
    const int bh = blockIdx.x >> 2, b = bh / a.Hh, h = bh - b * a.Hh;
    const int i = (blockIdx.x & 3) * 1024 + threadIdx.x * 4;
    float4 u[kMaxSegments];
    float dec[kMaxSegments];
#pragma unroll
    for (int s = 1; s < kMaxSegments; ++s) {
        const RowState rs = segment_state(a, b, h, plan.start(min(s, plan.n_seg - 1)));
        u[s] = *(const float4 *)rs.at(i);
        dec[s] = *rs.at(D * D + i / D);
    }
    float4 p = a.state_in ? *(const float4 *)(a.state_in + (int64_t)bh * D * D + i) : make_float4(0.f, 0.f, 0.f, 0.f);
    *(float4 *)segment_state(a, b, h, 0).at(i) = p;
#pragma unroll
    for (int s = 1; s < kMaxSegments; ++s) {
        if (s < plan.n_seg) {
            p = make_float4(fmaf(dec[s], p.x, u[s].x), fmaf(dec[s], p.y, u[s].y), fmaf(dec[s], p.z, u[s].z), fmaf(dec[s], p.w, u[s].w));
            *(float4 *)segment_state(a, b, h, plan.start(s)).at(i) = p;
        }
    }
}

// Few, long sequences are cut into segments of at least 8 chunks, the chunks dealt out evenly: one workgroup per compute
// unit (256 in all), or two where that at least doubles the number of segments (a chunk then takes 1.6 times as long).
// State pass and fold have to pay: 16 chunks off the walk's length, 24 with more than 128 workgroups, 30 with two per unit.
// Measured (us, one workgroup per sequence -> segments, tied key unless noted): 12 x 4096 tokens 120 -> 30 (16 segments),
// 12 x 3844 113 -> 30 (15), 24 x 2116 65 -> 31 (8), 40 x 2116 66 -> 37 (6; 8 of them: 41), 60 x 1024 35 -> 29 (4), 60 x 4096
// 122 -> 62 (8; 4: 72), 96 x 4096 123 -> 95 (5), 96 x 1444 49 -> 46 (5), 110 x 2116 70 -> 64 (4), fused layer 12 x 768 29 -> 27
// (3); not taken: 60 x 768 27 -> 28 (3), 80 x 1024 33 -> 34 (3), own key 34 -> 38, 128 x 1024 37 -> 42 (4), 128 x 1444
// 50 -> 52 (4), 192 x 2116 74 -> 91 (5).
SegPlan segment_plan(int64_t n_seq, int n_tokens)
{
    const int n_chunks = (n_tokens + C - 1) / C;
    auto segments = [&](int n_wg) {
        const int most = n_chunks / 8 < kMaxSegments ? n_chunks / 8 : kMaxSegments;
        return n_wg / n_seq < most ? (int)(n_wg / n_seq) : most;
    };
    const int g1 = segments(256), g2 = segments(512);
    const bool two = g2 >= 2 * g1;
    const int g = two ? g2 : g1;
    if (g < 3) return SegPlan{1, n_chunks, 0};
    const int saved = two ? n_chunks - 8 * n_chunks / (5 * g) : n_chunks - n_chunks / g;
    if (saved < (two ? 30 : n_seq * g > 128 ? 24 : 16)) return SegPlan{1, n_chunks, 0};
    static_assert(7 * C + 1 >= kRowStateTokens, "the rows of a segment of 8 chunks hold its incoming state");
    return SegPlan{g, n_chunks / g, n_chunks % g};
}

}  // namespace

bool forward_gated_chunk_fits(const ForwardArgs &a) { return a.in.stride_n <= kMaxStride; }

// The epilogue lengthens a tile's period of a workgroup that has a compute unit to itself by 0.4 us; a kernel of its own takes
// 3.2 us and 0.085 us a sequence and 1000 tokens, spread over the idle units.  us (forward and epilogue | forward, then kernel):
// 12 x 576 tokens 28.5 | 25.4, 33 x 400 22.2 | 21.5, 60 x 784 40.9 | 37.3, 80 x 1024 51.9 | 47.1, 96 x 784 41.8 | 39.8, but 12 x
// 128 10.5 | 11.4, 48 x 256 16.0 | 16.5, 96 x 400 22.5 | 24.4, 128 x 784 41.7 | 42.3, 256 x 1024 55 | 66, 512 x 576 53 | 76; in
// segments 12 x 4096 33.6 | 38.2, 96 x 4096 106 | 152.  In the whole layer's backward the three passes come behind it, which want
// full groups of eight sequences; without, the line lies lower (epilogue over kernel, the whole call: 33 x 320 1.02, 60 x 256
// 1.01, x 400 1.04, 67 x 400 1.03; 48 x 400 0.96, 80 x 400 1.00).
bool forward_gated_norm_backward_pays(int64_t n_seq, int n_tokens)
{
    if (n_seq >= 147 || segment_plan(n_seq, n_tokens).n_seg > 1) return true;
    return n_tokens <= (n_seq % 8 && n_seq < 80 ? 300 : 37600 / (147 - n_seq));
}

static hipError_t launch(const ForwardArgs &a, const NormBackwardArgs *nb, int *n_seg, hipStream_t s)
{
    if (a.d != D || a.io_dtype != LASAD_BF16 || a.n_tokens < 1 || !a.lam) return hipErrorInvalidValue;
    if ((a.fused_act && a.k) || (a.norm && !a.fused_act)) return hipErrorInvalidValue;      // the layer of Algorithm 1 ties the key to the gate
    const int64_t n_seq = (int64_t)a.B * a.Hh;
    if (n_seq > 0x7fffffff) return hipErrorInvalidValue;
    if (!forward_gated_chunk_fits(a)) return nb ? hipErrorInvalidValue : launch_forward_generic(a, s);      // (a lane's offsets in a chunk are 32 bits)
    const bool out16 = a.out_dtype == LASAD_BF16;
    const SegPlan plan = segment_plan(n_seq, a.n_tokens);
    if (n_seg) *n_seg = plan.n_seg;
    const NormBackwardArgs none{};
    if (plan.n_seg > 1) {
        const dim3 sgrid((unsigned)(n_seq * (plan.n_seg - 1)));
        if (a.fused_act) hipLaunchKernelGGL((gated_segment_state_kernel<0, 1>), sgrid, dim3(256), 0, s, a, plan);
        else if (a.k) hipLaunchKernelGGL((gated_segment_state_kernel<1, 0>), sgrid, dim3(256), 0, s, a, plan);
        else hipLaunchKernelGGL((gated_segment_state_kernel<0, 0>), sgrid, dim3(256), 0, s, a, plan);
        hipLaunchKernelGGL(gated_segment_fold_kernel, dim3((unsigned)(n_seq * 4)), dim3(256), 0, s, a, plan);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // One workgroup per compute unit: two loader groups (see above); more of them: one, and two workgroups per unit.  us, one
    // group -> two: tied key 96 x 256 tokens 13.0 -> 12.0, 192 x 1444 58 -> 52, 256 x 576 28.5 -> 26.3, 300 x 576 37.7 -> 42.5;
    // fused layer 200 x 576 30.5 -> 26.4.  A call of a few chunks is bound by its first loads, and a second group only adds
    // to them: own key 24 x 32 5.1 -> 6.0, x 64 6.4 -> 7.0, x 96 7.6 -> 8.0, x 160 10.0 -> 9.6; fused layer x 32 5.3 -> 5.7, x 96
    // 8.1 -> 7.9.
    const int64_t n_wg = n_seq * plan.n_seg;
    const int ng = n_wg <= 256 && a.n_tokens > (a.k ? 96 : 32) ? 2 : 1;
    const dim3 grid((unsigned)n_wg), block((1 + ng) * kThreads);
#define LASAD_LAUNCH1(O, K, F, N) do { \
        if (ng == 2) hipLaunchKernelGGL((forward_gated_chunk_kernel<O, K, F, N, 2>), grid, block, 0, s, a, plan, nb ? *nb : none); \
        else hipLaunchKernelGGL((forward_gated_chunk_kernel<O, K, F, N, 1>), grid, block, 0, s, a, plan, nb ? *nb : none); } while (0)
#define LASAD_LAUNCH(K, F, N) do { if (out16) LASAD_LAUNCH1(1, K, F, N); else LASAD_LAUNCH1(0, K, F, N); } while (0)
    if (nb) LASAD_LAUNCH1(0, 0, 1, 2);
    else if (a.norm) LASAD_LAUNCH(0, 1, 1);
    else if (a.fused_act) LASAD_LAUNCH(0, 1, 0);
    else if (a.k) LASAD_LAUNCH(1, 0, 0);
    else LASAD_LAUNCH(0, 0, 0);
#undef LASAD_LAUNCH
#undef LASAD_LAUNCH1
    return hipGetLastError();
}

hipError_t launch_forward_gated_chunk(const ForwardArgs &a, hipStream_t s) { return launch(a, nullptr, nullptr, s); }

hipError_t launch_forward_gated_norm_backward(const ForwardArgs &a, const NormBackwardArgs &nb, int *n_seg, hipStream_t s)
{
    if (!a.fused_act || a.norm || a.out_dtype != LASAD_F32) return hipErrorInvalidValue;
    return launch(a, &nb, n_seg, s);
}

}  // namespace lasad
