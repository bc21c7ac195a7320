// Chunked forward for the per-head decay on the bf16 matrix cores (gfx950 MFMA), bf16 storage, head dim 64: workgroups that have a
// compute unit to themselves, and with more sequences than units walk several, one after the other.  Chunks of 64 tokens; with
// e_i = E(i) - E(chunk's start), r_i = gamma^e_i, c_j = gamma^-e_j, f_j = gamma^(e_end - e_j):
//
//     o_i   = r_i ( q_i^T S + sum_{j<=i} c_j (q_i . k_j) v_j ),      S <- r_end S + sum_j k_j (f_j v_j)^T
//
// All computed operands (scores, S, f V) are bf16 hi + lo pairs against operands that are bf16 as they are: two MFMAs each.
//
// What bounds a lone workgroup is the longest wavefront between two barriers: a wavefront issues an instruction about every eight
// cycles alone on its SIMD, and four on a SIMD one every four to five together.  So the work of a chunk is dealt to many wavefronts
// with little each, and to few instructions in all (NV value tiles of 16 channels a workgroup, 4 / NV workgroups a sequence):
//   - one wavefront copies Q and K of the chunk three (two) periods on to LDS without a register in between;
//   - loader wavefronts turn V into V, f V hi and lo one chunk ahead;
//   - store wavefronts take the output tile of the chunk before to memory (and multiply it into the decay-gradient sums): apart from
//     the loads, as a load issued after a store is waited for with it;
//   - NV state wavefronts keep 16 columns of S each in accumulators and leave S^T, hi and lo, for the next chunk;
//   - output wavefronts take one query tile of 16 tokens each (the later ones, with more keys, half of its value channels or keys).
// One barrier a chunk; everything that one role leaves for another is doubled.
//
// Measured against the kernel this one replaced (10 or 12 wavefronts, 32 x 32 tiles, loaders that also moved Q and K), us a call,
// graph replay: 16 sequences of 256 tokens 8.0 -> 5.5 (NV 1), of 576 13.4 -> 8.1, 64 of 576 14.0 -> 9.4, 96 of 256 8.6 -> 7.3 (NV 2),
// 128 of 576 14.5 -> 11.5, 192 of 576 17.7 -> 15.1 (NV 4), 256 of 576 19.0 -> 18.2; three passes of a backward, 16 of 256 11.6 -> 8.8,
// 24 of 311 14.1 -> 11.5, 80 of 311 16.9 -> 14.8.  Per chunk: 1.2 us -> 0.5 (NV 1), 0.8 (NV 2); 1.65 -> 1.4 (NV 4, from memory).
// Stores apart from the loaders, NV 4 (and non-temporal ones in a backward too): three passes of 80 sequences of 576 tokens 23.7 ->
// 19.9 us, of 512 102 -> 89, a period 3340 -> 2870 cycles; NV 2, NV 1: 40 of 576 16.0 -> 15.0, 16 of 400 11.0 -> 10.7.
// Several sequences a workgroup without a pause, against the kernel of eight wavefronts with two workgroups a unit: 512 of 576 41.1 ->
// 37.6 us, 1000 of 576 81 -> 67; three passes, 512 of 576 102 -> 89, of 1024 200 -> 159, 96 of 4096 216 -> 178.
// Counters at 512 of 576: matrix cores busy 23 % of the SIMD cycles, vector ALU 40 %, LDS 44 %, wavefronts waiting 53 % of theirs.
// Scalar registers: the variants with the decay gradient spill 40 to 54 (18 in NV 4 without it), as five roles of one function share
// both argument structures; the state and output wavefronts' loops read none of them back.
// Dropped on the way: 32-token chunks (the latency of a period, about 1000 cycles, twice); compute wavefronts that own their state
// columns and form all scores themselves, as in the vector-decay kernels (more instructions than the kernel replaced); loaders that
// move Q and K through registers (16 wavefronts, 2000 cycles a chunk in the place of 1750).
#include <stdlib.h>

#include "lasad_gated_chunk.h"
#include "lasad_forward_mfma_common.h"
#include "lasad_recurrence.h"

namespace lasad {

namespace {

using gchunk::SlotMap;
using gchunk::SlotPtr;
using gchunk::causal_mask;
using gchunk::split_tiles;
using gchunk::state_channel;

constexpr int CT = 64;                 // tokens per chunk
constexpr int D = 64;                  // head dim

typedef __attribute__((address_space(3))) void LdsVoid;
template <int I> struct Const { static constexpr int value = I; };

// ---- Q and K of a chunk, copied from memory to LDS ----
// Rows of 128 bytes one after the other, their 16-byte pieces permuted by the row (the copy leaves 64 pieces of 16 bytes in a
// row, so a row cannot be moved, but which lane fetches what is free).  With this permutation sixteen lanes that are served
// together meet no bank conflict in the operands' row reads, and two-way ones in the transposing reads of K.
constexpr int kTile = CT * D;          // elements
__device__ __forceinline__ int turned(int r)           // what the piece's index is XORed with
{
    const int x = r >> 1;
    return (x & 1) | ((x & 2) << 1) | ((x & 4) >> 1);
}

// ---- V and f V of a chunk, in padded rows ----
template <int NV>
struct Slot {
    static constexpr int V = 0, Fh = 16 * NV, Fl = 32 * NV;
    static constexpr int ROW = 48 * NV + (NV == 1 ? 0 : 16);
    using Map = SlotMap<ROW>;
    static constexpr int kHalfs = CT / 16 * Map::kHalf;
};

// boundary tokens of a chunk (gchunk::RowBoundaries, for 64 of them)
struct Boundaries {
    uint64_t multiples;
    int W, step, first;
    __device__ __forceinline__ void init(int grid_w)
    {
        W = grid_w;
        multiples = 1;
        for (int k = grid_w; k < 64; k += grid_w) multiples |= 1ull << k;
        step = CT % grid_w;
    }
    __device__ __forceinline__ void begin(int start, int mode)
    {
        const int col0 = start % W;
        first = mode == LASAD_RESET_LAST_COL ? W - 1 - col0 : col0 ? W - col0 : 0;
        if (mode == LASAD_RESET_NONE) { multiples = 0; first = 0; }
    }
    __device__ __forceinline__ uint64_t mask() const { return first < CT ? multiples << first : 0ull; }
    __device__ __forceinline__ void advance()
    {
        first -= step;
        if (first < 0) first += W;
    }
};

// Chunks whose V the loaders hold in registers, and periods that a turn of their loop has (four: 1 to 3 % slower, for those past the end).
constexpr int kPeriods = 2;
// Tokens from the walk's last one on, at the most, that a load may be asked for (and gets zeros): the loaders fetch kPeriods chunks, one
// more, and then one a period for all periods, rounded up to whole turns of kPeriods; a chunk's own rows past the end add to that.
constexpr int kPast = (2 * kPeriods + 2) * CT;

// A walk's rows of one tensor as a buffer: rows before the first and past the last are read as zero and not written, without a
// branch (their offsets leave the range, below zero as unsigned numbers: forward_scalar_chunk_fits).
struct WalkRows {
    int step;                          // bytes from row to row (negative in a reversed pass)
    int first;                         // offset of row 0
    __device__ __forceinline__ WalkRows(int64_t stride, int n) : step((int)stride), first(stride < 0 ? -(n - 1) * (int)stride : 0) {}
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const char *row0, int n, int bytes) const      // bytes: of a row
    {
        const int span = (n - 1) * (step < 0 ? -step : step) + bytes;
        return __builtin_amdgcn_make_buffer_rsrc((void *)(row0 - first), 0, span, 0x00020000);
    }
};

template <bool NT>
__device__ __forceinline__ u32x4 buf_load(__amdgpu_buffer_rsrc_t r, int off)
{
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, NT ? 2 : 0));
}
template <bool NT>
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, int off, u32x4 x)
{
    __builtin_amdgcn_raw_buffer_store_b128(x, r, off, 0, NT ? 2 : 0);
}

// Wavefronts, in this order, number modulo 4 being the SIMD: the state's, output (NV 2: the two later query tiles by value tile, 96
// sequences of 576 tokens 11.4 -> 11.0 us; NV 1: the last one by half of the keys, 16 of 576 9.2 -> 8.1), loaders, stores, copy.
// (NV 4: the SIMDs with the two short query tiles have the stores.)
constexpr int out_waves(int nv) { return nv == 2 ? 6 : nv == 1 ? 5 : 4; }
constexpr int loader_waves(int nv) { return nv == 1 ? 2 : 4; }
constexpr int store_waves(int nv) { return nv == 1 ? 1 : 2; }
constexpr int all_waves(int nv) { return nv + out_waves(nv) + loader_waves(nv) + store_waves(nv) + 1; }

template <int OUT_BF16, int NV, int DOT>
struct Shape {
    static constexpr int kOut = out_waves(NV), kLoaders = loader_waves(NV), kStore = store_waves(NV), kWaves = all_waves(NV);
    static constexpr bool O16 = OUT_BF16 && !DOT && NV == 4;               // the output tile as bf16
    static constexpr int R = NV == 4 ? (O16 ? 3 : 2) : 4;                  // Q and K slots (six for NV 1: no gain)
    static constexpr int OS = O16 ? 16 * NV / 2 + 4 : 16 * NV + 4;         // output tile's row, floats
    using SM = SlotMap<2 * D + 16>;                                        // S^T, hi and lo
    static constexpr int kStateHalfs = NV * SM::kHalf;
    static constexpr int kPart = NV == 1 ? 17 * OS : 0;                    // floats: the last query tile's first half of the keys, and a row of zeros
    static constexpr int kBytes = 2 * kPart * 4 + R * 2 * kTile * 2 + 2 * Slot<NV>::kHalfs * 2 + 2 * kStateHalfs * 2 + 2 * CT * OS * 4;
};

// The state pass of a segment plan is dealt out finer than the segments: part i of a sequence, tokens t0 .. t1 - 1.
struct StatePart {
    int t0, t1;
    __device__ __forceinline__ StatePart(const ForwardArgs &a, int i)
    {
        const int seg = i / a.seg_parts, j = i - seg * a.seg_parts, len = (a.seg_chunks + a.seg_parts - 1) / a.seg_parts;
        t0 = (seg * a.seg_chunks + min(j * len, a.seg_chunks)) * CT;
        t1 = (seg * a.seg_chunks + min((j + 1) * len, a.seg_chunks)) * CT;
    }
};

// Whether the P items of a sequence stay on one XCD: not where some XCD would then have an item more than it has compute units, while
// the chip has enough (82 sequences, three passes: 33 items on two of the XCDs, 22.6 -> 17.0 us).
__host__ __device__ __forceinline__ bool by_xcd(int64_t n_blk, int P) { return (n_blk + 7) / 8 * P <= 32 || n_blk * P > 256; }

// With m.n_pass > 1 one of several independent passes; DOT: the variant that also takes the decay-gradient sums (MultiPass::x).
template <int OUT_BF16, int NV, int DOT>
__global__ void __launch_bounds__(all_waves(NV) * 64)
forward_scalar_chunk_kernel(ForwardArgs a, MultiPass m)
{
    using SL = Slot<NV>;
    using SH = Shape<OUT_BF16, NV, DOT>;
    using SM = typename SH::SM;
    constexpr int PARTS = 4 / NV, R = SH::R, OS = SH::OS, kCompute = NV + SH::kOut;
    constexpr bool MANY = NV == 4;
    // Rows touched once: non-temporal.  The workgroups of a sequence and the passes of a backward launch share what they read through
    // the L2.
    constexpr bool NTL = !DOT && PARTS == 1;
    constexpr int kRecBytes = recurrence_lds_floats<D>() * 4;
    constexpr int kTab = CT + 4;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[SH::kBytes > kRecBytes ? SH::kBytes : kRecBytes];
    __shared__ __attribute__((aligned(16))) float tabs[2][kTab];   // gamma^-e_j of the chunk's tokens, gamma^e_end
    uint16_t *const tiles = (uint16_t *)smem;                      // [slot][Q, K]
    uint16_t *const slots = tiles + R * 2 * kTile;
    uint16_t *const states = slots + 2 * SL::kHalfs;
    float *const outs = (float *)(states + 2 * SH::kStateHalfs);
    float *const parts = outs + 2 * CT * OS;

    // A workgroup's items are whole sequences of a pass, segments, or some value channels of one; MANY: it walks several, one after
    // the other (ids gridDim.x apart) without a pause, so that only the first one's loads are waited for.  The ids of a sequence's
    // items are 8 apart: they are walked at the same time on the same XCD (ids go round the 8 XCDs).
    const int G = a.n_segments, n_blk = a.B * a.Hh * G, P = PARTS * m.n_pass;
    struct Item { int blk, vp, pass; };
    auto item = [&](int i) {
        const uint32_t id = blockIdx.x + (uint32_t)i * gridDim.x;
        if (P == 1) return Item{(int)id, 0, 0};
        if (!by_xcd(n_blk, P)) return Item{(int)(id / P), (int)(id % P % PARTS), (int)(id % P / PARTS)};
        const uint32_t grp = id / (8 * P), r = id - grp * (8 * P);
        return Item{(int)(grp * 8 + (r & 7)), (int)((r >> 3) % PARTS), (int)((r >> 3) / PARTS)};
    };
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    uint64_t todo, rest;               // items walked in chunks; those with gamma <= 0.5, where c_j could overflow
    float lg_lane = 0.f;               // log2 gamma of item `lane`
    {
        const Item it = item(MANY ? lane : 0);
        const bool mine = it.blk < n_blk && (MANY || lane == 0);
        if (mine) lg_lane = log2f(a.gamma[it.blk / G % a.Hh]);
        todo = __ballot(mine && lg_lane * (float)CT > -64.0f);
        rest = __ballot(mine) & ~todo;
    }
    auto take = [](uint64_t &left) {
        const int i = __builtin_ctzll(left);
        left &= left - 1;
        return i;
    };
    auto log_gamma = [&](int i) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(lg_lane), i)); };
    const bool multi = m.n_pass > 1;
    const int seg = G > 1 ? item(0).blk % G : 0;
    const int seg_t0 = seg * a.seg_chunks * CT;
    const int n = min(a.seg_chunks * CT, a.n_tokens - seg_t0);
    const int n_chunks = (n + CT - 1) / CT;                                        // of an item
    const int n_all = MANY ? (int)__builtin_popcountll(todo) * n_chunks : n_chunks;
    // element offset of an item's first row in a layout
    auto first_row = [&](const lasad_layout_t &l, int bh) {
        const int b = bh / a.Hh, h = bh - b * a.Hh;
        return (int64_t)b * l.stride_b + (int64_t)h * l.stride_h + (int64_t)seg_t0 * l.stride_n;
    };
    auto walk_items = [&]() {
    if (wave == SH::kWaves - 1) {
        // ===================================== the copy of Q and K =====================================
        uint64_t items = todo;
        __amdgpu_buffer_rsrc_t rq, rk;
        int off[2], step, slot = 0, left;
        auto begin = [&]() {
            const Item it = item(take(items));
            const lasad_layout_t l = multi ? m.in[it.pass] : a.in;
            const WalkRows in(l.stride_n * 2, n);
            const int64_t base = first_row(l, it.blk / G) * 2;
            rq = in.rsrc((const char *)(multi ? m.q[it.pass] : a.q) + base, n, 128);
            rk = in.rsrc((const char *)(multi ? m.k[it.pass] : a.k) + base, n, 128);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int r = 8 * e + (lane >> 3);
                off[e] = in.first + r * in.step + ((lane & 7) ^ turned(r)) * 16;
            }
            step = in.step;
            left = n_chunks;
        };
        begin();
        auto copy = [&]() {                                    // the next chunk into the next slot
            char __attribute__((address_space(3))) *const at = (char __attribute__((address_space(3))) *)(tiles + slot * 2 * kTile);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rq, (LdsVoid *)(at + i * 1024), 16, off[i & 1], 0, 0, NTL ? 2 : 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (LdsVoid *)(at + kTile * 2 + i * 1024), 16, off[i & 1], 0, 0, NTL ? 2 : 0);
                off[i & 1] += 16 * step;
            }
            slot = slot + 1 == R ? 0 : slot + 1;
            if (MANY && --left == 0 && items) begin();
        };
        constexpr int kWait = 16 * (R - 2);                    // all but the last R - 2 chunks have arrived
        for (int i = 0; i < R - 1; ++i) copy();                // (past the end: zeros)
        __builtin_amdgcn_s_waitcnt(0x0f70 | (kWait & 15) | (kWait >> 4 << 14));
        __builtin_amdgcn_s_barrier();
        for (int chunk = 0; chunk < n_all; ++chunk) {
            if (chunk + R - 1 < n_all) {
                copy();
                __builtin_amdgcn_s_waitcnt(0x0f70 | (kWait & 15) | (kWait >> 4 << 14));
            } else {
                __builtin_amdgcn_s_waitcnt(0x0f70);
            }
            __builtin_amdgcn_s_barrier();
        }
        return;
    }
    SplitConst sc;
    sc.init();

    constexpr int PC = 2 * NV;                                 // pieces of eight channels a row
    const int pc = tid % PC;
    if (wave >= kCompute + SH::kLoaders) {
        // ===================================== store wavefronts =====================================
        constexpr int SROWS = SH::kStore * 64 / PC, SIT = CT / SROWS, E = OUT_BF16 ? 2 : 4;
        const int st = tid - 64 * (kCompute + SH::kLoaders), srow = st / PC;
        struct Tile { f32x4v u[SIT], w[SIT]; };
        auto read_tile = [&](Tile &t, int p) {
#pragma unroll
            for (int i = 0; i < SIT; ++i) {
                if (SH::O16) {
                    t.u[i] = *(const f32x4v *)(outs + p * CT * OS + (srow + i * SROWS) * OS + pc * 4);
                } else {
                    const float *tile = outs + p * CT * OS + (srow + i * SROWS) * OS + pc * 8;
                    t.u[i] = *(const f32x4v *)tile;
                    t.w[i] = *(const f32x4v *)(tile + 4);
                    if (NV == 1) {
                        const int r = srow + i * SROWS;
                        const float *const more = parts + p * SH::kPart + (r < CT - 16 ? 16 : r - (CT - 16)) * OS + pc * 8;
                        t.u[i] += *(const f32x4v *)more;
                        t.w[i] += *(const f32x4v *)(more + 4);
                    }
                }
            }
        };
        // One period behind the output: before the first tile there is one that leaves the range.  Decay-gradient sums: the fourth
        // tensor's rows, two periods ahead of their tile (one: the stores before them have to be through by then).
        uint64_t s_items = todo, x_items = todo;
        __amdgpu_buffer_rsrc_t ro, rx;
        int o_off = 0, o_step = 0, s_left = n_chunks + 1, x_off = 0, x_step = 0, x_left = 0;
        int t0 = -CT;                                              // token of the tile's first row
        float *sums = nullptr;
        float acc = 0.f, e_sign = 0.f, e_add = 0.f;
        int e_before = 0;
        Boundaries s_bounds;
        u32x4 x4[2][SIT];
        auto store_begin = [&]() {
            const Item it = item(take(s_items));
            const int bh = it.blk / G;
            const lasad_layout_t l = multi ? m.out[it.pass] : a.out;
            const WalkRows out(l.stride_n * E, n);
            ro = out.rsrc((char *)(multi ? m.o[it.pass] : a.o) + first_row(l, bh) * E, n, D * E);
            o_off = out.first + srow * out.step + (it.vp * 16 * NV + pc * 8) * E;
            o_step = out.step;
            if (DOT) {
                t0 = 0;
                e_before = 0;
                e_sign = e_add = 0.f;
                sums = nullptr;
                s_bounds.begin(m.start_pos[it.pass], a.mode);
                if (m.x[it.pass]) {
                    const int e_all = cum_exp(m.x_start_pos + a.n_tokens, a.grid_w, a.mode) - cum_exp(m.x_start_pos, a.grid_w, a.mode);
                    // in a reversed pass step i applies the decay of the token walked before it, the first step somebody else's
                    const int before = is_boundary(m.start_pos[it.pass] + 1, a.grid_w, a.mode) ? 0 : 1;
                    e_sign = m.x_rev[it.pass] ? -m.x_sign[it.pass] : m.x_sign[it.pass];
                    e_add = m.x_rev[it.pass] ? m.x_sign[it.pass] * (float)(e_all + before) : 0.f;
                    sums = m.x_sums + ((int64_t)it.pass * a.B * a.Hh + bh) * kDotSlots + it.vp * SH::kStore + (st >> 6);
                }
            }
        };
        auto x_begin = [&]() {
            const Item it = item(take(x_items));
            const lasad_layout_t l = m.in[it.pass];
            const WalkRows in(l.stride_n * 2, n);
            rx = in.rsrc((const char *)(m.x[it.pass] ? m.x[it.pass] : m.v[it.pass]) + first_row(l, it.blk / G) * 2, n, 128);
            x_off = in.first + srow * in.step + it.vp * (32 * NV) + pc * 16;
            x_step = in.step;
            x_left = n_chunks;
        };
        auto x_fetch = [&](u32x4 (&x)[SIT]) {
#pragma unroll
            for (int i = 0; i < SIT; ++i) x[i] = buf_load<false>(rx, x_off + i * SROWS * x_step);
            x_off += CT * x_step;
            if (MANY && --x_left == 0 && x_items) x_begin();
        };
        auto leave_sum = [&]() {
            if (sums) {
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
                if (lane == 0) {
                    sums[0] = acc;
                    for (int i = PARTS * SH::kStore; i < kDotSlots; i += PARTS * SH::kStore) sums[i] = 0.f;
                }
            }
            acc = 0.f;                                             // (also of an item without a sum: 0 * Inf there is not the next item's)
        };
        auto stores_begin = [&]() {
            if (DOT) s_bounds.init(a.grid_w);
            store_begin();
            o_off -= CT * o_step;
            if (DOT) {
                t0 = -CT;
                x_begin();
                x_fetch(x4[1]);
            }
        };
        auto store_tile = [&](const Tile &t, int p) {              // (tile p - 1 in the order of the walk)
            uint64_t bmask = 0;
            if (DOT) bmask = s_bounds.mask();
#pragma unroll
            for (int i = 0; i < SIT; ++i) {
                const int at = o_off + i * SROWS * o_step;
                const f32x4v &u = t.u[i], &w = t.w[i];
                if (SH::O16) {
                    buf_store<true>(ro, at, __builtin_bit_cast(u32x4, u));
                } else if (OUT_BF16) {
                    buf_store<true>(ro, at, u32x4{pack2(u[0], u[1]), pack2(u[2], u[3]), pack2(w[0], w[1]), pack2(w[2], w[3])});
                } else {
                    buf_store<true>(ro, at, __builtin_bit_cast(u32x4, u));
                    buf_store<true>(ro, at + 16, __builtin_bit_cast(u32x4, w));
                }
                if (DOT) {
                    float d = 0.f;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const f32x4v &y = j < 2 ? u : w;
                        d = fmaf(__uint_as_float(x4[p][i][j] << 16), y[2 * (j & 1)], d);
                        d = fmaf(__uint_as_float(x4[p][i][j] & 0xffff0000u), y[2 * (j & 1) + 1], d);
                    }
                    const int r = srow + i * SROWS, e = r + 1 - __builtin_popcountll(bmask & (~0ull >> (63 - r)));
                    const float weight = e_sign * (float)(e_before + e) + e_add;
                    acc = (uint32_t)(t0 + r) < (uint32_t)n ? fmaf(weight, d, acc) : acc;
                }
            }
            o_off += CT * o_step;
            if (DOT) {
                if (t0 >= 0) {                                     // (the tile before the first has no rows)
                    e_before += CT - __builtin_popcountll(bmask);
                    s_bounds.advance();
                }
                t0 += CT;
            }
            if (--s_left == 0 && s_items) {
                if (DOT) leave_sum();
                store_begin();
                s_left = n_chunks;
            }
            if (DOT) x_fetch(x4[p]);
        };
        stores_begin();
        __syncthreads();
        for (int c0 = 0; c0 <= n_all; c0 += 2) {               // (pairs of periods, as the loaders)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                Tile t;
                read_tile(t, (u + 1) & 1);
                store_tile(t, u);
                if (c0 + u < n_all) __syncthreads();
            }
        }
        if (DOT) leave_sum();
        return;
    }

    if (wave >= kCompute) {
        // ===================================== loader wavefronts =====================================
        constexpr int ROWS = SH::kLoaders * 64 / PC, IT = CT / ROWS;
        const int ld = tid - 64 * kCompute, row = ld / PC;
        constexpr int PF = kPeriods;
        struct Regs { u32x4 v[IT]; } r[PF];
        // the loads' own way through the items
        uint64_t f_items = todo;
        __amdgpu_buffer_rsrc_t rv;
        int v_off, v_step, f_left;
        auto fetch_begin = [&]() {
            const Item it = item(take(f_items));
            const lasad_layout_t l = multi ? m.in[it.pass] : a.in;
            const WalkRows in(l.stride_n * 2, n);
            rv = in.rsrc((const char *)(multi ? m.v[it.pass] : a.v) + first_row(l, it.blk / G) * 2, n, 128);
            v_off = in.first + row * in.step + it.vp * (32 * NV) + pc * 16;
            v_step = in.step;
            f_left = n_chunks;
        };
        fetch_begin();
        auto fetch = [&](Regs &x) {
#pragma unroll
            for (int i = 0; i < IT; ++i) x.v[i] = buf_load<NTL>(rv, v_off + i * ROWS * v_step);
            v_off += CT * v_step;
            if (MANY && --f_left == 0 && f_items) fetch_begin();
        };
#pragma unroll
        for (int i = 0; i < PF; ++i) fetch(r[i]);
        __builtin_amdgcn_sched_barrier(0);
        const uint64_t upto = ~0ull >> (63 - row);
        const int put = SL::Map::at(row, pc * 8);
        float *const tab_at = &tabs[0][pc == 0 ? row : CT];
        // the preparation's
        Boundaries bounds;
        bounds.init(a.grid_w);
        uint64_t p_items = todo;
        int p_left;                                            // tokens from the next chunk to be prepared on
        float lg;
        auto prepare_begin = [&]() {
            const int i = take(p_items), pass = item(i).pass;
            lg = log_gamma(i);
            const int start = multi ? m.start_pos[pass] : a.start_pos;
            bounds.begin(start + seg_t0, a.mode);
            p_left = n;
        };
        prepare_begin();
        auto prepare = [&](const Regs &x, int p) {
            const uint64_t bmask = bounds.mask();
            bounds.advance();
            const int nt = min(p_left, CT);
            p_left -= CT;
            const int e_end = nt - __builtin_popcountll(bmask & (~0ull >> (CT - nt)));
            const float end = __builtin_amdgcn_exp2f((float)e_end * lg);
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const uint64_t first = i == 0 ? upto : ((1ull << (ROWS & 63)) - 1) | upto << (ROWS & 63);      // (at most two rows a thread)
                const int e = row + i * ROWS + 1 - __builtin_popcountll(bmask & first);
                const float cj = __builtin_amdgcn_exp2f(-(float)e * lg), fj = cj * end;
                uint16_t *const s = slots + p * SL::kHalfs + put + i * (ROWS / 16) * SL::Map::kHalf;
                if (pc < 2) tab_at[p * kTab + (pc == 0 ? i * ROWS : 0)] = pc == 0 ? cj : end;
                *(u32x4 *)(s + SL::V) = x.v[i];
                u32x4 hi, lo;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    uint32_t hw, lw;
                    split2(__uint_as_float(x.v[i][w] << 16) * fj, __uint_as_float(x.v[i][w] & 0xffff0000u) * fj, hw, lw, sc);
                    hi[w] = hw;
                    lo[w] = lw;
                }
                *(u32x4 *)(s + SL::Fh) = hi;
                *(u32x4 *)(s + SL::Fl) = lo;
            }
            if (MANY && p_left <= 0 && p_items) prepare_begin();
        };
        if (NV == 1 && ld < 2 * OS) parts[(ld / OS) * SH::kPart + 16 * OS + ld % OS] = 0.f;
        prepare(r[0], 0);
        fetch(r[0]);
        __syncthreads();
        // Pairs of periods: with a way out between them the compiler waits for all loads at the loop's top.  (What is past the
        // end does nothing.)
        for (int c0 = 0; c0 <= n_all; c0 += PF) {
#pragma unroll
            for (int u = 0; u < PF; ++u) {
                const int chunk = c0 + u;
                if (chunk + 1 < n_all) prepare(r[(u + 1) % PF], (u + 1) & 1);
                fetch(r[(u + 1) % PF]);
                if (chunk < n_all) __syncthreads();
            }
        }
        return;
    }

    const int l16 = lane & 15, g = lane >> 4;
    const SlotPtr<SL::ROW> sp0(slots, lane);
    if (wave < NV) {
        // ===================================== state wavefronts =====================================
        const int col = 16 * wave;                             // value channels of this wavefront in the slot
        f32x4v accS[4];                                        // S[state_channel(t, g) + r][.. + l16]
        uint64_t items = todo;
        int left;
        int64_t s_off;
        float *state_out;
        auto begin = [&]() {
            const int i = take(items);
            const Item it = item(i);
            const int bh = it.blk / G;
            s_off = (int64_t)bh * D * D + it.vp * 16 * NV + col + l16;
            left = n_chunks;
            const float *const state_in = multi ? m.state_in[it.pass] : a.state_in;
            state_out = multi ? m.state_out[it.pass] : a.state_out;
#pragma unroll
            for (int t = 0; t < 4; ++t) accS[t] = f32x4v{0.f, 0.f, 0.f, 0.f};
            if (state_in) {
                const bool undo = multi ? m.first_decay_off[it.pass] : a.first_decay_off;
                const bool at_boundary = is_boundary((multi ? m.start_pos[it.pass] : a.start_pos) + 1, a.grid_w, a.mode);
                const float s_in = undo && !at_boundary ? 1.0f / a.gamma[bh % a.Hh] : 1.0f;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) accS[t][r] = s_in * state_in[s_off + (state_channel(t, g) + r) * D];
            }
            const float lg = log_gamma(i);
            for (int sp = 0; sp < seg * a.seg_parts; ++sp) {
                const StatePart part(a, sp);
                const int de = fwd::range_exponent(a.start_pos + part.t0, a.start_pos + part.t1, a.grid_w, a.mode);
                const float dec = de == 0 ? 1.0f : __builtin_amdgcn_exp2f((float)de * lg);
                const float *u = a.seg_states + ((int64_t)bh * (G - 1) * a.seg_parts + sp) * D * D + it.vp * 16 * NV + col + l16;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) accS[t][r] = fmaf(dec, accS[t][r], u[(state_channel(t, g) + r) * D]);
            }
        };
        auto finish = [&]() {
            if (!state_out || seg != G - 1) return;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) state_out[s_off + (state_channel(t, g) + r) * D] = accS[t][r];
        };
        begin();
        uint16_t *const st_put = states + SM::row(col + l16) + SM::piece(col + l16, g);
        auto publish = [&](int p) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint2 hi, lo;
                split2(accS[t][0], accS[t][1], hi.x, lo.x, sc);
                split2(accS[t][2], accS[t][3], hi.y, lo.y, sc);
                uint16_t *const d = st_put + p * SH::kStateHalfs + 32 * (t >> 1) + 4 * (t & 1);
                *(uint2 *)d = hi;
                *(uint2 *)(d + D) = lo;
            }
        };
        // K: rows 4 g + l16 / 4 (and 16, 32, 48 on), the tiles' channels
        const int kr = 4 * g + (l16 >> 2);
        const uint16_t *const k0 = tiles + kTile + kr * D + ((lane & 3) ^ turned(kr)) * 8;
        const uint16_t *const k1 = tiles + kTile + kr * D + (((lane & 3) + 4) ^ turned(kr)) * 8;
        publish(0);
        __syncthreads();
        int slot = 0;
        auto step = [&](auto parity, bool last) {
            constexpr int p = decltype(parity)::value;
            const float end = tabs[p][CT];
#pragma unroll
            for (int t = 0; t < 4; ++t) accS[t] *= end;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const SlotPtr<SL::ROW> sp(sp0, p * SL::kHalfs + kk * 2 * SL::Map::kHalf);
                const Frag fh = sp.tokens(SL::Fh + col), fl = sp.tokens(SL::Fl + col);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint16_t *const kp = (t >> 1 ? k1 : k0) + slot + kk * 32 * D + 4 * (t & 1);
                    Frag k;
                    k.h[0] = tr_read(kp);
                    k.h[1] = tr_read(kp + 16 * D);
                    accS[t] = mfma16(k, fh, accS[t]);
                    accS[t] = mfma16(k, fl, accS[t]);
                }
            }
            if (MANY && --left == 0 && !last) {
                finish();
                begin();
            }
            if (!last) publish(p ^ 1);
            slot = slot == (R - 1) * 2 * kTile ? 0 : slot + 2 * kTile;
            __syncthreads();
        };
        for (int chunk = 0; chunk < n_all; chunk += 2) {
            step(Const<0>(), chunk + 1 == n_all);
            if (chunk + 1 < n_all) step(Const<1>(), chunk + 2 == n_all);
        }
        finish();
        return;
    }

    // ===================================== output wavefronts =====================================
    const f32x4v zero4 = {0.f, 0.f, 0.f, 0.f};
    const uint16_t *const st_get = states + SM::row(l16) + SM::piece(l16, g);
    const uint16_t *const row0 = tiles + l16 * D + (g ^ turned(l16)) * 8, *const row1 = tiles + l16 * D + ((g + 4) ^ turned(l16)) * 8;
    __syncthreads();
    // query tile QT, value tiles C0 .. C0 + CN - 1; KEYS: 3 all keys of the chunk, 1 the first half of them alone, 2 the others
    auto walk = [&](auto tile, auto first, auto count, auto keys) {
        constexpr int KEYS = decltype(keys)::value;
        constexpr int QT = decltype(tile)::value, C0 = decltype(first)::value, CN = decltype(count)::value;
        int slot = 0;
        auto step = [&](auto parity) {
            constexpr int p = decltype(parity)::value;
            f32x4v pt[4] = {zero4, zero4, zero4, zero4}, o[CN];        // P^T[j][i] of the key tiles, O^T[n][i]
#pragma unroll
            for (int c = 0; c < CN; ++c) o[c] = zero4;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const uint16_t *const rows = (s ? row1 : row0) + slot;
                Frag q;
                q.u = *(const uint4 *)(rows + QT * 16 * D);
#pragma unroll
                for (int kt = 0; kt <= QT; ++kt) {
                    if (!(KEYS >> kt / 2 & 1)) continue;
                    Frag k;
                    k.u = *(const uint4 *)(rows + kTile + kt * 16 * D);
                    pt[kt] = mfma16(k, q, pt[kt]);
                }
#pragma unroll
                for (int c = 0; c < CN; ++c) {
                    if (!(KEYS & 2)) continue;
                    Frag sh, sl;
                    sh.u = *(const uint4 *)(st_get + p * SH::kStateHalfs + (C0 + c) * SM::kHalf + 32 * s);
                    sl.u = *(const uint4 *)(st_get + p * SH::kStateHalfs + (C0 + c) * SM::kHalf + D + 32 * s);
                    o[c] = mfma16(sh, q, o[c]);
                    o[c] = mfma16(sl, q, o[c]);
                }
            }
            const float osc = a.q_scale * __builtin_amdgcn_rcpf(tabs[p][16 * QT + l16]);
#pragma unroll
            for (int kt = 0; kt <= QT; ++kt)
                if (KEYS >> kt / 2 & 1) pt[kt] *= *(const f32x4v *)&tabs[p][16 * kt + 4 * g];
            if (KEYS >> QT / 2 & 1) causal_mask(pt[QT], lane);
#pragma unroll
            for (int kk = 0; kk <= QT / 2; ++kk) {
                if (!(KEYS >> kk & 1)) continue;
                const SlotPtr<SL::ROW> sk(sp0, p * SL::kHalfs + kk * 2 * SL::Map::kHalf);
                Frag ph, pl;
                split_tiles(pt[2 * kk], pt[2 * kk + 1], ph, pl, sc);   // (keys past the query tile: zero)
#pragma unroll
                for (int c = 0; c < CN; ++c) {
                    const Frag v = sk.tokens(SL::V + 16 * (C0 + c));
                    o[c] = mfma16(v, ph, o[c]);
                    o[c] = mfma16(v, pl, o[c]);
                }
            }
            if (SH::O16) {
                uint16_t *tile_at = (uint16_t *)outs + (p * CT + 16 * QT + l16) * 2 * OS + 4 * g;
#pragma unroll
                for (int c = 0; c < CN; ++c) {
                    o[c] *= osc;
                    *(uint2 *)(tile_at + 16 * (C0 + c)) = make_uint2(pack2(o[c][0], o[c][1]), pack2(o[c][2], o[c][3]));
                }
            } else {
                float *tile_at = (KEYS == 1 ? parts + p * SH::kPart : outs + p * CT * OS + 16 * QT * OS) + l16 * OS + 4 * g;
#pragma unroll
                for (int c = 0; c < CN; ++c) *(f32x4v *)(tile_at + 16 * (C0 + c)) = o[c] * osc;
            }
            slot = slot == (R - 1) * 2 * kTile ? 0 : slot + 2 * kTile;
            __syncthreads();
        };
        for (int chunk = 0; chunk < n_all; chunk += 2) {
            step(Const<0>());
            if (chunk + 1 < n_all) step(Const<1>());
        }
    };
    const int w = wave - NV;
    const Const<3> all;
    if constexpr (NV == 1) {
        if (w == 0) walk(Const<0>(), Const<0>(), Const<1>(), all);
        else if (w == 1) walk(Const<1>(), Const<0>(), Const<1>(), all);
        else if (w == 2) walk(Const<2>(), Const<0>(), Const<1>(), all);
        else if (w == 3) walk(Const<3>(), Const<0>(), Const<1>(), Const<1>());
        else walk(Const<3>(), Const<0>(), Const<1>(), Const<2>());
    } else if constexpr (NV == 2) {
        if (w == 0) walk(Const<0>(), Const<0>(), Const<2>(), all);
        else if (w == 1) walk(Const<1>(), Const<0>(), Const<2>(), all);
        else if (w == 2) walk(Const<2>(), Const<0>(), Const<1>(), all);
        else if (w == 3) walk(Const<2>(), Const<1>(), Const<1>(), all);
        else if (w == 4) walk(Const<3>(), Const<0>(), Const<1>(), all);
        else walk(Const<3>(), Const<1>(), Const<1>(), all);
    } else {
        if (w == 0) walk(Const<0>(), Const<0>(), Const<NV>(), all);
        else if (w == 1) walk(Const<1>(), Const<0>(), Const<NV>(), all);
        else if (w == 2) walk(Const<2>(), Const<0>(), Const<NV>(), all);
        else walk(Const<3>(), Const<0>(), Const<NV>(), all);
    }
    };
    if (todo) walk_items();
    if (!rest) return;
    // The fp32 recurrence, a whole sequence by four wavefronts, as many at a time as there are wavefronts for.  (One after the other: 512
    // sequences of 576 tokens 462 us, up to three at a time 221.  Against the kernels of eight and twelve wavefronts that had these
    // calls before, all heads such: forward 16 of 256 98 -> 85, 200 of 256 105 -> 92, 512 of 576 240 -> 221; three passes 16 of 256
    // 104 -> 97, 96 of 576 246 -> 235, 200 of 256 210 -> 129, 512 of 576 780 -> 589; 300 of 256 227 -> 232, one head in eight such 217 ->
    // 230: there a workgroup of four items has one for a second round.)
    constexpr int kSide = MANY ? SH::kWaves / (kRecThreads / 64) : 1;
    static_assert(kSide * kRecBytes <= (int)sizeof(smem), "a block of LDS for each");
    __syncthreads();
    const int side = wave / (kRecThreads / 64);
    if (side >= kSide || seg != 0) return;
    for (;;) {
        uint64_t mine = rest;
        for (int i = 0; i < side; ++i) mine &= mine - 1;       // (of none: none)
        if (!mine) return;
        const Item it = item(take(mine));
        if (it.vp != 0) return;                                // (a single item)
        ForwardArgs s = a;
        if (multi) {
            s.q = m.q[it.pass]; s.k = m.k[it.pass]; s.v = m.v[it.pass]; s.o = m.o[it.pass];
            s.in = m.in[it.pass]; s.out = m.out[it.pass]; s.start_pos = m.start_pos[it.pass];
            s.state_in = m.state_in[it.pass]; s.state_out = m.state_out[it.pass]; s.first_decay_off = m.first_decay_off[it.pass];
        }
        float *const lds = (float *)(smem + side * kRecBytes);
        const int rt = tid & (kRecThreads - 1);
        if (DOT) {
            fwd::recurrence_with_dot<OUT_BF16, true>(s, m, it.pass, it.blk / G, lds, rt);
            if (!m.x[it.pass]) {                               // (as many barriers as the passes with a sum)
                __syncthreads();
                __syncthreads();
            }
        } else {
            recurrence_sequence<D, 1, OUT_BF16, 0, true>(s, it.blk / G, lds, RecNoHook(), rt);
        }
        __syncthreads();
        for (int i = 0; i < kSide; ++i) rest &= rest - 1;
    }
}

// State pass of the segment plan: what a segment (all but the last) adds to the state, gamma^(E(end) - E(j)) k_j v_j^T summed over
// its tokens (bound by memory; a workgroup of four wavefronts that met at two barriers a chunk took 54 us a call where this one
// takes 36, 12 sequences of 4096 tokens in two segments; 96 of 4096 87 -> 69, and 64 with two workgroups a segment).  Weights from
// the segment's end on are at most 1, so nothing is ever rescaled, and a wavefront needs no other: it walks a quarter of the
// segment's chunks of 32 tokens in a slot of its own, all 64 x 64 of the state in its accumulators, without a barrier; the four
// states are added up at the end.
constexpr int kStateRow = 3 * D + 16;          // K, f V hi, lo
constexpr int kStateSlot = SlotMap<kStateRow>::kHalfs;
__global__ void __launch_bounds__(256, 2)
scalar_segment_state_kernel(ForwardArgs a)
{
    using Map = SlotMap<kStateRow>;
    constexpr int C = 32, kK = 0, kFh = D, kFl = 2 * D;
    __shared__ __attribute__((aligned(16))) unsigned char lds[4 * D * D * 4 > 4 * kStateSlot * 2 ? 4 * D * D * 4 : 4 * kStateSlot * 2];
    const int n_parts = (a.n_segments - 1) * a.seg_parts;
    const int bh = blockIdx.x / n_parts, part_i = blockIdx.x - bh * n_parts;
    const int b = bh / a.Hh, h = bh - b * a.Hh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const StatePart part(a, part_i);
    // chunks of 32 tokens of this wavefront (all full)
    const int n_chunks = (part.t1 - part.t0) / C, c_lo = n_chunks * wave / 4, c_hi = n_chunks * (wave + 1) / 4;
    const int64_t base = (int64_t)b * a.in.stride_b + (int64_t)h * a.in.stride_h + (int64_t)(part.t0 + c_lo * C) * a.in.stride_n;
    const int lr = lane >> 3, lc = lane & 7;       // rows r0 .. of a chunk: eight lanes a row, eight rows an instruction
    const int64_t step = 8 * a.in.stride_n, lane_off = lr * a.in.stride_n + lc * 8;
    const uint16_t *gk = (const uint16_t *)a.k + base + lane_off, *gv = (const uint16_t *)a.v + base + lane_off;
    u32x4 rk[4], rv[4];
    auto fetch = [&]() {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            rk[i] = *(const u32x4 *)(gk + i * step);
            rv[i] = *(const u32x4 *)(gv + i * step);
        }
        gk += 4 * step; gv += 4 * step;
    };
    if (c_lo < c_hi) fetch();
    __builtin_amdgcn_sched_barrier(0);
    const float lg = log2f(a.gamma[h]);
    SplitConst sc;
    sc.init();
    const int start = a.start_pos + part.t0 + c_lo * C;
    gchunk::RowBoundaries bounds;
    bounds.init(start, a.grid_w, a.mode, C);
    int to_end = fwd::range_exponent(start, a.start_pos + part.t1, a.grid_w, a.mode);     // exponent of the chunk's start
    uint16_t *const slot = (uint16_t *)lds + wave * kStateSlot;
    const SlotPtr<kStateRow> sp(slot, lane);
    f32x4v acc[4][4];                              // [key tile][value tile]
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[t][u] = f32x4v{0.f, 0.f, 0.f, 0.f};
    for (int c = c_lo; c < c_hi; ++c) {
        const uint32_t bmask = bounds.mask();
        bounds.advance();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 8 * i + lr;
            const int e = r + 1 - __builtin_popcount(bmask & (0xffffffffu >> (31 - r)));
            const float f = __builtin_amdgcn_exp2f((float)(to_end - e) * lg);
            uint16_t *const p = slot + Map::row(r) + Map::piece(r, lc);
            *(u32x4 *)(p + kK) = rk[i];
            u32x4 hi, lo;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t hw, lw;
                split2(__uint_as_float(rv[i][w] << 16) * f, __uint_as_float(rv[i][w] & 0xffff0000u) * f, hw, lw, sc);
                hi[w] = hw;
                lo[w] = lw;
            }
            *(u32x4 *)(p + kFh) = hi;
            *(u32x4 *)(p + kFl) = lo;
        }
        to_end -= C - __builtin_popcount(bmask);
        if (c + 1 < c_hi) fetch();
        Frag fh[4], fl[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) { fh[u] = sp.tokens(kFh + 16 * u); fl[u] = sp.tokens(kFl + 16 * u); }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const Frag k = sp.state_rows(kK, t);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[t][u] = mfma16(k, fh[u], acc[t][u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[t][u] = mfma16(k, fl[u], acc[t][u]);
        }
    }
    float *const sAcc = (float *)lds;              // [wave][64][64]
    __syncthreads();
    float *const mine = sAcc + wave * D * D;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[(state_channel(t, g) + r) * D + 16 * u + l16] = acc[t][u][r];
    __syncthreads();
    float *const out = a.seg_states + ((int64_t)bh * n_parts + part_i) * D * D;
    for (int i = threadIdx.x * 4; i < D * D; i += 1024) {
        const f32x4v *const p = (const f32x4v *)(sAcc + i);
        *(f32x4v *)(out + i) = (p[0] + p[D * D / 4]) + (p[2 * (D * D / 4)] + p[3 * (D * D / 4)]);
    }
}

}  // namespace

// The rows of a walk, and those past its end that loads are asked for (kPast), within 2^31 bytes.
bool forward_scalar_chunk_fits(const ForwardArgs &a)
{
    auto ok = [&](const lasad_layout_t &l, int elt) {
        return (l.stride_n < 0 ? -l.stride_n : l.stride_n) * elt < ((int64_t)1 << 31) / (a.n_tokens + kPast) - 4;
    };
    return ok(a.in, 2) && ok(a.out, a.out_dtype == LASAD_BF16 ? 2 : 4);
}

hipError_t launch_scalar_segment_state(const ForwardArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(scalar_segment_state_kernel, dim3((unsigned)((int64_t)a.B * a.Hh * (a.n_segments - 1) * a.seg_parts)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// As many workgroups a sequence (or segment) as still get a compute unit each (all of a sequence are on one XCD, of 32 units).  (64
// sequences of 576 tokens, NV 4, 2, 1: 14.1, 10.8, 9.4 us; 96 of 576: 14.4, 11.0, 16.4; 192 of 576: 15.0, 20.1.)
hipError_t launch_forward_scalar_chunk(const ForwardArgs &a, const MultiPass &m, hipStream_t s)
{
    if (a.d != D || a.io_dtype != LASAD_BF16 || a.n_tokens < 1 || (m.n_pass > 1 && a.n_segments != 1)) return hipErrorInvalidValue;
    const int64_t n_blk = (int64_t)a.B * a.Hh * a.n_segments;
    static const int split_env = [] { const char *e = getenv("LASAD_SPLIT"); return e ? atoi(e) : 0; }();
    const int split = split_env == 1 || split_env == 2 || split_env == 4 ? split_env
                      : (n_blk + 7) / 8 * m.n_pass <= 8 ? 4 : (n_blk + 7) / 8 * m.n_pass <= 16 ? 2 : 1;
    const int P = split * m.n_pass;
    int64_t n_wg = P > 1 && by_xcd(n_blk, P) ? (n_blk + 7) / 8 * 8 * P : n_blk * P;
    // A workgroup for each compute unit walks its sequences one after the other (at most 64: a lane each).
    if (split == 1 && a.n_segments == 1 && n_wg > 256) n_wg = n_wg <= 256 * 64 ? 256 : (n_wg + 511) / 512 * 8;
    if (n_wg > 0x7fffffff) return hipErrorInvalidValue;
    const bool dot = m.n_pass > 1 && (m.x[0] || m.x[1] || m.x[2]);
    const bool out16 = a.out_dtype == LASAD_BF16;
#define LASAD_LAUNCH(O, V, X) hipLaunchKernelGGL((forward_scalar_chunk_kernel<O, V, X>), dim3((unsigned)n_wg), dim3(all_waves(V) * 64), 0, s, a, m)
#define LASAD_LAUNCH1(V) do { \
        if (dot) { if (out16) LASAD_LAUNCH(1, V, 1); else LASAD_LAUNCH(0, V, 1); } \
        else { if (out16) LASAD_LAUNCH(1, V, 0); else LASAD_LAUNCH(0, V, 0); } } while (0)
    if (split == 4) LASAD_LAUNCH1(1);
    else if (split == 2) LASAD_LAUNCH1(2);
    else LASAD_LAUNCH1(4);
#undef LASAD_LAUNCH1
#undef LASAD_LAUNCH
    return hipGetLastError();
}

}  // namespace lasad
