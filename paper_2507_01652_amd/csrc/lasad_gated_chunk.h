// Building blocks of the chunked vector-decay kernels (bf16 storage, head dim 64): tiles of 32 tokens,
// loader wavefronts that prepare a chunk's operands in LDS one chunk ahead, and compute wavefronts that
// each own 16 columns of the state for the whole sequence.
//
// With A_i[c] = prod_{s<=i} lambda_s[c] over the tokens of a chunk (1 at a row boundary),
//     Q~ = q_scale q . A,   K~ = k / A,
//     o_i   = Q~_i^T S_prev + sum_{j<=i} (Q~_i . K~_j) v_j,      S_new = diag(A_end) (S_prev + K~^T V).
//
// A compute wavefront needs nothing from the others: it takes the chunk's 32 x 32 scores, masks and splits
// them in its own accumulators (which are an operand fragment of the next MFMA once the reduction index
// is enumerated in accumulator order), multiplies them with its 16 value channels, adds Q~ S from its own
// state accumulators and updates them.  State and scores never pass through LDS, and the only barrier is
// the one per chunk that hands over the loaders' tiles.  Every compute wavefront forms the scores (18 of
// its 42 MFMAs of 16 x 16 x 32): cheaper than an exchange and a second barrier.  (Two wavefronts of 32
// columns on 32 x 32 x 16 tiles: a quarter fewer vector instructions in all, but a longer chain per chunk
// and a wavefront less per SIMD to hide it: 57 against 49 us on the large fused-layer shape.)
//
// Enumeration of the reduction indices.  An operand fragment holds, per lane group g = lane / 16, eight
// elements of the reduction index; accumulators hold rows 4 g + r of a tile.  Tokens: elements 0..3 are
// tokens 4 g + e, elements 4..7 tokens 16 + 4 g + e (two score tiles).  Key channels: the rows of the
// four state tiles are enumerated so that a lane's rows of tiles 2 s and 2 s + 1 are the eight consecutive
// channels that a 16-byte row read of the other operand gives:
//     tile 2 s + h, row 4 g + r  <->  channel 32 s + 8 g + 4 h + r.
#pragma once

#include "lasad_mfma_util.h"
#include "lasad_internal.h"

namespace lasad {
namespace gchunk {

constexpr int C = 32;                  // tokens per chunk
constexpr int D = 64;                  // head dim
// One token's row of a chunk slot: its prepared operands side by side (bf16 elements), so that everything a lane
// reads or writes of a row lies within the immediate offsets of the LDS instructions.
//
// Where a row stands.  Sixteen lanes are served together: of a 16-byte read lanes 0-3, 12-15 (rows) and 20-27 (rows 4-11,
// the next 16 bytes), of an 8-byte write sixteen rows two apart.  Conflict-free are both with rows of 16 mod 32 elements
// (an even number of 16-byte pieces, twice an odd one), rows 8-15 (mod 16) half a bank turn on and with their 16-byte
// pieces swapped in pairs, and rows from 16 on two pieces on.  Cycles an instruction (eight wavefronts, one compute
// unit): 16-byte reads 4.4, transposing reads 2.7 and 4.2, 8-byte writes 8.2; plain rows of 164 words 8.1, 4.2, 6.1 and
// 16.1.  With those the conflicts were 960 of a lone workgroup's 1780 LDS cycles a chunk of 2500, now 290 of 1110.
// 24 sequences of 24 x 24 tokens, us: tied key 23.9 -> 21.3, own key 25.4 -> 22.1, backward 39.2 -> 34.6.
constexpr int kRow = 5 * D + 16;
constexpr int kColKh = 0, kColKl = D, kColQh = 2 * D, kColQl = 3 * D, kColV = 4 * D;
template <int ROW>
struct SlotMap {
    static_assert(ROW % 32 == 16, "see above");
    static constexpr int kHalf = 16 * ROW + 144;       // from a row to the one 16 on
    static constexpr int kHalfs = 32 * ROW + 208;      // the whole slot
    static __device__ __forceinline__ int row(int r) { return (r & 15) * ROW + 64 * ((r >> 3) & 1) + kHalf * (r >> 4); }
    // 16-byte piece of row r, from the row's start on
    static __device__ __forceinline__ int piece(int r, int i) { return 8 * (i ^ ((r >> 3) & 1)); }
    // four elements from column c on (a multiple of 4) of row r, from the slot's start on
    static __device__ __forceinline__ int at(int r, int c) { return row(r) + piece(r, c >> 3) + (c & 4); }
};
constexpr int kSlot = SlotMap<kRow>::kHalfs;
constexpr int OS = 68;                 // row stride (floats) of the output tile: 272 B
constexpr float kMaxInvDecay = 1.2676506e30f;      // 2^100: largest 1 / A of a chunk (see lasad_forward_gated_chunk.hip)

__device__ __forceinline__ int state_channel(int t, int g) { return 32 * (t >> 1) + 8 * g + 4 * (t & 1); }    // of row 4 g

// A sequence cut into segments that different workgroups walk (few, long sequences), whole chunks each, the first
// `longer` of them one chunk longer than the rest (the last chunk may be short of tokens).  A segment's incoming state
// P_g is formed by a state pass and a fold before the walk; in the forward it sits in the segment's own part of the
// output tensor until the segment's first tile is stored.
struct SegPlan {
    int n_seg, chunks, longer;         // n_seg = 1: no segments
    __host__ __device__ __forceinline__ int start(int seg) const { return (seg * chunks + (seg < longer ? seg : longer)) * C; }
};

// A 64 x 64 fp32 state and a vector of 64 after it, laid out over consecutive token rows of the output tensor: float i is
// in row i / row_floats (a row: 64 elements of the output type).
struct RowState {
    float *base;                       // first row
    int64_t stride;                    // floats from row to row
    int shift;                         // log2(row_floats): 5 (bf16 rows) or 6
    __device__ __forceinline__ float *at(int i) const { return base + (i >> shift) * stride + (i & ((1 << shift) - 1)); }
};
constexpr int kRowStateTokens = 130;   // rows it needs with bf16 output (65 with fp32)

// Running products of four values along the 16 lanes of a row: x becomes the inclusive product, e the exclusive
// one (1 in lane 0).  Lanes without a DPP source keep their value.  The four chains are interleaved, so every DPP
// source was written four instructions earlier; the s_nop covers what preceded the block.
#define GCHUNK_SCAN(ctrl)                                                                         \
    "v_mul_f32_dpp %0, %0, %0 " ctrl "\n v_mul_f32_dpp %1, %1, %1 " ctrl "\n"                     \
    "v_mul_f32_dpp %2, %2, %2 " ctrl "\n v_mul_f32_dpp %3, %3, %3 " ctrl "\n"
__device__ __forceinline__ void row_scan_mul4(float (&x)[4], float (&e)[4])
{
    e[0] = e[1] = e[2] = e[3] = 1.0f;
    asm("s_nop 1\n"
        GCHUNK_SCAN("row_shr:1 row_mask:0xf bank_mask:0xf")
        GCHUNK_SCAN("row_shr:2 row_mask:0xf bank_mask:0xf")
        GCHUNK_SCAN("row_shr:4 row_mask:0xf bank_mask:0xf")
        GCHUNK_SCAN("row_shr:8 row_mask:0xf bank_mask:0xf")
        "v_mov_b32_dpp %4, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n v_mov_b32_dpp %5, %1 row_shr:1 row_mask:0xf bank_mask:0xf\n"
        "v_mov_b32_dpp %6, %2 row_shr:1 row_mask:0xf bank_mask:0xf\n v_mov_b32_dpp %7, %3 row_shr:1 row_mask:0xf bank_mask:0xf\n"
        : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(e[0]), "+v"(e[1]), "+v"(e[2]), "+v"(e[3]));
}

// sum over the eight lanes of an aligned group, in every lane
__device__ __forceinline__ float sum8(float x)
{
    x += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0xB1, 0xf, 0xf, true));    // lane ^ 1
    x += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x4E, 0xf, 0xf, true));    // lane ^ 2
    x += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x141, 0xf, 0xf, true));   // the other quad
    return x;
}

__device__ __forceinline__ void unpack4(uint2 w, float (&f)[4])
{
    f[0] = __uint_as_float(w.x << 16); f[1] = __uint_as_float(w.x & 0xffff0000u);
    f[2] = __uint_as_float(w.y << 16); f[3] = __uint_as_float(w.y & 0xffff0000u);
}

// How a loader wavefront comes by its share of a tensor's 32 rows, tokens 2 pr, 2 pr + 1 and four channels a lane (pr = lane &
// 15) of the wavefront's sixteen: read as 16 bytes a lane, two lanes a row, and turned in LDS, in rows of its own that nobody
// else touches meanwhile (no barrier).  Read like that straight from memory, 8 bytes a lane in sixteen rows, a tile takes
// a compute unit 230 ns: the address unit spends about four cycles on every row that an instruction touches.  16 bytes in 32
// rows: 123 ns.  (Whole rows, 49 ns, would have to cross wavefronts.)
template <int ROW>
struct Turn {
    using Map = SlotMap<ROW>;
    int put, get;                      // elements from the tile's slot on, without the tensor's column
    __device__ __forceinline__ Turn(int lw, int lane)
    {
        const int m = lane >> 1;
        put = Map::row(m) + Map::piece(m, 2 * lw + (lane & 1));
        get = Map::at(2 * (lane & 15), 16 * lw + 4 * (lane >> 4));
    }
    __device__ __forceinline__ void write(uint16_t *slot, int col, u32x4 x) const { *(u32x4 *)(slot + put + col) = x; }
    __device__ __forceinline__ uint2 read(const uint16_t *slot, int col, int it) const { return *(const uint2 *)(slot + get + col + it * ROW); }
    static __device__ __forceinline__ int row(int lane) { return lane >> 1; }                       // what the lane reads from memory:
    static __device__ __forceinline__ int byte(int lw, int lane) { return 32 * lw + 16 * (lane & 1); }     // row, and where in it
};

// f as bf16 hi + lo, written to one row piece of two tiles
__device__ __forceinline__ void put_pair4(uint16_t *hi, uint16_t *lo, const float (&f)[4], const SplitConst &sc)
{
    uint2 h, l;
    split2(f[0], f[1], h.x, l.x, sc);
    split2(f[2], f[3], h.y, l.y, sc);
    *(uint2 *)hi = h;
    *(uint2 *)lo = l;
}

// Which of a chunk's 32 tokens sit on a row boundary (bit = token), advance_by tokens at a time, on the scalar unit: the
// boundary positions are every W-th one, so a mask is the pattern of multiples of W shifted to the chunk's first one.
struct RowBoundaries {
    uint64_t multiples;                // bits 0, W, 2 W, ...
    int W, step, first;                // first: chunk-local index of the first boundary token (W: none further on is nearer)
    __device__ __forceinline__ void init(int start, int grid_w, int mode, int advance_by)
    {
        W = grid_w;
        multiples = 1;
        for (int k = grid_w; k < 64; k += grid_w) multiples |= 1ull << k;
        step = advance_by % grid_w;
        const int col0 = start % grid_w;                     // column of the chunk's first token
        first = mode == LASAD_RESET_LAST_COL ? grid_w - 1 - col0 : col0 ? grid_w - col0 : 0;
        if (mode == LASAD_RESET_NONE) { multiples = 0; first = 0; }
    }
    __device__ __forceinline__ uint32_t mask() const { return first < C ? (uint32_t)(multiples << first) : 0u; }
    __device__ __forceinline__ void advance()                // to the next chunk
    {
        first -= step;
        if (first < 0) first += W;
    }
    __device__ __forceinline__ void retreat()                // to the chunk before
    {
        first += step;
        if (first >= W) first -= W;
    }
};

__device__ __forceinline__ float exp_neg(float x) { return __builtin_amdgcn_exp2f(x * -1.44269504088896340736f); }

// ---- compute wavefronts --------------------------------------------------------------------------

// A lane's places in a slot for its operand reads; everything else is immediate offsets.  The forward computes those of the
// first slot once and adds from there (2 % on the fused layer); in the backward, with two loader groups, that is 5 % slower.
template <int ROW = kRow>
struct SlotPtr {
    using Map = SlotMap<ROW>;
    const uint16_t *row, *tok, *st;
    __device__ __forceinline__ SlotPtr(const uint16_t *slot, int lane)
    {
        const int l16 = lane & 15, g = lane >> 4;
        const int r = 4 * g + (l16 >> 2);
        row = slot + Map::at(l16, 8 * g);
        tok = slot + Map::at(r, 4 * (lane & 3));
        st = slot + Map::at(r, 8 * (lane & 3));
    }
    __device__ __forceinline__ SlotPtr(const SlotPtr &first, int add) : row(first.row + add), tok(first.tok + add), st(first.st + add) {}
    // rows row0 + l16 (row0: 0 or 16), elements col + 32 s + 8 g ..
    __device__ __forceinline__ Frag rows(int row0, int col, int s) const
    {
        Frag f;
        f.u = *(const uint4 *)(row + (row0 ? Map::kHalf : 0) + col + 32 * s);
        return f;
    }
    // the 32 tokens for 16 columns from col in order / for the rows of state tile t
    __device__ __forceinline__ Frag tokens(int col) const { return pair(tok + col); }
    __device__ __forceinline__ Frag state_rows(int col, int t) const { return pair(st + col + 32 * (t >> 1) + 4 * (t & 1)); }
    __device__ __forceinline__ Frag pair(const uint16_t *p) const
    {
        Frag f;
        f.h[0] = tr_read(p);
        f.h[1] = tr_read(p + Map::kHalf);
        return f;
    }
};

// two accumulator tiles as one operand fragment over their rows, bf16 hi + lo
__device__ __forceinline__ void split_tiles(const f32x4v &t0, const f32x4v &t1, Frag &hi, Frag &lo, const SplitConst &sc)
{
    uint2 h, l;
    split2(t0[0], t0[1], h.x, l.x, sc);
    split2(t0[2], t0[3], h.y, l.y, sc);
    hi.h[0] = h; lo.h[0] = l;
    split2(t1[0], t1[1], h.x, l.x, sc);
    split2(t1[2], t1[3], h.y, l.y, sc);
    hi.h[1] = h; lo.h[1] = l;
}

// causal mask of a diagonal score tile P^T (this lane: query lane & 15, keys 4 g + r)
__device__ __forceinline__ void causal_mask(f32x4v &p, int lane)
{
    const int cq = (lane & 15) - 4 * (lane >> 4);
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = r <= cq ? p[r] : 0.f;
}

}  // namespace gchunk
}  // namespace lasad
