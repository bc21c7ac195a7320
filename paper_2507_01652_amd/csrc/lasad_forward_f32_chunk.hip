// Chunked scalar-decay forward for fp32 storage, head dim 64, on the fp32 matrix instruction
// v_mfma_f32_16x16x4_f32 (fp32 operands and sums: nothing is rounded to a shorter type).
//
// Over a chunk of 16 tokens, with e_i the number of decaying steps among its first i + 1 tokens,
//     o_i   = gamma^e_i q_i^T S_prev + sum_{j<=i} gamma^(e_i - e_j) (q_i . k_j) v_j
//     S_new = gamma^e_end S_prev     + sum_j      gamma^(e_end - e_j) k_j v_j^T.
// Every exponent is an integer from 0 to 16 and every power is used as it stands (none is a reciprocal), so any gamma goes
// this way, zero included; the 17 powers of a head are products in fp64, rounded once.
//
// A workgroup of four wavefronts walks a sequence; a wavefront owns 16 value channels, and its accumulators hold those
// columns of the state for the whole sequence.  Accumulator rows 4 g + r (g = lane / 16) of a tile are at the same time
// the A operand's reduction index of the next product when that is enumerated as 16 t + 4 g + r, so neither state nor scores
// pass through LDS; every wavefront forms the scores itself (16 of its 52 matrix instructions a chunk: cheaper than an
// exchange and a second barrier).  q, k and v go through LDS, 32 tokens a barrier, doubled, the next 32 in flight
// in registers.
//
// Bound by the chain from chunk to chunk on the compute units that have a sequence: 52 matrix instructions of 32 cycles a
// chunk and SIMD (0.8 us) and the LDS reads, decay and mask between them; 1.7 us a chunk in all, 0.5 of a chunk that is only
// taken into the state.  So few sequences are dealt to several workgroups each (Parts).  96 sequences of 256
// tokens: 22 us a call (27 with one workgroup each), 56 with the token-serial kernel (lasad_scan.h), which is left to the vector
// decay, to bf16 storage and to up to four tokens of few sequences; distance from fp64 results the same.  (The scores in
// wavefronts of their own beside those with the state: 31 in the place of 27; a test in the loop for steps without output: 36.)
#include "lasad_gated_chunk.h"

namespace lasad {

namespace {

constexpr int D = 64;
constexpr int T = 32;                  // tokens per barrier: gchunk::RowBoundaries counts in these
constexpr int kThreads = 256;
constexpr int RS = D + 4;              // row stride of the staged tiles: 16-byte reads of 16 rows fall on different banks
static_assert(T == gchunk::C, "row boundaries are counted 32 tokens at a time");

__device__ __forceinline__ f32x4v mfma_f32(float a, float b, f32x4v acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
}

// A sequence dealt to several workgroups: part p outputs steps first[p] .. first[p + 1] - 1 (of T tokens) and has to form the
// state before them by itself, from the steps before, in the same order and with the same operations as the part that outputs those.
constexpr int kMaxParts = 4;
struct Parts { int n, first[kMaxParts + 1]; };

template <int PARTS>
__global__ void __launch_bounds__(kThreads, PARTS ? 1 : 3)
forward_f32_chunk_kernel(ForwardArgs a, Parts parts)
{
    __shared__ __attribute__((aligned(16))) float tiles[2][3][T * RS];      // q, k, v
    __shared__ float pw[17];                                                // gamma^0 .. gamma^16
    const int bh = PARTS ? blockIdx.x / parts.n : blockIdx.x, part = PARTS ? blockIdx.x - bh * parts.n : 0;
    const int b = bh / a.Hh, h = bh - b * a.Hh;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l16 = lane & 15, g = lane >> 4;
    const int n = a.n_tokens;
    const int first = PARTS ? parts.first[part] : 0, n_steps = PARTS ? parts.first[part + 1] : (n + T - 1) / T;      // its steps

    if (tid < 17) {
        const double gm = a.gamma[h];
        double p = 1.0;
        for (int i = 0; i < tid; ++i) p *= gm;
        pw[tid] = (float)p;
    }

    // staging: thread = token tid / 16 (+ 16), channels 4 (tid % 16) ..
    const int srow = tid >> 4, scol = (tid & 15) * 4;
    const int64_t in_base = (int64_t)b * a.in.stride_b + (int64_t)h * a.in.stride_h + scol;
    const float *src[3] = {(const float *)a.q + in_base, (const float *)a.k + in_base, (const float *)a.v + in_base};
    f32x4v stage[3][2];
    auto fetch = [&](int step) {                   // (rows past the end re-read the last token)
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int64_t off = (int64_t)min(step * T + srow + 16 * it, n - 1) * a.in.stride_n;
#pragma unroll
            for (int x = 0; x < 3; ++x) stage[x][it] = *(const f32x4v *)(src[x] + off);
        }
    };
    auto put = [&](int step) {                     // rows past the end: zero
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const bool live = step * T + srow + 16 * it < n;
#pragma unroll
            for (int x = 0; x < 3; ++x)
                *(f32x4v *)&tiles[step & 1][x][(srow + 16 * it) * RS + scol] = live ? stage[x][it] : f32x4v{0.f, 0.f, 0.f, 0.f};
        }
    };

    const int col0 = 16 * wave;
    const int64_t s_off = (int64_t)bh * D * D + col0 + l16;
    f32x4v S[4];                                   // S[16 t + 4 g + r][col0 + l16]
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) S[t][r] = a.state_in ? a.state_in[s_off + (16 * t + 4 * g + r) * D] : 0.f;

    gchunk::RowBoundaries bounds;
    bounds.init(a.start_pos, a.grid_w, a.mode, T);
    float *const o_lane = (float *)a.o + (int64_t)b * a.out.stride_b + (int64_t)h * a.out.stride_h + col0 + 4 * g;

    // tokens of a step that decay (a row past the end does not)
    auto decaying = [&](int step) {
        uint32_t decays = ~bounds.mask();
        bounds.advance();
        if (n - step * T < T) decays &= (1u << (n - step * T)) - 1;
        if (step == 0 && a.first_decay_off) decays &= ~1u;
        return decays;
    };
    // S[c][n] <- gamma^e_end S + sum_j K[j][c] gamma^(e_end - e_j) V[j][n] over a chunk
    auto update = [&](const float *tk, float (&v)[4], int e_end, const int (&e_j)[4]) {
        const float r_end = pw[e_end];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] *= pw[e_end - e_j[r]];
#pragma unroll
        for (int t = 0; t < 4; ++t) S[t] *= r_end;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < 4; ++t) S[t] = mfma_f32(tk[(4 * g + r) * RS + 16 * t + l16], v[r], S[t]);
    };

    fetch(first);
    if (PARTS && first > 0) {                      // the state before the part: k and v only (full steps)
        f32x4v before[2][2];
        auto fetch_kv = [&](int step) {
#pragma unroll
            for (int it = 0; it < 2; ++it)
#pragma unroll
                for (int x = 0; x < 2; ++x) before[x][it] = *(const f32x4v *)(src[1 + x] + (int64_t)(step * T + srow + 16 * it) * a.in.stride_n);
        };
        auto put_kv = [&](int step) {
#pragma unroll
            for (int it = 0; it < 2; ++it)
#pragma unroll
                for (int x = 0; x < 2; ++x) *(f32x4v *)&tiles[step & 1][1 + x][(srow + 16 * it) * RS + scol] = before[x][it];
        };
        fetch_kv(0);
        put_kv(0);
        fetch_kv(min(1, first - 1));
        __syncthreads();
        for (int step = 0; step < first; ++step) {
            if (step + 1 < first) {
                put_kv(step + 1);
                fetch_kv(min(step + 2, first - 1));
            }
            const uint32_t decays = decaying(step);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const float *tk = &tiles[step & 1][1][16 * half * RS], *tv = &tiles[step & 1][2][16 * half * RS + col0];
                const uint32_t dm = (decays >> (16 * half)) & 0xffffu;
                int e_j[4];
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    e_j[r] = __builtin_popcount(dm & ((2u << (4 * g + r)) - 1));
                    v[r] = tv[(4 * g + r) * RS + l16];
                }
                update(tk, v, __builtin_popcount(dm), e_j);
            }
            __syncthreads();
        }
    }
    put(first);
    if (first + 1 < n_steps) fetch(first + 1);
    __syncthreads();
    for (int step = first; step < n_steps; ++step) {
        if (step + 1 < n_steps) {
            put(step + 1);
            if (step + 2 < n_steps) fetch(step + 2);
        }
        const int left = n - step * T;
        const uint32_t decays = decaying(step);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (half * 16 >= left) break;
            const float *tq = &tiles[step & 1][0][16 * half * RS], *tk = &tiles[step & 1][1][16 * half * RS];
            const float *tv = &tiles[step & 1][2][16 * half * RS + col0];
            const uint32_t dm = (decays >> (16 * half)) & 0xffffu;
            const int e_end = __builtin_popcount(dm);
            const int e_i = __builtin_popcount(dm & ((2u << l16) - 1));
            int e_j[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) e_j[r] = __builtin_popcount(dm & ((2u << (4 * g + r)) - 1));
            // ---- scores P^T[j][i] = sum_c K[j][c] Q[i][c], and O^T[n][i] = sum_c S[c][n] Q[i][c]: two chains each ----
            f32x4v p0 = {0.f, 0.f, 0.f, 0.f}, p1 = p0, o0 = p0, o1 = p0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const f32x4v q = *(const f32x4v *)&tq[l16 * RS + 16 * t + 4 * g];
                const f32x4v k = *(const f32x4v *)&tk[l16 * RS + 16 * t + 4 * g];
                p0 = mfma_f32(k[0], q[0], p0);
                o0 = mfma_f32(S[t][0], q[0], o0);
                p1 = mfma_f32(k[1], q[1], p1);
                o1 = mfma_f32(S[t][1], q[1], o1);
                p0 = mfma_f32(k[2], q[2], p0);
                o0 = mfma_f32(S[t][2], q[2], o0);
                p1 = mfma_f32(k[3], q[3], p1);
                o1 = mfma_f32(S[t][3], q[3], o1);
            }
            float v[4];                            // V[4 g + r][col0 + l16]
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = tv[(4 * g + r) * RS + l16];
            // ---- decay and causal mask (this lane: query l16, keys 4 g + r) ----
            const float r_i = pw[e_i];
            f32x4v o = (o0 + o1) * r_i, p = p0 + p1;
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = 4 * g + r <= l16 ? p[r] * pw[max(e_i - e_j[r], 0)] : 0.f;
            // ---- O^T[n][i] += sum_j V[j][n] P^T[j][i] ----
            uint32_t top = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) top = max(top, __float_as_uint(v[r]) & 0x7fffffffu);
            if (__builtin_expect(__any(top >= 0x7f800000u), 0)) {
                // an infinity or NaN among the values: its zero score would still make NaN of the queries before it
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const float pj = __shfl(p[j & 3], 16 * (j >> 2) + l16);
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[r] = j <= l16 ? fmaf(tv[j * RS + 4 * g + r], pj, o[r]) : o[r];
                }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) o = mfma_f32(v[r], p[r], o);
            }
            update(tk, v, e_end, e_j);
            const int tok = step * T + 16 * half + l16;
            if (tok < n) *(f32x4v *)(o_lane + (int64_t)tok * a.out.stride_n) = o * a.q_scale;
        }
        __syncthreads();
    }
    if (a.state_out && (!PARTS || part == parts.n - 1)) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) a.state_out[s_off + (16 * t + 4 * g + r) * D] = S[t][r];
    }
}

// As many parts as leave every workgroup a compute unit, dealt so that they end together.  us a call, one part -> parts: 12
// sequences of 256 tokens 27.2 -> 16.6 (four), of 1024 97 -> 52; 60 of 256 27.5 -> 18.3, of 1024 98 -> 57; 96 and 128 (two)
// of 256 28.5 -> 22.2 and 24.1, of 1024 98 -> 77.  Two parts in the place of four: 12 of 256 20.1, of 1024 70.
Parts deal(int64_t n_seq, int n_steps)
{
    constexpr float ratio = 0.35f;                 // of a step without output to one with it (0.2 and 0.5: up to 3 and 15 % slower)
    int g = (int)(256 / n_seq);
    if (g > kMaxParts) g = kMaxParts;
    if (g > n_steps / 2) g = n_steps / 2;
    if (g < 2) return Parts{1, {0, n_steps}};
    Parts p{g, {0}};
    for (float time = (float)n_steps / g;; time += 0.25f) {
        for (int i = 0; i < g; ++i) {
            const int more = (int)(time - ratio * p.first[i]);
            p.first[i + 1] = p.first[i] + (more > 0 ? more : 0);
            if (p.first[i + 1] > n_steps) p.first[i + 1] = n_steps;
        }
        if (p.first[g] == n_steps) break;
    }
    while (p.n > 1 && p.first[p.n - 1] == n_steps) --p.n;
    return p;
}

}  // namespace

hipError_t launch_forward_f32_chunk(const ForwardArgs &a, hipStream_t s)
{
    if (a.d != D || a.io_dtype != LASAD_F32 || a.out_dtype != LASAD_F32 || a.n_tokens < 1 || a.lam) return hipErrorInvalidValue;
    const int64_t n_seq = (int64_t)a.B * a.Hh;
    if (n_seq > 0x7fffffff) return hipErrorInvalidValue;
    // (a part reads the incoming state when another may have written the final one: not into the same memory)
    const float *in = a.state_in, *out = a.state_out;
    const bool in_place = in && out && in < out + n_seq * D * D && out < in + n_seq * D * D;
    const Parts parts = in_place ? Parts{1, {0}} : deal(n_seq, (a.n_tokens + T - 1) / T);
    if (parts.n > 1) hipLaunchKernelGGL(forward_f32_chunk_kernel<1>, dim3((unsigned)(n_seq * parts.n)), dim3(kThreads), 0, s, a, parts);
    else hipLaunchKernelGGL(forward_f32_chunk_kernel<0>, dim3((unsigned)n_seq), dim3(kThreads), 0, s, a, parts);
    return hipGetLastError();
}

}  // namespace lasad
