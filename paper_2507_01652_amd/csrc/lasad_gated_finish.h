// The last step of the vector-decay backward where dq and dk went through the workspace in fp32 (the token-serial walks,
// and sequences that the chunked kernels hand over to them):
//     r = q dq - k dk,   dlam_t = (boundary or first token ? 0 : (sum_{i >= t} r_i) / lambda_t) - (tied key: dk_t),
// and the stores of dq, dk, dlam in the caller's type (lasad_backward_gated.hip has the derivation).
#pragma once

#include "lasad_internal.h"

namespace lasad {

constexpr int kFinBlock = 64;          // tokens per step

template <int CH>
constexpr int finish_lds_floats() { return kFinBlock * (CH + 4) + 4 * CH + CH; }

// 16 CH threads walk tokens t_lo .. t_hi - 1 of sequence bh in blocks of 64 from the last block to the first,
// every thread holding four channels (of CH from ch0 on) of one token (16-byte loads; the next block's loads are in
// flight while this one is worked on).  Per block: r = q dq - k dk into LDS, suffix sums down the
// block's tokens per channel (four 16-token quarters side by side, then their totals), outputs,
// and the block's total joins the carry.  Every input is read once; the order of all sums is fixed.
// (fp64 sums were tried: no gain in accuracy, the error left is that of the fp32 dq and dk.)
template <int IN_BF16, int OUT_BF16, int CH>
struct FinishWalk {
    typedef float f4 __attribute__((ext_vector_type(4)));
    static constexpr int LPR = CH / 4;     // threads per token
    struct Item { f4 q, k, lam, dq, dk, dact; };     // dact: d(activation)/d(input) of q, fused activations only

    const GatedBackwardArgs &a;
    const float *dq32, *dk32;
    int tid, row, c4l;
    int64_t in_base, g_base, w_base, w_stride_n;

    __device__ __forceinline__ FinishWalk(const GatedBackwardArgs &args, const float *dq, const float *dk, int bh, int ch0)
        : a(args), dq32(dq), dk32(dk)
    {
        const int b = bh / a.Hh, h = bh - b * a.Hh;
        tid = threadIdx.x;
        row = tid / LPR;
        c4l = (tid % LPR) * 4;
        const int c4 = ch0 + c4l;
        in_base = (int64_t)b * a.in.stride_b + (int64_t)h * a.in.stride_h + c4;
        g_base = (int64_t)b * a.grad.stride_b + (int64_t)h * a.grad.stride_h + c4;
        w_base = ((int64_t)b * a.n_tokens * a.Hh + h) * a.d + c4;        // workspace: [B][n][Hh][d] fp32
        w_stride_n = (int64_t)a.Hh * a.d;
    }
    __device__ __forceinline__ f4 in4(const void *p, int t) const
    {
        const int64_t i = in_base + (int64_t)t * a.in.stride_n;
        if (IN_BF16) {
            const uint2 w = *(const uint2 *)((const uint16_t *)p + i);
            return f4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u),
                      __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u)};
        }
        return *(const f4 *)((const float *)p + i);
    }
    __device__ __forceinline__ void load(int t, Item &it) const
    {
        it.q = in4(a.q, t);
        it.lam = in4(a.lam, t);
        if (a.fused_act) {                 // q = SiLU(x), SiLU'(x) = s (1 + x (1 - s)) with s = sigmoid(x); lambda = sigmoid(z)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = it.q[e], sg = sigmoid_f32(x);
                it.q[e] = x * sg;
                it.dact[e] = sg * (1.0f + x * (1.0f - sg));
                it.lam[e] = sigmoid_f32(it.lam[e]);
            }
        }
        if (a.k) it.k = in4(a.k, t);
        else it.k = f4{1.0f, 1.0f, 1.0f, 1.0f} - it.lam;
        it.dq = *(const f4 *)(dq32 + w_base + t * w_stride_n);
        it.dk = *(const f4 *)(dk32 + w_base + t * w_stride_n);
    }
    __device__ __forceinline__ void put4(void *p, int t, f4 x) const
    {
        const int64_t i = g_base + (int64_t)t * a.grad.stride_n;
        if (OUT_BF16) {
            uint2 w;
            w.x = (uint32_t)float_to_bf16_bits(x[0]) | ((uint32_t)float_to_bf16_bits(x[1]) << 16);
            w.y = (uint32_t)float_to_bf16_bits(x[2]) | ((uint32_t)float_to_bf16_bits(x[3]) << 16);
            *(uint2 *)((uint16_t *)p + i) = w;
        } else {
            *(f4 *)((float *)p + i) = x;
        }
    }

    // sum of r over the tokens, per channel
    __device__ __forceinline__ void totals(int t_lo, int t_hi, float *out, float *lds) const
    {
        float (*sR)[CH + 4] = (float (*)[CH + 4])lds;
        f4 sum = f4{0.f, 0.f, 0.f, 0.f};
        for (int t0 = t_lo + (t_hi - 1 - t_lo) / kFinBlock * kFinBlock; t0 >= t_lo; t0 -= kFinBlock) {
            Item it;
            load(min(t0 + row, t_hi - 1), it);
            if (t0 + row < t_hi) sum += it.q * it.dq - it.k * it.dk;
        }
        *(f4 *)&sR[row][c4l] = sum;
        __syncthreads();
        if (tid < CH) {
            float acc = 0.f;
            for (int r2 = kFinBlock - 1; r2 >= 0; --r2) acc += sR[r2][tid];
            out[tid] = acc;
        }
    }

    // carry (threads 0 .. CH - 1): sum of r over the tokens from t_hi on
    __device__ __forceinline__ void walk(int t_lo, int t_hi, float carry, float *lds) const
    {
        float (*sR)[CH + 4] = (float (*)[CH + 4])lds;
        float (*sQtr)[CH] = (float (*)[CH])(lds + kFinBlock * (CH + 4));
        float *sCarry = lds + kFinBlock * (CH + 4) + 4 * CH;
        if (tid < CH) sCarry[tid] = carry;
        const int last0 = t_lo + (t_hi - 1 - t_lo) / kFinBlock * kFinBlock;
        Item cur;
        load(min(last0 + row, t_hi - 1), cur);
        for (int t0 = last0; t0 >= t_lo; t0 -= kFinBlock) {
            Item nxt = cur;
            if (t0 > t_lo) load(t0 - kFinBlock + row, nxt);
            const int t = t0 + row;
            const bool live = t < t_hi;
            f4 r = cur.q * cur.dq - cur.k * cur.dk;
            if (!live) r = f4{0.f, 0.f, 0.f, 0.f};
            *(f4 *)&sR[row][c4l] = r;
            __syncthreads();
            if (tid < 4 * CH) {            // suffix sums inside a quarter of the block, top down
                const int c = tid % CH, qtr = tid / CH;
                float acc = 0.f;
#pragma unroll
                for (int tt = 15; tt >= 0; --tt) {
                    acc += sR[16 * qtr + tt][c];
                    sR[16 * qtr + tt][c] = acc;
                }
                sQtr[qtr][c] = acc;
            }
            __syncthreads();
            {
                f4 suffix = *(const f4 *)&sR[row][c4l] + *(const f4 *)&sCarry[c4l];
                for (int q2 = 3; q2 > (row >> 4); --q2) suffix += *(const f4 *)&sQtr[q2][c4l];
                // (from a zero state the first token's decay multiplies nothing)
                const bool no_decay = (t == 0 && !a.state_in) || is_boundary(a.start_pos + t + 1, a.grid_w, a.mode);
                f4 dl = suffix / cur.lam;
                if (no_decay) dl = f4{0.f, 0.f, 0.f, 0.f};
                if (!a.k) dl -= cur.dk;
                f4 dqo = cur.dq;
                if (a.fused_act) {         // chain rule to the pre-activation inputs; sigmoid' = lambda (1 - lambda)
                    dl = dl * cur.lam * (f4{1.0f, 1.0f, 1.0f, 1.0f} - cur.lam);
                    dqo = dqo * cur.dact;
                }
                if (live) {
                    put4(a.dlam, t, dl);
                    put4(a.dq, t, dqo);
                    if (a.k) put4(a.dk, t, cur.dk);
                }
            }
            __syncthreads();
            if (tid < CH) sCarry[tid] += (sQtr[3][tid] + sQtr[2][tid]) + (sQtr[1][tid] + sQtr[0][tid]);
            cur = nxt;
        }
    }
};

}  // namespace lasad
