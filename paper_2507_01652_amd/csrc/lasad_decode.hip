// Recurrent decode step (Algorithm 1 loop body; Section 3.4 first equation):
//     S <- lambda S + k v^T,   o = q_scale * S^T q      for every (batch, head).
// 0.5 flop per byte: the kernel is a stream over the fp32 states (read once,
// written once, in place), so the design goal is HBM bandwidth.
//
// One 64-lane wavefront owns one d x d state, or a quarter of its rows (see launch_decode).  A lane
// reads 16-byte pieces (4 value channels) so that every wave-wide load covers whole contiguous
// rows of S; up to 16 loads per lane (the whole state at d = 64) are issued back to back
// before any arithmetic to keep many bytes in flight.  Each lane keeps the partial q-weighted column sums of
// the rows it touched; lanes that share a column group are then combined with
// cross-lane shuffles (no LDS round trip for the reduction).
//
// The states are touched exactly once per step, so their loads and stores carry
// the non-temporal hint (measured: 28.6 us instead of 33.6 us per step on 5120
// states, the same as a plain read-modify-write stream over the same bytes), and
// a workgroup is one state's wavefronts so that every wave starts as early as possible.
#include "lasad_internal.h"

namespace lasad {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float4 load_stream(const float4 *p)
{
    const f32x4 r = __builtin_nontemporal_load((const f32x4 *)p);
    return make_float4(r.x, r.y, r.z, r.w);
}

__device__ inline void store_stream(float4 *p, float4 x)
{
    const f32x4 r = {x.x, x.y, x.z, x.w};
    __builtin_nontemporal_store(r, (f32x4 *)p);
}

template <int IN_BF16>
__device__ inline float ld_in(const void *p, int64_t idx)
{
    if (IN_BF16) return bf16_bits_to_float(((const uint16_t *)p)[idx]);
    return ((const float *)p)[idx];
}

// GATED = 1: the decay is a vector over the key channels (row i of S is scaled by lambda[i],
// or by 1 at a row-boundary position) and the key is 1 - lambda unless a key is given
// (Section 3.4, Algorithm 1 as written).
// WV: wavefronts per state, each with D / WV of its rows; their sums meet in LDS.
template <int D, int IN_BF16, int OUT_BF16, int GATED, int WV>
__global__ void __launch_bounds__(WV * 64)
decode_kernel(DecodeArgs a)
{
    constexpr int CG = D / 4;        // column groups (float4) per row
    constexpr int RPP = 64 / CG;     // rows covered by one wave-wide load
    constexpr int P = D / RPP / WV;  // loads per lane for the wavefront's rows
    constexpr int PB = P < 16 ? P : 16;   // loads in flight per lane at a time
    __shared__ float sqk[WV][2 + GATED][D];
    __shared__ __attribute__((aligned(16))) float sSum[WV == 1 ? 1 : WV][WV == 1 ? 4 : D];

    const int wave = WV == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int bh = blockIdx.x;
    const int h = bh % a.Hh;
    const int cg = lane % CG, r0 = wave * (D / WV) + lane / CG;      // column group, first row
    const int64_t vec = (int64_t)bh * D;
    int pos = a.pos;
    if (a.pos_rows) {                // continuous batching: every batch row at its own raster position
        pos = a.pos_rows[bh / a.Hh];
        if (pos < 0 || pos >= a.grid_n) {      // inactive row: state untouched, output row zero (whole wave)
            if (threadIdx.x < CG) {
                if (OUT_BF16) *(ushort4 *)((uint16_t *)a.o + vec + cg * 4) = make_ushort4(0, 0, 0, 0);
                else *(float4 *)((float *)a.o + vec + cg * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            return;
        }
    }
    const int t = pos + 1;
    const bool boundary = is_boundary(t, a.grid_w, a.mode);
    const float lam = (boundary || GATED) ? 1.0f : a.gamma[h];

    float4 *S = (float4 *)(a.state + (int64_t)bh * D * D);

    // Global loads in issue order: the small q, k, v vectors, then the first
    // batch of state pieces; only then are q and k parked in LDS (fp32,
    // wave-private region) so that every lane can read any row's q_i, k_i.
    constexpr int NQ = (D + 63) / 64;
    float qr[NQ], kr[NQ], lr[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int c = lane + 64 * i;
        qr[i] = c < D ? ld_in<IN_BF16>(a.q, vec + c) : 0.f;
        if (GATED) {
            float l = c < D ? ld_in<IN_BF16>(a.lam, vec + c) : 1.f;
            if (a.fused_act) { l = sigmoid_f32(l); qr[i] = silu_f32(qr[i]); }     // Algorithm 1's activations
            kr[i] = a.k ? (c < D ? ld_in<IN_BF16>(a.k, vec + c) : 0.f) : 1.0f - l;   // key from the base decay
            lr[i] = boundary ? 1.0f : l;
        } else {
            kr[i] = c < D ? ld_in<IN_BF16>(a.k, vec + c) : 0.f;
            lr[i] = 1.0f;
        }
    }
    float4 vv;
    vv.x = ld_in<IN_BF16>(a.v, vec + cg * 4 + 0);
    vv.y = ld_in<IN_BF16>(a.v, vec + cg * 4 + 1);
    vv.z = ld_in<IN_BF16>(a.v, vec + cg * 4 + 2);
    vv.w = ld_in<IN_BF16>(a.v, vec + cg * 4 + 3);

    float4 s[PB];
#pragma unroll
    for (int p = 0; p < PB; ++p) s[p] = load_stream(&S[(r0 + p * RPP) * CG + cg]);

#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int c = lane + 64 * i;
        if (c < D) {
            sqk[wave][0][c] = qr[i];
            sqk[wave][1][c] = kr[i];
            if (GATED) sqk[wave][2][c] = lr[i];
        }
    }
    // wave-level ordering of the LDS writes above against the reads below
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int p0 = 0; p0 < P; p0 += PB) {
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int row = r0 + (p0 + p) * RPP;
            const float qi = sqk[wave][0][row], ki = sqk[wave][1][row];
            const float li = GATED ? sqk[wave][2][row] : lam;
            float4 x = s[p];
            x.x = fmaf(li, x.x, ki * vv.x);
            x.y = fmaf(li, x.y, ki * vv.y);
            x.z = fmaf(li, x.z, ki * vv.z);
            x.w = fmaf(li, x.w, ki * vv.w);
            store_stream(&S[row * CG + cg], x);
            acc.x = fmaf(qi, x.x, acc.x);
            acc.y = fmaf(qi, x.y, acc.y);
            acc.z = fmaf(qi, x.z, acc.z);
            acc.w = fmaf(qi, x.w, acc.w);
        }
        if (p0 + PB < P) {   // next batch of state pieces (d = 128 only)
#pragma unroll
            for (int p = 0; p < PB; ++p) s[p] = load_stream(&S[(r0 + (p0 + PB + p) * RPP) * CG + cg]);
        }
    }
    // combine the RPP lanes that share a column group (lane bits above log2(CG))
#pragma unroll
    for (int off = CG; off < 64; off <<= 1) {
        acc.x += __shfl_xor(acc.x, off, 64);
        acc.y += __shfl_xor(acc.y, off, 64);
        acc.z += __shfl_xor(acc.z, off, 64);
        acc.w += __shfl_xor(acc.w, off, 64);
    }
    if (WV > 1) {                    // ... and the wavefronts, in the first one
        if (lane < CG) *(float4 *)&sSum[wave][cg * 4] = acc;
        __syncthreads();
        if (wave != 0) return;
        acc = *(const float4 *)&sSum[0][cg * 4];
#pragma unroll
        for (int w = 1; w < WV; ++w) {
            const float4 x = *(const float4 *)&sSum[w][cg * 4];
            acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
        }
    }
    float qs = a.q_scale;
    if (GATED && a.norm) {           // Norm(o): root mean square over the D channels (lanes 0 .. CG-1 hold them)
        float ss = (acc.x * acc.x + acc.y * acc.y) + (acc.z * acc.z + acc.w * acc.w);
#pragma unroll
        for (int off = CG / 2; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 64);
        const float rstd = __builtin_amdgcn_rsqf(qs * qs * ss * (1.0f / D) + a.norm_eps);
        qs *= rstd;
        if (a.norm_w) {
            const float4 w4 = *(const float4 *)(a.norm_w + h * D + cg * 4);
            acc.x *= w4.x; acc.y *= w4.y; acc.z *= w4.z; acc.w *= w4.w;
        }
    }
    if (lane < CG) {
        if (OUT_BF16) {
            uint16_t *o = (uint16_t *)a.o + vec + cg * 4;
            ushort4 pk;
            pk.x = float_to_bf16_bits(qs * acc.x);
            pk.y = float_to_bf16_bits(qs * acc.y);
            pk.z = float_to_bf16_bits(qs * acc.z);
            pk.w = float_to_bf16_bits(qs * acc.w);
            *(ushort4 *)o = pk;
        } else {
            float *o = (float *)a.o + vec + cg * 4;
            *(float4 *)o = make_float4(qs * acc.x, qs * acc.y, qs * acc.z, qs * acc.w);
        }
    }
}

template <int D, int WV>
hipError_t launch_d(const DecodeArgs &a, hipStream_t s)
{
    const dim3 grid((unsigned)(a.B * a.Hh)), block(WV * 64);
    const bool in16 = a.io_dtype == LASAD_BF16, out16 = a.out_dtype == LASAD_BF16;
    if (a.lam) {
        if (in16 && out16) hipLaunchKernelGGL((decode_kernel<D, 1, 1, 1, WV>), grid, block, 0, s, a);
        else if (in16) hipLaunchKernelGGL((decode_kernel<D, 1, 0, 1, WV>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((decode_kernel<D, 0, 0, 1, WV>), grid, block, 0, s, a);
    } else {
        if (in16 && out16) hipLaunchKernelGGL((decode_kernel<D, 1, 1, 0, WV>), grid, block, 0, s, a);
        else if (in16) hipLaunchKernelGGL((decode_kernel<D, 1, 0, 0, WV>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((decode_kernel<D, 0, 0, 0, WV>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace

// Four wavefronts a state (d = 64) where the chip has a unit for each state, and the chain load, update, store of a lone wavefront is
// what a step waits for, and for so many states that their number of loads in flight counts again.  In between a fourth of
// the loads a wavefront with four times the wavefronts to start is slower.  us a step (graph replay), one | four wavefronts: 12
// states 3.06 | 2.86, 128 3.26 | 3.12, 256 3.91 | 3.81, fused layer 12 3.48 | 3.18, 256 3.95 | 3.84; 320 4.10 | 4.25, 512 4.60 | 4.70,
// 1024 6.9 | 7.8, 2048 13.0 | 13.1; 3072 18.9 | 18.6, 5120 30.1 | 29.1, 8192 46.8 | 44.7.  (A launch has room for 2^32 threads: states
// that fill the memory, 2^24 and more, keep one wavefront.)
hipError_t launch_decode(const DecodeArgs &a, hipStream_t s)
{
    const int64_t n_states = (int64_t)a.B * a.Hh;
    switch (a.d) {
        case 32: return launch_d<32, 1>(a, s);
        case 64: return n_states <= 256 || (n_states >= 3000 && n_states < 1 << 24) ? launch_d<64, 4>(a, s) : launch_d<64, 1>(a, s);
        case 128: return launch_d<128, 1>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lasad
