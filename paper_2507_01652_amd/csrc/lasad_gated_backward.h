// What the launcher of the vector-decay backward hands to its chunked kernels.
#pragma once

#include "lasad_gated_chunk.h"
#include "lasad_internal.h"
#include "lasad_scan.h"

namespace lasad {

constexpr int kMaxSegments = 16;       // of a sequence

struct GatedChunkArgs {
    GatedBackwardArgs b;
    float *dq32, *dk32;                // workspace, [B][n][Hh][64] fp32
    // incoming and final states of the walks ([B, Hh, d, d], [key channel][value channel]), or NULL
    const float *g_in;                 // dL/d(final state) / q_scale
    float *s_out, *g_out;              // S_n; the adjoint state at the first token / q_scale, without that token's decay
    const float *sink;                 // [sequence][d]: what every suffix sum of r starts from (cut: of the last segment), or NULL;
                                       //   of sequences whose dq walk did not hold the reversed walk forms it again
    gchunk::SegPlan cut;               // segments with a workgroup each
    // Parts of a segment at whose bounds the reversed walk takes the suffix sum from the states (bound j: the segment's chunks
    // j * count / n_part).
    int n_part;
    // [sequence][segment - 1]: the state before a segment; the adjoint state of its first token, with that token's decay,
    // / q_scale
    float *bounds_s, *bounds_g;
    float *parts_s;                    // [sequence][segment][part - 1]: the states before the parts, from the dq walk
    int *kept;                         // [sequence][segment]: whether the dq walk stayed in its range (else nothing of it holds)
    float *sinks;                      // cut: [sequence][kMaxSegments][d], what the suffix sums of a segment but the last start from
    // the same walks for the token-serial routine: dq, dv, dk
    ForwardArgs serial[3];
    scan::ScanRoles roles[3];

    __device__ __forceinline__ float *bound_s(int64_t bh, int i) const { return bounds_s + (bh * (cut.n_seg - 1) + i) * 4096; }
    __device__ __forceinline__ float *bound_g(int64_t bh, int i) const { return bounds_g + (bh * (cut.n_seg - 1) + i) * 4096; }
    __device__ __forceinline__ float *part_s(int64_t bh, int seg, int i) const { return parts_s + ((bh * cut.n_seg + seg) * (n_part - 1) + i) * 4096; }
    __device__ __forceinline__ const float *sink_of(int64_t bh, int seg) const
    {
        if (seg < cut.n_seg - 1) return sinks + (bh * kMaxSegments + seg) * 64;
        return sink ? sink + bh * 64 : nullptr;
    }
};

// the states at the bounds of the segments of `cut`
hipError_t launch_backward_gated_chunk_states(const GatedChunkArgs &p, hipStream_t s);
hipError_t launch_backward_gated_chunk_dq(const GatedChunkArgs &p, hipStream_t s);
hipError_t launch_backward_gated_chunk_reversed(const GatedChunkArgs &p, hipStream_t s);
bool backward_gated_chunk_fits(const GatedBackwardArgs &a);

}  // namespace lasad
