// Backward pass: parameter block and launcher.
#ifndef SWAA_BWD_H_
#define SWAA_BWD_H_

#include "swaa_common.h"

namespace swaa {

// delta_i = <dO_i, O_i> of the dQ kernels' rows: a lane holds 8 kSteps elements of its row's dO as B operands and
// reads the same of O at `o`; lanes l and l + 32 share a row.  The dQ kernels have every row's dO in
// registers once, so a launch of its own, which read dO and O for nothing else (268 MB in 42 us for 16384 tokens
// on 32 heads), is saved: backwards of 1000 to 9000 tokens are 1 to 2.6 % faster, longer ones 0.5 (100 tokens take 0.4 us
// longer: O is one more wait in the chain of a single workgroup).
template <int kSteps>
__device__ __forceinline__ float row_delta(const __bf16 *o, const bf16x8 (&dof)[kSteps]) {
    // eight products in a row, then pairs of sums: twelve additions deep for 128 elements, as far as the sums of a tree
    // over the lanes (64 in a row lose what is small beside a large product)
    bf16x8 of[kSteps];
#pragma unroll
    for (int ks = 0; ks < kSteps; ++ks) of[ks] = *reinterpret_cast<const bf16x8 *>(o + 16 * ks);
    __builtin_amdgcn_sched_barrier(0);  // (all of them asked for before the first is used)
    float part[kSteps];
#pragma unroll
    for (int ks = 0; ks < kSteps; ++ks) {
        part[ks] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) part[ks] += (float)dof[ks][e] * (float)of[ks][e];
    }
#pragma unroll
    for (int w = kSteps / 2; w > 0; w /= 2)
#pragma unroll
        for (int ks = 0; ks < w; ++ks) part[ks] += part[ks + w];
    return half_swap_sum(part[0]);
}

struct BwdParams {
    FwdParams f;  // q, k, v, lse, the mask and the forward's work decomposition; contiguous [B, H, N, D]
    const __bf16 *out;   // forward output
    const __bf16 *dout;  // upstream gradient, shaped like out
    __bf16 *dq;          // [B, Hq, N, D]
    __bf16 *dk;          // [B, Hkv, N, D]
    __bf16 *dv;          // [B, Hkv, N, D]
    float *delta;        // workspace, [B, Hq, N]
    int B, Hq, Hkv, N;
    int die_shift;  // of the dK/dV kernels' work list (dkv_main_item)
    // Key tiles (128 keys) that hold sink keys are seen by every later row.  Their rows
    // beyond the band are cut into n_seg segments of seg_tiles query tiles, each computed
    // by a workgroup of its own; the band part and the segments leave fp32 partial sums in
    // `partial` and a last kernel adds them.
    int n_sink_kt, n_seg, seg_tiles;
    // Where the key tiles are too few for the chip, the (head, query tile) steps of every one are cut into n_split pieces
    // (plan_bwd), each a workgroup's; then all key tiles leave partial sums: [B*Hkv][key tile][parts][2 (dK, dV)][128][D], the
    // parts being the pieces, then the segments (of key tiles that have them).
    int n_split;
    __host__ __device__ int parts(int kt) const { return kt < n_sink_kt ? n_split + n_seg : n_split > 1 ? n_split : 0; }
    __host__ __device__ long long first_part(int pair, int kt) const {
        const int sinks = kt < n_sink_kt ? kt : n_sink_kt, rest = n_split > 1 ? n_split : 0;
        const int n_kt = (N + 127) / 128;
        return (long long)pair * (n_sink_kt * (n_split + n_seg) + (n_kt - n_sink_kt) * rest) + sinks * (n_split + n_seg) + (kt - sinks) * rest;
    }
    float *partial;  // workspace, after delta
    // divisions the dK/dV workgroups make, as multiplications
    FastDiv div_kt, div_pairs, div_hkv, div_split, div_seg, div_sink_kt;
    FastDiv div_group;  // (and the dQ workgroups of short sequences)
};

// Fills die_shift, n_sink_kt, n_seg, seg_tiles, n_split and the reciprocals from the shape and mask fields.  pieces: key tiles may be cut into
// pieces (their partial sums take workspace).
void plan_bwd(BwdParams &p, int D, bool pieces);
// Floats of workspace the plan needs (delta + partial sums).
long long bwd_workspace_floats(const BwdParams &p, int D);

hipError_t launch_bwd(const BwdParams &p, int D, hipStream_t stream);
// dQ and delta, head dimension 128 (swaa_bwd_dq_pipelined.hip)
hipError_t launch_bwd_dq_pipelined_d128(const BwdParams &p, hipStream_t stream);

}  // namespace swaa

#endif  // SWAA_BWD_H_
