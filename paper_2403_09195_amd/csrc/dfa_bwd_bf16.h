// Pieces of the bf16 backward kernels: what a wave does with one 32 x 32 block of (walked row, own row) pairs.  The
// formulas and layouts are described at the head of dfa_bwd_bf16.hip.
#pragma once
#include "dfa_blocks.h"

namespace dfa {

// Every value of a 32-row block at or past list position nvalid becomes -inf (its P is then 0).
// Register v of lane (j, g) is block position 16*(v/8) + 8*g + v%8.
__device__ __forceinline__ void mask_rows(floatx16& s, int g, int nvalid) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
        if (16 * (v >> 3) + 8 * g + (v & 7) >= nvalid) s[v] = -INFINITY;
}

__device__ __forceinline__ floatx16 zero16() {
    floatx16 z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
    return z;
}

// packs 16 fp32 values into the two B operands (16-row steps) of the second product
__device__ __forceinline__ void pack_block(const float (&x)[16], u32x4 (&pb)[2]) {
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        const bf16x2 pr = {(__bf16)x[2 * v], (__bf16)x[2 * v + 1]};
        pb[v >> 2][v & 3] = __builtin_bit_cast(uint32_t, pr);
    }
}

// P and dS of one 32 x 32 block of the dk/dv kernel.  lp: lse (base-2 units) of the walked queries in LDS;
// register v of a lane is block position 16*(v/8) + 8*g + v%8, lp points at position 8*g.  dpd holds
// dP - delta already (the accumulators of dP start from -delta).  kBias: the pairs of this step count m
// times, log2 m = bias (see KeySeg).  The factor scale of dS goes onto the dk accumulator at the end.
template <bool kBias>
__device__ __forceinline__ void probs_block(const floatx16& s, const floatx16& dpd, const float* lp,
                                            float c, float bias, float (&pr)[16], float (&ds)[16]) {
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            const float4 l2 = *reinterpret_cast<const float4*>(lp + 16 * hf + e);
            const float l2a[4] = {l2.x, l2.y, l2.z, l2.w};
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int v = 8 * hf + e + x;
                pr[v] = __builtin_amdgcn_exp2f(fmaf(s[v], c, kBias ? bias - l2a[x] : -l2a[x]));
                ds[v] = pr[v] * dpd[v];
            }
        }
}

// -delta of the 32 walked queries of a block as the start value of the dP accumulators: register v of a
// lane is block position 16*(v/8) + 8*g + v%8, dl points at position 8*g.
__device__ __forceinline__ floatx16 load_ndelta(const float* dl) {
    floatx16 r;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            const float4 d = *reinterpret_cast<const float4*>(dl + 16 * hf + e);
            r[8 * hf + e] = d.x; r[8 * hf + e + 1] = d.y; r[8 * hf + e + 2] = d.z; r[8 * hf + e + 3] = d.w;
        }
    return r;
}

}  // namespace dfa
