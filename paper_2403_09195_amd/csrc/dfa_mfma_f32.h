// Device-side building blocks of the fp32 matrix-core kernels (gfx950): a wave's walk over 32-row blocks of a tile's
// key lists, the global->LDS copies of such a block and the two ways its rows are read back as MFMA operands.
//
// v_mfma_f32_32x32x2_f32 (lane = 32*g + j): A is 32 x 2 with row j, slot g in lane (j, g), B is 2 x 32 with slot g,
// column j, the result's register v of lane (j, g) is row kappa(v, g) = 8*(v/4) + 4*g + v%4, column j.  Which element of
// the contraction sits in which slot is free as long as A and B agree:
//   first products  (walked rows x tile rows, contraction over d): step (t, e) holds d = 8*t + 4*g + e, so a lane's
//                   operands are whole 16-byte chunks 2*t + g of one row;
//   second products (contraction over the 32 walked rows): step v holds walked row kappa(v, g), so the registers of a
//                   first product are the B operand as they stand and A is row kappa(v, g), column j of the walked rows.
#pragma once
#include "dfa_blocks.h"

namespace dfa {

constexpr int kF32BlockElems = kWalkBlock * kD;         // one block of one tensor in LDS: 8 KB
constexpr int kF32BlockBytes = kF32BlockElems * 4;
constexpr int kF32Copies = 8;                           // wave-level copies per block (1 KB = 4 rows each)

__device__ __forceinline__ floatx16 mfma_f32(float a, float b, const floatx16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Chunk swizzle of a block in LDS: 16-byte chunk c of row rho sits at chunk c ^ f32_swizzle(rho).  Sixteen consecutive
// rows spread one chunk column over all 64 banks (row reads), and rows rho and rho + 4, which the two halves of a wave
// read together in the second products, use different halves of the banks (column reads).
__device__ __forceinline__ int f32_swizzle(int rho) { return ((rho & 4) << 1) | ((rho & 8) >> 1) | (rho & 3); }

// Issues the copies of one block: rows first() + stride * i of a tensor with row pitch sn (elements); rows past the end
// of the list re-read its last one.
template <class Walk>
__device__ __forceinline__ void issue_block(const float* base, int64_t sn, const Walk& w, uint32_t lds_addr, int lane) {
    const uint32_t row_pitch = (uint32_t)(sn * 4);          // below 2^25, see check_forward_args
    const void* const ub = uniform_ptr(reinterpret_cast<const char*>(base) + (uint64_t)(uint32_t)w.first() * row_pitch);
    const uint32_t pitch = (uint32_t)w.seg.stride * row_pitch;
    const int chunk0 = (lane & 15) ^ (lane >> 4);
    if (w.rows() == kWalkBlock) {
        const uint32_t off = (uint32_t)(lane >> 4) * pitch;
#pragma unroll
        for (int u = 0; u < kF32Copies; ++u)
            copy16_to_lds(ub, off + 16u * (chunk0 ^ (((u & 1) << 3) | ((u & 2) << 1))) + 4 * u * pitch, lds_addr + 1024u * u);
    } else {
        const int room = w.rows() - 1;
#pragma unroll
        for (int u = 0; u < kF32Copies; ++u)
            copy16_to_lds(ub, (uint32_t)min(4 * u + (lane >> 4), room) * pitch + 16u * (chunk0 ^ (((u & 1) << 3) | ((u & 2) << 1))),
                          lds_addr + 1024u * u);
    }
}

// Rows past the end of a list become zeros in LDS, so that a second product's 0 weights meet finite values.
__device__ __forceinline__ void zero_tail(float* blk, int nvalid, int lane) {
    for (int x = lane; x < (kWalkBlock - nvalid) * (kD / 4); x += 64)
        *reinterpret_cast<float4*>(blk + nvalid * kD + 4 * x) = make_float4(0.f, 0.f, 0.f, 0.f);
    lds_reads_done();
}

// First product of a block: rows of `blk` (A) against 32 tile rows held as chunks 2*t + g (B).  Two chains: half the
// length of the sums.
__device__ __forceinline__ floatx16 rows_product(const float* blk, const float4 (&b)[8], int lane) {
    const int j = lane & 31, g = lane >> 5;
    const float* const row = blk + j * kD;
    const int c0 = g ^ f32_swizzle(j);
    floatx16 z, s0, s1;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float4 a = *reinterpret_cast<const float4*>(row + 4 * (c0 ^ (2 * t)));
        floatx16& s = t & 1 ? s1 : s0;
        s = mfma_f32(a.x, b[t].x, t < 2 ? z : s);
        s = mfma_f32(a.y, b[t].y, s);
        s = mfma_f32(a.z, b[t].z, s);
        s = mfma_f32(a.w, b[t].w, s);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) s0[v] += s1[v];
    return s0;
}

// Second product of a block: columns of `blk` (A) against the weights of its rows (B, a first product's registers).
__device__ __forceinline__ void cols_product(const float* blk, const float (&w)[16], floatx16 (&acc)[2], int lane) {
    const int i = lane & 31, g = lane >> 5;
    const int base = 4 * g * kD + 4 * ((i >> 2) ^ (8 * g)) + (i & 3);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int flip = (v & 3) | (v & 4), row = 8 * (v >> 2) + (v & 3);     // f32_swizzle(row) apart from g's bit
#pragma unroll
        for (int db = 0; db < 2; ++db)
            acc[db] = mfma_f32(blk[(base ^ (4 * (flip | (db << 3)))) + row * kD], w[v], acc[db]);
    }
}

// Tile rows held for the whole walk: their loads are waited for here and not inside the loop (where the compiler, which
// does not see the copies, would drain them with a wait sized for these loads).
__device__ __forceinline__ void pin(float4 (&x)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) asm volatile("" : "+v"(x[t].x), "+v"(x[t].y), "+v"(x[t].z), "+v"(x[t].w));
}

// Chunks 2*t + g of a row in global memory.
__device__ __forceinline__ void load_chunks(const float* row, int g, float4 (&x)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = *reinterpret_cast<const float4*>(row + 8 * t + 4 * g);
}

}  // namespace dfa
