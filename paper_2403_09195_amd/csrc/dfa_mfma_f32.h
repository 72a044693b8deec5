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
#include "dfa_device.h"
#include "dfa_mfma.h"

namespace dfa {

constexpr int kF32Waves = 4;                            // waves of a workgroup: one 32-row block of the tile, every wave a
                                                        // quarter of its key blocks
constexpr int kF32Block = 32;                           // walked rows per block
constexpr int kF32BlockElems = kF32Block * kD;          // one block of one tensor in LDS: 8 KB
constexpr int kF32BlockBytes = kF32BlockElems * 4;
constexpr int kF32Copies = 8;                           // wave-level copies per block (1 KB = 4 rows each)
constexpr int kF32RedPitch = kD + 4;                    // row pitch of the per-wave results in LDS (floats)
constexpr int kF32Dies = 8;                             // launch order of a plan: item i on die i mod 8
constexpr int kF32LaunchItems = 1 << 19;                // most items of one launch (16 workgroups of 256 threads each at most)

__device__ __forceinline__ floatx16 mfma_f32(float a, float b, const floatx16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Workgroup x of a launch of `parts` workgroups per item -> (item, part); the parts of an item stay on the item's die.
__device__ __forceinline__ void f32_item_of(int x, int parts, int& item, int& part) {
    const int group = x / (kF32Dies * parts), rem = x % (kF32Dies * parts);
    item = group * kF32Dies + rem % kF32Dies;
    part = rem / kF32Dies;
}

// The 32-row blocks of a tile's progressions, counted through; wave w takes blocks w, w + 4, w + 8, ...
struct BlockWalk {
    const KeySeg* segs;
    int nseg, s, t;              // progression, block within it
    KeySeg seg;

    // through the constant address space: a scalar load.  (After the copies' memory clobber the compiler takes a vector
    // load instead, whose wait would drain the copies in flight.)
    __device__ __forceinline__ void load() {
        typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
        const i32x4 x = *reinterpret_cast<const __attribute__((address_space(4))) i32x4*>(reinterpret_cast<uintptr_t>(segs + s));
        seg.key0 = x[0];
        seg.stride = x[1];
        seg.count = x[2];
        const int32_t mult = x[3];          // (the bit cast of an element in place would be that of element 0)
        seg.log2_mult = __builtin_bit_cast(float, mult);
    }
    __device__ __forceinline__ void settle() {
        while (s < nseg && t * kF32Block >= seg.count) {
            t -= (seg.count + kF32Block - 1) / kF32Block;
            if (++s < nseg) load();
        }
    }
    __device__ __forceinline__ void start(const KeySeg* list, int n, int wave) {
        segs = list;
        nseg = n;
        s = 0;
        t = wave;
        load();
        settle();
    }
    __device__ __forceinline__ void next() {
        t += kF32Waves;
        settle();
    }
    __device__ __forceinline__ bool valid() const { return s < nseg; }
    __device__ __forceinline__ int rows() const { return min(kF32Block, seg.count - t * kF32Block); }
    __device__ __forceinline__ int32_t first() const { return kept_row(seg.key0, seg.stride, t * kF32Block); }
};

// All LDS reads of this wave so far have returned; no memory access moves across.
__device__ __forceinline__ void lds_reads_done() {
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("" ::: "memory");
}
template <int N>
__device__ __forceinline__ void copies_left() {
    wait_vmcnt<N>();
    asm volatile("" ::: "memory");
}

// Chunk swizzle of a block in LDS: 16-byte chunk c of row rho sits at chunk c ^ f32_swizzle(rho).  Sixteen consecutive
// rows spread one chunk column over all 64 banks (row reads), and rows rho and rho + 4, which the two halves of a wave
// read together in the second products, use different halves of the banks (column reads).
__device__ __forceinline__ int f32_swizzle(int rho) { return ((rho & 4) << 1) | ((rho & 8) >> 1) | (rho & 3); }

// Issues the copies of one block: rows first() + stride * i of a tensor with row pitch sn (elements); rows past the end
// of the list re-read its last one.
__device__ __forceinline__ void issue_block(const float* base, int64_t sn, const BlockWalk& w, uint32_t lds_addr, int lane) {
    const void* const ub = uniform_ptr(base + (int64_t)w.first() * sn);
    const uint32_t pitch = (uint32_t)(w.seg.stride * sn * 4);
    const int room = w.rows() - 1;
    const int chunk0 = (lane & 15) ^ (lane >> 4);
#pragma unroll
    for (int u = 0; u < kF32Copies; ++u) {
        const int row = 4 * u + (lane >> 4);
        const int chunk = chunk0 ^ (((u & 1) << 3) | ((u & 2) << 1));
        copy16_to_lds(ub, (uint32_t)min(row, room) * pitch + 16u * chunk, lds_addr + 1024u * u);
    }
}

// Rows past the end of a list become zeros in LDS, so that a second product's 0 weights meet finite values.
__device__ __forceinline__ void zero_tail(float* blk, int nvalid, int lane) {
    for (int x = lane; x < (kF32Block - nvalid) * (kD / 4); x += 64)
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

// A wave's [32 rows][64 d] result, held transposed (lane (j, g), register v of half db: row j, d = 32*db + kappa(v, g)),
// into its own region of LDS.
__device__ __forceinline__ void result_to_lds(const floatx16 (&acc)[2], float* region, int lane) {
    const int j = lane & 31, g = lane >> 5;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int t = 0; t < 4; ++t)
            *reinterpret_cast<float4*>(region + j * kF32RedPitch + 32 * db + 8 * t + 4 * g) =
                make_float4(acc[db][4 * t], acc[db][4 * t + 1], acc[db][4 * t + 2], acc[db][4 * t + 3]);
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
