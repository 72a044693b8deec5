// Device-side building blocks of the fp32 kernels (gfx950): a wave's walk over 32-row blocks of a tile's key lists, the
// global->LDS copies of such a block and the two ways its rows are read back as MFMA operands.
//
// The products run on the bf16 matrix cores, whose rate is 16 times that of the fp32 ones: an fp32 number is the sum of three
// bf16 numbers, x = h + m + l, exactly (8 bits of its 24 each; h rounded to nearest, m and l cut off, so that |m| <= 2^-8 |x| and
// |l| < 2^-16 |x|), and of the nine partial products of two numbers the six of h h, h m, m h, m m, h l, l h are taken; m l, l m and l l
// together are below 2^-23 of the product, 2^-26.7 on average.  Every partial product is exact in the fp32 accumulator's input, and a
// step of 16 contraction slots is one accumulation where the fp32 instruction takes eight, so the sums are rounded less often: the
// error of the operator against fp64 is not larger than with v_mfma_f32_32x32x2_f32 (figures in the kernels).
// Operands that three parts do not hold go to fp32 products: the kernels then walk the workgroup's lists again.  Bits below 2^-133
// (bf16's least number; conversion, dot products and MFMAs of gfx950 keep numbers below 2^-126) are looked for in every operand as it is
// split; infinite and NaN operands and numbers that round up to 2^128 make a NaN (h - h) that reaches the result.  The softmax
// weights are not looked at: what theirs lose below 2^-133 is less than what the exponential does, which ends at 2^-126.
// A second walk of every workgroup makes a launch 2.0 to 2.3 times as long, forward or backward (q, k or v of N(0,1) 2^-120; one 1024^2
// image 127 -> 270 and 413 -> 935 us, two 512^2 images of 6 heads 15.8 -> 31.9 and 43.5 -> 88.5); one such key, which its own and every
// workgroup that walks it sees, 1.4 to 1.7 times.  The size of scores and weights sends nothing there (q of N(0,1) 16: 16.1 and 43.6 us).
//
// (Three bf16 numbers for one of fp32, products accumulated in fp32: G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype for Higher-Precision Computations", ARITH 2019.)
//
// Layouts (lane = 32*g + j).  v_mfma_f32_32x32x16_bf16: A is 32 x 16 with row j, slots 8*g .. +7 in lane (j, g), B 16 x 32 with the
// same slots, column j; v_mfma_f32_32x32x2_f32: one slot g.  The result's register v of lane (j, g) is row kappa(v, g) = 8*(v/4) +
// 4*g + v%4, column j, for both.  Which element of the contraction sits in which slot is free as long as A and B agree:
//   first products  (walked rows x tile rows, contraction over d): bf16 step kk, slot 8*g + e holds d = 16*kk + 8*g + e; fp32 step
//                   (t, e) holds d = 8*t + 4*g + e: a lane's operands are whole 16-byte chunks of one row;
//   second products (contraction over the 32 walked rows): bf16 step st, slot 8*g + e holds walked row kappa(8*st + e, g), fp32 step v
//                   row kappa(v, g), so the registers of a first product are the B operand as they stand and A is those
//                   rows, column j of the walked rows.
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

// The upper halves of two numbers: bf16, rounded towards zero.
__device__ __forceinline__ uint32_t high_halves(float lo, float hi) {
    return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo), 0x07060302u);
}

// Whether a lane has split a number that its parts do not hold: what is left after m is cut off has then bits below 2^-133, in the
// lower half of its word.  (One instruction for two numbers; without it one 1024^2 image takes 124.4 us for 125.2 forward, 412 for 415 backward.)
struct Lost {
    uint32_t bits = 0u;
    __device__ __forceinline__ void add(float a, float b) { bits |= __builtin_bit_cast(uint32_t, a) | __builtin_bit_cast(uint32_t, b); }
    __device__ __forceinline__ bool any() const { return (bits & 0xffffu) != 0u; }
};
// The same where there is no register to put it off (the dk/dv walk spills then).  Backward, us with / without the test: two 512^2 images, 6
// heads 43.6 / 43.2; windows of 32 to 256, 12 heads of 256 tokens 22.6 to 32.6 / 23.1 to 32.8 (4 images), 70 to 107 / 68 to 110 (16).
struct LostAtOnce : Lost {
    __device__ __forceinline__ void add(float a, float b) {
        Lost::add(a, b);
        asm volatile("" : "+v"(bits));
    }
};
struct Unchecked {
    __device__ __forceinline__ void add(float, float) {}
};

// 8 fp32 numbers as three bf16 operands.
struct Split8 {
    bf16x8 h, m, l;
};
// Two dot products with (-1, 0) and (0, -1) subtract a pair of parts from its numbers (exact: the difference fits fp32).  They take turns
// with the matrix cores, where other vector instructions run beside them, but are 4 instructions a pair where unpacking, masking
// and subtracting are 8, and the vector unit is the busier one (forward and backward of two 512^2 images, 6 heads: 60.5 us, 64.1 with
// the latter).  (The constants sit in scalar registers: as a literal operand the assembler's -1.0 is the pair (0, -1).)
template <class Check>
__device__ __forceinline__ Split8 split8(const float (&x)[8], Check& lost) {
    uint32_t c0 = 0x0000bf80u, c1 = 0xbf800000u;
    asm("" : "+s"(c0));
    asm("" : "+s"(c1));
    const bf16x2 n0 = __builtin_bit_cast(bf16x2, c0), n1 = __builtin_bit_cast(bf16x2, c1);
    u32x4 h, m, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bf16x2 hp = {(__bf16)x[2 * e], (__bf16)x[2 * e + 1]};
        const float r0 = __builtin_amdgcn_fdot2_f32_bf16(hp, n0, x[2 * e], false);
        const float r1 = __builtin_amdgcn_fdot2_f32_bf16(hp, n1, x[2 * e + 1], false);
        const uint32_t mw = high_halves(r0, r1);         // (a bit cast of m[e] would be that of element 0)
        const bf16x2 mp = __builtin_bit_cast(bf16x2, mw);
        m[e] = mw;
        h[e] = __builtin_bit_cast(uint32_t, hp);
        const float t0 = __builtin_amdgcn_fdot2_f32_bf16(mp, n0, r0, false), t1 = __builtin_amdgcn_fdot2_f32_bf16(mp, n1, r1, false);
        l[e] = high_halves(t0, t1);
        lost.add(t0, t1);
    }
    return Split8{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}
__device__ __forceinline__ floatx16 mfma_bf16(const bf16x8& a, const bf16x8& b, const floatx16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bool finite(float x) { return fabsf(x) <= 3.4028234e38f; }

// Tile rows held for the whole walk, as B operands of first products: row[16*kk + 8*g .. +7] split (LeanRows: the low parts in LDS,
// shared by the workgroup's waves, whose tile rows are the same), or chunks 2*t + g as they are.
struct SplitRows {
    static constexpr bool kPlain = false;
    Split8 k[4];
    __device__ __forceinline__ bf16x8 h(int kk) const { return k[kk].h; }
    __device__ __forceinline__ bf16x8 m(int kk) const { return k[kk].m; }
    __device__ __forceinline__ bf16x8 l(int kk, int) const { return k[kk].l; }
};
constexpr int kLowParts = 4 * 64;                       // bf16x8 of one tensor's low parts: [kk][lane]
struct LeanRows {
    static constexpr bool kPlain = false;
    bf16x8 hi[4], mid[4];
    bf16x8* low;
    __device__ __forceinline__ bf16x8 h(int kk) const { return hi[kk]; }
    __device__ __forceinline__ bf16x8 m(int kk) const { return mid[kk]; }
    __device__ __forceinline__ bf16x8 l(int kk, int lane) const { return low[64 * kk + lane]; }
};
struct PlainRows {
    static constexpr bool kPlain = true;
    float4 c[8];
};
template <class Check>
__device__ __forceinline__ void load_rows(const float* row, int g, SplitRows& x, Check& lost) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const float4 a = *reinterpret_cast<const float4*>(row + 16 * kk + 8 * g), b = *reinterpret_cast<const float4*>(row + 16 * kk + 8 * g + 4);
        x.k[kk] = split8({a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}, lost);
    }
}
// Every wave writes the same low parts; they can be read after the next barrier.
template <class Check>
__device__ __forceinline__ void load_rows(const float* row, int g, LeanRows& x, Check& lost) {
    SplitRows r;
    load_rows(row, g, r, lost);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        x.hi[kk] = r.k[kk].h;
        x.mid[kk] = r.k[kk].m;
        x.low[64 * kk + (threadIdx.x & 63)] = r.k[kk].l;
    }
}
template <class Check>
__device__ __forceinline__ void load_rows(const float* row, int g, PlainRows& x, Check&) {
#pragma unroll
    for (int t = 0; t < 8; ++t) x.c[t] = *reinterpret_cast<const float4*>(row + 8 * t + 4 * g);
}
// Their loads are waited for here and not inside the loop (where the compiler, which does not see the copies, would drain them
// with a wait sized for these loads).
__device__ __forceinline__ void pin(SplitRows& x) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(x.k[kk].h), "+v"(x.k[kk].m), "+v"(x.k[kk].l));
}
__device__ __forceinline__ void pin(LeanRows& x) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(x.hi[kk]), "+v"(x.mid[kk]));
}
__device__ __forceinline__ void pin(PlainRows& x) {
#pragma unroll
    for (int t = 0; t < 8; ++t) asm volatile("" : "+v"(x.c[t].x), "+v"(x.c[t].y), "+v"(x.c[t].z), "+v"(x.c[t].w));
}

// What a lane reads of a block for a first product (row j) and for a second one (column j of every 32 columns), as it stands in
// memory.  The whole block is in registers before its products start, so that the copies of the next one have all their
// time to land.
struct BlockRows {
    float4 c[8];                 // SplitRows, LeanRows: 2*kk + e is chunk 4*kk + 2*g + e; PlainRows: t is chunk 2*t + g
};
struct BlockCols {
    float x[2][16];              // [d block][step or slot v]: row kappa(v, g)
};
template <class Rows>
__device__ __forceinline__ BlockRows read_rows(const float* blk, const Rows&, int lane) {
    const int j = lane & 31, g = lane >> 5;
    const float* const row = blk + j * kD;
    const int c0 = (Rows::kPlain ? g : 2 * g) ^ f32_swizzle(j);
    BlockRows r;
#pragma unroll
    for (int t = 0; t < 8; ++t) r.c[t] = *reinterpret_cast<const float4*>(row + 4 * (c0 ^ (Rows::kPlain ? 2 * t : 4 * (t >> 1) + (t & 1))));
    return r;
}
__device__ __forceinline__ BlockCols read_cols(const float* blk, int lane) {
    const int i = lane & 31, g = lane >> 5;
    const int base = 4 * g * kD + 4 * ((i >> 2) ^ (8 * g)) + (i & 3);
    BlockCols r;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int flip = (v & 3) | (v & 4), row = 8 * (v >> 2) + (v & 3);     // f32_swizzle(row) apart from g's bit
#pragma unroll
        for (int db = 0; db < 2; ++db) r.x[db][v] = blk[(base ^ (4 * (flip | (db << 3)))) + row * kD];
    }
    return r;
}

// First product of a block: its rows (A) against 32 tile rows (B).  The five small partial products have a sum of their
// own, added to that of the large one at the end.
template <class Rows, class Check>
__device__ __forceinline__ floatx16 rows_product(const BlockRows& blk, const Rows& b, int lane, Check& lost) {
    floatx16 z, small, large;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const float4 x = blk.c[2 * kk], y = blk.c[2 * kk + 1];
        const Split8 a = split8({x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w}, lost);
        small = mfma_bf16(a.l, b.h(kk), kk == 0 ? z : small);
        large = mfma_bf16(a.h, b.h(kk), kk == 0 ? z : large);
        small = mfma_bf16(a.h, b.l(kk, lane), small);
        small = mfma_bf16(a.m, b.m(kk), small);
        small = mfma_bf16(a.m, b.h(kk), small);
        small = mfma_bf16(a.h, b.m(kk), small);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) large[v] += small[v];
    return large;
}

// Second product of a block: its columns (A) against the weights of its rows (B, a first product's registers).
// The five small partial products go to sums of their own, so that the large ones are rounded once per 16 rows.
struct SplitSum {
    floatx16 large[2], small[2];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int v = 0; v < 16; ++v) large[0][v] = large[1][v] = small[0][v] = small[1][v] = 0.f;
    }
    __device__ __forceinline__ void scale(float f) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            large[0][v] *= f;
            large[1][v] *= f;
            small[0][v] *= f;
            small[1][v] *= f;
        }
    }
    __device__ __forceinline__ void total(floatx16 (&sum)[2]) const {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            sum[0][v] = large[0][v] + small[0][v];
            sum[1][v] = large[1][v] + small[1][v];
        }
    }
};
struct PlainSum {
    floatx16 acc[2];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.f;
    }
    __device__ __forceinline__ void scale(float f) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            acc[0][v] *= f;
            acc[1][v] *= f;
        }
    }
    __device__ __forceinline__ void total(floatx16 (&sum)[2]) const {
        sum[0] = acc[0];
        sum[1] = acc[1];
    }
};
// All partial products in one sum, the small ones first: half the registers.
struct ChainSum : PlainSum {};

__device__ __forceinline__ void add_products(const Split8& a, const Split8& b, SplitSum& sum, int db) {
    sum.small[db] = mfma_bf16(a.l, b.h, sum.small[db]);
    sum.large[db] = mfma_bf16(a.h, b.h, sum.large[db]);
    sum.small[db] = mfma_bf16(a.h, b.l, sum.small[db]);
    sum.small[db] = mfma_bf16(a.m, b.m, sum.small[db]);
    sum.small[db] = mfma_bf16(a.m, b.h, sum.small[db]);
    sum.small[db] = mfma_bf16(a.h, b.m, sum.small[db]);
}
__device__ __forceinline__ void add_products(const Split8& a, const Split8& b, ChainSum& sum, int db) {
    sum.acc[db] = mfma_bf16(a.l, b.h, sum.acc[db]);
    sum.acc[db] = mfma_bf16(a.h, b.l, sum.acc[db]);
    sum.acc[db] = mfma_bf16(a.m, b.m, sum.acc[db]);
    sum.acc[db] = mfma_bf16(a.m, b.h, sum.acc[db]);
    sum.acc[db] = mfma_bf16(a.h, b.m, sum.acc[db]);
    sum.acc[db] = mfma_bf16(a.h, b.h, sum.acc[db]);
}
template <class Sum, class Check>
__device__ __forceinline__ void cols_product(const BlockCols& blk, const float (&w)[16], Sum& sum, Check& lost) {
    Unchecked weights;
#pragma unroll
    for (int st = 0; st < 2; ++st) {
        const Split8 b = split8({w[8 * st], w[8 * st + 1], w[8 * st + 2], w[8 * st + 3], w[8 * st + 4], w[8 * st + 5], w[8 * st + 6], w[8 * st + 7]}, weights);
#pragma unroll
        for (int db = 0; db < 2; ++db) {
            const float* const x = blk.x[db] + 8 * st;
            const Split8 a = split8({x[0], x[1], x[2], x[3], x[4], x[5], x[6], x[7]}, lost);
            add_products(a, b, sum, db);
        }
    }
}

// The same on the fp32 matrix cores.  Two chains in the first product: half the length of the sums.
template <class Check>
__device__ __forceinline__ floatx16 rows_product(const BlockRows& blk, const PlainRows& b, int, Check&) {
    floatx16 z, s0, s1;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float4 a = blk.c[t];
        floatx16& s = t & 1 ? s1 : s0;
        s = mfma_f32(a.x, b.c[t].x, t < 2 ? z : s);
        s = mfma_f32(a.y, b.c[t].y, s);
        s = mfma_f32(a.z, b.c[t].z, s);
        s = mfma_f32(a.w, b.c[t].w, s);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) s0[v] += s1[v];
    return s0;
}
template <class Check>
__device__ __forceinline__ void cols_product(const BlockCols& blk, const float (&w)[16], PlainSum& sum, Check&) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int db = 0; db < 2; ++db) sum.acc[db] = mfma_f32(blk.x[db][v], w[v], sum.acc[db]);
}

}  // namespace dfa
