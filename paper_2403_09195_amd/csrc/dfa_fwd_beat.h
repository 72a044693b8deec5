// One wave's work on a 32-key block in the bf16 forward kernels (gfx950): scores, softmax numerators, row sums and
// accumulation for 64 query rows (two 32-row blocks) as matrix-core products, woven into one instruction stream, and the
// online-softmax state's rare moves.  The layouts are described at the head of dfa_fwd_bf16.hip.
#pragma once
#include "dfa_device.h"
#include "dfa_mfma.h"

namespace dfa {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// If a lane's partial row sum of one 32-key block exceeds this, some exponent may have left
// the comfortable range and the reference exponent is moved up (see rebase_block).
constexpr float kRebaseThreshold = 256.0f;
// Reference exponent before the first score of a row (kernel variant for packed tiles): below any scaled score
// that fp32 holds with room to spare, and finite.
constexpr float kRefStart = -3.0e38f;

// Softmax numerators of one 32-key block against the current reference exponents m_ref (no
// row maximum is taken here): p = exp2(c*s - m_ref), rounded to bf16 (nearest even) and packed
// straight into the B operands of the second product; psum = the row sums of the block (whole rows:
// both lanes that share a query hold the same value), in fp32 over the unrounded values.  Plain form,
// used after a rebase; beat() takes the numerators the same way in its hand-ordered stream and has
// the matrix cores add them up.
__device__ __forceinline__ void exp_block(const floatx16 (&s)[2], float c, const float (&m_ref)[2],
                                          u32x4 (&pb)[2][2], float (&psum)[2]) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const float e0 = __builtin_amdgcn_exp2f(fmaf(s[qb][2 * v], c, -m_ref[qb]));
            const float e1 = __builtin_amdgcn_exp2f(fmaf(s[qb][2 * v + 1], c, -m_ref[qb]));
            const bf16x2 pr = {(__bf16)e0, (__bf16)e1};
            pb[qb][v >> 2][v & 3] = __builtin_bit_cast(uint32_t, pr);   // slots 2v%8, 2v%8+1 of step v/4
            a0 += e0;
            a1 += e1;
        }
        psum[qb] = wave_half_sum(a0 + a1);
    }
}

// Rare path of the online softmax: take the exact row maximum of this block, move the
// reference exponent up to it, rescale the running sum and the accumulator.
// kSkips: a query block may be skipping the progression in hand (m_ref = +inf, see the kernel): it stays as it is.
template <bool kSkips>
__device__ __forceinline__ void rebase_block(const floatx16 (&s)[2], float c, float (&m_ref)[2],
                                             float (&l_run)[2], floatx16 (&oacc)[2][2]) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        if (kSkips && m_ref[qb] == INFINITY) continue;      // wave-uniform: a block skips as a whole
        float mx = s[qb][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[qb][v]);
        mx = wave_half_max(mx);
        const float m_new = fmaxf(m_ref[qb], mx * c);
        const float alpha = __builtin_amdgcn_exp2f(m_ref[qb] - m_new);   // exp2(-inf) = 0 at the start
        m_ref[qb] = m_new;
        l_run[qb] *= alpha;
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[db][qb][v] *= alpha;
    }
}

// Lane constants of the LDS fragment reads.
struct FragLane {
    int k;        // element offset inside a 32-key K block of the 16-byte chunk for d-step 0; the chunk
                  // of d-step kk is (2*kk + g) ^ swizzle, i.e. this offset with 16*kk xor-ed in
    int v;        // element offset inside a 32-key V block of this lane's transposed-read address
};

// what a lane reads back as MFMA fragments
__device__ __forceinline__ FragLane frag_lane(int ln) {
    FragLane f;
    const int jj = ln & 31, gg = ln >> 5, i16 = ln & 15;
    f.k = jj * kRowElems + 8 * (gg ^ k_swizzle(jj));
    // transposed V fragments: within a 16-lane group lane i supplies the address of
    // V[R + i/4][C + 4*(i%4) ..] and receives V[R .. R+3][C + i]
    f.v = ((i16 >> 2) + 8 * gg) * kRowElems + 16 * ((ln >> 4) & 1) + 4 * (i16 & 3);
    return f;
}

// A operand of the row-sum products (v_mfma_f32_16x16x32_bf16 on a B operand of the second product, lane =
// 16*g4 + n): that instruction reads lane (n, g4) as contraction slots 8*g4 .. +7 of column n, so column n
// gathers the 8 keys each of lanes n, 16+n, 32+n, 48+n, which are query n of the block (slots 0-7 and
// 16-23) and query 16+n (slots 8-15 and 24-31).  Result row 4*g4 goes to register 0 of lane group g4:
// rows 0 and 8 select the slots of query n, rows 4 and 12 those of query 16+n, all other rows are zero,
// so register 0 of every lane receives the sum over all 16 keys of its own query.  (An infinite
// numerator of one query turns its neighbour's sum into NaN through a zero of the selector; either
// fails the test in settle(), which then redoes the block without the matrix cores.)
__device__ __forceinline__ bf16x8 row_sum_selector(int lane) {
    const int mrow = lane & 15, g4 = lane >> 4;
    const bool on = (mrow & 3) == 0 && ((mrow >> 2) & 1) == (g4 & 1);
    const uint32_t w = on ? 0x3f803f80u : 0u;
    return __builtin_bit_cast(bf16x8, u32x4{w, w, w, w});
}

// End of a key list: every score of a 32-key block at or past position nvalid becomes -inf.
// Register v of lane (j, g) is block position 16*(v/8) + 8*g + v%8.
__device__ __forceinline__ void mask_block(floatx16 (&s)[2], int g, int nvalid) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int pos = 16 * (v >> 3) + 8 * g + (v & 7);
        if (pos >= nvalid) {
            s[0][v] = -INFINITY;
            s[1][v] = -INFINITY;
        }
    }
}

// Scores of one 32-key block, S^T = K~ Q~^T, on their own (pipeline prologue).
__device__ __forceinline__ void scores_block(const uint16_t* kblk, const FragLane& fl, const bf16x8 (&qf)[2][4],
                                             floatx16 (&s)[2]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(kblk + (fl.k ^ (16 * kk)));
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            floatx16 z;
#pragma unroll
            for (int v = 0; v < 16; ++v) z[v] = 0.f;
            s[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[qb][kk], kk == 0 ? z : s[qb], 0, 0, 0);
        }
    }
}


// Second product of one 32-key block on its own (pipeline epilogue), for the 32-row blocks that take part.
__device__ __forceinline__ void accumulate_block(const uint16_t* vblk, const FragLane& fl, const u32x4 (&pb)[2][2],
                                                 floatx16 (&oacc)[2][2], bool first = true, bool second = true) {
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const bf16x8 vf = read_v_frag(vblk + fl.v + 16 * st * kRowElems + 32 * db);
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
                if (qb == 0 ? first : second)
                    oacc[db][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, pb[qb][st]), oacc[db][qb], 0, 0, 0);
        }
}

// The vector side of slot m of a beat's 18: exponents of score pair m, exponentials of pair m - 1, pair m - 2 rounded into its B-operand
// slot (a vector instruction that needs the result of the one just before it stalls the wave, so a pair moves one stage per slot).
// kSum: the numerators are added up before they are rounded.
template <bool kSum>
__device__ __forceinline__ void numerator_slot(int m, const floatx16 (&s_cur)[2], float c, const float (&m_ref)[2], float (&t)[16][2],
                                               u32x4 (&p_cur)[2][2], float (&sum)[2][2]) {
    if (m < 16) {
        const int qb = m >> 3, v = 2 * (m & 7);
        t[m][0] = fmaf(s_cur[qb][v], c, -m_ref[qb]);
        t[m][1] = fmaf(s_cur[qb][v + 1], c, -m_ref[qb]);
    }
    if (m >= 1 && m < 17) {
        t[m - 1][0] = __builtin_amdgcn_exp2f(t[m - 1][0]);
        t[m - 1][1] = __builtin_amdgcn_exp2f(t[m - 1][1]);
    }
    if (m >= 2) {
        const int q = m - 2, qb = q >> 3, pr = q & 7;
        const bf16x2 w = {(__bf16)t[q][0], (__bf16)t[q][1]};
        p_cur[qb][pr >> 2][pr & 3] = __builtin_bit_cast(uint32_t, w);
        if (kSum) {
            sum[qb][0] += t[q][0];
            sum[qb][1] += t[q][1];
        }
    }
}

// Row sums of the rounded numerators on the matrix cores (register 0 of rs), 16-key group by group: a group goes two slots after its last pair.
__device__ __forceinline__ void row_sum_group(int grp, const u32x4 (&p_cur)[2][2], const bf16x8& sel, floatx4 (&rs)[2]) {
    const int qb = grp >> 1, st = grp & 1;
    rs[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sel, __builtin_bit_cast(bf16x8, p_cur[qb][st]), st == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : rs[qb], 0, 0, 0);
}
__device__ __forceinline__ void row_sum_slot(int m, const u32x4 (&p_cur)[2][2], const bf16x8& sel, floatx4 (&rs)[2]) {
    if (m == 7 || m == 11 || m == 15) row_sum_group((m - 7) >> 2, p_cur, sel, rs);
}
// the last group, after the beat's slots, and the sums
__device__ __forceinline__ void row_sums(const u32x4 (&p_cur)[2][2], const bf16x8& sel, floatx4 (&rs)[2], float (&psum)[2]) {
    row_sum_group(3, p_cur, sel, rs);
    psum[0] = rs[0][0];
    psum[1] = rs[1][0];
}

// One pipeline beat (32 keys).  Three independent pieces of work are woven into one
// instruction stream, so that the matrix cores and the vector ALU of the SIMD are busy at the
// same time from within a single wave:
//   matrix cores : S^T of the NEXT block (K at k_next -> s_next), and O^T += V~^T P^T of the
//                  PREVIOUS block (V at v_prev, probabilities p_prev);
//   vector ALU   : softmax numerators of the CURRENT block (s_cur -> p_cur).
// The stream is laid out slot by slot: one MFMA, then the exponent, exponential and rounding
// instructions of three different score pairs (numerator_slot).  Whenever a 16-key group of p_cur is complete, one row-sum MFMA (selector `sel` times that group)
// adds it to psum: register 0 of its result is the sum over the group's 16 keys of the lane's query.
// Scheduling fences keep the compiler from regrouping the slots.
// kScores / kAccumulate: the beat has a next block to score / a previous block to accumulate (the first
// beat of a walk has no previous block, the last one no next block; their MFMAs and fragment reads are
// left out).
template <bool kScores, bool kAccumulate>
__device__ __forceinline__ void beat(const uint16_t* k_next, const uint16_t* v_prev, const FragLane& fl,
                                     const bf16x8 (&qf)[2][4], const floatx16 (&s_cur)[2], floatx16 (&s_next)[2],
                                     const u32x4 (&p_prev)[2][2], u32x4 (&p_cur)[2][2], floatx16 (&oacc)[2][2],
                                     float c, const float (&m_ref)[2], float (&psum)[2], const bf16x8& sel) {
    bf16x8 kf[2], vf[2];           // fragments of MFMA group r live in slot r & 1
    float t[16][2];                // exponents, then exponentials, of score pair q
    floatx4 rs[2];                 // row sums of the rounded numerators
    float no_sum[2][2];

    auto load_group = [&](int r) {     // group r: d-step r of the scores, (d block r/2, 16-key step r%2) of the accumulation
        if (kScores) kf[r & 1] = *reinterpret_cast<const bf16x8*>(k_next + (fl.k ^ (16 * r)));
        if (kAccumulate) vf[r & 1] = read_v_frag(v_prev + fl.v + 16 * (r & 1) * kRowElems + 32 * (r >> 1));
    };
    auto mfma = [&](int k) {           // MFMA k of the beat: group r = k/4; scores for query block 0, 1, then accumulation for 0, 1
        const int r = k >> 2, qb = k & 1;
        if ((k & 2) == 0) {
            if (!kScores) return;
            floatx16 z;
#pragma unroll
            for (int v = 0; v < 16; ++v) z[v] = 0.f;
            s_next[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[r & 1], qf[qb][r], r == 0 ? z : s_next[qb], 0, 0, 0);
        } else {
            if (!kAccumulate) return;
            const int db = r >> 1, st = r & 1;
            oacc[db][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[r & 1], __builtin_bit_cast(bf16x8, p_prev[qb][st]), oacc[db][qb], 0, 0, 0);
        }
    };

    load_group(0);
#pragma unroll
    for (int m = 0; m < 18; ++m) {
        // fragment reads run four slots ahead of their first MFMA
        if (m >= 2 && m < 14 && ((m - 2) & 3) == 0) load_group(((m - 2) >> 2) + 1);
        if (m >= 2 && m < 18) mfma(m - 2);
        numerator_slot<false>(m, s_cur, c, m_ref, t, p_cur, no_sum);
        row_sum_slot(m, p_cur, sel, rs);
        __builtin_amdgcn_sched_barrier(0);
    }
    row_sums(p_cur, sel, rs, psum);
}

// The wave-uniform end of a beat: accept the numerators, or (rarely) move the reference
// exponent and redo them.  oacc already holds every earlier block under the old reference.
template <bool kSkips>
__device__ __forceinline__ void settle(const floatx16 (&s_cur)[2], u32x4 (&p_cur)[2][2], float c, float (&m_ref)[2],
                                       float (&l_run)[2], floatx16 (&oacc)[2][2], float (&psum)[2]) {
    // written so that NaN (-inf - -inf before the first rebase) trips the test
    const bool calm = psum[0] <= kRebaseThreshold && psum[1] <= kRebaseThreshold;
    if (__builtin_expect(__ballot(!calm) != 0ull, 0)) {
        // one rebase always suffices for finite inputs (every p of the block is <= 1 after it)
        rebase_block<kSkips>(s_cur, c, m_ref, l_run, oacc);
        exp_block(s_cur, c, m_ref, p_cur, psum);
    }
    l_run[0] += psum[0];
    l_run[1] += psum[1];
}

}  // namespace dfa
