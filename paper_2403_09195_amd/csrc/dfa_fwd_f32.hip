// Fused dilated flash attention forward in fp32, on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: full fp32
// products and sums).
//
// Same plan and the same single online-softmax state per query row across all member branches as the bf16 kernel.
// A workgroup owns 32 query rows of a tile; its four waves walk the tile's key lists in blocks of 32 keys, wave w
// taking blocks w, w + 4, ..., each with an online softmax of its own, and merge their four partial results through
// LDS by their maxima and sums at the end.
//
// Bound: the fp32 matrix cores (64 FLOP per cycle and SIMD; 64 MFMAs of 64 cycles per 32 x 32 block of pairs beside
// some 1000 cycles of vector work, which the second wave of the SIMD covers).  One query block per workgroup gives a
// single 1024^2 image 1536 workgroups, enough to even out walks of 1024 to 2048 keys over 256 CUs; every operand read
// from LDS feeds one MFMA of 64 cycles, so LDS bandwidth is no issue and sharing a staged block between waves would save
// nothing but L2 reads.  A wave copies its own blocks global -> LDS, K and V into one buffer each: a buffer is
// refilled as soon as its product is through and has the other product's 2048 cycles to land, so no barrier and no
// second stage is needed.
//
// Measured, one 1024^2 image (12 heads x 4096 tokens, three branches): 160 us = 111 TFLOP/s of the distinct pairs, 70 % of
// the matrix cores' fp32 rate (one lane per query row on the vector units: 1048 us); error against fp64 2.3e-7 of the
// output's 2-norm (8.5e-7): a block's sums are added up on their own, so no chain of roundings is longer than 48.
#include "dfa_device.h"
#include "dfa_mfma_f32.h"

namespace dfa {

namespace {

template <bool kCut>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void dfa_fwd_f32_kernel(const FwdParams p, int n_items, int row_blocks) {
    __shared__ __attribute__((aligned(1024))) float lds[kWalkWaves][2 * kF32BlockElems];     // per wave: K block, V block
    __shared__ KeySeg records[kWalkWaves][kWalkRecords];

    hold_args(p);

    int item_index, sub;
    item_of_part(blockIdx.x, row_blocks, item_index, sub);
    if (item_index >= n_items) return;
    const Item item = load_item(p.items, item_index);
    const Tile tile = item.t;
    if (item.tile < 0 || sub * kWalkBlock >= tile.nrows) return;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int h = tile.h, b = item.b;
    const int32_t* const rows = p.rows + tile.row_begin + sub * kWalkBlock;
    const int nrows = min(kWalkBlock, tile.nrows - sub * kWalkBlock);

    // the row this thread writes: eight threads a row, 32 bytes each
    const int orow = tid >> 3, od = (tid & 7) * 8;
    const int64_t on = rows[min(orow, nrows - 1)];
    float* const out = static_cast<float*>(p.out) + (((int64_t)b * p.N + on) * p.H + h) * kD + od;
    float* const lse = p.lse ? p.lse + ((int64_t)b * p.H + h) * p.N + on : nullptr;

    if (tile.nseg == 0) {
        if (orow < nrows) {
            reinterpret_cast<float4*>(out)[0] = make_float4(0.f, 0.f, 0.f, 0.f);
            reinterpret_cast<float4*>(out)[1] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (lse && od == 0) *lse = -INFINITY;
        }
        return;
    }

    const float* const kp = static_cast<const float*>(p.k) + (int64_t)b * p.skb + (int64_t)h * p.skh;
    const float* const vp = static_cast<const float*>(p.v) + (int64_t)b * p.svb + (int64_t)h * p.svh;
    float* const k_lds = lds[wave];
    float* const v_lds = k_lds + kF32BlockElems;
    const uint32_t k_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, k_lds));
    const uint32_t v_addr = k_addr + kF32BlockBytes;

    const int64_t qn = rows[min(j, nrows - 1)];
    BlockWalk<kCut> w;
    w.start(p.segs + tile.seg_begin, tile.nseg, wave, records[wave]);
    float4 q[8];
    load_chunks(static_cast<const float*>(p.q) + (int64_t)b * p.sqb + qn * p.sqn + (int64_t)h * p.sqh, g, q);

    floatx16 acc[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;      // l_run: over the lane's own 16 keys of every block

    if (w.valid()) {
        issue_block(kp, p.skn, w, k_addr, lane);
        issue_block(vp, p.svn, w, v_addr, lane);
    }
    pin(q);
    while (w.valid()) {
        BlockWalk<kCut> nx = w;
        nx.next();
        const bool more = nx.valid();
        const int nvalid = w.rows();
        const float ln_mult = w.seg.log2_mult * kLn2;   // a key that counts m times: weight m exp(s) = exp(s + ln m)

        copies_left<kF32Copies>();                      // K is there, V may be on its way
        floatx16 s = rows_product(k_lds, q, lane);
        lds_reads_done();
        if (more) issue_block(kp, p.skn, nx, k_addr, lane);

        float mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = fmaf(s[v], p.scale, ln_mult);
        if (nvalid < kWalkBlock) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (8 * (v >> 2) + 4 * g + (v & 3) >= nvalid) s[v] = -INFINITY;
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[v]);
        const float m_new = fmaxf(m_run, wave_half_max(mx));
        const float m_use = m_new == -INFINITY ? 0.f : m_new;       // nothing but masked scores so far
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_use) * kLog2e);
        m_run = m_new;
        float pr[16], l0 = 0.f, l1 = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            pr[v] = __builtin_amdgcn_exp2f((s[v] - m_use) * kLog2e);
            (v & 1 ? l1 : l0) += pr[v];
        }
        l_run = fmaf(l_run, alpha, l0 + l1);

        if (more) copies_left<kF32Copies>();            // V is there, the next K may be on its way
        else copies_left<0>();
        if (nvalid < kWalkBlock) zero_tail(v_lds, nvalid, lane);
        // the block's sums on their own, added to the running ones once: shorter chains of roundings
        floatx16 blk[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) blk[0][v] = blk[1][v] = 0.f;
        cols_product(v_lds, pr, blk, lane);
        lds_reads_done();
        if (more) issue_block(vp, p.svn, nx, v_addr, lane);
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[db][v] = fmaf(acc[db][v], alpha, blk[db][v]);
        w = nx;
    }

    // merge of the four waves: a wave without a block has m = -inf, l = 0 and an accumulator of zeros
    l_run = wave_half_sum(l_run);
    float* const red = lds[wave];
    result_to_lds(acc, red, lane);
    if (g == 0) {
        red[kWalkBlock * kRedPitch + j] = m_run;
        red[kWalkBlock * kRedPitch + kWalkBlock + j] = l_run;
    }
    __syncthreads();
    if (orow >= nrows) return;
    float m = -INFINITY;
#pragma unroll
    for (int x = 0; x < kWalkWaves; ++x) m = fmaxf(m, lds[x][kWalkBlock * kRedPitch + orow]);
    const float m_use = m == -INFINITY ? 0.f : m;
    float l = 0.f;
    float4 o0 = make_float4(0.f, 0.f, 0.f, 0.f), o1 = o0;
#pragma unroll
    for (int x = 0; x < kWalkWaves; ++x) {
        const float* const r = lds[x];
        const float f = __builtin_amdgcn_exp2f((r[kWalkBlock * kRedPitch + orow] - m_use) * kLog2e);
        l = fmaf(r[kWalkBlock * kRedPitch + kWalkBlock + orow], f, l);
        const float4 a = *reinterpret_cast<const float4*>(r + orow * kRedPitch + od);
        const float4 c = *reinterpret_cast<const float4*>(r + orow * kRedPitch + od + 4);
        o0.x = fmaf(a.x, f, o0.x); o0.y = fmaf(a.y, f, o0.y); o0.z = fmaf(a.z, f, o0.z); o0.w = fmaf(a.w, f, o0.w);
        o1.x = fmaf(c.x, f, o1.x); o1.y = fmaf(c.y, f, o1.y); o1.z = fmaf(c.z, f, o1.z); o1.w = fmaf(c.w, f, o1.w);
    }
    const float inv = 1.0f / l;
    reinterpret_cast<float4*>(out)[0] = make_float4(o0.x * inv, o0.y * inv, o0.z * inv, o0.w * inv);
    reinterpret_cast<float4*>(out)[1] = make_float4(o1.x * inv, o1.y * inv, o1.z * inv, o1.w * inv);
    if (lse && od == 0) *lse = m + __builtin_amdgcn_logf(l) * kLn2;
}

}  // namespace

hipError_t launch_fwd_f32(const FwdParams& p, int n_items, int max_tile_rows, bool cut, hipStream_t st) {
    const int row_blocks = (max_tile_rows + kWalkBlock - 1) / kWalkBlock;
    for (int i0 = 0; i0 < n_items; i0 += kLaunchItems) {         // a grid holds fewer than 2^32 threads
        FwdParams q = p;
        q.items += i0;
        const int n = n_items - i0 < kLaunchItems ? n_items - i0 : kLaunchItems;
        const int groups = (n + kDies - 1) / kDies;
        hipLaunchKernelGGL(cut ? dfa_fwd_f32_kernel<true> : dfa_fwd_f32_kernel<false>, dim3((unsigned)groups * kDies * row_blocks), dim3(256), 0, st, q, n, row_blocks);
    }
    return hipGetLastError();
}

}  // namespace dfa
