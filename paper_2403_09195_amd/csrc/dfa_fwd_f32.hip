// Fused dilated flash attention forward in fp32.  The products run on the bf16 matrix cores, every operand as the sum of three bf16
// numbers (see dfa_mfma_f32.h), sums in fp32.
//
// Same plan and the same single online-softmax state per query row across all member branches as the bf16 kernel.
// A workgroup owns 32 query rows of a tile; its four waves walk the tile's key lists in blocks of 32 keys, wave w
// taking blocks w, w + 4, ..., each with an online softmax of its own, and merge their four partial results through
// LDS by their reference exponents and sums at the end.
//
// Bound: the matrix cores and the vector unit together.  A 32 x 32 block of pairs takes 48 MFMAs of 32 cycles and some 400 vector
// instructions, two thirds of them to split K, V and the weights (of which the subtractions take turns with the MFMAs); with fp32
// MFMAs the block took 64 of 64 cycles.  One query block per workgroup gives a single 1024^2 image 1536 workgroups, enough to even out
// walks of 1024 to 2048 keys over 256 CUs.  A wave copies its own blocks global -> LDS, K and V into one buffer each: a buffer is
// refilled as soon as its block is in registers and has the rest of the beat to land, so no barrier and no second stage is needed.
//
// Measured, one 1024^2 image (12 heads x 4096 tokens, three branches): 122 to 131 us depending on the box, 126 us =
// 141 TFLOP/s of the distinct pairs (160 us on the fp32 matrix cores, whose rate is 157 TFLOP/s); error against fp64 1.8e-7 of the output's 2-norm (2.3e-7), of lse 3.3e-8 (3.4e-8).
#include "dfa_device.h"
#include "dfa_mfma_f32.h"

namespace dfa {

namespace {

// Natural logarithm of 2^m l: the exponent of l goes to m, a = m + exponent with its rounding error e, so that what is left for
// the hardware's logarithm is below 1 in magnitude; ln 2 to twice fp32's digits.
__device__ __forceinline__ float log_sum(float m, float l) {
    const float k = (float)__builtin_amdgcn_frexp_expf(l), b = __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(l));
    const float a = m + k, kk = a - m, e = (m - (a - kk)) + (k - kk);
    if (!(fabsf(a) <= 3.4028234e38f) || !(fabsf(b) <= 3.4028234e38f)) return m + b;      // no key, or nothing that a number holds
    constexpr float kLn2Rest = 0.6931471805599453094 - (double)kLn2;
    return fmaf(a, kLn2, fmaf(a, kLn2Rest, (e + b) * kLn2));
}

// How far, in powers of two, a block's weights may pass the reference exponent before it is moved up (walks with fp32 products: not at
// all, so that values next to fp32's largest do not overflow for it).
template <class Rows> constexpr float kHeadroom = Rows::kPlain ? 0.f : 8.f;

// The walk of one wave over its share of the lists; its partial result (rows, maxima, sums) goes into its region of LDS.
// Rows, Sum: how the products are taken.  Returns whether the parts of an operand of this lane's leave something out.
template <class Rows, class Sum, bool kCut>
__device__ __forceinline__ bool walk(const FwdParams& p, const Tile& tile, int b, int64_t qn, float* k_lds, KeySeg* records, int wave, int lane) {
    const int j = lane & 31, g = lane >> 5, h = tile.h;
    const float* const kp = static_cast<const float*>(p.k) + (int64_t)b * p.skb + (int64_t)h * p.skh;
    const float* const vp = static_cast<const float*>(p.v) + (int64_t)b * p.svb + (int64_t)h * p.svh;
    float* const v_lds = k_lds + kF32BlockElems;
    const uint32_t k_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, k_lds));
    const uint32_t v_addr = k_addr + kF32BlockBytes;

    BlockWalk<kCut> w;
    w.start(p.segs + tile.seg_begin, tile.nseg, wave, records);
    Lost lost;
    Rows q;
    load_rows(static_cast<const float*>(p.q) + (int64_t)b * p.sqb + qn * p.sqn + (int64_t)h * p.sqh, g, q, lost);

    Sum acc;
    acc.clear();
    const float c = p.scale * kLog2e;          // scores in base-2 units (scale > 0)
    float m_ref = -INFINITY, l_run = 0.f;      // l_run: over the lane's own 16 keys of every block

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
        const float mult = rintf(__builtin_amdgcn_exp2f(w.seg.log2_mult));         // a key that counts m times has weight m exp2(t)

        copies_left<kF32Copies>();                      // K is there, V may be on its way
        const BlockRows kr = read_rows(k_lds, q, lane);
        lds_reads_done();
        if (more) issue_block(kp, p.skn, nx, k_addr, lane);
        floatx16 s = rows_product(kr, q, lane, lost);

        if (nvalid < kWalkBlock) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (8 * (v >> 2) + 4 * g + (v & 3) >= nvalid) s[v] = -INFINITY;
        }
        // (rounded to fp32 before the reference is taken off: the largest score then has weight 1 exactly)
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] *= c;
        float t_max = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) t_max = fmaxf(t_max, s[v]);
        t_max = wave_half_max(t_max);
        // The reference exponent moves only where weights would pass 2^kHeadroom: fp32 holds them as exactly as those below 1.
        if (__ballot(!(t_max <= m_ref + kHeadroom<Rows>)) != 0ull) {
            const float m_new = fmaxf(m_ref, t_max);
            const float alpha = m_ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_ref - m_new);
            m_ref = m_new;
            l_run *= alpha;
            acc.scale(alpha);
        }
        const float ref = m_ref == -INFINITY ? 0.f : m_ref;        // nothing but masked or infinitely low scores so far
        float pr[16], l0 = 0.f, l1 = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) pr[v] = __builtin_amdgcn_exp2f(s[v] - ref);
        if (mult != 1.f) {
#pragma unroll
            for (int v = 0; v < 16; ++v) pr[v] *= mult;
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) (v & 1 ? l1 : l0) += pr[v];
        l_run += l0 + l1;

        if (more) copies_left<kF32Copies>();            // V is there, the next K may be on its way
        else copies_left<0>();
        if (nvalid < kWalkBlock) zero_tail(v_lds, nvalid, lane);
        const BlockCols vc = read_cols(v_lds, lane);
        lds_reads_done();
        if (more) issue_block(vp, p.svn, nx, v_addr, lane);
        cols_product(vc, pr, acc, lost);
        w = nx;
    }

    l_run = wave_half_sum(l_run);
    floatx16 sum[2];
    acc.total(sum);
    result_to_lds(sum, k_lds, lane);
    if (g == 0) {
        k_lds[kWalkBlock * kRedPitch + j] = m_ref;
        k_lds[kWalkBlock * kRedPitch + kWalkBlock + j] = l_run;
    }
    return lost.any();
}

// kPlain: fp32 products from the start, for plans whose lists are one block each: a single block is not worth the code of both walks,
// which a short launch has to fetch (windows of 32, four images of 256 tokens, 12 heads: 7.7 us, split 8.1; windows of 64 9.5 / 9.3).
template <bool kCut, bool kPlain>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void dfa_fwd_f32_kernel(const FwdParams p, int n_items, int row_blocks) {
    __shared__ __attribute__((aligned(1024))) float lds[kWalkWaves][2 * kF32BlockElems];     // per wave: K block, V block
    __shared__ KeySeg records[kWalkWaves][kWalkRecords];
    __shared__ __attribute__((aligned(16))) uint32_t odd_lds[kWalkWaves];

    hold_args(p);

    int item_index, sub;
    item_of_part(blockIdx.x, row_blocks, item_index, sub);
    if (item_index >= n_items) return;
    const Item item = load_item(p.items, item_index);
    const Tile tile = item.t;
    if (item.tile < 0 || sub * kWalkBlock >= tile.nrows) return;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31;
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

    const int64_t qn = rows[min(j, nrows - 1)];
    // merge of the four waves: a wave without a block has m = -inf, l = 0 and an accumulator of zeros.  Returns whether a
    // result of this thread's is not finite.
    auto merge = [&]() {
        __syncthreads();
        bool odd = false;
        if (orow < nrows) {
            float m = -INFINITY;
#pragma unroll
            for (int x = 0; x < kWalkWaves; ++x) m = fmaxf(m, lds[x][kWalkBlock * kRedPitch + orow]);
            const float m_use = m == -INFINITY ? 0.f : m;
            float l = 0.f, o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int x = 0; x < kWalkWaves; ++x) {
                const float* const r = lds[x];
                const float f = __builtin_amdgcn_exp2f(r[kWalkBlock * kRedPitch + orow] - m_use);
                l = fmaf(r[kWalkBlock * kRedPitch + kWalkBlock + orow], f, l);
                const float4 lo = *reinterpret_cast<const float4*>(r + orow * kRedPitch + od);
                const float4 hi = *reinterpret_cast<const float4*>(r + orow * kRedPitch + od + 4);
                const float a[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = fmaf(a[e], f, o[e]);
            }
            const float inv = 1.0f / l, row_lse = log_sum(m, l);
            odd = !finite(row_lse);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                o[e] *= inv;
                odd |= !finite(o[e]);
            }
            reinterpret_cast<float4*>(out)[0] = make_float4(o[0], o[1], o[2], o[3]);
            reinterpret_cast<float4*>(out)[1] = make_float4(o[4], o[5], o[6], o[7]);
            if (lse && od == 0) *lse = row_lse;
        }
        return odd;
    };
    if constexpr (!kPlain) {
        const bool lost = walk<SplitRows, SplitSum, kCut>(p, tile, b, qn, lds[wave], records[wave], wave, lane);
        const bool wave_odd = __ballot(merge() | lost) != 0ull;
        if (lane == 0) odd_lds[wave] = wave_odd;
        __syncthreads();                                      // everyone has read the partial results as well
        const u32x4 odd_any = *reinterpret_cast<const u32x4*>(odd_lds);
        end_unless(odd_any[0] | odd_any[1] | odd_any[2] | odd_any[3]);
    }
    walk<PlainRows, PlainSum, kCut>(p, tile, b, qn, lds[wave], records[wave], wave, lane);
    merge();
}

}  // namespace

hipError_t launch_fwd_f32(const FwdParams& p, int n_items, int max_tile_rows, bool cut, bool one_block, hipStream_t st) {
    const int row_blocks = (max_tile_rows + kWalkBlock - 1) / kWalkBlock;
    const auto kernel = one_block ? &dfa_fwd_f32_kernel<true, true> : cut ? &dfa_fwd_f32_kernel<true, false> : &dfa_fwd_f32_kernel<false, false>;
    for (int i0 = 0; i0 < n_items; i0 += kLaunchItems) {         // a grid holds fewer than 2^32 threads
        FwdParams q = p;
        q.items += i0;
        const int n = n_items - i0 < kLaunchItems ? n_items - i0 : kLaunchItems;
        const int groups = (n + kDies - 1) / kDies;
        hipLaunchKernelGGL(kernel, dim3((unsigned)groups * kDies * row_blocks), dim3(256), 0, st, q, n, row_blocks);
    }
    return hipGetLastError();
}

}  // namespace dfa
