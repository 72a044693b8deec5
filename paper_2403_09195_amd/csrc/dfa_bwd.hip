// Backward of the fused dilated attention: dq, dk, dv for a gradient dout of the merged output.
//
// The paper states no backward pass; this is the chain rule on Eq. 2 and the branch merge.  The
// merged operator is a softmax over the multiset union of a row's key lists, so with the merged
// lse of the forward pass, P(n, j) = exp(scale q_n.k_j - lse_n) per (branch, n, j) pair and
// delta_n = dout_n . out_n:
//   dv_j += P dout_n,   ds = P (dout_n . v_j - delta_n),   dq_n += scale ds k_j,   dk_j += scale ds q_n.
// P is recomputed from lse, nothing of the forward pass is stored besides out and lse.  Where the
// plan visits a pair once for the m branches that hold it, P carries the factor m (every formula
// above is linear in P).
//
// This file: the per-row preparation of the fp32 path (delta, and lse in base-2 units; the bf16 path does it in
// its dq kernel) and the fp32 path, whose products run on the bf16 matrix cores with every operand as the sum of three bf16
// numbers (see dfa_mfma_f32.h).  bf16 operands go to the kernels of dfa_bwd_bf16.hip.  In a segment the kept rows are queries
// and keys alike, so a tile's key lists are also the lists of queries that see its rows as keys: the dq workgroups walk them as
// keys, the dk/dv workgroups walk them as queries, and no gradient needs an atomic or a second pass over partial sums.
//
// Bound: the matrix cores and the vector unit together (a 32 x 32 block of pairs takes 72 MFMAs of 32 cycles for dq and 96 for
// dk and dv, and as much again to split the operands).  As in the forward a workgroup owns 32 rows of a tile and its four waves a
// quarter of the walked 32-row blocks each (small images are what fp32 training runs on: 12 heads of 1024 rows are 384 workgroups
// for either gradient kernel).  The dq and the dk/dv workgroups ride in one launch, so that together they fill the chip.
// Buffers are refilled as soon as a block's last product with them is through, each landing under a product with the other
// one.  The dk/dv workgroups hold 64 registers of split tile rows and the low parts in LDS, where the four waves share them: with all of
// them in registers the walk spills.
// Measured, forward and backward of two 512^2 images (6 heads x 1024 tokens): 60 to 64 us depending on the box (fp32 matrix
// cores 74 us), error of the gradients
// against fp64 3.6e-7 of their 2-norm (4.3e-7).
#include "dfa_device.h"
#include "dfa_mfma_f32.h"
#include <type_traits>

namespace dfa {

namespace {

// ndelta[b][h][n] = -(dout[b][n][h][:] . out[b][n][h][:]) and lse2 = lse * log2(e); 16 lanes per row, 4 d each.
// grid = (16 * rows of one image / 256, B): one image is indexed with 32-bit arithmetic.
__global__ __launch_bounds__(256)
void bwd_delta_kernel(const float* out, const float* dout, const float* lse, float* ndelta, float* lse2, int32_t H, int32_t N) {
    const uint32_t x = blockIdx.x * 256u + threadIdx.x;
    const uint32_t t = x >> 4;                                       // n * H + h
    const int part = (int)(x & 15u);
    const bool in = t < (uint32_t)N * (uint32_t)H;
    const int64_t b = blockIdx.y;
    const int64_t rowid = b * N * H + t;                             // (b, n, h) flattened
    float s = 0.f;
    if (in) {
        const float4 a = *reinterpret_cast<const float4*>(out + rowid * kD + 4 * part);
        const float4 g = *reinterpret_cast<const float4*>(dout + rowid * kD + 4 * part);
        s = (a.x * g.x + a.y * g.y) + (a.z * g.z + a.w * g.w);
    }
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1) s += __shfl_xor(s, m, 16);
    if (in && part == 0) {
        const uint32_t n = t / (uint32_t)H, h = t - n * (uint32_t)H;
        const int64_t at = (b * H + h) * N + n;
        ndelta[at] = -s;
        lse2[at] = lse[at] * kLog2e;
    }
}

// What a workgroup works on: 32 rows of a tile.
struct BwdBlock {
    Tile tile;
    int b, h, nrows;
    const int32_t* rows;
    KeySeg* records;             // LDS, kWalkRecords per wave
};

// dS of a pair, P times the difference of dP and delta.  As weights of split products they carry 2^60 in place of `scale`, so that their
// parts hold what fp32 holds (small gradients, weights of exp2(-100)), and the sums are put right at the end; differences past
// 2^67 overflow and go to fp32 products, which take `scale` at once.
template <class Rows>
__device__ __forceinline__ float score_grad(const BwdParams& p, float pr, float diff) {
    return Rows::kPlain ? pr * diff * p.scale : pr * (diff * 0x1p60f);
}
template <class Rows>
__device__ __forceinline__ float sum_factor(const BwdParams& p) { return Rows::kPlain ? 1.f : p.scale * 0x1p-60f; }
constexpr float kLeastScale = 0x1p-60f;             // below it that factor would leave fp32's normal numbers: fp32 products

// Sum of the four waves' [32][64] results times `factor`, written to rows of a contiguous [B, N, H, D] tensor.  Every wave has
// finished with its own region of LDS.  Returns whether a value of this thread's is not finite.
__device__ __forceinline__ bool write_sum(const BwdParams& p, const BwdBlock& k, float (*lds)[2 * kF32BlockElems], int tid,
                                          const floatx16 (&acc)[2], void* grad, float factor) {
    asm volatile("" : "+v"(tid));                     // nothing of what follows is worked out before the walk and kept: its registers are full
    result_to_lds(acc, lds[tid >> 6], tid & 63);
    __syncthreads();
    const int row = tid >> 3, d = (tid & 7) * 8;
    bool odd = false;
    if (row < k.nrows) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), c = a;
#pragma unroll
        for (int x = 0; x < kWalkWaves; ++x) {
            const float4 u = *reinterpret_cast<const float4*>(lds[x] + row * kRedPitch + d);
            const float4 v = *reinterpret_cast<const float4*>(lds[x] + row * kRedPitch + d + 4);
            a.x += u.x; a.y += u.y; a.z += u.z; a.w += u.w;
            c.x += v.x; c.y += v.y; c.z += v.z; c.w += v.w;
        }
        a.x *= factor; a.y *= factor; a.z *= factor; a.w *= factor;
        c.x *= factor; c.y *= factor; c.z *= factor; c.w *= factor;
        float4* const dst = reinterpret_cast<float4*>(static_cast<float*>(grad) +
                                                      (((int64_t)k.b * p.N + k.rows[row]) * p.H + k.h) * kD + d);
        dst[0] = a;
        dst[1] = c;
        odd = !(finite(a.x) & finite(a.y) & finite(a.z) & finite(a.w) & finite(c.x) & finite(c.y) & finite(c.z) & finite(c.w));
    }
    return odd;
}

// dq of the block's rows: they are queries, the lists are walked as keys.
template <class Rows, class Sum, bool kCut>
__device__ __forceinline__ bool dq_block(const BwdParams& p, const BwdBlock& k, float (*lds)[2 * kF32BlockElems], int tid) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31, g = lane >> 5;
    const float* const kb = static_cast<const float*>(p.k) + (int64_t)k.b * p.skb + (int64_t)k.h * p.skh;
    const float* const vb = static_cast<const float*>(p.v) + (int64_t)k.b * p.svb + (int64_t)k.h * p.svh;
    float* const k_lds = lds[wave];
    float* const v_lds = k_lds + kF32BlockElems;
    const uint32_t k_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, k_lds));
    const uint32_t v_addr = k_addr + kF32BlockBytes;

    const int64_t n = k.rows[min(j, k.nrows - 1)];
    BlockWalk<kCut> w;
    w.start(p.segs + k.tile.seg_begin, k.tile.nseg, wave, k.records + wave * kWalkRecords);
    LostAtOnce lost;
    Unchecked checked;                                   // second products: their rows have gone through a first one
    Rows q, go;
    load_rows(static_cast<const float*>(p.q) + (int64_t)k.b * p.sqb + n * p.sqn + (int64_t)k.h * p.sqh, g, q, lost);
    load_rows(static_cast<const float*>(p.dout) + (((int64_t)k.b * p.N + n) * p.H + k.h) * kD, g, go, lost);
    const int64_t at = ((int64_t)k.b * p.H + k.h) * p.N + n;
    float my_l = p.lse2[at], my_d = p.ndelta[at];

    Sum acc;
    acc.clear();

    if (w.valid()) {
        issue_block(vb, p.svn, w, v_addr, lane);
        issue_block(kb, p.skn, w, k_addr, lane);
    }
    pin(q);
    pin(go);
    asm volatile("" : "+v"(my_l), "+v"(my_d));
    while (w.valid()) {
        BlockWalk<kCut> nx = w;
        nx.next();
        const bool more = nx.valid();
        const int nvalid = w.rows();
        const float bias = w.seg.log2_mult;

        copies_left<kF32Copies>();                       // V is there
        const floatx16 dp = rows_product(read_rows(v_lds, go, lane), go, lane, lost);
        lds_reads_done();
        if (more) issue_block(vb, p.svn, nx, v_addr, lane);
        if (more) copies_left<kF32Copies>();             // K is there
        else copies_left<0>();
        if (nvalid < kWalkBlock) zero_tail(k_lds, nvalid, lane);
        const floatx16 s = rows_product(read_rows(k_lds, q, lane), q, lane, lost);
        float ds[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float pr = __builtin_amdgcn_exp2f(fmaf(s[v] * p.scale, kLog2e, bias) - my_l);
            ds[v] = score_grad<Rows>(p, pr, dp[v] + my_d);
        }
        if (nvalid < kWalkBlock) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (8 * (v >> 2) + 4 * g + (v & 3) >= nvalid) ds[v] = 0.f;
        }
        cols_product(read_cols(k_lds, lane), ds, acc, checked);   // dq += ds k
        lds_reads_done();
        if (more) issue_block(kb, p.skn, nx, k_addr, lane);
        w = nx;
    }
    floatx16 sum[2];
    acc.total(sum);
    return write_sum(p, k, lds, tid, sum, p.dq, sum_factor<Rows>(p)) | lost.any() | !(p.scale >= kLeastScale);
}

// dk and dv of the block's rows: they are keys, the lists are walked as queries.
template <class Rows, class Sum, bool kCut>
__device__ __forceinline__ bool dkdv_block(const BwdParams& p, const BwdBlock& k, float (*lds)[2 * kF32BlockElems],
                                           float (*stat_lds)[64], bf16x8 (*low_lds)[kLowParts], int tid) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31, g = lane >> 5;
    const float* const qb = static_cast<const float*>(p.q) + (int64_t)k.b * p.sqb + (int64_t)k.h * p.sqh;
    const float* const gb = static_cast<const float*>(p.dout) + ((int64_t)k.b * p.N * p.H + k.h) * kD;   // row n at n * H * D
    const int64_t gpitch = (int64_t)p.H * kD;
    float* const q_lds = lds[wave];
    float* const g_lds = q_lds + kF32BlockElems;
    const float* const stat = stat_lds[wave];            // lse2 of the block's 32 queries, then -delta
    const uint32_t q_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, q_lds));
    const uint32_t g_addr = q_addr + kF32BlockBytes;
    const uint32_t stat_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, stat));
    const float* const my_stat = (g == 0 ? p.lse2 : p.ndelta) + ((int64_t)k.b * p.H + k.h) * p.N;

    const int64_t n = k.rows[min(j, k.nrows - 1)];
    BlockWalk<kCut> w;
    w.start(p.segs + k.tile.seg_begin, k.tile.nseg, wave, k.records + wave * kWalkRecords);
    LostAtOnce lost;
    Unchecked checked;                                   // second products: their rows have gone through a first one
    Rows kr, vr;
    if constexpr (std::is_same<Rows, LeanRows>::value) {
        kr.low = low_lds[0];
        vr.low = low_lds[1];
    }
    load_rows(static_cast<const float*>(p.k) + (int64_t)k.b * p.skb + n * p.skn + (int64_t)k.h * p.skh, g, kr, lost);
    load_rows(static_cast<const float*>(p.v) + (int64_t)k.b * p.svb + n * p.svn + (int64_t)k.h * p.svh, g, vr, lost);

    Sum dk, dv;
    dk.clear();
    dv.clear();

    auto issue_q = [&](const BlockWalk<kCut>& w) {             // 9 copies
        issue_block(qb, p.sqn, w, q_addr, lane);
        copy4_to_lds(my_stat + (w.first() + w.seg.stride * min(j, w.rows() - 1)), stat_addr);
    };
    if (w.valid()) {
        issue_block(gb, gpitch, w, g_addr, lane);
        issue_q(w);
    }
    pin(kr);
    pin(vr);
    __syncthreads();                                     // the low parts are there
    while (w.valid()) {
        BlockWalk<kCut> nx = w;
        nx.next();
        const bool more = nx.valid();
        const int nvalid = w.rows();
        const float bias = w.seg.log2_mult;

        copies_left<kF32Copies + 1>();                   // dout is there
        if (nvalid < kWalkBlock) zero_tail(g_lds, nvalid, lane);
        const floatx16 dp = rows_product(read_rows(g_lds, vr, lane), vr, lane, lost);
        copies_left<0>();                                // q and the row statistics are there
        if (nvalid < kWalkBlock) zero_tail(q_lds, nvalid, lane);
        const floatx16 s = rows_product(read_rows(q_lds, kr, lane), kr, lane, lost);
        float pr[16], ds[16];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float4 l = *reinterpret_cast<const float4*>(stat + 8 * t + 4 * g);
            const float4 nd = *reinterpret_cast<const float4*>(stat + 32 + 8 * t + 4 * g);
            const float lv[4] = {l.x, l.y, l.z, l.w}, dv4[4] = {nd.x, nd.y, nd.z, nd.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int v = 4 * t + e;
                pr[v] = __builtin_amdgcn_exp2f(fmaf(s[v] * p.scale, kLog2e, bias) - lv[e]);
                ds[v] = score_grad<Rows>(p, pr[v], dp[v] + dv4[e]);
            }
        }
        if (nvalid < kWalkBlock) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (8 * (v >> 2) + 4 * g + (v & 3) >= nvalid) pr[v] = ds[v] = 0.f;
        }
        cols_product(read_cols(g_lds, lane), pr, dv, checked);    // dv += P dout
        lds_reads_done();
        if (more) issue_block(gb, gpitch, nx, g_addr, lane);
        cols_product(read_cols(q_lds, lane), ds, dk, checked);    // dk += ds q
        lds_reads_done();
        if (more) issue_q(nx);
        w = nx;
    }
    floatx16 sum[2];
    dv.total(sum);
    const bool odd = write_sum(p, k, lds, tid, sum, p.dv, 1.f);
    __syncthreads();
    dk.total(sum);
    return odd | write_sum(p, k, lds, tid, sum, p.dk, sum_factor<Rows>(p)) | lost.any() | !(p.scale >= kLeastScale);
}

template <bool kCut>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void bwd_f32_kernel(const BwdParams p, int n_items, int row_blocks) {
    __shared__ __attribute__((aligned(1024))) float lds[kWalkWaves][2 * kF32BlockElems];
    __shared__ __attribute__((aligned(256))) float stat_lds[kWalkWaves][64];
    __shared__ KeySeg records[kWalkWaves][kWalkRecords];
    __shared__ bf16x8 low_lds[2][kLowParts];
    __shared__ int odd_lds[kWalkWaves];

    hold_args(p);
    int item_index, part;
    item_of_part(blockIdx.x, 2 * row_blocks, item_index, part);
    if (item_index >= n_items) return;
    const int sub = part >> 1;
    const Item item = load_item(p.items, item_index);
    if (item.tile < 0 || sub * kWalkBlock >= item.t.nrows) return;
    const int tid = threadIdx.x;
    BwdBlock k;
    k.tile = item.t;
    k.b = item.b;
    k.h = item.t.h;
    k.nrows = min(kWalkBlock, item.t.nrows - sub * kWalkBlock);
    k.records = records[0];
    k.rows = p.rows + item.t.row_begin + sub * kWalkBlock;

    if (item.t.nseg == 0) {                  // rows that no branch keeps take and give no gradient
        floatx16 zero[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) zero[0][v] = zero[1][v] = 0.f;
        write_sum(p, k, lds, tid, zero, part & 1 ? p.dq : p.dv, 1.f);
        if (!(part & 1)) {
            __syncthreads();
            write_sum(p, k, lds, tid, zero, p.dk, 1.f);
        }
        return;
    }
    // operands that parts do not hold, results that are not finite: the same with fp32 products
    const bool odd = part & 1 ? dq_block<SplitRows, ChainSum, kCut>(p, k, lds, tid) : dkdv_block<LeanRows, ChainSum, kCut>(p, k, lds, stat_lds, low_lds, tid);
    const bool wave_odd = __ballot(odd) != 0ull;
    if ((tid & 63) == 0) odd_lds[tid >> 6] = wave_odd;
    __syncthreads();                         // everyone has read the partial sums as well
    if (!(odd_lds[0] | odd_lds[1] | odd_lds[2] | odd_lds[3])) return;
    if (part & 1) dq_block<PlainRows, PlainSum, kCut>(p, k, lds, tid);
    else dkdv_block<PlainRows, PlainSum, kCut>(p, k, lds, stat_lds, low_lds, tid);
}

}  // namespace

// fp32 operands: the per-row preparation, then both gradients' workgroups in one launch.  bf16 operands go to the
// matrix-core kernels of dfa_bwd_bf16.hip, whose dq kernel prepares the per-row values itself.
hipError_t launch_bwd(const BwdParams& p, int n_items, int max_tile_rows, bool cut, int32_t B, bool bf16, hipStream_t st) {
    if (bf16) return launch_bwd_bf16(p, n_items, st);
    hipLaunchKernelGGL(bwd_delta_kernel, dim3((unsigned)(((int64_t)p.N * p.H * 16 + 255) / 256), B), dim3(256), 0, st,
                       static_cast<const float*>(p.out), static_cast<const float*>(p.dout), p.lse, p.ndelta, p.lse2, p.H, p.N);
    const int row_blocks = (max_tile_rows + kWalkBlock - 1) / kWalkBlock;
    for (int i0 = 0; i0 < n_items; i0 += kLaunchItems) {         // a grid holds fewer than 2^32 threads
        BwdParams q = p;
        q.items += i0;
        const int n = n_items - i0 < kLaunchItems ? n_items - i0 : kLaunchItems;
        const int groups = (n + kDies - 1) / kDies;
        hipLaunchKernelGGL(cut ? bwd_f32_kernel<true> : bwd_f32_kernel<false>, dim3((unsigned)groups * kDies * 2 * row_blocks), dim3(256), 0, st, q, n, row_blocks);
    }
    return hipGetLastError();
}

}  // namespace dfa
