// Backward of the fused dilated attention for bf16 operands, for launches that do not fill the chip (the rule is
// short_backward_plan's).  Formulas and operand layouts are those of dfa_bwd_bf16.hip.
//
// A small launch leaves -delta and lse in base-2 units of every row in the workspace, one more works out all gradients: a
// workgroup owns 64 rows of dq, or 32 rows of dk and dv, and its four waves walk a quarter of the tile's 32-row blocks
// each (wave w takes blocks w, w + 4, ...); the four partial sums are added through LDS in fp32, in the same order every
// time.  A wave copies its own blocks, two ahead, and waits for nobody until that sum; the list comes cut into blocks,
// whose records a wave reads in one trip to memory at the start and keeps in LDS.
//
// Bound: latency.  With one wave on a SIMD a block's steps (fragments, first products, exponentials, second products) follow
// one another; the second workgroup of the CU fills the gaps.  Two workgroups to a CU are 512 slots, and a launch per gradient
// (dq working out delta) ended each on a round of its own that was nearly empty: one image of 2500 tokens, 12 heads has 528 dq
// and 1056 dk/dv workgroups.  Forward and backward of that image 81.7 -> 73.7 us in one launch for all gradients, of four images
// of 1024 tokens, 6 heads 37.6 -> 34.9 us.
#include "dfa_bwd_bf16.h"

namespace dfa {

namespace {

constexpr int kBuffers = 2;                        // blocks of each of the two walked tensors in a wave's LDS
constexpr int kPairElems = 2 * kBlockElems;        // one block of both tensors
constexpr int kPairBytes = kPairElems * 2;
constexpr int kMostBlocks = 64;                    // of one wave's share

__device__ __forceinline__ KeySeg read_record(const KeySeg* records, int t) {
    const KeySeg r = records[min(t, kMostBlocks - 1)];
    KeySeg k;
    k.key0 = __builtin_amdgcn_readfirstlane(r.key0);
    k.stride = __builtin_amdgcn_readfirstlane(r.stride);
    k.count = __builtin_amdgcn_readfirstlane(r.count);
    k.log2_mult = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, r.log2_mult)));
    return k;
}

// Sum of the four waves' [32][64] results, times `scale`, written to rows of a contiguous [B, N, H, D] tensor (`grad`
// points at image b, head h; `rows` in LDS).  Every wave has finished with its own region of LDS.
__device__ __forceinline__ void write_sum(const floatx16 (&acc)[2], uint16_t (*lds)[kBuffers * kPairElems], int tid, const int32_t* rows,
                                          int nrows, uint16_t* grad, int64_t row_pitch, float scale) {
    result_to_lds(acc, reinterpret_cast<float*>(lds[tid >> 6]), tid & 63);
    __syncthreads();
    const int row = tid >> 3, d = (tid & 7) * 8;
    if (row < nrows) {
        float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < kWalkWaves; ++x) {
            const float* const r = reinterpret_cast<const float*>(lds[x]) + row * kRedPitch + d;
            const float4 lo = *reinterpret_cast<const float4*>(r), hi = *reinterpret_cast<const float4*>(r + 4);
            const float a[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] += a[e];
        }
        bf16x8 ob;
#pragma unroll
        for (int e = 0; e < 8; ++e) ob[e] = (__bf16)(o[e] * scale);
        *reinterpret_cast<bf16x8*>(grad + (int64_t)rows[row] * row_pitch + d) = ob;
    }
}

// What a workgroup keeps in LDS: two of them fit a CU.
struct ShortLds {
    uint16_t blocks[kWalkWaves][kBuffers * kPairElems];
    float stats[kWalkWaves][kBuffers][2 * kWalkBlock];         // dk/dv: lse and -delta of a block
    KeySeg records[kWalkWaves][kMostBlocks];
    int32_t rows[kShortRows];
};
static_assert(sizeof(ShortLds) <= 80 * 1024, "two workgroups to a CU");
static_assert(sizeof(ShortLds::blocks) / kWalkWaves >= kWalkBlock * kRedPitch * 4, "a wave's results fit its blocks");

// -delta = -(dout . out) and lse in base-2 units of every row: 8 lanes a row, 16 bytes each.  grid = (8 * rows of one image /
// 256, B): one image is indexed with 32-bit arithmetic.
__global__ __launch_bounds__(256)
void bwd_rows_short_kernel(const BwdParams p) {
    const uint32_t x = blockIdx.x * 256u + threadIdx.x, t = x >> 3;      // t = n * H + h
    const bool in = t < (uint32_t)p.N * (uint32_t)p.H;
    const uint32_t h = t % (uint32_t)p.H, n = t / (uint32_t)p.H;
    const int64_t stat = ((int64_t)blockIdx.y * p.H + h) * p.N + n;
    float part = 0.f, lse = 0.f;
    if (in) {
        const int64_t at = ((int64_t)blockIdx.y * p.N * p.H + t) * kD + 8 * (x & 7u);
        const bf16x8 go = *reinterpret_cast<const bf16x8*>(static_cast<const uint16_t*>(p.dout) + at);
        const bf16x8 oo = *reinterpret_cast<const bf16x8*>(static_cast<const uint16_t*>(p.out) + at);
        if ((x & 7u) == 0) lse = p.lse[stat];
#pragma unroll
        for (int e = 0; e < 8; ++e) part = fmaf((float)go[e], (float)oo[e], part);
    }
    part += __shfl_xor(part, 1, 8);
    part += __shfl_xor(part, 2, 8);
    part += __shfl_xor(part, 4, 8);
    if (in && (x & 7u) == 0) {
        p.lse2[stat] = lse * kLog2e;
        p.ndelta[stat] = -part;
    }
}

// dq of 64 rows: they are queries, the lists are walked as keys.
__device__ __forceinline__ void dq_short(const BwdParams& p, ShortLds& mem, const Item& item) {
    uint16_t (*const lds)[kBuffers * kPairElems] = mem.blocks;
    int32_t* const row_lds = mem.rows;
    if (item.tile < 0) return;
    const Tile tile = item.t;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int h = tile.h, b = item.b;
    const int32_t* const rows = p.rows + tile.row_begin;
    const int64_t out_bh = ((int64_t)b * p.N * p.H + h) * kD, g_pitch = (int64_t)p.H * kD;   // contiguous [B, N, H, D]
    uint16_t* const grad = static_cast<uint16_t*>(p.dq) + out_bh;

    if (tile.nseg == 0) {                              // rows that no branch keeps take and give no gradient
        for (int x = tid; x < tile.nrows * 8; x += 64 * kWalkWaves)
            *reinterpret_cast<u32x4*>(grad + (int64_t)rows[x >> 3] * g_pitch + 8 * (x & 7)) = u32x4{0u, 0u, 0u, 0u};
        return;
    }

    const uint16_t* const qp = static_cast<const uint16_t*>(p.q) + (int64_t)b * p.sqb + (int64_t)h * p.sqh;
    const BlockSource k_src = block_source(static_cast<const uint16_t*>(p.k) + (int64_t)b * p.skb + (int64_t)h * p.skh, p.skn);
    const BlockSource v_src = block_source(static_cast<const uint16_t*>(p.v) + (int64_t)b * p.svb + (int64_t)h * p.svh, p.svn);
    const BlockLane cl = block_lane<BlockOrder::kWalked>(lane);
    const uint16_t* const gp = static_cast<const uint16_t*>(p.dout) + out_bh;
    const int64_t stat_bh = ((int64_t)b * p.H + h) * p.N;

    // one trip to memory for the records and the row numbers, one for everything these lead to
    KeySeg* const records = mem.records[wave];
    const KeySeg my_record = p.segs[tile.seg_begin + min(wave + kWalkWaves * lane, tile.nseg - 1)];
    const int32_t row[2] = {rows[min(j, tile.nrows - 1)], rows[min(kWalkBlock + j, tile.nrows - 1)]};
    if (tid < kShortRows) row_lds[tid] = rows[min(tid, tile.nrows - 1)];
    records[lane] = my_record;                         // read back by this wave alone
    const int n = (tile.nseg - wave + kWalkWaves - 1) / kWalkWaves;
    const uint32_t addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, lds[wave]));
    auto issue = [&](const KeySeg& blk, int buf) {
        issue_block_rows<BlockOrder::kWalked>(k_src, blk.key0, blk.stride, blk.count, addr + buf * kPairBytes, cl);
        issue_block_rows<BlockOrder::kWalked>(v_src, blk.key0, blk.stride, blk.count, addr + buf * kPairBytes + kBlockBytes, cl);
    };
    KeySeg cur = read_record(records, 0), nx = read_record(records, 1);
    float my_l2[2], my_nd[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        my_l2[blk] = p.lse2[stat_bh + row[blk]];
        my_nd[blk] = p.ndelta[stat_bh + row[blk]];
    }
    // the tile's own rows as B operands (16 d x 32 rows): lane (j, g) holds row j, d 16*kk + 8*g .. +7
    bf16x8 qf[2][4], gf[2][4];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            qf[blk][kk] = *reinterpret_cast<const bf16x8*>(qp + row[blk] * p.sqn + 16 * kk + 8 * g);
            gf[blk][kk] = *reinterpret_cast<const bf16x8*>(gp + row[blk] * g_pitch + 16 * kk + 8 * g);
        }
    if (n > 0) issue(cur, 0);
    if (n > 1) issue(nx, 1);

    const int frag = j * kRowElems + 8 * (g ^ stage_swizzle(j));
    const TransposedLane tl = transposed_lane(lane);
    const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, p.scale * kLog2e)));
    floatx16 acc[2][2];                                // [own 32-row block][d block], transposed
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int db = 0; db < 2; ++db) acc[blk][db] = zero16();

    // pinned: the compiler waits for the own rows here and places no vector-memory wait of its own in the loop (it does
    // not see the copies, and a wait sized for these loads would drain them)
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            asm volatile("" : "+v"(qf[blk][kk]));
            asm volatile("" : "+v"(gf[blk][kk]));
        }
        asm volatile("" : "+v"(my_l2[blk]));
        asm volatile("" : "+v"(my_nd[blk]));
    }

    for (int t = 0; t < n; ++t) {
        const KeySeg nx2 = read_record(records, t + 2);
        if (t + 1 < n) copies_left<2 * kBlockCopies>(); else copies_left<0>();
        const uint16_t* const kb = lds[wave] + (t & 1) * kPairElems;
        const uint16_t* const vb = kb + kBlockElems;
        floatx16 s[2], dp[2];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const bf16x8 kfr = *reinterpret_cast<const bf16x8*>(kb + (frag ^ (16 * kk)));
            const bf16x8 vfr = *reinterpret_cast<const bf16x8*>(vb + (frag ^ (16 * kk)));
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                s[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr, qf[blk][kk], kk == 0 ? zero16() : s[blk], 0, 0, 0);
                dp[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr, gf[blk][kk], kk == 0 ? zero16() : dp[blk], 0, 0, 0);
            }
        }
        u32x4 pb[2][2];                                // [own block][16-key step], packed bf16 pairs of dS
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            if (cur.count < kWalkBlock) mask_rows(s[blk], g, cur.count);
            const float off = cur.log2_mult - my_l2[blk];      // pairs that count m times: P carries the factor m
            float ds[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float pr = __builtin_amdgcn_exp2f(fmaf(s[blk][v], c, off));
                ds[v] = pr * (dp[blk][v] + my_nd[blk]);        // the factor scale goes onto the accumulator at the end
            }
            pack_block(ds, pb[blk]);
        }
        // dQ^T[d][query] += K~^T[d][key] . dS^T[key][query]
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                const bf16x8 kt = read_transposed(kb + 16 * st * kRowElems, tl, db);
#pragma unroll
                for (int blk = 0; blk < 2; ++blk)
                    acc[blk][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt, __builtin_bit_cast(bf16x8, pb[blk][st]), acc[blk][db], 0, 0, 0);
            }
        lds_reads_done();
        if (t + 2 < n) issue(nx2, t & 1);
        cur = nx;
        nx = nx2;
    }

#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        if (blk * kWalkBlock >= tile.nrows) break;     // uniform for the workgroup
        if (blk > 0) __syncthreads();                  // everyone has read the first block
        write_sum(acc[blk], lds, tid, row_lds + blk * kWalkBlock, tile.nrows - blk * kWalkBlock, grad, g_pitch, p.scale);
    }
}

// dk and dv of 32 rows, half `sub` of the tile: they are keys, the lists are walked as the queries that see them.
__device__ __forceinline__ void dkdv_short(const BwdParams& p, ShortLds& mem, const Item& item, int sub) {
    uint16_t (*const lds)[kBuffers * kPairElems] = mem.blocks;
    float (*const stats)[kBuffers][2 * kWalkBlock] = mem.stats;
    int32_t* const row_lds = mem.rows;
    if (item.tile < 0 || sub * kWalkBlock >= item.t.nrows) return;
    const Tile tile = item.t;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int h = tile.h, b = item.b;
    const int32_t* const rows = p.rows + tile.row_begin + sub * kWalkBlock;
    const int nrows = min(kWalkBlock, tile.nrows - sub * kWalkBlock);
    const int64_t out_bh = ((int64_t)b * p.N * p.H + h) * kD, g_pitch = (int64_t)p.H * kD;   // contiguous [B, N, H, D]
    uint16_t* const grad_k = static_cast<uint16_t*>(p.dk) + out_bh;
    uint16_t* const grad_v = static_cast<uint16_t*>(p.dv) + out_bh;

    if (tile.nseg == 0) {                              // rows that no branch keeps take and give no gradient
        if (tid < nrows * 8) {
            const int64_t at = (int64_t)rows[tid >> 3] * g_pitch + 8 * (tid & 7);
            *reinterpret_cast<u32x4*>(grad_k + at) = u32x4{0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4*>(grad_v + at) = u32x4{0u, 0u, 0u, 0u};
        }
        return;
    }

    const BlockSource q_src = block_source(static_cast<const uint16_t*>(p.q) + (int64_t)b * p.sqb + (int64_t)h * p.sqh, p.sqn);
    const BlockSource g_src = block_source(static_cast<const uint16_t*>(p.dout) + out_bh, g_pitch);
    const BlockLane cl = block_lane<BlockOrder::kWalked>(lane);
    const uint16_t* const kp = static_cast<const uint16_t*>(p.k) + (int64_t)b * p.skb + (int64_t)h * p.skh;
    const uint16_t* const vp = static_cast<const uint16_t*>(p.v) + (int64_t)b * p.svb + (int64_t)h * p.svh;
    const int64_t stat_bh = ((int64_t)b * p.H + h) * p.N;

    KeySeg* const records = mem.records[wave];
    const KeySeg my_record = p.segs[tile.seg_begin + min(wave + kWalkWaves * lane, tile.nseg - 1)];
    const int64_t row = rows[min(j, nrows - 1)];
    if (tid < kWalkBlock) row_lds[tid] = (int32_t)row;
    // the own rows as B operands (16 d x 32 rows): lane (j, g) holds row j, d 16*kk + 8*g .. +7
    bf16x8 kf[4], vf[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        kf[kk] = *reinterpret_cast<const bf16x8*>(kp + row * p.skn + 16 * kk + 8 * g);
        vf[kk] = *reinterpret_cast<const bf16x8*>(vp + row * p.svn + 16 * kk + 8 * g);
    }
    records[lane] = my_record;                         // read back by this wave alone
    const int n = (tile.nseg - wave + kWalkWaves - 1) / kWalkWaves;
    const uint32_t addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, lds[wave]));
    const uint32_t stat_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, stats[wave][0]));
    const float* const lane_stat = (g ? p.ndelta : p.lse2) + stat_bh;       // lanes 0 to 31 bring lse, 32 to 63 -delta
    auto issue = [&](const KeySeg& blk, int buf) {
        issue_block_rows<BlockOrder::kWalked>(q_src, blk.key0, blk.stride, blk.count, addr + buf * kPairBytes, cl);
        issue_block_rows<BlockOrder::kWalked>(g_src, blk.key0, blk.stride, blk.count, addr + buf * kPairBytes + kBlockBytes, cl);
        copy4_to_lds(lane_stat + (blk.key0 + (int64_t)blk.stride * min(j, blk.count - 1)), stat_addr + buf * (2 * kWalkBlock * 4));
    };
    constexpr int kCopies = 2 * kBlockCopies + 1;
    KeySeg cur = read_record(records, 0), nx = read_record(records, 1);
    if (n > 0) issue(cur, 0);
    if (n > 1) issue(nx, 1);

    const int frag = j * kRowElems + 8 * (g ^ stage_swizzle(j));
    const TransposedLane tl = transposed_lane(lane);
    const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, p.scale * kLog2e)));
    floatx16 dk_acc[2], dv_acc[2];                     // [d block], transposed: lane = own row
#pragma unroll
    for (int db = 0; db < 2; ++db) dk_acc[db] = dv_acc[db] = zero16();
    // pinned, as in the dq kernel
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        asm volatile("" : "+v"(kf[kk]));
        asm volatile("" : "+v"(vf[kk]));
    }

    for (int t = 0; t < n; ++t) {
        const KeySeg nx2 = read_record(records, t + 2);
        if (t + 1 < n) copies_left<kCopies>(); else copies_left<0>();
        const uint16_t* const qb = lds[wave] + (t & 1) * kPairElems;
        const uint16_t* const gb = qb + kBlockElems;
        const float* const st_l = stats[wave][t & 1] + 8 * g;
        floatx16 s, dp = load_ndelta(st_l + kWalkBlock);       // dp ends up as dP - delta
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const bf16x8 qfr = *reinterpret_cast<const bf16x8*>(qb + (frag ^ (16 * kk)));
            const bf16x8 gfr = *reinterpret_cast<const bf16x8*>(gb + (frag ^ (16 * kk)));
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qfr, kf[kk], kk == 0 ? zero16() : s, 0, 0, 0);
            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gfr, vf[kk], dp, 0, 0, 0);
        }
        if (cur.count < kWalkBlock) mask_rows(s, g, cur.count);
        float pr[16], ds[16];
        if (cur.log2_mult == 0.f) probs_block<false>(s, dp, st_l, c, 0.f, pr, ds);
        else probs_block<true>(s, dp, st_l, c, cur.log2_mult, pr, ds);
        u32x4 pp[2], ps[2];
        pack_block(pr, pp);
        pack_block(ds, ps);
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                const bf16x8 qt = read_transposed(qb + 16 * st * kRowElems, tl, db);
                const bf16x8 gt = read_transposed(gb + 16 * st * kRowElems, tl, db);
                dv_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gt, __builtin_bit_cast(bf16x8, pp[st]), dv_acc[db], 0, 0, 0);
                dk_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qt, __builtin_bit_cast(bf16x8, ps[st]), dk_acc[db], 0, 0, 0);
            }
        lds_reads_done();
        if (t + 2 < n) issue(nx2, t & 1);
        cur = nx;
        nx = nx2;
    }

    write_sum(dk_acc, lds, tid, row_lds, nrows, grad_k, g_pitch, p.scale);     // dk = scale dS^T q
    __syncthreads();                                   // everyone has read dk
    write_sum(dv_acc, lds, tid, row_lds, nrows, grad_v, g_pitch, 1.0f);
}

// The dq workgroups (an item each, padded to a multiple of the dies), then the dk/dv workgroups: the longer ones start first.
__global__ __launch_bounds__(64 * kWalkWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void bwd_short_kernel(const BwdParams p, int n_items, int n_dq) {
    __shared__ __attribute__((aligned(1024))) ShortLds mem;
    hold_args(p);
    if ((int)blockIdx.x < n_dq) {
        if ((int)blockIdx.x < n_items) dq_short(p, mem, load_item(p.items, blockIdx.x));
        return;
    }
    int item_index, sub;
    item_of_part((int)blockIdx.x - n_dq, kShortDkdvParts, item_index, sub);
    if (item_index < n_items) dkdv_short(p, mem, load_item(p.items, item_index), sub);
}

}  // namespace

hipError_t launch_bwd_short(const BwdParams& p, int n_items, int32_t B, hipStream_t st) {
    const int64_t lanes = (int64_t)p.N * p.H * 8;
    hipLaunchKernelGGL(bwd_rows_short_kernel, dim3((unsigned)((lanes + 255) / 256), B), dim3(256), 0, st, p);
    for (int i0 = 0; i0 < n_items; i0 += kLaunchItems) {         // a grid holds fewer than 2^32 threads
        BwdParams q = p;
        q.items += i0;
        const int n = n_items - i0 < kLaunchItems ? n_items - i0 : kLaunchItems;
        const int n_dq = (n + kDies - 1) / kDies * kDies;
        hipLaunchKernelGGL(bwd_short_kernel, dim3((unsigned)short_backward_workgroups(n)), dim3(64 * kWalkWaves), 0, st, q, n, n_dq);
    }
    return hipGetLastError();
}

}  // namespace dfa
