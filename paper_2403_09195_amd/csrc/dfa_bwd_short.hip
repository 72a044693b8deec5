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
// The rows that a workgroup owns are the same for its four waves: a quarter copied to LDS by each, whole lines, where every wave loaded its
// fragments itself before (32 lines touched per load, 16 loads a wave for dq: 2.8 us from the row numbers to the last one issued), and the
// waves' sums go out behind one barrier.  Backward alone, us, before / now: four images of 1024 tokens, 6 heads 23.9 / 20.6, one of 2500, 12 heads
// 47.6 / 42.9, one of 256 9.2 / 8.4, 16 of 512 90.7 / 78.3.
// Tiles of a few rows or one short list pay for rows and waves that there are not: rows past 32 that a tile does not have and waves without a block write no
// results and are not added up, no second dk/dv workgroup is launched where no tile has more than 32 rows.  Four branches, us, own rows loaded by every
// wave / copied / copied so: 106 images of 34 tokens, 2 heads 114 / 125 / 83, 22 of 13, 12 heads 69 / 73 / 49, 8 of 64, 12 heads 28.2 / 28.1 / 20.0, one of 256 9.5 / 8.4 / 8.2, of 2500 52.1 / 42.7 / 42.7.
#include "dfa_bwd_bf16.h"

namespace dfa {

namespace {

constexpr int kBuffers = 2;                        // blocks of each of the two walked tensors in a wave's LDS
constexpr int kPairElems = 2 * kBlockElems;        // one block of both tensors
constexpr int kPairBytes = kPairElems * 2;
constexpr int kMostBlocks = 64;                    // of one wave's share
constexpr int kStatRows = 64;                      // tokens of one head per workgroup of the launch for -delta and lse

__device__ __forceinline__ KeySeg read_record(const KeySeg* records, int t) {
    const KeySeg r = records[min(t, kMostBlocks - 1)];
    KeySeg k;
    k.key0 = __builtin_amdgcn_readfirstlane(r.key0);
    k.stride = __builtin_amdgcn_readfirstlane(r.stride);
    k.count = __builtin_amdgcn_readfirstlane(r.count);
    k.log2_mult = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, r.log2_mult)));
    return k;
}

// What a workgroup keeps in LDS: two of them fit a CU.
struct ShortLds {
    uint16_t blocks[kWalkWaves][kBuffers * kPairElems];
    float stats[kWalkWaves][kBuffers][2 * kWalkBlock];         // dk/dv: lse and -delta of a block
    KeySeg records[kWalkWaves][kMostBlocks];
    uint16_t own[kShortRows * kRowElems];                      // dq: query rows; dk/dv: key rows, then value rows
    int32_t rows[kShortRows];
};
static_assert(sizeof(ShortLds) <= 80 * 1024, "two workgroups to a CU");
static_assert(sizeof(ShortLds::blocks) / kWalkWaves >= kShortRows * kD * 4, "a wave's results fit its blocks");

// The two [32][64] results of a wave that walked (n blocks) into its blocks' place, rows 0 to 31 and, if `both`, 32 to 63: what sum_of_waves adds up.
__device__ __forceinline__ void results_to_lds(const floatx16 (&first)[2], const floatx16 (&second)[2], ShortLds& mem, int tid, int n, bool both) {
    float* const mine = reinterpret_cast<float*>(mem.blocks[tid >> 6]);
    if (n > 0) {
        half_to_lds(first[0], first[1], mine, 0, tid & 63);
        if (both) half_to_lds(second[0], second[1], mine, 1, tid & 63);
    }
    __syncthreads();
}
// Row tid / 4 of the sum of the first `walkers` waves' results times `scale`, this thread's 16 d of it (see result_chunk), to dst[od ..] and
// dst[od + 32 ..].
__device__ __forceinline__ void sum_of_waves(const ShortLds& mem, int tid, int walkers, float scale, uint16_t* dst) {
    const int row = tid >> 2, od = (tid & 3) * 8;
    float o[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) o[e] = 0.f;
    auto add = [&](int x) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 a = result_chunk(reinterpret_cast<const float*>(mem.blocks[x]), row, od, i);
            o[4 * i] += a.x;
            o[4 * i + 1] += a.y;
            o[4 * i + 2] += a.z;
            o[4 * i + 3] += a.w;
        }
    };
    if (walkers == kWalkWaves) {
#pragma unroll
        for (int x = 0; x < kWalkWaves; ++x) add(x);
    } else {
        for (int x = 0; x < walkers; ++x) add(x);
    }
    bf16x8 ob[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) ob[e >> 3][e & 7] = (__bf16)(o[e] * scale);
    *reinterpret_cast<bf16x8*>(dst + od) = ob[0];
    *reinterpret_cast<bf16x8*>(dst + od + 32) = ob[1];
}

// One wave-level copy of eight of the workgroup's own rows, LDS rows 8 * u8 .. +7 of a [rows][64] tile with stage_swizzle's chunks: lane L brings
// 16 bytes of row 8 * u8 + L / 8, `row` in memory.
__device__ __forceinline__ void copy_own_rows(const uint16_t* base, int64_t sn, int32_t row, int u8, uint32_t lds_addr, int lane) {
    const int slot = 8 * u8 + (lane >> 3);
    copy16_to_lds(base + row * sn + 8 * ((lane & 7) ^ stage_swizzle(slot)), lds_addr);
}

// -delta = -(dout . out) and lse in base-2 units of every row: 8 lanes a row, 16 bytes each, a workgroup takes kStatRows tokens of one head and
// writes whole lines.  (32 rows in memory order, of all heads, wrote 4 bytes to each of H lines; forward and backward of one image of 2500 tokens, 12 heads 60.2 /
// 59.6 us.  What is left of its 3 to 5 us is the trip to memory for what the forward has just written.)
__global__ __launch_bounds__(256)
void bwd_rows_short_kernel(const BwdParams p) {
    constexpr int kRows = 32, kTurns = kStatRows / kRows;
    const int part = threadIdx.x & 7, n0 = blockIdx.x * kStatRows + (threadIdx.x >> 3), h = blockIdx.y;
    const int64_t b = blockIdx.z, stat = (b * p.H + h) * p.N;
    bf16x8 go[kTurns], oo[kTurns];
    float lse[kTurns];
#pragma unroll
    for (int u = 0; u < kTurns; ++u) {
        if ((int)blockIdx.x * kStatRows + kRows * u >= p.N) break;
        const int n = min(n0 + kRows * u, p.N - 1);
        const int64_t at = ((b * p.N + n) * p.H + h) * kD + 8 * part;
        go[u] = *reinterpret_cast<const bf16x8*>(static_cast<const uint16_t*>(p.dout) + at);
        oo[u] = *reinterpret_cast<const bf16x8*>(static_cast<const uint16_t*>(p.out) + at);
        lse[u] = p.lse[stat + n];
    }
#pragma unroll
    for (int u = 0; u < kTurns; ++u) {
        const int n = n0 + kRows * u;
        if ((int)blockIdx.x * kStatRows + kRows * u >= p.N) break;
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) sum = fmaf((float)go[u][e], (float)oo[u][e], sum);
        sum += __shfl_xor(sum, 1, 8);
        sum += __shfl_xor(sum, 2, 8);
        sum += __shfl_xor(sum, 4, 8);
        if (n < p.N && part == 0) {
            p.lse2[stat + n] = lse[u] * kLog2e;
            p.ndelta[stat + n] = -sum;
        }
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
    int32_t copy_row[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) copy_row[u] = rows[min(16 * wave + 8 * u + (lane >> 3), tile.nrows - 1)];
    const int32_t lane_row = rows[min(lane, tile.nrows - 1)];
    if (tid < kShortRows) row_lds[tid] = lane_row;
    records[lane] = my_record;                         // read back by this wave alone
    const int n = (tile.nseg - wave + kWalkWaves - 1) / kWalkWaves;
    const uint32_t addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, lds[wave]));
    auto issue_keys = [&](const KeySeg& blk, int buf) {
        issue_block_rows<BlockOrder::kWalked>(k_src, blk.key0, blk.stride, blk.count, addr + buf * kPairBytes, cl);
    };
    auto issue_values = [&](const KeySeg& blk, int buf) {
        issue_block_rows<BlockOrder::kWalked>(v_src, blk.key0, blk.stride, blk.count, addr + buf * kPairBytes + kBlockBytes, cl);
    };
    // The tile's own rows, a quarter copied by each wave: queries and (in the waves' places for the values of their second blocks, which
    // are fetched once everyone has read them) dout; their lse by the first wave, -delta by the second.
    {
        const uint32_t own_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, mem.own)) + 2048u * wave;
        const uint32_t stat_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, mem.stats)) + 256u * wave;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            copy_own_rows(qp, p.sqn, copy_row[u], u, own_addr + 1024u * u, lane);
            copy_own_rows(gp, g_pitch, copy_row[u], u, addr + kPairBytes + kBlockBytes + 1024u * u, lane);
        }
        if (wave < 2) copy4_to_lds((wave == 0 ? p.lse2 : p.ndelta) + stat_bh + lane_row, stat_addr);
    }
    KeySeg cur = read_record(records, 0), nx = read_record(records, 1);
    if (n > 0) {
        issue_keys(cur, 0);
        issue_values(cur, 0);
    }
    if (n > 1) {
        issue_keys(nx, 1);
        copies_left<3 * kBlockCopies>();
    } else if (n > 0) {
        copies_left<2 * kBlockCopies>();
    } else {
        copies_left<0>();
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // everyone's own rows are there
    const int frag = j * kRowElems + 8 * (g ^ stage_swizzle(j));
    // as B operands (16 d x 32 rows): lane (j, g) holds row j, d 16*kk + 8*g .. +7
    bf16x8 qf[2][4], gf[2][4];
    float my_l2[2], my_nd[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        const uint16_t* const g_rows = lds[2 * blk + (j >> 4)] + kPairElems + kBlockElems - 16 * (j >> 4) * kRowElems;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            qf[blk][kk] = *reinterpret_cast<const bf16x8*>(mem.own + kWalkBlock * blk * kRowElems + (frag ^ (16 * kk)));
            gf[blk][kk] = *reinterpret_cast<const bf16x8*>(g_rows + (frag ^ (16 * kk)));
        }
        my_l2[blk] = (&mem.stats[0][0][0])[kWalkBlock * blk + j];
        my_nd[blk] = (&mem.stats[0][0][0])[kShortRows + kWalkBlock * blk + j];
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // everyone has read them
    if (n > 1) issue_values(nx, 1);

    const TransposedLane tl = transposed_lane(lane);
    const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, p.scale * kLog2e)));
    floatx16 acc[2][2];                                // [own 32-row block][d block], transposed
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int db = 0; db < 2; ++db) acc[blk][db] = zero16();

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
        if (t + 2 < n) {
            issue_keys(nx2, t & 1);
            issue_values(nx2, t & 1);
        }
        cur = nx;
        nx = nx2;
    }

    results_to_lds(acc[0], acc[1], mem, tid, n, tile.nrows > kWalkBlock);
    if (tid >> 2 < tile.nrows) sum_of_waves(mem, tid, min(tile.nseg, kWalkWaves), p.scale, grad + (int64_t)row_lds[tid >> 2] * g_pitch);
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
    const int32_t copy_row = rows[min(8 * wave + (lane >> 3), nrows - 1)];
    if (tid < kWalkBlock) row_lds[tid] = rows[min(tid, nrows - 1)];
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
    // the own rows, a quarter of keys and values copied by each wave
    {
        const uint32_t own_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, mem.own)) + 1024u * wave;
        copy_own_rows(kp, p.skn, copy_row, wave, own_addr, lane);
        copy_own_rows(vp, p.svn, copy_row, wave, own_addr + kBlockBytes, lane);
    }
    KeySeg cur = read_record(records, 0), nx = read_record(records, 1);
    if (n > 0) issue(cur, 0);
    if (n > 1) issue(nx, 1);
    if (n > 1) copies_left<2 * kCopies>();
    else if (n > 0) copies_left<kCopies>();
    else copies_left<0>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // everyone's own rows are there

    const int frag = j * kRowElems + 8 * (g ^ stage_swizzle(j));
    // as B operands (16 d x 32 rows): lane (j, g) holds row j, d 16*kk + 8*g .. +7
    bf16x8 kf[4], vf[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        kf[kk] = *reinterpret_cast<const bf16x8*>(mem.own + (frag ^ (16 * kk)));
        vf[kk] = *reinterpret_cast<const bf16x8*>(mem.own + kBlockElems + (frag ^ (16 * kk)));
    }
    const TransposedLane tl = transposed_lane(lane);
    const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, p.scale * kLog2e)));
    floatx16 dk_acc[2], dv_acc[2];                     // [d block], transposed: lane = own row
#pragma unroll
    for (int db = 0; db < 2; ++db) dk_acc[db] = dv_acc[db] = zero16();

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

    results_to_lds(dk_acc, dv_acc, mem, tid, n, true);
    const int own = (tid >> 2) & (kWalkBlock - 1);     // threads 0 to 127 write dk = scale dS^T q, the others dv
    if (own < nrows)
        sum_of_waves(mem, tid, min(tile.nseg, kWalkWaves), tid < 128 ? p.scale : 1.0f, (tid < 128 ? grad_k : grad_v) + (int64_t)row_lds[own] * g_pitch);
}

// The dq workgroups (an item each, padded to a multiple of the dies), then the dk/dv workgroups: the longer ones start first.
__global__ __launch_bounds__(64 * kWalkWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void bwd_short_kernel(const BwdParams p, int n_items, int n_dq, int parts) {
    __shared__ __attribute__((aligned(1024))) ShortLds mem;
    hold_args(p);
    if ((int)blockIdx.x < n_dq) {
        if ((int)blockIdx.x < n_items) dq_short(p, mem, load_item(p.items, blockIdx.x));
        return;
    }
    int item_index, sub;
    // (both counts as constants: the division by a variable one took 0.3 us of the 43 of one image of 2500 tokens)
    if (parts == 1) item_of_part((int)blockIdx.x - n_dq, 1, item_index, sub);
    else item_of_part((int)blockIdx.x - n_dq, kShortDkdvParts, item_index, sub);
    if (item_index < n_items) dkdv_short(p, mem, load_item(p.items, item_index), sub);
}

}  // namespace

hipError_t launch_bwd_short(const BwdParams& p, int n_items, int max_tile_rows, int32_t B, hipStream_t st) {
    hipLaunchKernelGGL(bwd_rows_short_kernel, dim3((unsigned)((p.N + kStatRows - 1) / kStatRows), p.H, B), dim3(256), 0, st, p);
    const int parts = short_dkdv_parts(max_tile_rows);
    for (int i0 = 0; i0 < n_items; i0 += kLaunchItems) {         // a grid holds fewer than 2^32 threads
        BwdParams q = p;
        q.items += i0;
        const int n = n_items - i0 < kLaunchItems ? n_items - i0 : kLaunchItems;
        const int n_dq = (n + kDies - 1) / kDies * kDies;
        hipLaunchKernelGGL(bwd_short_kernel, dim3((unsigned)short_backward_workgroups(n, parts)), dim3(64 * kWalkWaves), 0, st, q, n, n_dq, parts);
    }
    return hipGetLastError();
}

}  // namespace dfa
