// Fused dilated flash attention forward, bf16, for launches that do not fill the chip (one image, small images; the rule is
// short_plan's).
//
// Same arithmetic as dfa_fwd_bf16.hip, whose beat it runs (reference exponent moved only when a block's sums ask for it,
// probabilities rounded to bf16, row sums over the rounded values on the matrix cores), another split of the work: a
// workgroup owns 64 query rows and its four waves walk a quarter of the tile's 32-key blocks each (wave w takes blocks w,
// w + 4, ...), every wave with an online softmax of its own; the four partial results are merged through LDS in fp32, and
// nothing but out and lse is written.
//
// Bound: latency.  Such a launch is as long as one workgroup's start, walk and end, so the walk is cut by four where the rows
// are, not by more workgroups that have to meet in memory (partial rows written, read back and merged by a second launch).
// A wave copies its own blocks and waits for nobody until the merge.  The list comes cut into blocks: one record each, all of a
// wave's records read in one trip to memory at the start and kept in LDS.  Two workgroups to a CU (registers); a beat takes
// 0.65 us then and as much with one: a wave's own chain of wait, products and exponentials, not the rate of the copies (four
// waves' 32 KB in that time are 23 bytes per clock and CU; copies from L2 alone reach 52 to 57).  Eight waves that share the copies of a block for 128 rows
// need a barrier per beat and were slower (one image of 2500 tokens, 12 heads: 32.5 against 23.0 us).
// Measured, us against 256-row tiles with split walks: three images of 1500 tokens, 6 heads 18.2 / 25.7; one of 2500, 12
// heads 23.0 / 27.2 (18.9 now that the rests of its row groups share tiles); one of 4096, 6 heads 19.6 / 26.4.
#include "dfa_blocks.h"
#include "dfa_fwd_beat.h"

namespace dfa {

namespace {

constexpr int kBuffers = 4;                // 32-key blocks in a wave's LDS: two of K, two of V

// One 32-key block of a wave's share of the list.  Wave-uniform, in scalar registers.
struct Block {
    int32_t key0;
    int32_t stride_count;      // stride | count << 24; count 0: past the share's end, a copy of its last block without a valid key
    float log2_mult[2];        // of the keys' multiplicity for either 32-row block of the tile; -inf: they are skipped
    __device__ __forceinline__ int stride() const { return stride_count & 0xffffff; }
    __device__ __forceinline__ int count() const { return stride_count >> 24; }
};

// Lane L's record of the wave's share.
__device__ __forceinline__ u32x4 load_record(const FwdParams& p, const Tile& tile, int wave, int lane) {
    const int i = wave + kWalkWaves * lane, last = tile.nseg - 1;
    const int x = tile.seg_begin + (i <= last ? i : last >= wave ? last - ((last - wave) & (kWalkWaves - 1)) : 0);
    const KeySeg r = p.segs[x];
    const float2 m = *reinterpret_cast<const float2*>(p.block_mult + (int64_t)kTileBlocks * x);
    return u32x4{(uint32_t)r.key0, (uint32_t)(r.stride | ((i <= last ? r.count : 0) << 24)), __builtin_bit_cast(uint32_t, m.x),
                 __builtin_bit_cast(uint32_t, m.y)};
}
__device__ __forceinline__ Block read_block(const u32x4* records, int t) {
    const u32x4 r = records[min(t, 63)];
    Block b;
    b.key0 = __builtin_amdgcn_readfirstlane(r[0]);
    b.stride_count = __builtin_amdgcn_readfirstlane(r[1]);
    b.log2_mult[0] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(r[2]));
    b.log2_mult[1] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(r[3]));
    return b;
}

__global__ __launch_bounds__(64 * kWalkWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void dfa_fwd_short_kernel(const FwdParams p) {
    __shared__ __attribute__((aligned(1024))) uint16_t lds[kWalkWaves][kBuffers * kBlockElems];     // per wave: K, K, V, V
    __shared__ u32x4 records_all[kWalkWaves][64];
    __shared__ int32_t row_lds[kShortRows];
    __shared__ __attribute__((aligned(16))) uint32_t skips_lds[kWalkWaves], odd_lds[kWalkWaves];

    hold_args(p);
    const Item item = load_item(p.items, blockIdx.x);
    if (item.tile < 0) return;
    const Tile tile = item.t;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int h = tile.h, b = item.b;
    const int32_t* const rows = p.rows + tile.row_begin;

    uint16_t* const out = static_cast<uint16_t*>(p.out) + ((int64_t)b * p.N * p.H + h) * kD;     // row n adds n * H * D
    float* const lse = p.lse ? p.lse + ((int64_t)b * p.H + h) * p.N : nullptr;

    if (tile.nseg == 0) {                      // rows that no branch keeps (such tiles hold no filler slots)
        for (int x = tid; x < tile.nrows * 8; x += 64 * kWalkWaves)
            *reinterpret_cast<u32x4*>(out + (int64_t)rows[x >> 3] * p.H * kD + 8 * (x & 7)) = u32x4{0u, 0u, 0u, 0u};
        if (lse && tid < tile.nrows) lse[rows[tid]] = -INFINITY;
        return;
    }

    const BlockSource k_src = block_source(static_cast<const uint16_t*>(p.k) + (int64_t)b * p.skb + (int64_t)h * p.skh, p.skn);
    const BlockSource v_src = block_source(static_cast<const uint16_t*>(p.v) + (int64_t)b * p.svb + (int64_t)h * p.svh, p.svn);
    const BlockLane k_lane = block_lane<BlockOrder::kKeys>(lane), v_lane = block_lane<BlockOrder::kValues>(lane);
    const uint32_t k_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, lds[wave]));
    const uint32_t v_addr = k_addr + 2 * kBlockBytes;

    // the share's records and the rows of the Q fragments in one trip to memory, the fragments and the first blocks in the next
    u32x4* const records = records_all[wave];
    const u32x4 my_record = load_record(p, tile, wave, lane);
    if (tid < kShortRows) row_lds[tid] = rows[min(tid, tile.nrows - 1)];
    // Q fragments: B operand of S^T, lane (j, g) holds Q[row j][16*kk + 8*g .. +7]
    bf16x8 qf[2][4];
    auto load_q = [&](int j, int g, int last) {
        // a filler slot of a packed tile holds ~n of a row n of its group: loaded like any row, never stored
        int32_t q_row[2] = {rows[min(j, last)], rows[min(kWalkBlock + j, last)]};
        q_row[0] ^= q_row[0] >> 31;
        q_row[1] ^= q_row[1] >> 31;
        const uint16_t* const qp = static_cast<const uint16_t*>(p.q) + (int64_t)b * p.sqb + (int64_t)h * p.sqh;
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) qf[qb][kk] = *reinterpret_cast<const bf16x8*>(qp + (int64_t)q_row[qb] * p.sqn + 16 * kk + 8 * g);
    };
    load_q(j, g, tile.nrows - 1);
    records[lane] = my_record;                 // read back by this wave alone
    // blocks are walked in pairs: a wave with an odd number of them, or none, ends on a block that is masked as a whole
    const int n_pairs = max((tile.nseg - wave + 2 * kWalkWaves - 1) / (2 * kWalkWaves), 1);
    Block blk[3];                              // blocks t, t + 1 and t + 2 of the walk
#pragma unroll
    for (int x = 0; x < 3; ++x) blk[x] = read_block(records, x);
    auto issue_k = [&](const Block& b, int buf) { issue_block_rows<BlockOrder::kKeys>(k_src, b.key0, b.stride(), b.count(), k_addr + buf * kBlockBytes, k_lane); };
    auto issue_v = [&](const Block& b, int buf) { issue_block_rows<BlockOrder::kValues>(v_src, b.key0, b.stride(), b.count(), v_addr + buf * kBlockBytes, v_lane); };
    issue_k(blk[0], 0);
    issue_k(blk[1], 1);
    // does either block skip a key of the share?
    constexpr uint32_t kMinusInf = 0xff800000u;
    const bool skips = __ballot(my_record[2] == kMinusInf || my_record[3] == kMinusInf) != 0ull;
    if (lane == 0) skips_lds[wave] = skips;

    const FragLane fl = frag_lane(lane);
    const bf16x8 sel = row_sum_selector(lane);
    const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, p.scale * kLog2e)));

    floatx16 oacc[2][2];                       // [d block][query block], O^T layout
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[db][qb][v] = 0.f;
    // Per 32-row block: the reference exponent less log2 m of the keys in hand (a key that counts m times adds log2 m to
    // its score); while the block skips its keys, m_ref is +inf (every numerator an exact 0) and the reference waits in m_kept.
    float m_ref[2] = {kRefStart, kRefStart}, m_kept[2] = {kRefStart, kRefStart}, bias_cur[2] = {0.f, 0.f}, l_run[2] = {0.f, 0.f};

    // pinned: the compiler waits for the Q loads here and places no vector-memory wait of its own in the walk (it does
    // not see the copies, and a wait sized for these loads would drain them)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(qf[qb][kk]));

    // Beat t turns block t's scores into numerators, scores block t + 1 and accumulates block t - 1; buffers go by the
    // parity of the block (odd = t & 1), left = blocks from t on.
    int count = kWalkBlock;                    // valid keys of block t - 1
    // rows past the end of a block become zeros in its V buffer, so that the weights 0 they get meet finite values
    auto zero_tail = [&](int buf, int valid) {
        int ln = lane;                         // its address is worked out here, not kept in a register
        asm volatile("" : "+v"(ln));
        for (int x = ln; x < (kWalkBlock - valid) * 8; x += 64)
            *reinterpret_cast<u32x4*>(lds[wave] + buf * kBlockElems + valid * kRowElems + 8 * x) = u32x4{0u, 0u, 0u, 0u};
    };
    auto before = [&](int t, int odd, int left, floatx16 (&s)[2]) {
        lds_reads_done();                      // K of block t and V of block t - 2 have been read
        if (left > 2) issue_k(blk[2], odd);
        issue_v(blk[0], odd);
        const Block cur = blk[0];
        const int prev_count = count;
        count = cur.count();
        blk[0] = blk[1];
        blk[1] = blk[2];
        blk[2] = read_block(records, t + 3);
        if (left > 2) copies_left<8>(); else copies_left<4>();       // K of block t + 1 and V of block t - 1 are there
        if (prev_count < kWalkBlock) zero_tail(odd ? 2 : 3, prev_count);
        if (count < kWalkBlock) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            mask_block(s, ln >> 5, count);
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            const float now = cur.log2_mult[qb];
            if (now != bias_cur[qb]) {         // wave-uniform
                const float ref = bias_cur[qb] > -INFINITY ? m_ref[qb] + bias_cur[qb] : m_kept[qb];
                if (now > -INFINITY) {
                    m_ref[qb] = ref - now;
                } else {
                    m_kept[qb] = ref;
                    m_ref[qb] = INFINITY;
                }
                bias_cur[qb] = now;
            }
        }
    };
    const uint16_t* const k0 = lds[wave];
    const uint16_t* const k1 = k0 + kBlockElems;
    const uint16_t* const v0 = k0 + 2 * kBlockElems;
    const uint16_t* const v1 = k0 + 3 * kBlockElems;

    floatx16 s_a[2], s_b[2];
    u32x4 p_a[2][2], p_b[2][2];
    float psum[2];
    copies_left<4>();                          // K of block 0
    scores_block(k0, fl, qf, s_a);
    before(0, 0, 2 * n_pairs, s_a);
    beat<true, false>(k1, v1, fl, qf, s_a, s_b, p_b, p_a, oacc, c, m_ref, psum, sel);
    settle<true>(s_a, p_a, c, m_ref, l_run, oacc, psum);
    for (int s = 0; s + 1 < n_pairs; ++s) {
        before(2 * s + 1, 1, 3, s_b);
        beat<true, true>(k0, v0, fl, qf, s_b, s_a, p_a, p_b, oacc, c, m_ref, psum, sel);
        settle<true>(s_b, p_b, c, m_ref, l_run, oacc, psum);
        before(2 * s + 2, 0, 2 * (n_pairs - s) - 2, s_a);
        beat<true, true>(k1, v1, fl, qf, s_a, s_b, p_b, p_a, oacc, c, m_ref, psum, sel);
        settle<true>(s_a, p_a, c, m_ref, l_run, oacc, psum);
    }
    before(2 * n_pairs - 1, 1, 1, s_b);
    beat<false, true>(k0, v0, fl, qf, s_b, s_a, p_a, p_b, oacc, c, m_ref, psum, sel);
    settle<true>(s_b, p_b, c, m_ref, l_run, oacc, psum);
    copies_left<0>();
    if (count < kWalkBlock) zero_tail(3, count);
    accumulate_block(v1, fl, p_b, oacc);
    lds_reads_done();

    // Merge of the four waves, one 32-row block after the other: a wave without a key for a row has a row sum and an
    // accumulator of zeros under the start exponent, whose weight is an exact 0.
    static_assert(sizeof(lds[0]) >= (kWalkBlock * kRedPitch + 2 * kWalkBlock) * 4, "a wave's results fit its buffers");
    float* const red = reinterpret_cast<float*>(lds[wave]);
    // the lane's number worked out afresh: nothing that only this part needs is carried through the walk, which has no register left
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int orow = 8 * wave + (ln >> 3), od = (ln & 7) * 8;        // eight threads a row, 16 bytes each
    for (int apart = 0;; apart = 1) {
        u32x4 skips_any;
        bool odd = false;                                     // a result of this thread's is not finite
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            if (qb * kWalkBlock >= tile.nrows) break;         // uniform for the workgroup
            if (qb > 0) __syncthreads();                      // everyone has read the first block
            const floatx16 mine[2] = {oacc[0][qb], oacc[1][qb]};
            result_to_lds(mine, red, ln);
            if (ln < kWalkBlock) {
                red[kWalkBlock * kRedPitch + ln] = bias_cur[qb] > -INFINITY ? m_ref[qb] + bias_cur[qb] : m_kept[qb];
                red[kWalkBlock * kRedPitch + kWalkBlock + ln] = l_run[qb];
            }
            __syncthreads();
            if (qb == 0) skips_any = *reinterpret_cast<const u32x4*>(skips_lds);
            const int slot = qb * kWalkBlock + orow;
            const int32_t n_out = row_lds[slot];
            if (slot >= tile.nrows || n_out < 0) continue;
            float m = kRefStart;
#pragma unroll
            for (int x = 0; x < kWalkWaves; ++x) m = fmaxf(m, reinterpret_cast<const float*>(lds[x])[kWalkBlock * kRedPitch + orow]);
            float l = 0.f, o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int x = 0; x < kWalkWaves; ++x) {
                const float* const r = reinterpret_cast<const float*>(lds[x]);
                const float f = __builtin_amdgcn_exp2f(r[kWalkBlock * kRedPitch + orow] - m);
                l = fmaf(r[kWalkBlock * kRedPitch + kWalkBlock + orow], f, l);
                const float4 lo = *reinterpret_cast<const float4*>(r + orow * kRedPitch + od);
                const float4 hi = *reinterpret_cast<const float4*>(r + orow * kRedPitch + od + 4);
                const float a[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = fmaf(a[e], f, o[e]);
            }
            const float inv = 1.0f / l;
            bf16x8 ob;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                ob[e] = (__bf16)(o[e] * inv);
                odd |= !(fabsf(o[e]) <= 3.4028234e38f);
            }
            *reinterpret_cast<bf16x8*>(out + (int64_t)n_out * p.H * kD + od) = ob;
            if (lse && od == 0) lse[n_out] = (m + __builtin_amdgcn_logf(l)) * kLn2;
        }

        // A 32-row block that skips keys still scores them and multiplies their values by weights 0, which makes NaN of what is not
        // finite.  A tile with such a result walks its list once more, one block of keys at a time and without the blocks that skip it.
        // (No register of the walk above and hardly any time: one 256^2 image 6.66 us with and without, one 800^2 image 17.4, four 512^2
        // images of 6 heads, forward and backward, 35.05 and 34.95.)
        if (apart) return;
        end_unless(skips_any[0] | skips_any[1] | skips_any[2] | skips_any[3]);
        const bool wave_odd = __ballot(odd) != 0ull;
        if (ln == 0) odd_lds[wave] = wave_odd;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");     // everyone has read the partial results; the stores may be on their way
        const u32x4 odd_any = *reinterpret_cast<const u32x4*>(odd_lds);
        end_unless(odd_any[0] | odd_any[1] | odd_any[2] | odd_any[3]);
        int last = __builtin_amdgcn_readfirstlane(tile.nrows - 1);
        asm volatile("" : "+s"(last));
        load_q(ln & 31, ln >> 5, last);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            m_ref[qb] = kRefStart;
            bias_cur[qb] = l_run[qb] = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[0][qb][v] = oacc[1][qb][v] = 0.f;
        }
        for (int t = 0; wave + kWalkWaves * t < tile.nseg; ++t) {        // at most kShortBlocks / kWalkWaves: every block has its record
            const Block cur = read_block(records, t);
            issue_k(cur, 0);
            issue_v(cur, 0);
            copies_left<0>();
            if (cur.count() < kWalkBlock) zero_tail(2, cur.count());
            lds_reads_done();
            scores_block(k0, fl, qf, s_a);
            if (cur.count() < kWalkBlock) mask_block(s_a, ln >> 5, cur.count());
            const bool on[2] = {cur.log2_mult[0] > -INFINITY, cur.log2_mult[1] > -INFINITY};
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                if (on[qb]) {
                    m_ref[qb] += bias_cur[qb] - cur.log2_mult[qb];
                    bias_cur[qb] = cur.log2_mult[qb];
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v) s_a[qb][v] = -INFINITY;
                }
            }
            exp_block(s_a, c, m_ref, p_a, psum);
            settle<false>(s_a, p_a, c, m_ref, l_run, oacc, psum);
            accumulate_block(v0, fl, p_a, oacc, on[0], on[1]);
            lds_reads_done();
        }
    }
}

}  // namespace

hipError_t launch_fwd_short(const FwdParams& p, int n_items, hipStream_t st) {
    hipLaunchKernelGGL(dfa_fwd_short_kernel, dim3(n_items), dim3(64 * kWalkWaves), 0, st, p);
    return hipGetLastError();
}

}  // namespace dfa
