// Fused dilated flash attention forward, bf16, for launches that do not fill the chip (one image, small images; the rule is
// short_plan's).
//
// Same arithmetic as dfa_fwd_bf16.hip (reference exponent moved only when a block's sums ask for it,
// probabilities rounded to bf16, row sums over the rounded values on the matrix cores), another split of the work: a
// workgroup owns 64 query rows and its four waves walk a quarter of the tile's 32-key blocks each (wave w takes blocks w,
// w + 4, ...), every wave with an online softmax of its own; the four partial results are merged through LDS in fp32, and
// nothing but out and lse is written.
//
// Bound: a wave's own chain.  Such a launch is as long as one workgroup's start, walk and end, so the walk is cut by four where the rows
// are, not by more workgroups that have to meet in memory (partial rows written, read back and merged by a second launch).
// A wave copies its own blocks and waits for nobody until the merge.  The list comes cut into blocks: one record each, all of a
// wave's records read with the item and the row numbers in one trip to memory (ShortStart) and kept in LDS.  Two workgroups to a CU (registers, LDS).  A beat takes some 1700
// cycles with one wave on a SIMD and 2100 with two: 1200 for its 20 MFMAs, 32 exponentials and the rest of the softmax, the others for
// the next blocks' addresses, records and waits; the waits themselves are 40, and rings of three or four blocks (one workgroup to a CU) were
// slower (one image of 2000 tokens, 3 heads 16.5 us, 18.1 and 18.7).  Eight waves that share the copies of a block for 128 rows
// need a barrier per beat and were slower (one image of 2500 tokens, 12 heads: 32.5 against 23.0 us).
// Measured, us, before the query rows were copied once for all waves, the halves of a beat took turns, the merge took all rows at once and the
// first reference was taken ahead / now: one 256^2 image, 12 heads 6.66 / 6.13, of 512^2 8.4 / 7.8, four of 1024 tokens, 6 heads 9.9 / 8.4, three of
// 1500, 6 heads 14.05 / 13.1, one of 2500, 12 heads 15.5 / 14.3 (the start in one trip not counted yet).  Against 256-row tiles with split walks, in the launch order of before: three
// images of 1500 tokens, 6 heads 18.2 / 25.7; one of 2500, 12 heads 23.0 / 27.2; one of 4096, 6 heads 19.6 / 26.4.
#include "dfa_blocks.h"
#include "dfa_fwd_beat.h"
#include <type_traits>

namespace dfa {

namespace {

// One 32-key block of a wave's share of the list.  Wave-uniform, in scalar registers.
struct Block {
    int32_t key0;
    int32_t stride_count;      // these as in ShortRecord
    float log2_mult[2];
    __device__ __forceinline__ int stride() const { return stride_count & 0xffffff; }
    __device__ __forceinline__ int count() const { return (stride_count >> 24) & 0x3f; }
    __device__ __forceinline__ bool turns() const { return stride_count < 0; }
};
__device__ __forceinline__ Block block_of(const u32x4& r, int from_lane) {
    Block b;
    b.key0 = __builtin_amdgcn_readlane(r[0], from_lane);
    b.stride_count = __builtin_amdgcn_readlane(r[1], from_lane);
    const uint32_t m0 = __builtin_amdgcn_readlane(r[2], from_lane), m1 = __builtin_amdgcn_readlane(r[3], from_lane);
    b.log2_mult[0] = __builtin_bit_cast(float, m0);
    b.log2_mult[1] = __builtin_bit_cast(float, m1);
    return b;
}
__device__ __forceinline__ Block read_block(const u32x4* records, int t) { return block_of(records[min(t, 63)], 0); }

// Waits until at most the youngest `blocks` blocks of this wave's copies are on their way.
template <int kMost>
__device__ __forceinline__ void blocks_left(int blocks) {
    if constexpr (kMost == 0) {
        copies_left<0>();
    } else {
        if (blocks >= kMost) copies_left<kBlockCopies * kMost>();
        else blocks_left<kMost - 1>(blocks);
    }
}

// The beat of dfa_fwd_beat.h with the scores of the next block first and the accumulation of the previous one behind them, so that either
// needs its operand half a beat later, or frees it half a beat sooner.  `values` waits for the previous block's values, `keys`
// refills the buffer that the next block's keys leave.  The first beat of a walk (nothing to accumulate) adds up the numerators before
// they are rounded, as exp_block does.
template <bool kScores, bool kAccumulate, class Values, class Keys>
__device__ __forceinline__ void beat_halves(const uint16_t* k_next, const uint16_t* v_prev, const FragLane& fl, const bf16x8 (&qf)[2][4],
                                            const floatx16 (&s_cur)[2], floatx16 (&s_next)[2], const u32x4 (&p_prev)[2][2], u32x4 (&p_cur)[2][2],
                                            floatx16 (&oacc)[2][2], float c, const float (&m_ref)[2], float (&psum)[2], const bf16x8& sel,
                                            Values values, Keys keys) {
    bf16x8 f[4];                   // fragments: i < 4 d-step i of the keys, then (d block, 16-key step) i - 4 of the values, in f[i & 3]
    float t[16][2];
    floatx4 rs[2];
    float sum[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
    auto load = [&](int i) {
        if (i < 4) {
            if (kScores) f[i & 3] = *reinterpret_cast<const bf16x8*>(k_next + (fl.k ^ (16 * i)));
        } else if (kAccumulate) {
            f[i & 3] = read_v_frag(v_prev + fl.v + 16 * (i & 1) * kRowElems + 32 * ((i - 4) >> 1));
        }
    };
    auto mfma = [&](int k) {
        const int i = k >> 1, qb = k & 1;
        if (i < 4) {
            if (!kScores) return;
            floatx16 z;
#pragma unroll
            for (int v = 0; v < 16; ++v) z[v] = 0.f;
            s_next[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i & 3], qf[qb][i], i == 0 ? z : s_next[qb], 0, 0, 0);
        } else {
            if (!kAccumulate) return;
            const int db = (i - 4) >> 1, st = i & 1;
            oacc[db][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i & 3], __builtin_bit_cast(bf16x8, p_prev[qb][st]), oacc[db][qb], 0, 0, 0);
        }
    };
    load(0);
    load(1);
#pragma unroll
    for (int m = 0; m < 18; ++m) {
        if (m == 6) values();
        if (m >= 2 && m <= 12 && m % 2 == 0) load(m / 2 + 1);
        if (m >= 2) mfma(m - 2);
        numerator_slot<!kAccumulate>(m, s_cur, c, m_ref, t, p_cur, sum);
        if (kAccumulate) row_sum_slot(m, p_cur, sel, rs);
        __builtin_amdgcn_sched_barrier(0);
        if (m == 9) keys();                             // the MFMAs with the last of the keys are behind us
    }
    if (kAccumulate) {
        row_sums(p_cur, sel, rs, psum);
    } else {
        psum[0] = wave_half_sum(sum[0][0] + sum[0][1]);
        psum[1] = wave_half_sum(sum[1][0] + sum[1][1]);
    }
}

// The reference exponents of a walk's first block, taken before its numerators (which settle() would otherwise take twice: 0.1 us).
__device__ __forceinline__ void first_reference(const floatx16 (&s)[2], float c, float (&m_ref)[2]) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        float mx = s[qb][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[qb][v]);
        m_ref[qb] = fmaxf(m_ref[qb], wave_half_max(mx) * c);         // +inf, of a block that skips these keys, stays
    }
}

__global__ __launch_bounds__(64 * kWalkWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void dfa_fwd_short_kernel(const FwdParams p) {
    __shared__ __attribute__((aligned(1024))) uint16_t lds[kWalkWaves][4 * kBlockElems];     // per wave: K, K, V, V
    __shared__ __attribute__((aligned(1024))) uint16_t q_lds[kShortRows * kRowElems];
    __shared__ u32x4 records_all[kWalkWaves][64];
    __shared__ float stats[kWalkWaves][2][kShortRows];                                                   // merge: references and sums
    __shared__ int32_t row_lds[kShortRows];
    __shared__ __attribute__((aligned(16))) uint32_t skips_lds[kWalkWaves], odd_lds[kWalkWaves];

    hold_args(p);
    asm volatile("" ::"s"(p.starts), "s"(p.start_bytes));
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // All that the workgroup starts from in one trip to memory; the query rows and the first blocks come in the next.  (Item
    // first, rows and records behind it, us / now: one image of 256 tokens, 12 heads 6.16 / 6.02, three of 1500, 6 heads 13.1 / 12.6.)
    const char* const start = p.starts + (int64_t)blockIdx.x * p.start_bytes;
    const Item item = load_item(reinterpret_cast<const Item*>(start), 0);
    const int32_t* const rows = reinterpret_cast<const ShortStart*>(start)->rows;
    const int per_wave = (p.start_bytes - (int)sizeof(ShortStart)) / (int)(sizeof(ShortRecord) * kWalkWaves);
    u32x4 my_record = *reinterpret_cast<const u32x4*>(start + sizeof(ShortStart) + sizeof(ShortRecord) * (wave * per_wave + min(lane, per_wave - 1)));
    // (a filler slot of a packed tile holds ~n of a row n of its group: loaded like any row, never stored)
    int32_t q_row[2] = {rows[16 * wave + (lane >> 3)], rows[16 * wave + 8 + (lane >> 3)]}, my_row = rows[lane];
    asm volatile("" : "+v"(my_record), "+v"(q_row[0]), "+v"(q_row[1]), "+v"(my_row));
    if (item.tile < 0) return;
    const Tile tile = item.t;
    const int h = tile.h, b = item.b;

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
    const uint16_t* const q_src = static_cast<const uint16_t*>(p.q) + (int64_t)b * p.sqb + (int64_t)h * p.sqh;
    const BlockLane k_lane = block_lane<BlockOrder::kKeys>(lane), v_lane = block_lane<BlockOrder::kValues>(lane);
    const uint32_t k_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, lds[wave]));
    const uint32_t v_addr = k_addr + 2 * kBlockBytes;

    u32x4* const records = records_all[wave];
#pragma unroll
    for (int u = 0; u < 2; ++u) q_row[u] ^= q_row[u] >> 31;
    if (tid < kShortRows) row_lds[tid] = my_row;
    // The query rows are the same for all four waves: a quarter copied by each, whole lines.  (A wave that loaded its fragments itself
    // touched 32 lines with every load, 32 loads of them to a workgroup.)
    {
        const uint32_t q_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)DFA_LDS_PTR(void, q_lds)) + 2048u * wave;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int slot = 8 * u + (lane >> 3);
            copy16_to_lds(q_src + (int64_t)q_row[u] * p.sqn + 8 * ((lane & 7) ^ k_swizzle(slot)), q_addr + 1024u * u);
        }
    }
    // blocks are walked in pairs: a wave with an odd number of them, or none, ends on a block that is masked as a whole
    const int n_pairs = max((tile.nseg - wave + 2 * kWalkWaves - 1) / (2 * kWalkWaves), 1), n_blocks = 2 * n_pairs;
    Block blk[4];                              // blocks t .. t + 3 of the walk
#pragma unroll
    for (int x = 0; x < 4; ++x) blk[x] = block_of(my_record, x);
    auto issue_k = [&](const Block& b, int buf) { issue_block_rows<BlockOrder::kKeys>(k_src, b.key0, b.stride(), b.count(), k_addr + buf * kBlockBytes, k_lane); };
    auto issue_v = [&](const Block& b, int buf) { issue_block_rows<BlockOrder::kValues>(v_src, b.key0, b.stride(), b.count(), v_addr + buf * kBlockBytes, v_lane); };
    issue_k(blk[0], 0);
    issue_k(blk[1], 1);
    records[lane] = my_record;                 // read back by this wave alone
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

    // Q fragments: B operand of S^T, lane (j, g) holds Q[row j][16*kk + 8*g .. +7]
    bf16x8 qf[2][4];
    copies_left<2 * kBlockCopies>();           // this wave's share of the query rows is there
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) qf[qb][kk] = *reinterpret_cast<const bf16x8*>(q_lds + 32 * qb * kRowElems + (fl.k ^ (16 * kk)));

    // Beat t turns block t's scores into numerators, scores block t + 1 and accumulates block t - 1.  K of block t + 3 is fetched from the
    // middle of the beat on, V of block t + 1 from its end; buffers go by the parity of the block, left = blocks from t on.
    int count = kWalkBlock;                    // valid keys of block t - 1
    // rows past the end of a block become zeros in its V buffer, so that the weights 0 they get meet finite values
    auto zero_tail = [&](int buf, int valid) {
        int ln = lane;                         // its address is worked out here, not kept in a register
        asm volatile("" : "+v"(ln));
        for (int x = ln; x < (kWalkBlock - valid) * 8; x += 64)
            *reinterpret_cast<u32x4*>(lds[wave] + (2 + buf) * kBlockElems + valid * kRowElems + 8 * x) = u32x4{0u, 0u, 0u, 0u};
    };
    // block t comes up: its keys' places past the end are masked, the references follow its multiplicities
    auto enter = [&](floatx16 (&s)[2]) {
        const Block& cur = blk[0];
        if (!cur.turns()) return;
        if (cur.count() < kWalkBlock) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            mask_block(s, ln >> 5, cur.count());
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
    u32x4 coming;                              // record of block t + 4, on its way from LDS from the middle of beat t on
    // the end of beat t, odd = t & 1: V of block t + 1, and on to that block
    auto leave = [&](int odd, int left) {
        if (left > 1) issue_v(blk[1], odd ^ 1);
        count = blk[0].count();
        blk[0] = blk[1];
        blk[1] = blk[2];
        blk[2] = blk[3];
        blk[3] = block_of(coming, 0);
    };
    const uint16_t* const k_buf = lds[wave];
    const uint16_t* const v_buf = k_buf + 2 * kBlockElems;
    float psum[2];
    auto step = [&](auto first, auto last, int odd, int t, int left, floatx16 (&s_cur)[2], floatx16 (&s_next)[2], const u32x4 (&p_prev)[2][2],
                    u32x4 (&p_cur)[2][2]) {
        constexpr bool kFirst = decltype(first)::value, kLast = decltype(last)::value;
        if (!kFirst) enter(s_cur);
        // K of block t + 1 is there; sent for after it: V of block t - 1, K of block t + 2 if there is one, V of block t
        if (!kLast) blocks_left<3>(min(left, 3) - (kFirst ? 1 : 0));
        const int valid = count;
        auto values = [&]() {
            if (kFirst) return;
            blocks_left<2>(left > 2 ? 2 : 1);  // V of block t - 1; after it K of block t + 2 if there is one, V of block t
            if (valid < kWalkBlock) zero_tail(odd ^ 1, valid);
        };
        auto keys = [&]() {
            coming = records[min(t + 4, 63)];
            if (!kLast && left > 3) issue_k(blk[3], odd ^ 1);
        };
        beat_halves<!kLast, !kFirst>(k_buf + (odd ^ 1) * kBlockElems, v_buf + (odd ^ 1) * kBlockElems, fl, qf, s_cur, s_next, p_prev, p_cur, oacc, c, m_ref,
                                     psum, sel, values, keys);
        settle<true>(s_cur, p_cur, c, m_ref, l_run, oacc, psum);
        leave(odd, left);
    };
    floatx16 s_a[2], s_b[2];
    u32x4 p_a[2][2], p_b[2][2];
    using Yes = std::true_type;
    using No = std::false_type;
    copies_left<kBlockCopies>();               // K of block 0
    scores_block(k_buf, fl, qf, s_a);
    lds_reads_done();
    if (n_blocks > 2) issue_k(blk[2], 0);
    issue_v(blk[0], 0);
    enter(s_a);
    first_reference(s_a, c, m_ref);
    step(Yes{}, No{}, 0, 0, n_blocks, s_a, s_b, p_b, p_a);
    for (int s = 0; s + 1 < n_pairs; ++s) {
        step(No{}, No{}, 1, 2 * s + 1, n_blocks - 2 * s - 1, s_b, s_a, p_a, p_b);
        step(No{}, No{}, 0, 2 * s + 2, n_blocks - 2 * s - 2, s_a, s_b, p_b, p_a);
    }
    step(No{}, Yes{}, 1, n_blocks - 1, 1, s_b, s_a, p_a, p_b);
    copies_left<0>();
    if (count < kWalkBlock) zero_tail(1, count);
    accumulate_block(v_buf + kBlockElems, fl, p_b, oacc);
    lds_reads_done();

    // Merge of the four waves: a wave without a key for a row has a row sum and an accumulator of zeros under the start exponent,
    // whose weight is an exact 0.  All 64 rows at once, four threads a row: one barrier, and the chains of exponentials and divisions of
    // the two 32-row blocks side by side (1.2 us; 1.6 where the blocks took turns, with 256 threads to 32 rows).
    static_assert(sizeof(lds[0]) >= kShortRows * kD * 4, "a wave's results fit its buffers");
    float* const red = reinterpret_cast<float*>(lds[wave]);
    // the lane's number worked out afresh: nothing that only this part needs is carried through the walk, which has no register left
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int orow = 16 * wave + (ln >> 2), od = (ln & 3) * 8;       // a thread's row and its first 8 d; 8 more at od + 32
    for (int apart = 0;; apart = 1) {
        bool odd = false;                                     // a result of this thread's is not finite
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            if (qb * kWalkBlock >= tile.nrows) break;         // uniform for the workgroup
            const int r = kWalkBlock * qb + (ln & 31);
            half_to_lds(oacc[0][qb], oacc[1][qb], red, qb, ln);
            if (ln < kWalkBlock) {
                stats[wave][0][r] = bias_cur[qb] > -INFINITY ? m_ref[qb] + bias_cur[qb] : m_kept[qb];
                stats[wave][1][r] = l_run[qb];
            }
        }
        __syncthreads();
        const u32x4 skips_any = *reinterpret_cast<const u32x4*>(skips_lds);
        const int32_t n_out = row_lds[orow];
        if (orow < tile.nrows && n_out >= 0) {
            float m = kRefStart;
#pragma unroll
            for (int x = 0; x < kWalkWaves; ++x) m = fmaxf(m, stats[x][0][orow]);
            float l = 0.f, o[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) o[e] = 0.f;
#pragma unroll
            for (int x = 0; x < kWalkWaves; ++x) {
                const float f = __builtin_amdgcn_exp2f(stats[x][0][orow] - m);
                l = fmaf(stats[x][1][orow], f, l);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 a = result_chunk(reinterpret_cast<const float*>(lds[x]), orow, od, i);
                    o[4 * i] = fmaf(a.x, f, o[4 * i]);
                    o[4 * i + 1] = fmaf(a.y, f, o[4 * i + 1]);
                    o[4 * i + 2] = fmaf(a.z, f, o[4 * i + 2]);
                    o[4 * i + 3] = fmaf(a.w, f, o[4 * i + 3]);
                }
            }
            const float inv = 1.0f / l;
            bf16x8 ob[2];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                ob[e >> 3][e & 7] = (__bf16)(o[e] * inv);
                odd |= !(fabsf(o[e]) <= 3.4028234e38f);
            }
            uint16_t* const dst = out + (int64_t)n_out * p.H * kD + od;
            *reinterpret_cast<bf16x8*>(dst) = ob[0];
            *reinterpret_cast<bf16x8*>(dst + 32) = ob[1];
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
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                qf[qb][kk] = *reinterpret_cast<const bf16x8*>(q_lds + 32 * qb * kRowElems + (frag_lane(ln).k ^ (16 * kk)));
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
            if (cur.count() < kWalkBlock) zero_tail(0, cur.count());
            lds_reads_done();
            scores_block(k_buf, fl, qf, s_a);
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
            accumulate_block(v_buf, fl, p_a, oacc, on[0], on[1]);
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
