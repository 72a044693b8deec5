// Projections either side of the attention operator inside an encoder layer (the ViT
// self-attention block of section 3.1: a fused QKV projection before the operator, an output
// projection after it): y = x . w^T, bf16 operands on the gfx950 matrix cores, fp32
// accumulation, result rounded to bf16 (nearest even).
//
// One workgroup of 8 waves owns a 256 x BN tile of y (BN = 256 or 128) and walks K in steps
// of 64.  Both operand tiles have their K elements contiguous in memory (x rows and w rows),
// so both go global -> LDS as 128-byte rows (global_load_lds, 16 bytes per lane, no staging
// registers) into two alternating stages, with the 16-byte chunks of a row XOR-swizzled so
// that the fragment reads are free of bank conflicts, and both are read back as 16-byte MFMA
// fragments.  What limits the kernel is the byte rate of the CU's vector memory path (copies in,
// results out), so the tile is as large as LDS allows and the results leave as whole 128-byte
// lines.
//
// Matrix-core mapping (v_mfma_f32_16x16x32_bf16; lane = 16*g4 + r16): A operand = 16 weight rows (output
// features) x 32 k, B operand = 32 k x 16 x-rows, each lane supplying 8 consecutive k of row r16.  The result
// then has one x-row (one row of y) per lane and 4 consecutive output features in its 4 registers.  A wave
// computes 128 rows x BN/4 features: per 32 k it reads 8 + BN/64 fragments and issues 8 * BN/64 MFMAs.  (The
// 32x32x16 instruction does the same work in half as many issues but with twice the accumulator traffic
// per FLOP; under this part's power limit the 16x16x32 form is the faster one: 115 us against 123 us on the
// QKV projection of the stack workload.)
// Epilogue: each wave rounds its results to bf16, lays them out row-major in its own piece of
// LDS (the stages are free by then) and stores them 16 bytes per lane, eight lanes to a row.
#include "dfa_device.h"
#include "dfa_mfma.h"

namespace dfa {

namespace {

constexpr int kLinBM = 256;                // rows of y per workgroup
constexpr int kLinBK = 64;                 // k elements per stage: one 128-byte LDS row
constexpr int kLinStages = 2;

typedef float floatx4 __attribute__((ext_vector_type(4)));

// 16-byte chunk swizzle: chunk c of LDS row rho sits at chunk c ^ swizzle(rho).  Eight consecutive
// rows then spread one chunk column over all 64 banks (a fragment read takes row r16 of a 16-row block).
__device__ __forceinline__ int lin_swizzle(int rho) { return rho & 7; }

// The 256 x BN tile of y at (m0, n0): y[m][n] = sum_k x[m][k] * w[n][k].  lds: the workgroup's LDS (two stages
// of a 256-row x tile and a BN-row w tile).
template <int BN>
__device__ __forceinline__ void linear_tile(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                                            uint16_t* __restrict__ y, int K, int64_t ldx, int64_t ldw, int64_t ldy,
                                            int64_t m0, int64_t n0, char* lds) {
    constexpr int NT = BN / 64;            // 16-feature blocks per wave
    constexpr uint32_t kXStageBytes = kLinBM * kLinBK * 2, kWStageBytes = BN * kLinBK * 2;
    constexpr uint32_t kXBytes = kLinStages * kXStageBytes;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r16 = lane & 15, g4 = lane >> 4;

    // ---- copies: a copy fills 8 rows of 128 bytes; lane L lands at row L/8, chunk L%8 and fetches
    // the source chunk that the swizzle puts there.  Wave `wave` fills x rows 32*wave .. +31
    // (4 copies) and w rows (BN/8)*wave .. (BN/64 copies: 4 + BN/64 per wave and stage); both starts are multiples of 8, so
    // the swizzle of row 8u + L/8 of a wave's share is L/8.
    const int r8 = lane >> 3;
    const int chunk = (lane & 7) ^ lin_swizzle(r8);
    const uint32_t x_off = (uint32_t)(r8 * ldx * 2 + 16 * chunk);      // byte offset of this lane inside an 8-row group
    const uint32_t w_off = (uint32_t)(r8 * ldw * 2 + 16 * chunk);
    const uint32_t lds_addr = (uint32_t)(uintptr_t)DFA_LDS_PTR(void, &lds[0]);

    auto issue = [&](int ks, int stage) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int row = 32 * wave + 8 * u;
            copy16_to_lds(uniform_ptr(x + (m0 + row) * ldx + (int64_t)ks * kLinBK), x_off,
                       lds_addr + stage * kXStageBytes + row * 128);
        }
#pragma unroll
        for (int u = 0; u < BN / 64; ++u) {
            const int row = (BN / 8) * wave + 8 * u;
            copy16_to_lds(uniform_ptr(w + (n0 + row) * ldw + (int64_t)ks * kLinBK), w_off,
                       lds_addr + kXBytes + stage * kWStageBytes + row * 128);
        }
    };

    // ---- fragments: lane (j, g) reads row j of a 32-row block, chunk (2*kk + g) ^ swizzle(j)
    const int wm = wave >> 2, wn = wave & 3;
    const int frag = r16 * kLinBK + 8 * (g4 ^ lin_swizzle(r16));       // element offset for k half 0; half 1 xors 32 in
    const int x_rows = 128 * wm, w_rows = (BN / 4) * wn;               // first row of this wave in the two tiles

    floatx4 acc[NT][8];                    // [16-feature block][16-row block]: lane (g4, r16), register i = y[row r16][feature 4*g4 + i]
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < 8; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int n_k = K / kLinBK;
    issue(0, 0);
    for (int ks = 0; ks < n_k; ++ks) {
        const int stage = ks & 1;
        wait_vmcnt<0>();       // this wave's share of stage ks has landed
        __syncthreads();           // everyone's has, and everyone is done reading the other stage
        if (ks + 1 < n_k) issue(ks + 1, stage ^ 1);
        const uint16_t* xs = reinterpret_cast<const uint16_t*>(lds + stage * kXStageBytes) + x_rows * kLinBK;
        const uint16_t* ws = reinterpret_cast<const uint16_t*>(lds + kXBytes + stage * kWStageBytes) + w_rows * kLinBK;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) {
            bf16x8 wf[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                wf[nt] = *reinterpret_cast<const bf16x8*>(ws + 16 * nt * kLinBK + (frag ^ (32 * kh)));
#pragma unroll
            for (int mh = 0; mh < 2; ++mh) {
                bf16x8 xf[4];
#pragma unroll
                for (int m4 = 0; m4 < 4; ++m4)
                    xf[m4] = *reinterpret_cast<const bf16x8*>(xs + 16 * (4 * mh + m4) * kLinBK + (frag ^ (32 * kh)));
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int m4 = 0; m4 < 4; ++m4)
                        acc[nt][4 * mh + m4] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nt], xf[m4], acc[nt][4 * mh + m4], 0, 0, 0);
            }
        }
    }

    // ---- epilogue.  Lane (g4, r16) holds row x_rows + 16*mt + r16 of the tile; its registers 0..3 of
    // block nt are features w_rows + 16*nt + 4*g4 .. +3.  Each wave transposes 64 rows at a time through
    // its own piece of LDS: rows of BN/4 features (64 or 128 bytes) at a pitch of 16 bytes more, written 8
    // bytes per lane, read back 16 bytes per lane with consecutive lanes along a row, and stored as whole
    // rows of the wave's tile.
    __syncthreads();               // every wave is done with the stages
    constexpr int kRowBytes = (BN / 4) * 2, kPitch = kRowBytes + 16, kLanesPerRow = kRowBytes / 16;
    constexpr int kRowsPerStore = 64 / kLanesPerRow;
    char* mine = lds + wave * (64 * kPitch);
    const int srow = lane / kLanesPerRow, schunk = lane % kLanesPerRow;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int m4 = 0; m4 < 4; ++m4)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const floatx4& a = acc[nt][4 * half + m4];
                const bf16x4 o = {(__bf16)a[0], (__bf16)a[1], (__bf16)a[2], (__bf16)a[3]};
                *reinterpret_cast<bf16x4*>(mine + (16 * m4 + r16) * kPitch + (16 * nt + 4 * g4) * 2) = o;
            }
        // the wave reads only what it wrote itself: LDS operations of a wave complete in order
#pragma unroll
        for (int s = 0; s < 64 / kRowsPerStore; ++s) {
            const int row = s * kRowsPerStore + srow;                      // row within this half
            const u32x4 v = *reinterpret_cast<const u32x4*>(mine + row * kPitch + 16 * schunk);
            uint16_t* dst = y + (m0 + x_rows + 64 * half + row) * ldy + n0 + w_rows + 8 * schunk;
            *reinterpret_cast<u32x4*>(dst) = v;
        }
    }
}

// ---- the resident form used by the projections -------------------------------------------------------------
// One workgroup per CU stays for the whole launch and works through its CU's tiles one after the other.  The
// tiles of a launch all cost the same, so the fixed round-robin deal below is also the balanced one, and a
// resident workgroup can do what a fresh one cannot: fetch the first k-step of its next tile while the last
// k-step of the current one is computed, so that neither the first trip to memory of a tile nor the write-out of
// the one before it leaves the CU's matrix cores idle.
// LDS: two stages of a 256-row x tile and a (up to) 256-row w tile, at fixed places whatever the width of the
// tile in hand, and a piece per wave for the write-out (16 rows at a time), apart from the stages because the
// next tile's first stage is already arriving while the results leave.
constexpr uint32_t kResXStage = kLinBM * kLinBK * 2;                 // 32 KB
constexpr uint32_t kResWStage = 256 * kLinBK * 2;                    // 32 KB (a 128-feature tile uses half)
constexpr uint32_t kResWBase = kLinStages * kResXStage;
constexpr uint32_t kResOutBase = kResWBase + kLinStages * kResWStage;
constexpr int kResOutPitch = 64 * 2 + 16;                            // a wave's 64 features of one row, padded
constexpr uint32_t kResLdsBytes = kResOutBase + 8 * 16 * kResOutPitch;

// One work item of a die's list: local index j < wide: the 256-feature tile j; beyond, the halves of the tiles
// after them (see launch_tiles).  Returns false past the end of the die's list.
struct ResItem {
    int64_t m0, n0;
    bool wide;
};
__device__ __forceinline__ bool res_item(int die, int j, int per_die, int wide_per_die, int tiles_m, int tiles_n, int bn,
                                         ResItem* it) {
    const bool whole = bn == 128 || j < wide_per_die;
    const int in_die = whole ? j : wide_per_die + (j - wide_per_die) / 2;
    const int t = die * per_die + in_die;
    if (in_die >= per_die || t >= tiles_m * tiles_n) return false;
    it->m0 = (int64_t)(t / tiles_n) * kLinBM;
    it->n0 = (int64_t)(t % tiles_n) * bn + (whole ? 0 : 128 * ((j - wide_per_die) & 1));
    it->wide = whole && bn == 256;
    return true;
}

// Copy u of a k-step (4 of x, BN / 64 of w per wave) into stage `stage`; xb, wb: the tile's operands at that k-step.
template <int BN>
__device__ __forceinline__ void res_copy(int u, const uint16_t* xb, const uint16_t* wb, int64_t ldx, int64_t ldw, int stage,
                                         int wave, uint32_t x_off, uint32_t w_off, uint32_t lds_addr) {
    if (u < 4) {
        const int row = 32 * wave + 8 * u;
        copy16_to_lds(uniform_ptr(xb + (int64_t)row * ldx), x_off, lds_addr + stage * kResXStage + row * 128);
    } else {
        const int row = (BN / 8) * wave + 8 * (u - 4);
        copy16_to_lds(uniform_ptr(wb + (int64_t)row * ldw), w_off, lds_addr + kResWBase + stage * kResWStage + row * 128);
    }
}
// All copies of the first k-step of the tile at (m0, n0).
template <int BN>
__device__ __forceinline__ void res_first(const uint16_t* x, const uint16_t* w, int64_t ldx, int64_t ldw, int64_t m0, int64_t n0,
                                          int stage, int wave, uint32_t x_off, uint32_t w_off, uint32_t lds_addr) {
#pragma unroll
    for (int u = 0; u < 4 + BN / 64; ++u) res_copy<BN>(u, x + m0 * ldx, w + n0 * ldw, ldx, ldw, stage, wave, x_off, w_off, lds_addr);
}

// All k-steps and the write-out of one tile whose first k-step is already on its way into stage `stage`
// (updated to the stage the next tile starts in).  `next`: the tile to prefetch during the last k-step, if any.
template <int BN>
__device__ __forceinline__ void res_tile(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                                         uint16_t* __restrict__ y, int K, int64_t ldx, int64_t ldw, int64_t ldy,
                                         const ResItem& cur, bool have_next, const ResItem& next, int& stage, char* lds) {
    constexpr int NT = BN / 64;            // 16-feature blocks per wave
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r16 = lane & 15, g4 = lane >> 4;
    const int r8 = lane >> 3;
    const int chunk = (lane & 7) ^ lin_swizzle(r8);
    const uint32_t x_off = (uint32_t)(r8 * ldx * 2 + 16 * chunk);
    const uint32_t w_off = (uint32_t)(r8 * ldw * 2 + 16 * chunk);
    const uint32_t lds_addr = (uint32_t)(uintptr_t)DFA_LDS_PTR(void, &lds[0]);
    const int wm = wave >> 2, wn = wave & 3;
    const int frag = r16 * kLinBK + 8 * (g4 ^ lin_swizzle(r16));
    const int x_rows = 128 * wm, w_rows = (BN / 4) * wn;

    floatx4 acc[NT][8];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < 8; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int n_k = K / kLinBK;
    for (int ks = 0; ks < n_k; ++ks) {
        wait_vmcnt<0>();           // this wave's share of stage ks has landed (and the stores of the tile before have left)
        __syncthreads();           // everyone's has, and everyone is done reading the other stage
        // The copies of the next k-step: half of them here, half a quarter of a step later.  Behind the other waves' in the
        // vector-memory queue a copy holds up its wave's MFMAs; too late, and the next step waits for it.  (32768 x 2304 x 768: all
        // here 118.9 us, in halves 114.4, over three quarters of the step 117.6, over all of it 119.1.)
        const bool inner = ks + 1 < n_k;
        const uint16_t* const xb = x + cur.m0 * ldx + (int64_t)(ks + 1) * kLinBK;
        const uint16_t* const wb = w + cur.n0 * ldw + (int64_t)(ks + 1) * kLinBK;
        constexpr int kCopies = 4 + BN / 64;
        if (!inner && have_next) { // the next tile's first k-step, under this tile's last one and its write-out
            if (next.wide) res_first<256>(x, w, ldx, ldw, next.m0, next.n0, stage ^ 1, wave, x_off, w_off, lds_addr);
            else res_first<128>(x, w, ldx, ldw, next.m0, next.n0, stage ^ 1, wave, x_off, w_off, lds_addr);
        }
        const uint16_t* xs = reinterpret_cast<const uint16_t*>(lds + stage * kResXStage) + x_rows * kLinBK;
        const uint16_t* ws = reinterpret_cast<const uint16_t*>(lds + kResWBase + stage * kResWStage) + w_rows * kLinBK;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) {
            bf16x8 wf[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                wf[nt] = *reinterpret_cast<const bf16x8*>(ws + 16 * nt * kLinBK + (frag ^ (32 * kh)));
#pragma unroll
            for (int mh = 0; mh < 2; ++mh) {
                if (kh == 0 && inner) {
#pragma unroll
                    for (int u = mh * kCopies / 2; u < (mh + 1) * kCopies / 2; ++u)
                        res_copy<BN>(u, xb, wb, ldx, ldw, stage ^ 1, wave, x_off, w_off, lds_addr);
                }
                bf16x8 xf[4];
#pragma unroll
                for (int m4 = 0; m4 < 4; ++m4)
                    xf[m4] = *reinterpret_cast<const bf16x8*>(xs + 16 * (4 * mh + m4) * kLinBK + (frag ^ (32 * kh)));
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int m4 = 0; m4 < 4; ++m4)
                        acc[nt][4 * mh + m4] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nt], xf[m4], acc[nt][4 * mh + m4], 0, 0, 0);
            }
        }
        stage ^= 1;
    }

    // ---- write-out, 16 rows of the wave's tile at a time through the wave's own piece of LDS: lane (g4, r16) holds
    // row 16*mt + r16, features 16*nt + 4*g4 .. +3; written 8 bytes per lane, read back 16 bytes per lane with
    // consecutive lanes along a row, stored as whole rows of the wave's tile.  No barrier: the piece belongs to
    // this wave alone, and LDS operations of a wave complete in order.
    constexpr int kRowBytes = (BN / 4) * 2, kLanesPerRow = kRowBytes / 16, kRowsPerStore = 64 / kLanesPerRow;
    char* mine = lds + kResOutBase + wave * (16 * kResOutPitch);
    const int srow = lane / kLanesPerRow, schunk = lane % kLanesPerRow;
#pragma unroll
    for (int mt = 0; mt < 8; ++mt) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const floatx4& a = acc[nt][mt];
            const bf16x4 o = {(__bf16)a[0], (__bf16)a[1], (__bf16)a[2], (__bf16)a[3]};
            *reinterpret_cast<bf16x4*>(mine + r16 * kResOutPitch + (16 * nt + 4 * g4) * 2) = o;
        }
#pragma unroll
        for (int s = 0; s < (16 + kRowsPerStore - 1) / kRowsPerStore; ++s) {
            const int row = s * kRowsPerStore + srow;                      // row within these 16
            if (kRowsPerStore <= 16 || row < 16) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(mine + row * kResOutPitch + 16 * schunk);
                uint16_t* dst = y + (cur.m0 + x_rows + 16 * mt + row) * ldy + cur.n0 + w_rows + 8 * schunk;
                *reinterpret_cast<u32x4*>(dst) = v;
            }
        }
    }
}

// Requires M % 256 == 0, N % BN == 0, K % 64 == 0, every row of x, w and y starting on a 16-byte boundary.
// Workgroup i stays on CU (i / dies) of die i % dies; tiles (256 x BN) are numbered band by band and dealt so that one
// die walks all feature tiles of a row band before moving on (the x band is then read from memory once per die, w stays
// in its L2), the CUs of a die taking them round-robin.  When the last round of a die would be at most half full
// (wide tiles only), its tiles are cut into two 128-feature halves, which fill the die for a round half as long: the
// first `wide_per_die` items of a die are whole tiles, the others halves.
template <int BN>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void linear_bf16_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w, uint16_t* __restrict__ y,
                        int K, int64_t ldx, int64_t ldw, int64_t ldy, int tiles_m, int tiles_n, int wide_per_die, int dies,
                        int cus_per_die) {
    __shared__ __attribute__((aligned(1024))) char lds[kResLdsBytes];
    const int die = blockIdx.x % dies, cu = blockIdx.x / dies;
    const int per_die = (tiles_m * tiles_n + dies - 1) / dies;
    ResItem cur, next;
    int j = cu;
    if (!res_item(die, j, per_die, wide_per_die, tiles_m, tiles_n, BN, &cur)) return;
    // the first tile's first k-step
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, r8 = lane >> 3;
        const int chunk = (lane & 7) ^ lin_swizzle(r8);
        const uint32_t x_off = (uint32_t)(r8 * ldx * 2 + 16 * chunk), w_off = (uint32_t)(r8 * ldw * 2 + 16 * chunk);
        const uint32_t lds_addr = (uint32_t)(uintptr_t)DFA_LDS_PTR(void, &lds[0]);
        if (cur.wide) res_first<256>(x, w, ldx, ldw, cur.m0, cur.n0, 0, wave, x_off, w_off, lds_addr);
        else res_first<128>(x, w, ldx, ldw, cur.m0, cur.n0, 0, wave, x_off, w_off, lds_addr);
    }
    int stage = 0;
    for (;;) {                     // ends: j grows by cus_per_die >= 1 every trip, res_item fails past the die's list
        j += cus_per_die;
        const bool have_next = res_item(die, j, per_die, wide_per_die, tiles_m, tiles_n, BN, &next);
        if (cur.wide) res_tile<256>(x, w, y, K, ldx, ldw, ldy, cur, have_next, next, stage, lds);
        else res_tile<128>(x, w, y, K, ldx, ldw, ldy, cur, have_next, next, stage, lds);
        if (!have_next) break;
        cur = next;
    }
}

// ---- the resident form of 128-row tiles ---------------------------------------------------------------------------
// 128 x BN tiles (launch_linear_bf16 says when).  A workgroup of 4 waves, one per SIMD, stays for the whole launch and works
// through its CU's tiles one after the other, as one stream of 64-k steps: stage i + S of the ring is fetched as soon as every
// wave has stage i in registers, whichever tile it belongs to, so neither the first trip to memory of a tile nor the write-out
// of the one before it stops the copies.  A wave computes 64 rows x BN/2 features; the barrier of a step stands where every wave has
// the whole of its slot in registers, ahead of the products that use them.  The k-steps' addresses are counted along: a division by
// the number of feature tiles in every step cost up to 0.08 us.
// Bound, with all CUs at it: the copies (40 to 57 bytes per clock and CU) beside the MFMAs (whose power takes the clock to some
// 2 GHz).  A 64-k step of a 128 x 288 tile takes 0.90 us: its MFMAs alone 0.71, its copies alone 0.57.  A copy waits in the
// vector-memory queue behind the other waves' and its wave's MFMAs with it, so the wide tiles (288, 192) spread the copies of a step over
// all of it (0.97 us with all of them behind the barrier), one 16-feature block against the four 16-row blocks at a time, and store
// from the registers (two lane-group exchanges give every lane 16 contiguous bytes of a row).  The steps of the narrow tiles are too short
// for that: walked the same way, 64 features took 780 to 800 cycles a step without copies (two halves: 710) and the stores 130 more, 0.5 us
// of a launch of 6 steps; with all copies behind the barrier a step takes 790 cycles in both forms.
// Before / now, us: 4096 x 2304 x 768 (256 x 256 tiles on 144 CUs / 256 tiles of 128 x 288) 21.5 / 18.1; 1024 x 1152 x 384 5.1 / 5.1,
// 1024 x 768 x 768 (64 features) 7.3 / 6.9, 4096 x 768 x 768 (96) 9.4 / 8.9, 3072 x 1152 x 384 (128) 7.0 / 6.8.
constexpr int kStreamBM = 128;
template <int BN> constexpr uint32_t kStreamStageBytes = (kStreamBM + BN) * kLinBK * 2;
template <int BN> constexpr int kStreamStages = BN == 288 ? 3 : BN >= 128 ? 4 : BN == 96 ? 5 : 6;      // 160, 163, 131, 143 and 147 KB

// Rows (16-lane groups) 1 and 3 of `a` change places with rows 0 and 2 of `b`.
__device__ __forceinline__ void swap_lane_rows(uint32_t& a, uint32_t& b) {
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}

// Two 16 x 16 results, lane (g4, r16) with features 4*g4 .. +3 of row r16 of either, as 16 bytes: lane groups 0 and 2 receive
// features 0 .. 7 and 8 .. 15 of `a`'s row r16, groups 1 and 3 those of `b`'s.
__device__ __forceinline__ u32x4 pack_pair(const floatx4& a, const floatx4& b) {
    const bf16x2 a0 = {(__bf16)a[0], (__bf16)a[1]}, a1 = {(__bf16)a[2], (__bf16)a[3]};
    const bf16x2 b0 = {(__bf16)b[0], (__bf16)b[1]}, b1 = {(__bf16)b[2], (__bf16)b[3]};
    uint32_t x0 = __builtin_bit_cast(uint32_t, a0), x1 = __builtin_bit_cast(uint32_t, a1);
    uint32_t y0 = __builtin_bit_cast(uint32_t, b0), y1 = __builtin_bit_cast(uint32_t, b1);
    swap_lane_rows(x0, y0);
    swap_lane_rows(x1, y1);
    return u32x4{x0, x1, y0, y1};
}

// (512 threads in the launch bounds keep the compiler within 256 registers: above that it moves the accumulators through the
// second half of the register file, two copies per product.)
template <int BN>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void linear_stream_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w, uint16_t* __restrict__ y,
                          int K, int64_t ldx, int64_t ldw, int64_t ldy, int part_n, int part_shift, int per_die, int part_tiles, int cus_per_die) {
    constexpr int BM = kStreamBM, S = kStreamStages<BN>, MT = 4, NT = BN / 32;        // 16-row / 16-feature blocks per wave
    constexpr int kXCopies = BM / 32, kCopies = kXCopies + BN / 32;                   // copies per wave and stage
    constexpr uint32_t kStage = kStreamStageBytes<BN>, kWBase = BM * kLinBK * 2;
    constexpr bool kWide = BN >= 192;
    constexpr int kPitch = BN + 16;                                                   // bytes: BN / 2 features of a row, padded
    __shared__ __attribute__((aligned(1024))) char lds[S * kStage + (kWide ? 0 : 4 * 16 * kPitch)];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r16 = lane & 15, g4 = lane >> 4;
    const int r8 = lane >> 3;
    const int chunk = (lane & 7) ^ lin_swizzle(r8);
    const uint32_t x_step = (uint32_t)(16 * ldx), w_step = (uint32_t)(16 * ldw);      // bytes per 8 rows
    const uint32_t x_off = (uint32_t)(((BM / 4) * wave + r8) * ldx * 2) + 16u * chunk;
    const uint32_t w_off = (uint32_t)(((BN / 4) * wave + r8) * ldw * 2) + 16u * chunk;
    const uint32_t lds_addr = (uint32_t)(uintptr_t)DFA_LDS_PTR(void, &lds[0]);
    const int wm = wave >> 1, wn = wave & 1;

    // this workgroup's tiles: first, first + cus_per_die, ... of its die's list.  A group of 2^part_shift dies has a run of the tiles
    // (numbered band by band, part_n to a band), each die of it a share of the features.  (Die and place come as the grid's dimensions and the
    // shares from the host: a launch waits for every division before its first copy, 0.17 us for five of them.)
    const int die = blockIdx.x, tile_n0 = (die & ((1 << part_shift) - 1)) * part_n;
    const int die_first = (die >> part_shift) * per_die, die_tiles = min(per_die, part_tiles - die_first);
    const int first = blockIdx.y;
    if (first >= die_tiles) return;
    const int n_k = K / kLinBK;
    const int total = ((die_tiles - first - 1) / cus_per_die + 1) * n_k;             // k-steps of all its tiles

    // the stream of copies
    int ij = first, iks = 0, issued = 0;
    const uint16_t *xt, *wt;                                                          // the tile in hand at k-step iks
    auto tile_start = [&]() {
        const int t = die_first + ij;
        xt = x + (int64_t)(t / part_n) * BM * ldx;
        wt = w + (int64_t)(tile_n0 + t % part_n) * BN * ldw;
    };
    tile_start();
    auto copy = [&](int u, uint32_t at) {
        if (u < kXCopies) copy16_to_lds(uniform_ptr(xt), x_off + u * x_step, at + ((BM / 4) * wave + 8 * u) * 128);
        else copy16_to_lds(uniform_ptr(wt), w_off + (u - kXCopies) * w_step, at + kWBase + ((BN / 4) * wave + 8 * (u - kXCopies)) * 128);
    };
    auto stage_issued = [&]() {
        xt += kLinBK;
        wt += kLinBK;
        if (++iks == n_k) { iks = 0; ij += cus_per_die; tile_start(); }
        ++issued;
    };
    // waits until all but the youngest `ahead` stages of this wave's copies have landed (stores of a tile before count as
    // well: the wait is then longer than it has to be, never shorter)
    auto landed = [&](int ahead) {
        // (S - 2 at most)
        if (S > 5 && ahead >= 4) wait_vmcnt<(S > 5 ? 4 : 0) * kCopies>();
        else if (S > 4 && ahead >= 3) wait_vmcnt<(S > 4 ? 3 : 0) * kCopies>();
        else if (S > 3 && ahead >= 2) wait_vmcnt<(S > 3 ? 2 : 0) * kCopies>();
        else if (S > 2 && ahead >= 1) wait_vmcnt<kCopies>();
        else wait_vmcnt<0>();
    };

    // fragments: row r16 of a 16-row block, chunk (4 * half + g4) ^ swizzle
    const int frag = r16 * kLinBK + 8 * (g4 ^ lin_swizzle(r16));
    auto x_frag = [&](int slot, int half, int mt) {
        return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const uint16_t*>(lds + slot * kStage) + ((BM / 2) * wm + 16 * mt) * kLinBK + (frag ^ (32 * half)));
    };
    auto w_frag = [&](int slot, int half, int nt) {
        return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const uint16_t*>(lds + slot * kStage + kWBase) + ((BN / 2) * wn + 16 * nt) * kLinBK + (frag ^ (32 * half)));
    };

    for (int s = 0; s < S && s < total; ++s) {
#pragma unroll
        for (int u = 0; u < kCopies; ++u) copy(u, lds_addr + s * kStage);
        stage_issued();
    }
    landed(issued - 1);
    asm volatile("s_barrier" ::: "memory");

    floatx4 acc[NT][MT];                   // [16-feature block][16-row block], as in linear_tile
    auto clear = [&]() {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    int step = 0, slot = 0;
    if constexpr (kWide) {
        // A group: one weight fragment, four MFMAs of 16 cycles.  Weight fragments are read kAhead groups before their use, the x
        // fragments of a half as far before it starts; the ring's length divides a step's groups.
        constexpr int kGroups = 2 * NT, kAhead = NT == 9 ? 4 : 3, kRing = NT == 9 ? 6 : 4, kMeet = kGroups - kAhead;
        static_assert(kGroups % kRing == 0 && kAhead < kRing && kAhead <= NT, "a fragment's place in the ring is its group's, in every step");
        bf16x8 wf[kRing], xf[2][MT];
        auto read_w = [&](int sl, int i) { wf[i % kRing] = w_frag(sl, i / NT, i % NT); };
        auto read_x = [&](int sl, int half) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xf[half][mt] = x_frag(sl, half, mt);
        };
        read_x(0, 0);
#pragma unroll
        for (int i = 0; i < kAhead; ++i) read_w(0, i);
        int fill = 0;
        bool more = false;                 // a stage is being fetched into slot `fill`
        for (int j = first; j < die_tiles; j += cus_per_die) {
            clear();
            for (int ks = 0; ks < n_k; ++ks, ++step) {
                const int next_slot = slot + 1 == S ? 0 : slot + 1;
#pragma unroll
                for (int i = 0; i < kGroups; ++i) {
                    if (i == kMeet) {
                        // every wave has the whole of this slot in registers, and stage step + 1 has landed for every wave
                        if (more) stage_issued();
                        landed(issued - step - 2);
                        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                        more = issued < total;
                        fill = slot;
                    }
                    // past the last step: an old slot, not used
                    const int r = i + kAhead;
                    if (i % NT == NT - kAhead) read_x(i < NT ? slot : next_slot, i < NT ? 1 : 0);
                    read_w(r < kGroups ? slot : next_slot, r % kGroups);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[i % NT][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i % kRing], xf[i / NT][mt], acc[i % NT][mt], 0, 0, 0);
                    const int g = (i + kGroups - kMeet) % kGroups;
                    if (more) {
#pragma unroll
                        for (int u = g * kCopies / kGroups; u < (g + 1) * kCopies / kGroups; ++u) copy(u, lds_addr + fill * kStage);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                slot = next_slot;
            }
            // Write-out straight from the registers: pairs of feature blocks, 64 contiguous bytes of every row per store; a last single one
            // by pairs of row blocks.
            const int t = die_first + j;
            uint16_t* const yt = y + ((int64_t)(t / part_n) * BM + (BM / 2) * wm + r16) * ldy + (tile_n0 + t % part_n) * BN + (BN / 2) * wn + 8 * (g4 >> 1);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt + 1 < NT; nt += 2)
                    *reinterpret_cast<u32x4*>(yt + (int64_t)16 * mt * ldy + 16 * (nt + (g4 & 1))) = pack_pair(acc[nt][mt], acc[nt + 1][mt]);
            if (NT % 2 != 0) {
#pragma unroll
                for (int mt = 0; mt < MT; mt += 2)
                    *reinterpret_cast<u32x4*>(yt + (int64_t)16 * (mt + (g4 & 1)) * ldy + 16 * (NT - 1)) = pack_pair(acc[NT - 1][mt], acc[NT - 1][mt + 1]);
            }
        }
    } else {
        // The fragments of a 32-k half are read under the MFMAs of the half before, also across the step's barrier, behind which all copies
        // into the freed slot go out: these steps are short, and every branch in them shows.
        struct Frags { bf16x8 w[NT], x[MT]; };
        auto read = [&](Frags& f, int sl, int half) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) f.w[nt] = w_frag(sl, half, nt);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) f.x[mt] = x_frag(sl, half, mt);
        };
        auto multiply = [&](const Frags& f) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[nt], f.x[mt], acc[nt][mt], 0, 0, 0);
        };
        // the reads of one half spread over the MFMAs of the other
        auto weave = [&]() {
#pragma unroll
            for (int i = 0; i < MT + NT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, MT * NT / (MT + NT), 0);
            }
        };
        Frags f0, f1;
        read(f0, 0, 0);
        for (int j = first; j < die_tiles; j += cus_per_die) {
            clear();
            for (int ks = 0; ks < n_k; ++ks, ++step) {
                read(f1, slot, 1);
                multiply(f0);
                weave();
                const int next_slot = slot + 1 == S ? 0 : slot + 1;
                // every wave has the whole of this slot in registers, and stage step + 1 has landed for every wave
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                landed(issued - step - 2);
                asm volatile("s_barrier" ::: "memory");
                if (issued < total) {
#pragma unroll
                    for (int u = 0; u < kCopies; ++u) copy(u, lds_addr + slot * kStage);
                    stage_issued();
                }
                read(f0, next_slot, 0);    // past the last step: an old slot, not used
                multiply(f1);
                weave();
                slot = next_slot;
            }
            // Write-out, 16 rows of the wave's tile at a time through its own piece of LDS.  No barrier: the piece belongs to this wave
            // alone, and LDS operations of a wave complete in order.
            const int t = die_first + j;
            const int64_t m0 = (int64_t)(t / part_n) * BM + (BM / 2) * wm, n0 = (int64_t)(tile_n0 + t % part_n) * BN + (BN / 2) * wn;
            constexpr int kLanesPerRow = BN / 16, kChunks = 16 * kLanesPerRow;             // 16-byte pieces of BN / 2 features
            char* const mine = lds + S * kStage + wave * (16 * kPitch);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const floatx4& a = acc[nt][mt];
                    const bf16x4 o = {(__bf16)a[0], (__bf16)a[1], (__bf16)a[2], (__bf16)a[3]};
                    *reinterpret_cast<bf16x4*>(mine + r16 * kPitch + (16 * nt + 4 * g4) * 2) = o;
                }
#pragma unroll
                for (int c0 = 0; c0 < kChunks; c0 += 64) {
                    const int c = c0 + lane, row = c / kLanesPerRow, ch = c % kLanesPerRow;
                    if (kChunks % 64 == 0 || c < kChunks)
                        *reinterpret_cast<u32x4*>(y + (m0 + 16 * mt + row) * ldy + n0 + 8 * ch) =
                            *reinterpret_cast<const u32x4*>(mine + row * kPitch + 16 * ch);
                }
            }
        }
    }
}

template <int BN>
hipError_t launch_stream(const void* x, const void* w, void* y, int64_t M, int32_t N, int32_t K,
                         int64_t ldx, int64_t ldw, int64_t ldy, const ChipShape& chip, hipStream_t st) {
    const int dies = chip.dies > 0 ? chip.dies : 1, cus_per_die = chip.cus / dies > 0 ? chip.cus / dies : 1;
    const int tiles_n = N / BN, tiles_m = (int)(M / kStreamBM);
    // Two dies with half the feature tiles each fetch less, and keep it more easily, than each with all (8192 x 2304 x 768 34.3 ->
    // 31.9 us, 4096 x 2304 x 768 18.7 -> 18.5), where that deals the dies the same number of tiles.  Not for narrow tiles, whose weights are
    // small beside the rows that two dies then fetch (6144 x 384 x 384 6.4 us, 5.9 without; 1024 x 2304 x 768 8.5 / 8.6).
    const int parts = BN >= 192 && tiles_n % 2 == 0 && dies % 2 == 0 && tiles_m % (dies / 2) == 0 ? 2 : 1;
    const int per_die = (tiles_m * tiles_n + dies - 1) / dies;
    // dies along x: workgroups go to the dies in turn, x first
    hipLaunchKernelGGL((linear_stream_kernel<BN>), dim3(dies, per_die < cus_per_die ? per_die : cus_per_die), dim3(256), 0, st,
                       static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w), static_cast<uint16_t*>(y),
                       K, ldx, ldw, ldy, tiles_n / parts, parts - 1, per_die, tiles_m * (tiles_n / parts), cus_per_die);
    return hipGetLastError();
}

// A batch of independent products of one shape: workgroup (t, z) computes tile t of matrix z = z0 * batch_inner + z1,
// whose operands start at x + z0 * xs0 + z1 * xs1 (elements), and likewise for w and y.  Plain tile order.
template <int BN>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void linear_bf16_batched_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w, uint16_t* __restrict__ y,
                                int K, int64_t ldx, int64_t ldw, int64_t ldy, int tiles_n, int batch_inner,
                                int64_t xs0, int64_t xs1, int64_t ws0, int64_t ws1, int64_t ys0, int64_t ys1) {
    __shared__ __attribute__((aligned(1024))) char lds[kLinStages * (kLinBM + BN) * kLinBK * 2];
    const int z0 = blockIdx.y / batch_inner, z1 = blockIdx.y % batch_inner;
    const int64_t m0 = (int64_t)(blockIdx.x / tiles_n) * kLinBM, n0 = (int64_t)(blockIdx.x % tiles_n) * BN;
    linear_tile<BN>(x + z0 * xs0 + z1 * xs1, w + z0 * ws0 + z1 * ws1, y + z0 * ys0 + z1 * ys1, K, ldx, ldw, ldy, m0, n0, lds);
}

template <int BN>
hipError_t launch_tiles(const void* x, const void* w, void* y, int64_t M, int32_t N, int32_t K,
                        int64_t ldx, int64_t ldw, int64_t ldy, const ChipShape& chip, hipStream_t st) {
    const int dies = chip.dies > 0 ? chip.dies : 1, cus_per_die = chip.cus / dies > 0 ? chip.cus / dies : 1;
    const int tiles_m = (int)(M / kLinBM), tiles_n = N / BN;
    const int per_die = (tiles_m * tiles_n + dies - 1) / dies;
    // wide tiles: whole rounds of a die's CUs as they are, a last round that is at most half full in halves
    const int rem = per_die % cus_per_die;
    const int wide_per_die = (BN == 256 && rem > 0 && 2 * rem <= cus_per_die) ? per_die - rem : per_die;
    const int items_per_die = wide_per_die + 2 * (per_die - wide_per_die);
    const int wg_per_die = items_per_die < cus_per_die ? items_per_die : cus_per_die;      // one resident workgroup per CU
    hipLaunchKernelGGL((linear_bf16_kernel<BN>), dim3(wg_per_die * dies), dim3(512), 0, st,
                       static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w), static_cast<uint16_t*>(y),
                       K, ldx, ldw, ldy, tiles_m, tiles_n, wide_per_die, dies, cus_per_die);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_linear_bf16(const void* x, const void* w, void* y, int64_t M, int32_t N, int32_t K,
                              int64_t ldx, int64_t ldw, int64_t ldy, const ChipShape& chip, hipStream_t st) {
    // One workgroup per CU at a time, so a launch lasts as long as the CU with most tiles.  Per round of tiles the small forms
    // cost about as much as the bytes they fetch, 64 (BM + BN) per k-step and CU; 256 x 256, 128 x 288 and 128 x 192 tiles
    // more (their MFMAs show), 128 x 192 ones less where K is long enough to make up for their start.  Fitted over 256 to 32768
    // rows and 384 to 2304 features (K = 384 and 768): on 50 of 52 shapes the least estimate is the fastest form or within 4 % of it,
    // which is what two runs differ by (16384 x 1152 x 384 22.2 us, 21.0 with 192; 32768 x 384 x 384 17.8, 16.0 with 128).
    // Rows x features x K, us, 256 x 256 / 256 x 128 / 128 x 288 / 128 x 192 / 128 x 128 / 128 x 96 / 128 x 64 tiles:
    // 2048 x 2304 x 768 14.3 / 13.5 / 15.8 / 13.1 / 16.7 / 14.4 / 16.6, 4096 x 2304 x 768 20.9 / 25.7 / 18.7 / 22.0 / 24.0 / 21.5 / 25.8,
    // 8192 x 2304 x 768 34.1 / 39.2 / 32.2 / 33.6 / 39.3 / 40.1 / 44.3, 16384 x 2304 x 768 56.8 / 65.7 / 61.4 / 64.2 / 70.4 / 78.2 / 87.6,
    // 4096 x 768 x 768 13.7 / 12.9 / - / 12.5 / 9.6 / 9.1 / 12.1, 6144 x 768 x 768 14.2 / 13.4 / - / 13.1 / 16.6 / 14.7 / 16.5,
    // 5120 x 1152 x 384 - / 9.5 / 11.5 / 9.8 / 10.7 / 10.2 / 10.9, 8192 x 1152 x 384 - / 16.3 / 13.1 / 15.3 / 14.8 / 13.9 / 16.2.
    const int64_t dies = chip.dies > 0 ? chip.dies : 1, cus = chip.cus / dies > 0 ? chip.cus / dies : 1;
    auto per_die = [&](int bm, int bn) { return ((M / bm) * (N / bn) + dies - 1) / dies; };
    auto rounds = [&](int bm, int bn) { return (per_die(bm, bn) + cus - 1) / cus; };
    int64_t least = rounds(256, 128) * (256 + 128);
    int form = 0;                                                   // 256 x 128
    auto consider = [&](int f, int64_t cost) {
        if (cost < least) { least = cost; form = f; }
    };
    if (N % 256 == 0) {
        // a last round that is at most half full goes in 128-feature halves (launch_tiles)
        const int64_t rem = per_die(256, 256) % cus, halves = rem > 0 && 2 * rem <= cus;
        consider(256, (rounds(256, 256) - halves) * 655 + halves * (256 + 128));
    }
    // their copy lanes address up to 288 rows with 32-bit byte offsets
    if (ldx < (1 << 22) && ldw < (1 << 22)) {
        if (N % 288 == 0) consider(288, rounds(128, 288) * 515);
        if (N % 192 == 0) consider(192, rounds(128, 192) * (K >= 512 ? 375 : 400));
        consider(128, rounds(128, 128) * (128 + 128));
        if (N % 96 == 0) consider(96, rounds(128, 96) * (128 + 96));
        consider(64, rounds(128, 64) * (128 + 64));
    }
    switch (form) {
        case 288: return launch_stream<288>(x, w, y, M, N, K, ldx, ldw, ldy, chip, st);
        case 192: return launch_stream<192>(x, w, y, M, N, K, ldx, ldw, ldy, chip, st);
        case 256: return launch_tiles<256>(x, w, y, M, N, K, ldx, ldw, ldy, chip, st);
        case 128: return launch_stream<128>(x, w, y, M, N, K, ldx, ldw, ldy, chip, st);
        case 96: return launch_stream<96>(x, w, y, M, N, K, ldx, ldw, ldy, chip, st);
        case 64: return launch_stream<64>(x, w, y, M, N, K, ldx, ldw, ldy, chip, st);
        default: return launch_tiles<128>(x, w, y, M, N, K, ldx, ldw, ldy, chip, st);
    }
}

hipError_t launch_linear_bf16_batched(const void* x, const void* w, void* y, int64_t M, int32_t N, int32_t K,
                                      int64_t ldx, int64_t ldw, int64_t ldy, int32_t batch_outer, int32_t batch_inner,
                                      int64_t xs0, int64_t xs1, int64_t ws0, int64_t ws1, int64_t ys0, int64_t ys1,
                                      hipStream_t st) {
    const uint16_t* xp = static_cast<const uint16_t*>(x);
    const uint16_t* wp = static_cast<const uint16_t*>(w);
    uint16_t* yp = static_cast<uint16_t*>(y);
    const dim3 block(512);
    if (N % 256 == 0) {
        const dim3 grid((unsigned)((M / kLinBM) * (N / 256)), (unsigned)(batch_outer * batch_inner));
        hipLaunchKernelGGL((linear_bf16_batched_kernel<256>), grid, block, 0, st, xp, wp, yp, K, ldx, ldw, ldy, N / 256,
                           batch_inner, xs0, xs1, ws0, ws1, ys0, ys1);
    } else if (N % 128 == 0) {
        const dim3 grid((unsigned)((M / kLinBM) * (N / 128)), (unsigned)(batch_outer * batch_inner));
        hipLaunchKernelGGL((linear_bf16_batched_kernel<128>), grid, block, 0, st, xp, wp, yp, K, ldx, ldw, ldy, N / 128,
                           batch_inner, xs0, xs1, ws0, ws1, ys0, ys1);
    } else {
        const dim3 grid((unsigned)((M / kLinBM) * (N / 64)), (unsigned)(batch_outer * batch_inner));
        hipLaunchKernelGGL((linear_bf16_batched_kernel<64>), grid, block, 0, st, xp, wp, yp, K, ldx, ldw, ldy, N / 64,
                           batch_inner, xs0, xs1, ws0, ws1, ys0, ys1);
    }
    return hipGetLastError();
}

}  // namespace dfa
