// Device-side building blocks of the kernels whose waves walk 32-row blocks of a tile's key lists on their own (small
// launches, fp32), and of the transposed reads of swizzled stages (gfx950).
#pragma once
#include "dfa_device.h"
#include "dfa_mfma.h"

namespace dfa {

constexpr int kRedPitch = kD + 4;          // row pitch of the per-wave results in LDS (floats)
constexpr int kBlockElems = kWalkBlock * kRowElems;      // one bf16 block of one tensor in LDS: 4 KB
constexpr int kBlockBytes = kBlockElems * 2;
constexpr int kBlockCopies = 4;            // wave-level copies per bf16 block (1 KB = 8 rows each)

// Workgroup x of a launch of `parts` workgroups per item -> (item, part); the parts of an item stay on the item's die.
__device__ __forceinline__ void item_of_part(int x, int parts, int& item, int& part) {
    const int group = x / (kDies * parts), rem = x % (kDies * parts);
    item = group * kDies + rem % kDies;
    part = rem / kDies;
}

// A wave's share of a list: its 32-row blocks wave, wave + 4, ..., the one in hand in scalar registers.
// kCut: the list is cut into blocks.  Their records come 64 at a time in one trip to memory (a lane each) and wait in LDS of
// the wave's own.  Otherwise the blocks are counted through the list's progressions, read one by one: plans whose cut lists
// would take too much memory (kMaxCutRecords).
constexpr int kWalkRecords = 64;
template <bool kCut>
struct BlockWalk;
template <>
struct BlockWalk<true> {
    const KeySeg* list;
    KeySeg* records;
    int nseg, i;                 // block in hand
    int t;                       // its place in `records`
    KeySeg seg;

    __device__ __forceinline__ void fetch() { records[threadIdx.x & 63] = list[min(i + kWalkWaves * (int)(threadIdx.x & 63), nseg - 1)]; }
    __device__ __forceinline__ void read() {
        const KeySeg r = records[t];
        seg.key0 = __builtin_amdgcn_readfirstlane(r.key0);
        seg.stride = __builtin_amdgcn_readfirstlane(r.stride);
        seg.count = __builtin_amdgcn_readfirstlane(r.count);
        seg.log2_mult = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, r.log2_mult)));
    }
    __device__ __forceinline__ void start(const KeySeg* l, int n, int wave, KeySeg* lds) {
        list = l;
        records = lds;
        nseg = n;
        i = wave;
        t = 0;
        fetch();
        read();
    }
    __device__ __forceinline__ void next() {
        i += kWalkWaves;
        if (++t == kWalkRecords) {
            t = 0;
            if (i < nseg) fetch();
        }
        read();
    }
    __device__ __forceinline__ bool valid() const { return i < nseg; }
    __device__ __forceinline__ int rows() const { return seg.count; }
    __device__ __forceinline__ int32_t first() const { return seg.key0; }
};
template <>
struct BlockWalk<false> {
    const KeySeg* segs;
    int nseg, s, t;              // progression, block within it
    KeySeg seg;

    // through the constant address space: a scalar load.  (After the copies' memory clobber the compiler takes a vector
    // load instead, whose wait would drain the copies in flight.)
    __device__ __forceinline__ void load() {
        typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
        const i32x4 x = *reinterpret_cast<const __attribute__((address_space(4))) i32x4*>(reinterpret_cast<uintptr_t>(segs + s));
        seg.key0 = x[0];
        seg.stride = x[1];
        seg.count = x[2];
        const int32_t mult = x[3];          // (the bit cast of an element in place would be that of element 0)
        seg.log2_mult = __builtin_bit_cast(float, mult);
    }
    __device__ __forceinline__ void settle() {
        while (s < nseg && t * kWalkBlock >= seg.count) {
            t -= (seg.count + kWalkBlock - 1) / kWalkBlock;
            if (++s < nseg) load();
        }
    }
    __device__ __forceinline__ void start(const KeySeg* list, int n, int wave, KeySeg*) {
        segs = list;
        nseg = n;
        s = 0;
        t = wave;
        load();
        settle();
    }
    __device__ __forceinline__ void next() {
        t += kWalkWaves;
        settle();
    }
    __device__ __forceinline__ bool valid() const { return s < nseg; }
    __device__ __forceinline__ int rows() const { return min(kWalkBlock, seg.count - t * kWalkBlock); }
    __device__ __forceinline__ int32_t first() const { return kept_row(seg.key0, seg.stride, t * kWalkBlock); }
};

// All LDS reads of this wave so far have returned; no memory access moves across.
__device__ __forceinline__ void lds_reads_done() {
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("" ::: "memory");
}
template <int N>
__device__ __forceinline__ void copies_left() {
    wait_vmcnt<N>();
    asm volatile("" ::: "memory");
}

// The wave ends here if x is zero (the same in every lane).  In place: the compiler's own end of the kernel lies behind the code that
// is skipped, and fetching it takes longer than the branch saves (short forward of one 256^2 image 6.66 us, 7.0 that way).
__device__ __forceinline__ void end_unless(uint32_t x) {
    const uint32_t s = __builtin_amdgcn_readfirstlane(x);
    asm volatile("s_cmp_lg_u32 %0, 0\n\ts_cbranch_scc1 .Lgo_on%=\n\ts_endpgm\n.Lgo_on%=:" ::"s"(s) : "scc", "memory");
}

// 16-byte chunk swizzle of a stage: chunk c of LDS row rho sits at chunk c ^ stage_swizzle(rho).  Any map of bits
// 1 to 3 of rho onto 0 .. 7 spreads one chunk column of sixteen consecutive rows over all 64 banks (row reads); with bit
// 1 on the chunk's top bit, the 32 lanes that read 64 bytes of each of four consecutive rows (transposed reads)
// are spread over all banks too.
__device__ __forceinline__ int stage_swizzle(int rho) { return ((rho & 2) << 1) | ((rho & 4) >> 1) | ((rho & 8) >> 3); }

// Element offsets of a lane's transposed reads inside a 16-row group of a stage: 32-d block db, walked positions
// (lane & 15) / 4 + 8 * g (+ 4 for the second half), which sigma puts into LDS rows (lane & 15) / 4 + 4 * g (+ 8).
struct TransposedLane {
    int lo[2], hi[2];
};
__device__ __forceinline__ TransposedLane transposed_lane(int lane) {
    const int g = lane >> 5, row = ((lane & 15) >> 2) + 4 * g;
    const int chunk = (2 * ((lane >> 4) & 1) + ((lane >> 1) & 1)) ^ stage_swizzle(row);
    const int lo = row * kRowElems + 8 * chunk + 4 * (lane & 1);
    TransposedLane t;
    t.lo[0] = lo;
    t.lo[1] = lo ^ 32;                            // db = 1: chunk + 4
    t.hi[0] = (lo ^ 8) + 8 * kRowElems;           // eight rows down: the swizzle's lowest bit
    t.hi[1] = (lo ^ 40) + 8 * kRowElems;
    return t;
}
__device__ __forceinline__ bf16x8 read_transposed(const uint16_t* rows16, const TransposedLane& t, int db) {
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(DFA_LDS_PTR(short4v, rows16 + t.lo[db]));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(DFA_LDS_PTR(short4v, rows16 + t.hi[db]));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// A tensor whose rows a wave copies block by block: rows n of one image and head start at base + n * pitch.  (The entry
// points take no row pitch of 2^25 bytes or more, see check_forward_args.)
struct BlockSource {
    const char* base;
    uint32_t pitch;
};
__device__ __forceinline__ BlockSource block_source(const uint16_t* base, int64_t sn) {
    return BlockSource{reinterpret_cast<const char*>(base), (uint32_t)(sn * 2)};
}

// What a lane fetches of a block: copy u fills LDS rows 8*u .. +7, lane L lands at row 8*u + L/8, chunk L%8.
struct BlockLane {
    int pos;               // list position of the lane's row in copy 0
    uint32_t chunk;        // byte offset of its 16-byte chunk
};

// Issues the copies of one bf16 block into a wave's own LDS: rows key0 + stride * i, permuted and swizzled as kOrder says;
// rows past the end of the block re-read its last one (a block without a valid row: its first).
// kWalked: rows permuted by sigma (swap bits 2 and 3), chunks by stage_swizzle: read back as rows or transposed;
// kKeys, kValues: the layouts of the forward's beat (sigma and k_swizzle; list order, chunks in place).
enum class BlockOrder { kWalked, kKeys, kValues };
template <BlockOrder kOrder>
__device__ __forceinline__ BlockLane block_lane(int lane) {
    const int r = lane >> 3, c = lane & 7;
    BlockLane l;
    l.pos = kOrder == BlockOrder::kValues ? r : (r & 3) | ((r & 4) << 1);
    l.chunk = 16u * (kOrder == BlockOrder::kValues ? c : c ^ (kOrder == BlockOrder::kKeys ? r >> 1 : stage_swizzle(r)));
    return l;
}
template <BlockOrder kOrder>
__device__ __forceinline__ void issue_block_rows(const BlockSource& src, int key0, int stride, int count, uint32_t lds_addr, const BlockLane& l) {
    const void* const first = uniform_ptr(src.base + (uint64_t)(uint32_t)key0 * src.pitch);
    const uint32_t pitch = (uint32_t)stride * src.pitch;
    constexpr uint32_t kFlip = kOrder == BlockOrder::kValues ? 0u : kOrder == BlockOrder::kKeys ? 64u : 16u;     // swizzle bit of LDS row bit 3
    auto row_of = [](int u) { return kOrder == BlockOrder::kValues ? 8 * u : ((u & 1) << 2) | ((u & 2) << 3); };
    if (count == kWalkBlock) {
        const uint32_t off = (uint32_t)l.pos * pitch;
#pragma unroll
        for (int u = 0; u < kBlockCopies; ++u) copy16_to_lds(first, off + (l.chunk ^ (kFlip * (u & 1))), row_of(u) * pitch, lds_addr + 1024u * u);
    } else {
        const int room = max(count - 1, 0);
#pragma unroll
        for (int u = 0; u < kBlockCopies; ++u)
            copy16_to_lds(first, (uint32_t)min(l.pos + row_of(u), room) * pitch + (l.chunk ^ (kFlip * (u & 1))), lds_addr + 1024u * u);
    }
}

// A wave's [32 rows][64 d] result, held transposed (lane (j, g), register v of half db: row j, d = 32*db + kappa(v, g)),
// into its own region of LDS.
__device__ __forceinline__ void result_to_lds(const floatx16 (&acc)[2], float* region, int lane) {
    const int j = lane & 31, g = lane >> 5;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int t = 0; t < 4; ++t)
            *reinterpret_cast<float4*>(region + j * kRedPitch + 32 * db + 8 * t + 4 * g) =
                make_float4(acc[db][4 * t], acc[db][4 * t + 1], acc[db][4 * t + 2], acc[db][4 * t + 3]);
}

// The same for 64 rows, unpadded: 16-byte chunk c of row r sits at chunk c ^ result_swizzle(r).  Sixteen consecutive rows spread a chunk column
// over all banks (these writes), four consecutive rows and every other chunk do so too (the merges' reads: four threads a row).
__device__ __forceinline__ int result_swizzle(int row) {
    return (row & 1) | ((row & 2) << 2) | ((row & 4) >> 1) | ((row & 8) >> 1);
}
// half 0: rows 0 to 31, half 1: rows 32 to 63
__device__ __forceinline__ void half_to_lds(const floatx16& d0, const floatx16& d1, float* region, int half, int lane) {
    const int r = kWalkBlock * half + (lane & 31);
    const floatx16 acc[2] = {d0, d1};
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int t = 0; t < 4; ++t)
            *reinterpret_cast<float4*>(region + r * kD + 4 * ((8 * db + 2 * t + (lane >> 5)) ^ result_swizzle(r))) =
                make_float4(acc[db][4 * t], acc[db][4 * t + 1], acc[db][4 * t + 2], acc[db][4 * t + 3]);
}
// Chunk i of the four that a thread takes of a row: d = od .. od + 7 and 32 further on, od = 8 * (thread & 3).
__device__ __forceinline__ float4 result_chunk(const float* region, int row, int od, int i) {
    return *reinterpret_cast<const float4*>(region + row * kD + 4 * ((od / 4 + (i & 1) + 4 * (i & 2)) ^ result_swizzle(row)));
}

}  // namespace dfa
