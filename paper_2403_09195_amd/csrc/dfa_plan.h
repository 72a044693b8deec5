// Launch plan of the fused dilated-attention kernels: host-side construction.
//
// Query rows of one head are grouped by the set of (branch, segment) pairs that keep them
// (section 3.1, Eq. 1: a row is kept by branch (w, r) iff n mod r equals the head's start
// offset, and its keys are the kept rows of segment floor(n / w)).  Rows of one group share
// one key list per member branch, so a tile of such rows runs a single online softmax over
// the concatenated key lists - which is exactly the log-sum-exp merge of the branches.
#pragma once
#include <cstdint>
#include <vector>
#include "../../include/dfa.h"

namespace dfa {

constexpr int kTileRows = 256;   // query rows per workgroup (4 waves x 64 rows)
constexpr int kTileBlocks = 8;   // a wave's 64 rows are two blocks of 32, each with its own softmax state
constexpr int kBlockRows = 32;
constexpr int kWalkBlock = 32;   // keys per piece of a list cut into blocks (see cut_blocks)
constexpr int kWalkWaves = 4;    // waves that share such a list
constexpr int kPackWindow = 32;  // row groups (in signature order) after a group that are tried as its tile mates
constexpr int kShortRows = 64;   // query rows per workgroup of the short-launch kernels
constexpr int kDies = 8;         // launch order of a plan: item i on die i mod 8
constexpr int kLaunchItems = 1 << 19;    // most items of one launch (at most 16 workgroups of 256 threads each: a grid
                                         // holds fewer than 2^32 threads)
constexpr int kDkdvRows = 128;   // bf16 backward, full tiles: rows of a dk/dv workgroup; a tile is up to kDkdvParts of them
constexpr int kDkdvParts = kTileRows / kDkdvRows;
constexpr int kShortDkdvParts = kShortRows / kWalkBlock;     // bf16 backward, short launches: dk/dv workgroups of a tile
constexpr int kFwdWorkgroupsPerCu = 2;   // workgroups of the bf16 forward kernel that fit one compute unit
constexpr int kTailItemsPerDie = 96;     // launch order: items at the end of a die's list that go heaviest first
constexpr int kMaxTileSegs = 32; // key progressions per tile (the kernels hold a tile's list in LDS)
constexpr int kMaxCoalesceLcm = 64;   // largest common period of a tile's dilation rates that is coalesced

// One arithmetic progression of a tile's key list: keys key0 + stride * j, j < count.  Either the
// kept keys of one segment of one branch (multiplicity 1), or, where the member branches of a
// tile keep some keys more than once, a piece of their multiset union in which every key has the
// same multiplicity m: the key is then visited once and its softmax weight multiplied by m, which
// is what visiting it m times adds up to.  log2_mult = log2(m) is added to the scaled score.
struct KeySeg {
    int32_t key0, stride, count;
    float log2_mult;
};
struct Tile {
    int32_t h;          // head
    int32_t row_begin;  // first entry in the row list
    int32_t nrows;      // 1 .. kTileRows: slots of the tile (a packed tile's list has entries < 0, see HostPlan::rows)
    int32_t seg_begin;  // first entry in the key-segment list
    int32_t nseg;       // 0 = rows kept by no branch (output 0, lse -inf)
    int32_t n_steps;    // 64-key steps of the whole list: sum of ceil(count / 64)
};
struct Item {        // one workgroup of the launch
    int32_t tile;    // -1 = padding, nothing to do
    int32_t b;       // batch index
    Tile t;          // copy of tiles[tile]: a workgroup reads what it needs to start in one load
};

// What the planner needs to know of the chip: workgroup i of a launch runs on die i mod dies (each
// die has its own L2).  The library reads both numbers from the device; the default is the MI355X.
struct ChipShape {
    int32_t dies = 8;
    int32_t cus = 256;
    int32_t fwd_slots() const { return cus * kFwdWorkgroupsPerCu; }          // forward workgroups resident at once
    int32_t fwd_slots_per_die() const { return fwd_slots() / (dies > 0 ? dies : 1); }
};

// Split launches (few workgroups, see split_plan): workgroup g of the launch walks share `part` of `nparts` of the
// 64-key steps of launch item `item` and leaves its partial result in block `block` of the workspace
// (kSplitBlockBytes: out [256 rows][64] in fp16, each row divided by its largest magnitude, then lse [256] and
// those row scales [256] in fp32; rows in tile order).
struct SplitWg {
    int32_t item;           // -1 = padding
    int32_t part_nparts;    // part | nparts << 16
    int32_t block;
};
struct ItemParts {          // per launch item: its blocks are first_block .. first_block + nparts - 1 (nparts = 0: padding)
    int32_t first_block;
    int32_t nparts;
};
constexpr int kSplitBlockBytes = kTileRows * (DFA_HEAD_DIM * 2 + 8);
constexpr int kMaxSplit = 4;             // most shares a tile is cut into
constexpr int kMinShareSteps = 8;        // a share of fewer 64-key steps is not worth a partial result and its merge

// What a workgroup of the short forward starts from, all at one address known from its index: its launch item, the rows of its 64 slots (past the
// tile's last slot that one again), then short_records(longest list) records for each wave: blocks wave, wave + 4, ... of the list, the
// last one again without a valid key where the share has ended.
struct ShortRecord {
    int32_t key0;
    int32_t stride_count;    // stride | count << 24 | kTurn; count 0: past the share's end
    float log2_mult[2];      // of the keys' multiplicity for either 32-row block of the tile; -inf: they are skipped
};
constexpr int32_t kTurn = (int32_t)0x80000000;     // the block is not full, or other multiplicities than those of the share's block before
struct ShortStart {
    Item item;
    int32_t rows[kShortRows];
};
inline int32_t short_records(int32_t longest) { return (longest + kWalkWaves - 1) / kWalkWaves + 1; }
inline size_t short_start_bytes(int32_t longest) { return sizeof(ShortStart) + sizeof(ShortRecord) * kWalkWaves * short_records(longest); }

struct HostPlan {
    std::vector<Tile> tiles;
    std::vector<int64_t> tile_pairs;     // (query, key) pairs of each tile
    // token positions, tile after tile.  A tile that packs several row groups starts each group on a 32-row block of
    // its own; the slots in between hold ~n of a row n of the group (valid to load, never stored).
    std::vector<int32_t> rows;
    std::vector<KeySeg> segs;
    std::vector<int32_t> seg_mult;   // multiplicity of each entry of segs (packed tiles: the largest of its blocks)
    std::vector<int32_t> block_mult; // [segs][kTileBlocks]: multiplicity for the rows of each 32-row block, 0 = they skip the keys
    bool packed_tiles = false;       // some tile packs several row groups (block_mult differs between blocks, filler slots)
    std::vector<Item> items;
    bool whole_units = false;            // the launch order keeps all tiles of an (image, head) on one die
    std::vector<SplitWg> split_wgs;      // empty: the launch is not split
    std::vector<ItemParts> item_parts;
};

// Lays the starts of a short forward plan out, item after item.
std::vector<char> pack_starts(const HostPlan& plan);

// Validates the branch list (DFA_OK or a negative status).  offsets: [nb][H] or nullptr.
int check_branches(int32_t H, int32_t N, const dfa_branch_t* br, int32_t nb, const int32_t* offsets);

// Start offset of head h in branch x.
inline int32_t head_offset(const int32_t* offsets, int32_t H, int32_t x, int32_t h, int32_t r) {
    return offsets ? offsets[(int64_t)x * H + h] : h % r;
}

// Builds tiles, row lists, key segments and the launch order for B images.
// order_mode: 3 = default (see dfa_plan.cpp), 0 to 2 are alternatives kept for measurement.
// pack: row groups of fewer than eight 32-row blocks may share a tile (only the bf16 forward kernel reads such
// tiles: it takes its multiplicities per block from block_mult).
// tile_blocks: 32-row blocks of a tile, kTileBlocks or less.
// pack_tails: the rows past a group's last full tile may share a tile too (they then walk the union of two lists).
void build_plan(int32_t B, int32_t H, int32_t N, const dfa_branch_t* br, int32_t nb,
                const int32_t* offsets, int order_mode, const ChipShape& chip, bool pack, HostPlan* plan,
                int tile_blocks = kTileBlocks, bool pack_tails = false);

// Launches of the bf16 forward kernel with fewer workgroups than half the chip's slots are as long as their longest
// tile's walk.  There the walks are cut: every tile gets one workgroup, then the workgroup slots left over go one by
// one to the tile whose shares are longest (up to kMaxSplit shares, none shorter than kMinShareSteps), and a second,
// small launch merges the partial results of the tiles that were cut by their log-sum-exp weights (a tile left whole
// is written out by its one workgroup).  Launches that fill more than half the slots are left alone: cutting their
// longest walks fills every CU with two workgroups, which slows every step by more than the shorter walks save
// (two 1024^2 images: 54.7 us against 46.1 us).  The shares go to the dies in runs like the
// items they come from, the longest of a die first.  Fills plan->split_wgs / item_parts, or
// leaves them empty when the launch is not to be split.
void split_plan(HostPlan* plan, const ChipShape& chip);

// Cuts every progression into pieces of at most kWalkBlock keys, the form the kernels read whose waves walk blocks of a
// list on their own: piece i of a tile is one 16-byte record at a known place, whatever the progressions' lengths.  A piece
// of one key has stride 0, so that every stride is below the token count.  The short forward keeps strides in 24 bits;
// short_backward_plan takes the same bound, which its kernels do not need: past it a launch is long.
constexpr int32_t kMaxCutStride = 1 << 24;
void cut_blocks(HostPlan* plan);

// What cut_blocks would make of a plan: records of all its lists, and of the longest one.
struct CutSize {
    int64_t records = 0;
    int64_t longest = 0;
};
CutSize cut_size(const HostPlan& plan);
// A cut list takes 16 bytes per 32 keys where a progression took 16 bytes in all, and a plan has a list per row group: many
// small groups with long lists (a branch over the whole image beside narrow windows) would take gigabytes at
// some 100 000 tokens.  Plans past this many records (4 MB) keep their lists whole; such launches are long and lose nothing by it.
constexpr int64_t kMaxCutRecords = 1 << 18;
// The fp32 kernels give a workgroup 32 rows, every tile as many workgroups as the largest has.  A launch with part-filled tiles
// would start workgroups without rows and deal the others unevenly to the CUs; it takes a plan of 32-row tiles, unless it
// is long anyway (such a plan holds 32 bytes per workgroup).  Measured, us, forward / backward, 32-row tiles against 256-row ones: two
// images of 1024 tokens, 6 heads 19.8 / 55.2 against 31.1 / 56.3, four 31.3 / 86.4 against 42.8 / 90.9, one of 2500, 12 heads
// 74.1 / 239.8 against 99.7 / 268.4, 16 of 1024, 12 heads 289.6 / 643.8 against 289.5 / 642.3; tiles that are all full: one of
// 4096, 12 heads 162.3 / 545.0 against 160.2 / 543.4.  `plan`: the plain plan of 256-row tiles.
constexpr size_t kMaxRowTiles = 1 << 14;
bool wants_row_tiles(const HostPlan& plan);

// Launches that do not fill the chip are as long as one workgroup's start, walk and end.  The short-launch forward kernel cuts
// the walk by four inside the workgroup and gives it a quarter of the rows, but copies every key block for 64 rows where the
// other kernels copy it for 256.  It is considered up to two and a quarter times as many workgroups as there are slots, where no list has
// more than kShortBlocks blocks, and taken where it is estimated to be the faster one (kShortMargin).
constexpr int kShortBlocks = 64;
// Plans of more workgroups than start at once, or of up to a quarter more than there are CUs, are tried with the rests of row groups sharing
// tiles: fewer workgroups, some of which walk the union of two lists.  That is taken where the lists have kTailBlocks blocks or
// more on average and the workgroups become 4 % fewer (then they are worth more than some longer walks), where there are too many workgroups for
// the form otherwise, or where it brings them within the bound and no list gets longer.  Over 266 drawn shapes that this changes 1.14 times
// as fast in the mean, 24 of them slower by more than 3 % and 14 % at worst (one of 1576 tokens, 9 heads, with offsets 14.0 / 16.2): which
// of the two plans is the shorter there the lists' lengths alone do not tell, and rules on their growth lost as much elsewhere.  us, apart / sharing:
// one image of 2312 tokens, 12 heads (528 / 480 workgroups) 22.6 / 18.5, of 2219 (560 / 520) 27.0 / 21.9, one of 2332, 6 heads
// (264 / 240) 15.8 / 13.6, one of 2229, 12 heads, in whole tiles before, (528) 36.5 / 20.9; short lists that get longer: one of 1386, 16
// heads, four branches (552 / 504, 12 blocks on average) 14.9 / 17.0, one of 654, 16 heads (288 / 256, 9 blocks) 9.9 / 11.2.
constexpr int kTailBlocks = 19;
// Both times are estimated, in us, by sums that are linear in the plan: workgroups, with and without keys, the 32-key blocks or 64-key steps of all
// lists, and of the longest one.  A sum each for: short launches of one workgroup to a CU, of one round, of one round beside workgroups without keys, and
// of more; split launches; packed and whole tiles of one to a CU, one round and more.  Fitted to 1731 launches (3 to 16 heads, 200 to 8192 tokens, 1
// to 16 images, windows, single dilated branches, two to four branches), with residuals of 6 to 9 % for the short form (12 % beside workgroups without
// keys), 3 to 6 % for tiles of one to a CU and 9 to 14 % for the rest.  The margins keep the launches with whose estimates they
// are wrong most where they would be without the form; whole tiles of one step always stay (one of 256 tokens, windows of 32, 6 images of 6
// heads 5.4 / 7.2), and of split launches none of up to nine eighths of the slots.  On 897 other drawn launches the choice differs from that by
// estimates fitted to earlier kernels on 87, which run 1.23 times as fast in the mean, two slower by more than 3 % (0.91 at worst: 11 of 259 tokens,
// 12 heads 17.7 / 19.4).  us, tiles or split / short: 7 images of 1152 tokens, 3 heads, four branches 30.9 / 14.4; 2 of 875, 16 heads 24.8 / 13.6;
// one of 4736, 8 heads, windows of 1184 at rate 3 13.2 / 8.2; 3 of 1024, 12 heads 17.0 / 14.1; left as they are: one of 4096, 12 heads, split 30.6 / 31.8;
// 10 of 959, 6 heads, windows of 191 12.2 / 14.3.
// (Packed tiles of more than one to a CU: fitted again to 399 launches of 1 to 32 heads and 16 tokens on.  Lists of a few steps had been estimated up to a
// fifth too long, and the short form was taken where it is the slower one: 23 images of 98 tokens, 4 heads, two branches 12.4 us in tiles, 14.9
// short.  Of 1600 launches the choice is more than 5 % slower than the other form on 47, where it was on 61, and 0.4 % in the mean.)
// With one workgroup to a CU, lists that do not fill their last step stay with the short kernel whatever the times: it clears the rows past a list's
// end, where the 256-row kernel gives them weight 0, which makes NaN of an infinite value, and its start outweighs the walk by 2 us at most.
constexpr double kShortMargin = 1.05;
constexpr double kIdleMargin = 1.25;      // one round of workgroups with keys, and others that need a second one
constexpr double kWholeMargin = 1.15;     // more than a round, against tiles of one row group each
bool short_plan(int32_t B, int32_t H, int32_t N, const dfa_branch_t* br, int32_t nb, const int32_t* offsets,
                int order_mode, const ChipShape& chip, const HostPlan& full, HostPlan* plan);

// The same for the backward.  The kernels of dfa_bwd_bf16.hip walk a tile's whole list in one workgroup and spend as much on
// a part-filled tile as on a full one; those of dfa_bwd_short.hip cut the walk by four and have 64-row tiles, but copy a block
// for 64 (dq) or 32 rows (dk, dv).  Both times, in us, are linear in the plan: 64-row tiles, with and without keys, 32 x 32 blocks of pairs and the
// longest list, in a sum each for up to two rounds of workgroups and for more; 256-row tiles, steps and the longest list, in a sum each for one tile
// to a CU, one round and more.  (In the middle one tiles weigh less than nothing: of the same steps, more tiles are shorter walks.  Fitted without
// that, to 498 calls, it sends 86 of 3010 elsewhere, to no gain in the mean and 1.65 times the time at worst.)  Fitted to 900 calls (200 to 4096 tokens, 3 to 16 heads, 1 to 16 images, one to four branches), with residuals of 6 to 8 %
// (short) and 7 to 12 % (full); below 16 us a call is bound by its host side.  On these the choice costs 0.4 % against the faster form of each, where
// estimates fitted to earlier kernels cost 1.6 %: it differs on 67, which run 1.18 times as fast in the mean, three slower by more than 3 % (0.93 at
// worst).  Past kFewTiles 64-row tiles the earlier ones stay (of 3010 launches, most of them past that, 326 would be more than 5 % shorter in the other
// form since tiles of a few rows got shorter there; 4 % in the mean): 15 + the larger of 3.2 per step of the longest list and
// 0.0164 per step of all 256-row tiles, against 10 + 0.024 per 64-row tile + 0.00105 per block of pairs.  us, full / short: 8 images of 384 tokens, 12 heads,
// windows of 54 32.1 / 22.5; 64 of 64, 8 heads 20.4 / 16.2; 7 of 521, 12 heads, one window 64.3 / 47.6; 2 of 3520, 8 heads, windows of 1173 at rate 3 36.2 / 26.1.
// `full` is the plain plan of 256-row tiles.
constexpr int kShortBackwardBlocks = 256;
constexpr double kShortBackwardMargin = 0.97;
constexpr double kFewTiles = 1280;
// dk/dv workgroups of every tile of a plan whose tiles have up to max_tile_rows rows (tiles of up to 32 have no second half: an empty workgroup
// still waits for a place on a CU)
inline int short_dkdv_parts(int max_tile_rows) { return max_tile_rows > kWalkBlock ? kShortDkdvParts : 1; }
// workgroups of the launch that works out all gradients of n_items launch items: dq ones, padded to whole rounds of the dies, then dk/dv ones
inline int64_t short_backward_workgroups(int64_t n_items, int parts) { return (n_items + kDies - 1) / kDies * kDies * (1 + parts); }
bool short_backward_plan(int32_t B, int32_t H, int32_t N, const dfa_branch_t* br, int32_t nb, const int32_t* offsets,
                         int order_mode, const ChipShape& chip, const HostPlan& full, HostPlan* plan);

}  // namespace dfa
