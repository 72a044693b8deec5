#include "dfa_plan.h"

#include <algorithm>
#include <deque>
#include <array>
#include <cmath>
#include <map>
#include <numeric>

namespace dfa {

namespace {

int64_t steps_of(const std::vector<KeySeg>& segs) {
    int64_t n = 0;
    for (const KeySeg& s : segs) n += (s.count + 63) / 64;
    return n;
}

// Multiplicities of one progression's keys for the (up to kTileBlocks) row groups of a tile; 0 = the group's rows
// do not attend to these keys.
using MultVec = std::array<int32_t, kTileBlocks>;

// The multiset union of the progressions in `plain` rewritten as progressions in which every key has one
// multiplicity.  A tile of one row group has one plain progression per member branch; a tile that packs several
// row groups has the distinct progressions of all of them, and member[g] says which ones group g's rows attend
// to (bit x = plain[x]): a key's multiplicity is then a number per group.  With L the least common multiple of
// the strides, a residue class mod L is either inside or outside each progression's own class, so along one
// class the multiplicities only change where a progression starts or ends.  Classes covered by the same
// progressions are joined into coarser strides where they line up.
// Returns false (outputs untouched) when L is too large, the list would not fit a tile, or no 64-key step
// would be saved against walking the plain progressions one after the other.
bool coalesce(const std::vector<KeySeg>& plain, const std::vector<uint32_t>& member, std::vector<KeySeg>* out,
              std::vector<MultVec>* out_mult) {
    const int ns = (int)plain.size(), ng = (int)member.size();
    if (ns < 2 || ns > 32) return false;
    int64_t L = 1;
    for (const KeySeg& s : plain) {
        L = std::lcm<int64_t>(L, s.stride);
        if (L > kMaxCoalesceLcm) return false;
    }
    std::vector<int64_t> last(ns);
    for (int x = 0; x < ns; ++x) last[x] = plain[x].key0 + (int64_t)(plain[x].count - 1) * plain[x].stride;

    std::vector<uint32_t> mask_of(L, 0);
    for (int64_t rho = 0; rho < L; ++rho)
        for (int x = 0; x < ns; ++x)
            if ((rho - plain[x].key0) % plain[x].stride == 0) mask_of[rho] |= 1u << x;

    std::vector<KeySeg> segs;
    std::vector<MultVec> mult;
    std::vector<char> used(L, 0);
    for (int64_t rho0 = 0; rho0 < L; ++rho0) {
        const uint32_t mask = mask_of[rho0];
        if (used[rho0] || mask == 0) continue;
        // where the multiplicity can change along these classes
        std::vector<int64_t> cuts;
        for (int x = 0; x < ns; ++x)
            if (mask >> x & 1) {
                cuts.push_back(plain[x].key0);
                cuts.push_back(last[x] + 1);
            }
        std::sort(cuts.begin(), cuts.end());
        cuts.erase(std::unique(cuts.begin(), cuts.end()), cuts.end());
        // the classes with this mask, as progressions (a mod g), smallest stride first
        for (int64_t g = 1; g <= L; ++g) {
            if (L % g) continue;
            for (int64_t a = 0; a < g; ++a) {
                bool all = true;
                for (int64_t rho = a; rho < L && all; rho += g) all = !used[rho] && mask_of[rho] == mask;
                if (!all) continue;
                for (int64_t rho = a; rho < L; rho += g) used[rho] = 1;
                size_t open = segs.size();                      // pieces of this (a mod g) start here
                for (size_t c = 0; c + 1 < cuts.size(); ++c) {
                    const int64_t lo = cuts[c], hi = cuts[c + 1];
                    uint32_t cover = 0;                             // progressions that hold the keys of [lo, hi) in these classes
                    for (int x = 0; x < ns; ++x)
                        if ((mask >> x & 1) && plain[x].key0 <= lo && hi - 1 <= last[x]) cover |= 1u << x;
                    if (cover == 0) continue;
                    MultVec m{};
                    for (int gi = 0; gi < ng; ++gi) m[gi] = __builtin_popcount(cover & member[gi]);
                    const int64_t key0 = lo + (((a - lo) % g) + g) % g;
                    if (key0 >= hi) continue;
                    const int32_t count = (int32_t)((hi - 1 - key0) / g + 1);
                    if (segs.size() > open && mult.back() == m &&
                        segs.back().key0 + (int64_t)segs.back().count * g == key0) {
                        segs.back().count += count;             // the progression runs on with the same multiplicity
                    } else {
                        segs.push_back(KeySeg{(int32_t)key0, (int32_t)g, count, std::log2((float)std::max(m[0], 1))});
                        mult.push_back(m);
                    }
                }
            }
        }
    }
    if ((int)segs.size() > kMaxTileSegs || steps_of(segs) >= steps_of(plain)) return false;
    // ascending first keys: consecutive steps then read neighbouring rows
    std::vector<size_t> order(segs.size());
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](size_t i, size_t j) { return segs[i].key0 < segs[j].key0; });
    out->clear();
    out_mult->clear();
    for (size_t i : order) {
        out->push_back(segs[i]);
        out_mult->push_back(mult[i]);
    }
    return true;
}

// Rows of one head that share their key lists: the same parts of the same branches keep them.
struct RowGroup {
    std::vector<int32_t> rows;
    std::vector<KeySeg> plain;        // one progression per member branch
    std::vector<int64_t> plain_id;    // which (branch, part) each one is
    std::vector<KeySeg> list;         // what a tile of these rows alone walks
    std::vector<MultVec> list_mult;   // entry 0: the multiplicity of the progression's keys
    int64_t key_lo = 0, key_hi = -1;  // first and last key of its progressions
};

int blocks_of(const RowGroup& g) { return ((int)g.rows.size() + kBlockRows - 1) / kBlockRows; }

// Key list of a tile whose rows come from the groups in `pack` (group i of the pack = entry i of the
// multiplicities): the coalesced union of their progressions where that saves steps, else the distinct
// progressions one after the other.  False when the list would not fit a tile.
bool tile_list(const std::vector<const RowGroup*>& pack, std::vector<KeySeg>* list, std::vector<MultVec>* mult) {
    std::vector<KeySeg> plain;
    std::vector<int64_t> ids;
    std::vector<uint32_t> member(pack.size(), 0);
    for (size_t gi = 0; gi < pack.size(); ++gi)
        for (size_t x = 0; x < pack[gi]->plain.size(); ++x) {
            size_t at = std::find(ids.begin(), ids.end(), pack[gi]->plain_id[x]) - ids.begin();
            if (at == ids.size()) {
                if (ids.size() == 32) return false;
                ids.push_back(pack[gi]->plain_id[x]);
                plain.push_back(pack[gi]->plain[x]);
            }
            member[gi] |= 1u << at;
        }
    if (coalesce(plain, member, list, mult)) return true;
    if ((int)plain.size() > kMaxTileSegs) return false;
    list->assign(plain.begin(), plain.end());
    mult->assign(plain.size(), MultVec{});
    for (size_t x = 0; x < plain.size(); ++x)
        for (size_t gi = 0; gi < pack.size(); ++gi) (*mult)[x][gi] = member[gi] >> x & 1;
    return true;
}

}  // namespace

int check_branches(int32_t H, int32_t N, const dfa_branch_t* br, int32_t nb, const int32_t* offsets) {
    if (nb < 1 || nb > DFA_MAX_BRANCHES) return DFA_ERR_BRANCHES;
    if (!br) return DFA_ERR_NULL;
    if (H <= 0 || N <= 0) return DFA_ERR_SHAPE;
    for (int x = 0; x < nb; ++x) {
        const int32_t w = br[x].w, r = br[x].r;
        if (r < 1 || w < 1) return DFA_ERR_SHAPE;
        if (offsets)
            for (int h = 0; h < H; ++h) {
                const int32_t o = offsets[(int64_t)x * H + h];
                if (o < 0 || o >= r) return DFA_ERR_SHAPE;
            }
    }
    return DFA_OK;
}

void build_plan(int32_t B, int32_t H, int32_t N, const dfa_branch_t* br, int32_t nb,
                const int32_t* offsets, int order_mode, const ChipShape& chip, bool pack, HostPlan* plan,
                int tile_blocks, bool pack_tails) {
    const int kNumXcd = std::max(chip.dies, 1);
    const int kSlotsPerDie = std::max(chip.fwd_slots_per_die(), 1);
    plan->tiles.clear();
    plan->rows.clear();
    plan->segs.clear();
    plan->seg_mult.clear();
    plan->block_mult.clear();
    plan->items.clear();
    plan->packed_tiles = false;
    const size_t tile_rows = (size_t)tile_blocks * kBlockRows;

    std::vector<int64_t>& tile_cost = plan->tile_pairs;
    tile_cost.clear();
    // appends a key list; block_group[w] = which entry of a progression's multiplicities the rows of block w take (-1: none)
    auto add_list = [&](const std::vector<KeySeg>& list, const std::vector<MultVec>& mult, const int (&block_group)[kTileBlocks]) {
        const int32_t seg_begin = (int32_t)plan->segs.size();
        plan->segs.insert(plan->segs.end(), list.begin(), list.end());
        for (const MultVec& m : mult) {
            int32_t most = 0;
            for (int w = 0; w < kTileBlocks; ++w) {
                const int32_t mw = block_group[w] < 0 ? 0 : m[block_group[w]];
                plan->block_mult.push_back(mw);
                most = std::max(most, mw);
            }
            plan->seg_mult.push_back(most);
        }
        return seg_begin;
    };
    // heads with the same start offsets in every branch have the same rows, lists and tiles: the later one's tiles
    // are copies of the earlier one's (pointing at the same rows and progressions) under its own head number
    std::map<std::vector<int32_t>, std::pair<size_t, size_t>> tiles_of_offsets;
    for (int32_t h = 0; h < H; ++h) {
        std::vector<int32_t> head_key(nb);
        for (int x = 0; x < nb; ++x) head_key[x] = head_offset(offsets, H, x, h, br[x].r);
        const auto twin = tiles_of_offsets.find(head_key);
        if (twin != tiles_of_offsets.end()) {
            for (size_t t = twin->second.first; t < twin->second.second; ++t) {
                Tile copy = plan->tiles[t];
                copy.h = h;
                plan->tiles.push_back(copy);
                tile_cost.push_back(tile_cost[t]);
            }
            continue;
        }
        const size_t first_tile = plan->tiles.size();
        // signature of a row: for each branch the part that keeps it, or -1
        std::map<std::vector<int32_t>, RowGroup> by_sig;
        std::vector<int32_t> sig(nb);
        for (int32_t n = 0; n < N; ++n) {
            for (int x = 0; x < nb; ++x) {
                const int32_t o = head_offset(offsets, H, x, h, br[x].r);
                const int32_t part = n / br[x].w, pos = n - part * br[x].w - o;   // position inside the part
                sig[x] = (pos >= 0 && pos % br[x].r == 0) ? part : -1;
            }
            by_sig[sig].rows.push_back(n);
        }
        std::vector<RowGroup*> groups;
        for (auto& kv : by_sig) {
            const std::vector<int32_t>& s = kv.first;
            RowGroup& g = kv.second;
            for (int x = 0; x < nb; ++x) {
                if (s[x] < 0) continue;
                const int32_t o = head_offset(offsets, H, x, h, br[x].r);
                // kept keys of the part: first, first + r, ... below the end of the part (the last part
                // is shorter when w does not divide N)
                const int64_t first = (int64_t)s[x] * br[x].w + o;
                const int64_t end = std::min<int64_t>((int64_t)(s[x] + 1) * br[x].w, N);
                const int32_t count = (int32_t)((end - 1 - first) / br[x].r + 1);   // >= 1: a row of the part is kept
                g.plain.push_back(KeySeg{(int32_t)first, br[x].r, count, 0.f});
                g.plain_id.push_back((int64_t)x * ((int64_t)N + 1) + s[x]);
                const int64_t last_key = first + (int64_t)(count - 1) * br[x].r;
                if (g.key_hi < g.key_lo) {
                    g.key_lo = first;
                    g.key_hi = last_key;
                } else {
                    g.key_lo = std::min(g.key_lo, first);
                    g.key_hi = std::max(g.key_hi, last_key);
                }
            }
            // keys that several member branches keep are visited once, weighted by how many keep them
            if (!g.plain.empty()) tile_list({&g}, &g.list, &g.list_mult);
            groups.push_back(&g);
        }

        // The rows past a group's last full tile as a group of their own (same lists), which may share a tile like any other.
        std::deque<RowGroup> tails;
        if (pack_tails) {
            std::vector<RowGroup*> cut;
            for (RowGroup* g : groups) {
                cut.push_back(g);
                const size_t rest = g->rows.size() % tile_rows;
                if (g->plain.empty() || g->rows.size() < tile_rows || rest == 0) continue;
                tails.push_back(*g);
                tails.back().rows.assign(g->rows.end() - rest, g->rows.end());
                g->rows.resize(g->rows.size() - rest);
                cut.push_back(&tails.back());
            }
            groups.swap(cut);
        }

        // Row groups that fill only part of a tile.  Where such groups attend to many of the same keys (rows of one
        // window of a narrow branch that differ in which wider, dilated branches also keep them), a tile takes
        // several of them, each in 32-row blocks of its own (half a wave: the unit that has its own softmax state in the
        // kernel): the tile walks the union of their lists once, and a block whose
        // rows do not attend to a progression masks its scores (multiplicity 0).  A group joins a tile when at least
        // half the steps of the shorter of the two lists are saved.
        const size_t G = groups.size();
        std::vector<char> done(G, 0);
        for (size_t i = 0; i < G; ++i) {
            if (done[i]) continue;
            done[i] = 1;
            const RowGroup& g = *groups[i];
            const bool small = pack && !g.plain.empty() && blocks_of(g) < tile_blocks;
            std::vector<const RowGroup*> members = {&g};
            std::vector<KeySeg> list = g.list;
            std::vector<MultVec> list_mult = g.list_mult;
            int blocks = blocks_of(g);
            int64_t key_lo = g.key_lo, key_hi = g.key_hi;
            while (small && blocks < tile_blocks) {
                int64_t best = -1, best_saved = 0;
                std::vector<KeySeg> best_list;
                std::vector<MultVec> best_mult;
                const int64_t have = steps_of(list);
                for (size_t j = i + 1; j < std::min(G, i + 1 + kPackWindow); ++j) {
                    const RowGroup& c = *groups[j];
                    if (done[j] || c.plain.empty() || blocks + blocks_of(c) > tile_blocks) continue;
                    if (c.key_hi < key_lo || key_hi < c.key_lo) continue;      // no key in common: nothing to save
                    std::vector<const RowGroup*> trial = members;
                    trial.push_back(&c);
                    std::vector<KeySeg> tl;
                    std::vector<MultVec> tm;
                    if (!tile_list(trial, &tl, &tm)) continue;
                    const int64_t own = steps_of(c.list), saved = have + own - steps_of(tl);
                    if (saved * 2 < std::min(have, own) || saved <= best_saved) continue;
                    best = (int64_t)j;
                    best_saved = saved;
                    best_list.swap(tl);
                    best_mult.swap(tm);
                }
                if (best < 0) break;
                done[best] = 1;
                members.push_back(groups[best]);
                blocks += blocks_of(*groups[best]);
                key_lo = std::min(key_lo, groups[best]->key_lo);
                key_hi = std::max(key_hi, groups[best]->key_hi);
                list.swap(best_list);
                list_mult.swap(best_mult);
            }
            const int32_t nseg = (int32_t)list.size();
            if (members.size() == 1) {
                // tiles of one group: cut its rows into tiles that share the list; every block takes entry 0
                const int block_group[kTileBlocks] = {0, 0, 0, 0, 0, 0, 0, 0};
                const int32_t seg_begin = add_list(list, list_mult, block_group);
                int64_t keys = 0;
                for (const KeySeg& sg : list) keys += sg.count;
                for (size_t lo = 0; lo < g.rows.size(); lo += tile_rows) {
                    const int32_t cnt = (int32_t)std::min<size_t>(tile_rows, g.rows.size() - lo);
                    Tile t{h, (int32_t)plan->rows.size(), cnt, seg_begin, nseg, (int32_t)steps_of(list)};
                    plan->rows.insert(plan->rows.end(), g.rows.begin() + lo, g.rows.begin() + lo + cnt);
                    plan->tiles.push_back(t);
                    tile_cost.push_back(keys * cnt);
                }
                continue;
            }
            // one tile of several groups: each starts on a block of its own; the slots between the end of a group and
            // the next block hold ~row of the group's last row (a valid row to load, never stored)
            plan->packed_tiles = true;
            int block_group[kTileBlocks] = {-1, -1, -1, -1, -1, -1, -1, -1};
            const int32_t row_begin = (int32_t)plan->rows.size();
            int w0 = 0;
            int64_t pairs = 0;
            for (size_t gi = 0; gi < members.size(); ++gi) {
                const RowGroup& m = *members[gi];
                if (gi > 0) {
                    const int32_t filler = ~members[gi - 1]->rows.back();
                    while ((int32_t)plan->rows.size() - row_begin < w0 * kBlockRows) plan->rows.push_back(filler);
                }
                plan->rows.insert(plan->rows.end(), m.rows.begin(), m.rows.end());
                for (int w = 0; w < blocks_of(m); ++w) block_group[w0 + w] = (int)gi;
                w0 += blocks_of(m);
                for (size_t x = 0; x < list.size(); ++x)
                    pairs += (int64_t)list[x].count * (list_mult[x][gi] ? 1 : 0) * (int64_t)m.rows.size();
            }
            const int32_t seg_begin = add_list(list, list_mult, block_group);
            plan->tiles.push_back(Tile{h, row_begin, (int32_t)plan->rows.size() - row_begin, seg_begin, nseg, (int32_t)steps_of(list)});
            tile_cost.push_back(pairs);
        }
        tiles_of_offsets[head_key] = {first_tile, plan->tiles.size()};
    }

    // Launch order.  Workgroup i runs on die i mod 8, each die has its own L2, and the tiles
    // of one (b, h) read the same K/V rows: keep a (b, h) unit on one die when there are
    // enough units to balance the dies, otherwise give every die a run of tiles.  Within a die the
    // heaviest tiles go first so the tail of the launch is made of short ones.
    const int32_t T = (int32_t)plan->tiles.size();
    std::vector<std::vector<int32_t>> tiles_of_head(H);
    std::vector<int64_t> head_cost(H, 0);
    for (int32_t t = 0; t < T; ++t) {
        tiles_of_head[plan->tiles[t].h].push_back(t);
        head_cost[plan->tiles[t].h] += tile_cost[t];
    }
    std::vector<std::vector<Item>> per_die(kNumXcd);
    std::vector<int64_t> die_cost(kNumXcd, 0);
    auto lightest = [&]() {
        return (int)(std::min_element(die_cost.begin(), die_cost.end()) - die_cost.begin());
    };
    // whole units per die when that balances the dies to within an eighth (always with 4 units per die or more);
    // every die then reads only its own units' K/V rows from memory
    const int64_t units = (int64_t)B * H;
    const bool by_unit = plan->whole_units = units >= 4 * kNumXcd ||
                         (units >= kNumXcd && ((units + kNumXcd - 1) / kNumXcd) * kNumXcd * 8 <= units * 9);
    // Fewer units: the tiles one after the other, unit by unit and within a unit by their first row, cut into a run of the same number for
    // every die: the tiles of a run share most of their K/V rows, which the die then reads once.  Only where that balances the dies to
    // within a thirty-second; otherwise single tiles are spread.  (12 heads, us, spread / runs: one 1024^2 image, forward 32.1 / 30.0, one 800^2
    // image, forward and backward 69.4 / 64.2, two 512^2 images of 6 heads in fp32 60.9 / 58.3; one image of 10122 tokens 242 / 153.  Of 890 drawn
    // launches those of 64 tiles and more take 0.91 to 0.99 of the time of spread ones, those of fewer the same.  So would the runs that the bound
    // turns away, up to two fifths apart in pairs, and so do those whose dies are that far apart in steps: it could be wider.)
    auto by_runs = [&]() {
        const int64_t total = (int64_t)T * B;
        int64_t at = 0, all = 0;
        for (auto& tiles : tiles_of_head)
            std::stable_sort(tiles.begin(), tiles.end(),
                             [&](int32_t a, int32_t c) { return plan->rows[plan->tiles[a].row_begin] < plan->rows[plan->tiles[c].row_begin]; });
        for (int32_t b = 0; b < B; ++b)
            for (int32_t h = 0; h < H; ++h)
                for (int32_t t : tiles_of_head[h]) {
                    const int d = (int)(at++ * kNumXcd / total);
                    per_die[d].push_back(Item{t, b, plan->tiles[t]});
                    die_cost[d] += tile_cost[t];
                    all += tile_cost[t];
                }
        if (*std::max_element(die_cost.begin(), die_cost.end()) * kNumXcd <= all + all / 32) return true;
        for (auto& v : per_die) v.clear();
        std::fill(die_cost.begin(), die_cost.end(), 0);
        return false;
    };
    if (by_unit) {
        for (int32_t b = 0; b < B; ++b)
            for (int32_t h = 0; h < H; ++h) {
                const int d = lightest();
                for (int32_t t : tiles_of_head[h]) per_die[d].push_back(Item{t, b, plan->tiles[t]});
                die_cost[d] += head_cost[h];
            }
    } else if (!by_runs()) {
        std::vector<int32_t> order(T);
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(),
                         [&](int32_t a, int32_t c) { return tile_cost[a] > tile_cost[c]; });
        for (int32_t t : order)
            for (int32_t b = 0; b < B; ++b) {
                const int d = lightest();
                per_die[d].push_back(Item{t, b, plan->tiles[t]});
                die_cost[d] += std::max<int64_t>(tile_cost[t], 1);
            }
    }
    // Order inside a die.  Mode 3 (default): unit after unit, each unit's tiles heaviest first, so
    // that the workgroups running at the same time read the same K/V rows from the die's L2 and
    // every row comes from HBM about once; only the last kTailItemsPerDie items of the die are
    // ordered heaviest first as one group, so that the launch ends on short tiles (long lists only).  Mode 2: the
    // multi-progression tiles of one unit together, the single-progression tiles of all units
    // last as filler.  Mode 1: strictly unit after unit.  Mode 0: heaviest first overall.
    size_t longest = 0;
    const size_t die_cus = std::max<size_t>(kSlotsPerDie / kFwdWorkgroupsPerCu, 1);
    auto more_pairs = [&](const Item& a, const Item& c) { return tile_cost[a.tile] > tile_cost[c.tile]; };
    // By the length of their walks, which a tile with few rows takes as long for as a full one.  (By pairs such a tile came last and ended the
    // launch: 2 images of 1318 tokens, 9 heads 19.2 us, by length 15.)
    auto longer = [&](const Item& a, const Item& c) {
        const int32_t sa = plan->tiles[a.tile].n_steps, sc = plan->tiles[c.tile].n_steps;
        return sa != sc ? sa > sc : tile_cost[a.tile] > tile_cost[c.tile];
    };
    for (auto& v : per_die) {
        // a die with fewer than four items per workgroup slot is too short a list for mode 3's
        // unit-after-unit body to balance: it gets mode 2
        if (order_mode == 3 && v.size() < 4 * (size_t)kSlotsPerDie) order_mode = 2;
        const bool at_once = order_mode == 2 && v.size() <= (size_t)kSlotsPerDie;
        if (order_mode == 0 || !by_unit || at_once) {
            std::stable_sort(v.begin(), v.end(), longer);
            if (pack && at_once && v.size() > die_cus) {       // pack: a forward launch in bf16, one workgroup per item
                // Workgroups i and i + die_cus share a compute unit.  The longest have one to themselves, of the others a long one goes with a
                // short one.  (us, by length alone / so: 3 images of 2879 tokens, 3 heads 20.6 / 19.5, 12 heads of 1059 13.3 / 12.5; units dealt
                // whole, unit by unit / so: 2 images of 865 tokens, 12 heads 12.6 / 11.0, 3 of 905, windows of 150 11.4 / 8.7.  Backward launches,
                // which start more workgroups per item, lose 4 to 7 % by it.)
                const size_t twos = v.size() - die_cus;
                std::reverse(v.end() - twos, v.end());
                std::rotate(v.begin(), v.begin() + (die_cus - twos), v.begin() + die_cus);
            }
        } else {
            // v is unit-major already; sort each unit's run by cost, then (mode 2) move the
            // single-segment tiles behind everything else, keeping their order
            size_t lo = 0;
            while (lo < v.size()) {
                size_t hi = lo;
                while (hi < v.size() && v[hi].b == v[lo].b &&
                       plan->tiles[v[hi].tile].h == plan->tiles[v[lo].tile].h) ++hi;
                std::stable_sort(v.begin() + lo, v.begin() + hi, more_pairs);
                lo = hi;
            }
            if (order_mode == 2)
                std::stable_partition(v.begin(), v.end(),
                                      [&](const Item& a) { return plan->tiles[a.tile].nseg > 1; });
            if (order_mode == 3) {
                const size_t tail = std::min<size_t>(v.size(), kTailItemsPerDie);
                std::stable_sort(v.end() - tail, v.end(), more_pairs);
            }
        }
        longest = std::max(longest, v.size());
    }
    plan->items.reserve(longest * kNumXcd);
    for (size_t p = 0; p < longest; ++p)
        for (int d = 0; d < kNumXcd; ++d)
            plan->items.push_back(p < per_die[d].size() ? per_die[d][p] : Item{-1, 0, Tile{0, 0, 0, 0, 0, 0}});
}

void split_plan(HostPlan* plan, const ChipShape& chip) {
    plan->split_wgs.clear();
    plan->item_parts.clear();
    const int64_t slots = chip.fwd_slots(), n_items = (int64_t)plan->items.size();
    if (n_items == 0 || n_items * 2 > slots) return;
    std::vector<int32_t> parts(n_items, 0);
    int64_t total = 0;
    for (int64_t i = 0; i < n_items; ++i)
        if (plan->items[i].tile >= 0) {
            parts[i] = 1;
            ++total;
        }
    // One more share for the tile with the longest shares, as long as slots are left and the shares stay long enough.  Of several tiles with the
    // same shares the one with the most pairs comes first, then the first tile, then the first image; where whole units are dealt to the dies, the
    // first unit of every die tile by tile, then the second.  (By the tiles, not by the place in the launch: how a row is rounded then does
    // not change with the order of a launch.)
    const int64_t dies = std::max(chip.dies, 1), heads = plan->tiles.back().h + 1;
    std::vector<int32_t> by_pairs(plan->tiles.size()), rank(plan->tiles.size());
    std::iota(by_pairs.begin(), by_pairs.end(), 0);
    std::stable_sort(by_pairs.begin(), by_pairs.end(), [&](int32_t t, int32_t u) { return plan->tile_pairs[t] > plan->tile_pairs[u]; });
    {
        std::vector<int32_t> next(heads, 0);
        for (int32_t t : by_pairs) rank[t] = plan->whole_units ? next[plan->tiles[t].h]++ : next[0]++;
    }
    auto place = [&](int64_t i) {
        const Item& it = plan->items[i];
        const int64_t unit = it.b * heads + it.t.h;
        return plan->whole_units ? std::array<int64_t, 4>{it.t.nseg <= 1, unit / dies, rank[it.tile], unit % dies} : std::array<int64_t, 4>{0, 0, rank[it.tile], it.b};
    };
    std::vector<int64_t> by_work;
    for (int64_t i = 0; i < n_items; ++i)
        if (parts[i]) by_work.push_back(i);
    std::sort(by_work.begin(), by_work.end(), [&](int64_t i, int64_t k) { return place(i) < place(k); });
    bool any = false;
    while (total < slots) {
        int64_t best = -1;
        int32_t best_share = 0;
        for (int64_t i : by_work) {
            if (parts[i] >= kMaxSplit) continue;
            const int32_t steps = plan->items[i].t.n_steps;
            if (steps / (parts[i] + 1) < kMinShareSteps) continue;
            const int32_t share = (steps + parts[i] - 1) / parts[i];
            if (share > best_share) {
                best_share = share;
                best = i;
            }
        }
        if (best < 0) break;
        ++parts[best];
        ++total;
        any = true;
    }
    if (!any) return;
    std::vector<SplitWg> wgs;
    plan->item_parts.assign(n_items, ItemParts{0, 0});
    for (int64_t d = 0; d < dies; ++d)
        for (int64_t i = d; i < n_items; i += dies) {
            plan->item_parts[i] = ItemParts{(int32_t)wgs.size(), parts[i]};
            for (int32_t x = 0; x < parts[i]; ++x) wgs.push_back(SplitWg{(int32_t)i, x | (parts[i] << 16), (int32_t)wgs.size()});
        }
    // The shares die after die in the items' order, cut into a run of the same number for every die: the shares of a tile, and the tiles that read
    // the same K/V rows, are on a die but where a run ends.  Where a compute unit then walks longer, the shares of every length are cut so on
    // their own (the rest of a length goes to the dies with the fewest shares so far): a die has as many of every length as any other.
    // (us, all in one run per die / every length on its own: 2 images of 8043 tokens, windows of 4021, whose last tokens are a tile of
    // one step 37.6 / 27.4; one list over all tokens, tiles of two and of three shares: 8 heads of 6464 112 / 91, 2 images of 2486, 10 heads 50.8 /
    // 43.5; 12 heads of 4096, three branches, shares of 8 to 11 steps 34.4 / 34.6.)
    auto share_steps = [&](const SplitWg& g) { return plan->items[g.item].t.n_steps / (double)(g.part_nparts >> 16); };
    auto longer = [&](const SplitWg& a, const SplitWg& c) { return share_steps(a) > share_steps(c); };
    using Dies = std::vector<std::vector<SplitWg>>;
    auto runs = [&](Dies* of_die, size_t lo, size_t hi) {
        std::vector<int64_t> run(dies, (int64_t)(hi - lo) / dies);
        for (int64_t rest = (int64_t)(hi - lo) % dies; rest > 0; --rest) {
            int64_t fewest = 0;
            for (int64_t d = 1; d < dies; ++d)
                if ((int64_t)(*of_die)[d].size() + run[d] < (int64_t)(*of_die)[fewest].size() + run[fewest]) fewest = d;
            ++run[fewest];
        }
        for (int64_t d = 0; d < dies; lo += run[d++]) (*of_die)[d].insert((*of_die)[d].end(), wgs.begin() + lo, wgs.begin() + lo + run[d]);
    };
    const size_t die_cus = std::max(chip.cus / (int32_t)dies, 1);
    auto longest_unit = [&](const Dies& of_die) {              // workgroups i, i + die_cus, ... of a die share a compute unit
        double most = 0;
        for (const auto& v : of_die)
            for (size_t cu = 0; cu < std::min(die_cus, v.size()); ++cu) {
                double steps = 0;
                for (size_t x = cu; x < v.size(); x += die_cus) steps += share_steps(v[x]);
                most = std::max(most, steps);
            }
        return most;
    };
    Dies of_die(dies), by_length(dies);
    runs(&of_die, 0, wgs.size());
    for (auto& v : of_die) std::stable_sort(v.begin(), v.end(), longer);
    std::stable_sort(wgs.begin(), wgs.end(), longer);
    for (size_t lo = 0, hi = 0; lo < wgs.size(); lo = hi) {
        while (hi < wgs.size() && share_steps(wgs[hi]) == share_steps(wgs[lo])) ++hi;
        runs(&by_length, lo, hi);
    }
    if (longest_unit(of_die) > longest_unit(by_length)) of_die.swap(by_length);
    size_t longest = 0;
    for (const auto& v : of_die) longest = std::max(longest, v.size());
    plan->split_wgs.assign(longest * dies, SplitWg{-1, 0, 0});
    for (int64_t d = 0; d < dies; ++d)
        for (size_t x = 0; x < of_die[d].size(); ++x) plan->split_wgs[x * dies + d] = of_die[d][x];
}

CutSize cut_size(const HostPlan& plan) {
    CutSize size;
    std::vector<char> seen(plan.segs.size() + 1, 0);
    for (const Tile& t : plan.tiles) {
        if (t.nseg == 0 || seen[t.seg_begin]) continue;      // tiles of one group share their list
        seen[t.seg_begin] = 1;
        int64_t records = 0;
        for (int32_t x = t.seg_begin; x < t.seg_begin + t.nseg; ++x) records += ((int64_t)plan.segs[x].count + kWalkBlock - 1) / kWalkBlock;
        size.records += records;
        size.longest = std::max(size.longest, records);
    }
    return size;
}

void cut_blocks(HostPlan* plan) {
    std::vector<KeySeg> segs;
    std::vector<int32_t> mult, block_mult;
    std::map<int32_t, std::pair<int32_t, int32_t>> cut;      // seg_begin -> first piece, number of pieces
    auto cut_list = [&](Tile& t) {
        if (t.nseg == 0) return;
        auto it = cut.find(t.seg_begin);                     // tiles of one group share their list
        if (it == cut.end()) {
            const int32_t begin = (int32_t)segs.size();
            for (int32_t x = t.seg_begin; x < t.seg_begin + t.nseg; ++x) {
                const KeySeg& s = plan->segs[x];
                for (int32_t k = 0; k < s.count; k += kWalkBlock) {
                    const int32_t count = std::min(kWalkBlock, s.count - k);
                    segs.push_back(KeySeg{s.key0 + s.stride * k, count > 1 ? s.stride : 0, count, s.log2_mult});
                    mult.push_back(plan->seg_mult[x]);
                    block_mult.insert(block_mult.end(), plan->block_mult.begin() + (size_t)x * kTileBlocks,
                                      plan->block_mult.begin() + (size_t)(x + 1) * kTileBlocks);
                }
            }
            it = cut.emplace(t.seg_begin, std::make_pair(begin, (int32_t)segs.size() - begin)).first;
        }
        t.seg_begin = it->second.first;
        t.nseg = it->second.second;
    };
    for (Tile& t : plan->tiles) cut_list(t);
    for (Item& i : plan->items)
        if (i.tile >= 0) i.t = plan->tiles[i.tile];
    plan->segs.swap(segs);
    plan->seg_mult.swap(mult);
    plan->block_mult.swap(block_mult);
}

bool wants_row_tiles(const HostPlan& plan) {
    if (plan.items.size() > kMaxRowTiles / kTileBlocks) return false;
    int64_t tiles = 0, filled = 0, most = 0;           // 32-row blocks: with rows, and of the largest tile
    for (const Item& i : plan.items)
        if (i.tile >= 0) {
            const int64_t blocks = (i.t.nrows + kBlockRows - 1) / kBlockRows;
            ++tiles;
            filled += blocks;
            most = std::max(most, blocks);
        }
    return tiles * most > filled;
}

namespace {

// What short_plan estimates the times by: workgroups with keys (one of rows that no branch keeps is over at once), the 32-key blocks
// and 64-key steps of all their lists, and the steps of the longest one.
struct LaunchSize {
    int64_t live = 0, blocks = 0, steps = 0;
    int32_t longest = 0;
};
LaunchSize launch_size(const HostPlan& plan) {
    LaunchSize size;
    for (const Item& i : plan.items)
        if (i.tile >= 0 && i.t.nseg > 0) {
            ++size.live;
            for (int32_t x = 0; x < i.t.nseg; ++x) size.blocks += (plan.segs[i.t.seg_begin + x].count + kWalkBlock - 1) / kWalkBlock;
            size.steps += i.t.n_steps;
            size.longest = std::max(size.longest, i.t.n_steps);
        }
    return size;
}

}  // namespace

bool short_plan(int32_t B, int32_t H, int32_t N, const dfa_branch_t* br, int32_t nb, const int32_t* offsets,
                int order_mode, const ChipShape& chip, const HostPlan& full, HostPlan* plan) {
    const size_t near = (size_t)chip.fwd_slots() * 9 / 8, most = (size_t)chip.fwd_slots() * 9 / 4;
    // 64 rows to a workgroup: more rows than this cannot fit
    if ((uint64_t)B * H * N > (uint64_t)most * kShortRows || full.items.size() > most || N >= kMaxCutStride) return false;
    build_plan(B, H, N, br, nb, offsets, order_mode, chip, true, plan, kShortRows / kBlockRows);
    // A little more than one round of workgroups, or than one to a CU: fewer of them where the rests of row groups share tiles (see
    // kTailBlocks).
    const int64_t slots = chip.fwd_slots(), one = slots / kFwdWorkgroupsPerCu;
    const LaunchSize apart = launch_size(*plan);
    if ((apart.live > one && apart.live <= one * 5 / 4) || apart.live > slots) {
        HostPlan shared;
        build_plan(B, H, N, br, nb, offsets, order_mode, chip, true, &shared, kShortRows / kBlockRows, true);
        const int64_t live = launch_size(shared).live, bound = apart.live > slots ? slots : one;
        const int64_t longest = cut_size(shared).longest;
        // (padding for the dies included, the plan must not leave the range that it is in apart)
        if (longest <= kShortBlocks && (plan->items.size() > near || shared.items.size() <= near) && ((apart.blocks >= kTailBlocks * apart.live && 25 * live <= 24 * apart.live) ||
                                        (plan->items.size() > near && shared.items.size() <= near) ||
                                        (live <= bound && longest <= cut_size(*plan).longest)))
            *plan = std::move(shared);
    }
    const int32_t longest = (int32_t)cut_size(*plan).longest;
    if (plan->items.size() > most || longest > kShortBlocks) return false;
    const LaunchSize size = launch_size(*plan), whole = launch_size(full);
    const bool split = !full.split_wgs.empty();
    cut_blocks(plan);
    const bool one_to_a_cu = size.live <= one;
    if (!split && one_to_a_cu && plan->items.size() <= near && std::any_of(full.segs.begin(), full.segs.end(), [](const KeySeg& s) { return s.count % 64 != 0; })) return true;
    if (split && plan->items.size() <= near) return true;
    if (!split && !full.packed_tiles && whole.longest <= 1) return false;
    // packed tiles that are full walk like tiles of one group
    const bool shared = full.packed_tiles && std::any_of(full.tiles.begin(), full.tiles.end(), [](const Tile& t) { return t.nrows != kTileRows; });
    // us, see kShortMargin
    const double per_slot = 512.0 / slots;
    const double items = per_slot * plan->items.size(), live = per_slot * size.live, blocks = per_slot * size.blocks;
    const double tiles = per_slot * full.items.size(), steps = per_slot * whole.steps;
    const bool one_round = (int64_t)plan->items.size() <= slots, live_fit = size.live <= slots;
    const double short_us = one_to_a_cu ? 5.2 + 0.0016 * items + 0.184 * longest
                            : one_round ? 6.3 + 0.0004 * blocks + 0.113 * longest
                            : live_fit  ? 5.7 + 0.0029 * items + 0.00012 * blocks + 0.186 * longest
                                        : 4.9 + 0.0025 * items + 0.0057 * live + 0.00053 * blocks + 0.052 * longest;
    const bool few = (int64_t)full.items.size() <= one, fit = (int64_t)full.items.size() <= slots;
    const double other_us = split               ? (shared ? 23.3 + 0.002 * steps : 12.6 + 0.0043 * steps)
                            : full.packed_tiles ? (few   ? 6.9 + 0.0025 * tiles + 0.00012 * steps + 1.27 * whole.longest
                                                   : fit ? 6.8 + 0.0023 * steps + 1.06 * whole.longest
                                                         : 5.0 + 0.0053 * steps + 0.74 * whole.longest)
                            : few ? 4.1 + 0.002 * tiles + 0.0002 * steps + 1.2 * whole.longest
                            : fit ? 3.6 + 0.005 * tiles + 0.0025 * steps + 0.86 * whole.longest
                                  : 5.5 + 0.0031 * tiles + 0.0037 * steps + 0.65 * whole.longest;
    const double margin = live_fit && plan->items.size() > near && !one_to_a_cu && !split ? kIdleMargin : !live_fit && !(split ? shared : full.packed_tiles) ? kWholeMargin : kShortMargin;
    return short_us * margin < other_us;
}

std::vector<char> pack_starts(const HostPlan& plan) {
    int32_t longest = 0;
    for (const Tile& t : plan.tiles) longest = std::max(longest, t.nseg);
    const size_t bytes = short_start_bytes(longest);
    const int32_t per_wave = short_records(longest);
    std::vector<char> out(plan.items.size() * bytes, 0);
    for (size_t i = 0; i < plan.items.size(); ++i) {
        const Item& item = plan.items[i];
        ShortStart* const start = reinterpret_cast<ShortStart*>(out.data() + i * bytes);
        start->item = item;
        if (item.tile < 0) continue;
        const Tile& t = item.t;
        for (int32_t x = 0; x < kShortRows; ++x) start->rows[x] = plan.rows[t.row_begin + std::min(x, t.nrows - 1)];
        if (t.nseg == 0) continue;
        ShortRecord* const records = reinterpret_cast<ShortRecord*>(start + 1);
        auto log2_mult = [&](int32_t x, int block) {
            const int32_t m = plan.block_mult[(size_t)(t.seg_begin + x) * kTileBlocks + block];
            return m > 0 ? std::log2((float)m) : -INFINITY;
        };
        for (int32_t wave = 0; wave < kWalkWaves; ++wave)
            for (int32_t r = 0; r < per_wave; ++r) {
                const int32_t at = wave + kWalkWaves * r, last = t.nseg - 1;
                const int32_t x = at <= last ? at : last >= wave ? last - (last - wave) % kWalkWaves : 0;
                const KeySeg& seg = plan.segs[t.seg_begin + x];
                const int32_t count = at <= last ? seg.count : 0;
                ShortRecord& rec = records[wave * per_wave + r];
                rec.key0 = seg.key0;
                bool turn = r == 0 || count < kWalkBlock;
                for (int blk = 0; blk < 2; ++blk) {
                    rec.log2_mult[blk] = log2_mult(x, blk);
                    turn = turn || rec.log2_mult[blk] != log2_mult(at - kWalkWaves, blk);
                }
                rec.stride_count = seg.stride | (count << 24) | (turn ? kTurn : 0);
            }
    }
    return out;
}

bool short_backward_plan(int32_t B, int32_t H, int32_t N, const dfa_branch_t* br, int32_t nb, const int32_t* offsets,
                         int order_mode, const ChipShape& chip, const HostPlan& full, HostPlan* plan) {
    if (N >= kMaxCutStride) return false;
    // us for the call on 256 CUs, see dfa_plan.h
    const int64_t slots = chip.fwd_slots(), one = slots / kFwdWorkgroupsPerCu;
    const double per_slot = 512.0 / slots;
    const LaunchSize whole = launch_size(full);
    const double items = per_slot * full.items.size(), steps = per_slot * whole.steps;
    const double full_us = whole.live <= one     ? 11.6 + 0.0027 * items + 0.0035 * steps + 2.88 * whole.longest
                           : whole.live <= slots ? 14.3 - 0.0071 * items + 0.0153 * steps + 0.43 * whole.longest
                                                 : 9.2 + 0.01 * items + 0.0122 * steps + 0.7 * whole.longest;
    const double long_us = 15.0 + std::max(3.2 * whole.longest, 0.0164 * steps);        // past kFewTiles
    if (0.02 * items > std::max(full_us, long_us)) return false;          // there are at least as many 64-row tiles
    build_plan(B, H, N, br, nb, offsets, order_mode, chip, false, plan, kShortRows / kBlockRows);
    const CutSize size = cut_size(*plan);
    if (size.longest > kShortBackwardBlocks || size.records > kMaxCutRecords) return false;
    cut_blocks(plan);
    int64_t tiles = 0, live = 0, blocks = 0;
    for (const Item& i : plan->items)
        if (i.tile >= 0) {
            ++tiles;
            live += i.t.nseg > 0;
            blocks += (int64_t)i.t.nseg * ((i.t.nrows + kBlockRows - 1) / kBlockRows);
        }
    if (per_slot * tiles > kFewTiles) return 10.0 + per_slot * (0.024 * tiles + 0.00105 * blocks) < long_us;
    const double short_us = live * (1 + kShortDkdvParts) <= 2 * slots ? 14.8 + 0.00075 * per_slot * blocks
                                                                      : 4.7 + per_slot * (0.0077 * tiles + 0.0135 * live + 0.00097 * blocks) + 0.098 * size.longest;
    return short_us * kShortBackwardMargin < full_us;
}

}  // namespace dfa
