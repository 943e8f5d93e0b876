// Memory-safety fuzz of the decode plan builder (host code only; built with the address and undefined-behaviour
// sanitizers by tests/test_library_host.py).  Random forests with the sharing structure forks produce - a
// thread's table is its root path's blocks, refcounts count the live holders, internal nodes end on block
// boundaries - are planned under random geometry and policy parameters; the plan is checked for coverage:
// every row group of every listed thread must be shown exactly the blocks of its thread's table, once, and
// every index in the plan must lie inside its array (the sanitizers watch the builder's own accesses), every list says
// how many of its tiles are full, and a call that is not one of few units has the plan of a pool without such units.
#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>
#include <set>
#include <vector>

#include "plan.hpp"

using namespace apar;

#define CHECK(c)                                                                   \
    do {                                                                           \
        if (!(c)) {                                                                \
            std::fprintf(stderr, "seed %d: check failed: %s (line %d)\n", seed, #c, __LINE__); \
            return 1;                                                              \
        }                                                                          \
    } while (0)

template <class T>
static bool same_table(const std::vector<T>& a, const std::vector<T>& b) {
    return a.size() == b.size() && (a.empty() || std::memcmp(a.data(), b.data(), a.size() * sizeof(T)) == 0);
}

static int n_few = 0, n_packed = 0;  // plans of calls of few units, those that were packed

static int one(int seed) {
    std::mt19937 rng(seed);
    auto rnd = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    // forest: node = (parent, own blocks); leaves are the threads
    struct Node { int parent; std::vector<int32_t> blocks; int last_valid; std::vector<int> kids; };
    std::vector<Node> nodes;
    int32_t next_block = 0;
    const bool small = seed % 2;  // (the size of calls of few units)
    const int n_roots = rnd(1, 3), max_nodes = rnd(4, small ? 60 : 400);
    for (int r = 0; r < n_roots; ++r) nodes.push_back(Node{-1, {}, 16, {}});
    while ((int)nodes.size() < max_nodes) {
        const int p = rnd(0, (int)nodes.size() - 1);
        const int fan = rnd(1, rng() % 8 == 0 ? (small ? 20 : 200) : 6);
        for (int k = 0; k < fan; ++k) {
            nodes[p].kids.push_back((int)nodes.size());
            nodes.push_back(Node{p, {}, 16, {}});
        }
    }
    for (Node& nd : nodes) {
        const bool leaf = nd.kids.empty();
        const int nb = leaf ? rnd(0, 6) : rnd(1, rng() % 6 == 0 ? 300 : 5);  // a leaf may have no block of its own
        for (int b = 0; b < nb; ++b) nd.blocks.push_back(next_block++);
        nd.last_valid = (leaf && nb > 0) ? rnd(1, 16) : 16;
    }
    // a leaf without blocks of its own under a parent: it ends at the parent's segment.  Roots that are leaves need a block.
    for (Node& nd : nodes)
        if (nd.parent < 0 && nd.kids.empty() && nd.blocks.empty()) nd.blocks.push_back(next_block++);
    // a node all of whose children end at it (threads listed right after their fork) may end on an open block
    for (Node& nd : nodes) {
        if (nd.kids.empty()) continue;
        bool all_end_here = true;
        for (int k : nd.kids) all_end_here = all_end_here && nodes[k].kids.empty() && nodes[k].blocks.empty();
        if (all_end_here) nd.last_valid = rnd(1, 16);
    }
    std::vector<int32_t> refcount(next_block + 8, 0);
    std::vector<std::vector<int32_t>> tables;
    std::vector<int64_t> lens;
    for (size_t i = 0; i < nodes.size(); ++i) {
        if (!nodes[i].kids.empty()) continue;
        std::vector<int> path;
        for (int a = (int)i; a >= 0; a = nodes[a].parent) path.push_back(a);
        std::vector<int32_t> t;
        for (auto it = path.rbegin(); it != path.rend(); ++it) t.insert(t.end(), nodes[*it].blocks.begin(), nodes[*it].blocks.end());
        for (int32_t b : t) refcount[b] += 1;
        const int lv = nodes[i].blocks.empty() ? nodes[nodes[i].parent].last_valid : nodes[i].last_valid;
        tables.push_back(t);
        lens.push_back((int64_t)(t.size() - 1) * 16 + lv);
    }
    const int n = (int)tables.size();
    std::vector<int> order(n);
    for (int i = 0; i < n; ++i) order[i] = i;
    std::shuffle(order.begin(), order.end(), rng);
    std::vector<PlanThreadView> views(n);
    for (int i = 0; i < n; ++i) views[i] = PlanThreadView{tables[order[i]].data(), (int32_t)tables[order[i]].size(), lens[order[i]]};
    std::vector<int32_t> seg_of(refcount.size(), -1);
    PlanHost ph;
    for (int round = 0; round < 3; ++round) {
        PlanParams prm{};
        const int rpts[] = {1, 2, 4, 5, 8, 16, 20, 40, 64};
        prm.rows_per_thread = rpts[rng() % 9];
        const int caps[] = {1, 2, 5, 16, 64, 512};
        prm.max_unit_tiles = caps[rng() % 6];
        prm.allow_direct = rng() % 8 != 0;
        prm.fuse = rng() % 8 != 0;
        prm.inline_shared = rng() % 2;
        const int mrows[] = {0, 1, 64, 256};
        prm.matrix_min_rows = mrows[rng() % 4];
        const int mblk[] = {1, 3, 128};
        prm.matrix_min_blocks = mblk[rng() % 3];
        prm.open_cost = rnd(1, 3);
        const int units[] = {0, 1, 40, 1024};
        prm.few_units = units[rng() % 4];
        prm.few_row_tiles = rnd(1, 2);
        const int again[] = {0, 100, 3000, INT_MAX};
        prm.few_again = again[rng() % 4];
        prm.few_again_wide = again[rng() % 4];
        prm.few_again_narrow = again[rng() % 4];
        prm.few_small = again[rng() % 4];
        prm.few_open_cost = rnd(1, 2);
        if (round == 2) {  // as a pool asks for them, but for the blocks of a unit
            prm.allow_direct = prm.fuse = prm.inline_shared = true;
            prm.matrix_min_rows = 256, prm.matrix_min_blocks = 128;
            prm.few_units = 1024;
        }
        CHECK(build_plan(views.data(), n, refcount.data(), seg_of.data(), prm, ph) == 0);
        for (int32_t x : seg_of) CHECK(x == -1);
        if (!ph.few_row_tiles && prm.few_units > 0) {  // another call's plan is the one without such units
            PlanParams none = prm;
            none.few_units = 0;
            PlanHost general;
            CHECK(build_plan(views.data(), n, refcount.data(), seg_of.data(), none, general) == 0);
            CHECK(same_table(ph.wgs, general.wgs) && same_table(ph.tiles, general.tiles) && ph.path_ids == general.path_ids &&
                  ph.path_ofs == general.path_ofs && ph.dfs_threads == general.dfs_threads && ph.n_partial_rows == general.n_partial_rows);
        }
        const int n_sl = (prm.rows_per_thread + 15) / 16;
        // coverage: row group -> multiset of (block, valid)
        std::vector<std::map<int32_t, int>> seen((size_t)n * n_sl);
        const size_t n_tiles = ph.tiles.size();
        auto show = [&](const TileRef& t, int base, int g, int& err) {
            const int lo = t.meta & 1023, hi = (t.meta >> 10) & 1023, valid = (t.meta >> 20) & 31;
            if (valid < 1 || valid > 16 || lo >= hi) err = 1;
            if (g - base >= lo && g - base < hi) seen[g][t.blk] += valid;
        };
        CHECK(ph.few_row_tiles >= 0 && ph.few_row_tiles <= (prm.few_units > 0 ? prm.few_row_tiles : 0));
        n_few += ph.few_row_tiles > 0;
        if (ph.few_row_tiles) {  // no more tiles listed again than allowed
            int64_t listed = 0;
            for (const WgDesc& wg : ph.wgs)
                for (const WaveItem& wi : wg.w) listed += wi.n_tiles;
            CHECK(listed - ph.unique_blocks <= (ph.few_row_tiles == 1 ? prm.few_again : prm.few_again_wide));
            int64_t again_narrow = 0;  // in trees of at most 64 rows: `listed` over the units of threads that share such a root, less the trees' blocks
            std::map<int32_t, std::pair<int, std::set<int32_t>>> trees;  // by a tree's first block: its threads, its blocks
            for (int i = 0; i < n; ++i) {
                auto& tree = trees[tables[i][0]];
                tree.first += 1;
                tree.second.insert(tables[i].begin(), tables[i].end());
            }
            const int slices = (prm.rows_per_thread + 15) / 16, per_tile = 16 / ((prm.rows_per_thread + slices - 1) / slices);
            for (const WgDesc& wg : ph.wgs)
                if (const int32_t root = tables[order[ph.dfs_threads[wg.grp_base / slices]]][0]; trees[root].first * slices <= 4 * per_tile)
                    for (const WaveItem& wi : wg.w) again_narrow += wi.n_tiles;
            for (const auto& [root, tree] : trees)
                if (tree.first * slices <= 4 * per_tile) again_narrow -= (int64_t)tree.second.size();
            CHECK(ph.few_row_tiles == 1 || again_narrow <= prm.few_again_narrow || ph.unique_blocks <= prm.few_small);
        }
        if (ph.few_row_tiles && !ph.any_partial && ph.tiles.size() < 832 && n < 832) {  // (such may go along packed)
            for (const TileRef& t : ph.tiles) {
                const TileRef u = unpack_few_tile(pack_few_tile(t));
                CHECK((t.meta >> 20) == 0 || (u.blk == t.blk && u.meta == t.meta));  // (0: room behind a list)
            }
            for (const WgDesc& wg : ph.wgs)
                for (int k = 0; k < 4; ++k) {
                    const WaveItem& wi = wg.w[k];
                    uint32_t w[kFewWaveWords];
                    pack_few_wave(wi, wg.n_full[k], w);
                    int n_full;
                    const WaveItem u = unpack_few_wave(w[0], w[1], n_full);
                    CHECK(u.n_grp == wi.n_grp && (wi.n_grp == 0 || (u.tile_ofs == wi.tile_ofs && u.n_tiles == wi.n_tiles && u.grp_lo == wi.grp_lo &&
                                                                    u.flags == wi.flags && n_full == std::min(wg.n_full[k], wi.n_tiles))));
                }
            n_packed += 1;
        }
        for (const WgDesc& wg : ph.wgs) {
            // which kernel takes the unit: all of a call's are for the one without shared lists or none is
            if (ph.few_row_tiles) CHECK(wg.n_coop == 0 && (wg.row_tiles & 255) <= ph.few_row_tiles);
            else CHECK((wg.row_tiles & 255) != 2 || !(wg.w[0].flags & kWaveSplit));
            CHECK(wg.coop_ofs >= 0 && wg.n_coop >= 0 && (size_t)wg.coop_ofs + wg.n_coop <= n_tiles);
            for (int k = 0; k < 4; ++k) {
                const WaveItem& wi = wg.w[k];
                CHECK(wi.n_grp >= 0 && wi.n_tiles >= 0);
                if (wi.n_grp == 0) continue;
                CHECK(wi.tile_ofs >= 0 && (size_t)wi.tile_ofs + wi.n_tiles <= n_tiles);
                CHECK(wi.grp_lo >= 0 && wi.grp_lo + wi.n_grp <= n * n_sl);
                int err = 0;
                for (int g = wi.grp_lo; g < wi.grp_lo + wi.n_grp; ++g) {
                    for (int t = 0; t < wg.n_coop; ++t) show(ph.tiles[wg.coop_ofs + t], wg.grp_base, g, err);
                    for (int t = 0; t < wi.n_tiles; ++t) show(ph.tiles[wi.tile_ofs + t], wi.grp_lo, g, err);
                }
                CHECK(!err);
                // a list's full tiles come first, and as many as the descriptor says
                const int n_full = std::min(wg.n_full[k], wi.n_tiles);
                for (int t = 0; t < wi.n_tiles; ++t) CHECK((((ph.tiles[wi.tile_ofs + t].meta >> 20) & 31) == 16) == (t < n_full));
            }
        }
        CHECK((int)ph.dfs_threads.size() == n);
        for (int rank = 0; rank < n; ++rank) {
            const int i = ph.dfs_threads[rank];
            CHECK(i >= 0 && i < n);
            const std::vector<int32_t>& tb = tables[order[i]];
            const int64_t len = lens[order[i]];
            for (int sl = 0; sl < n_sl; ++sl) {
                const std::map<int32_t, int>& got = seen[(size_t)rank * n_sl + sl];
                CHECK(got.size() == tb.size());
                int64_t total = 0;
                for (int32_t b : tb) {
                    auto it = got.find(b);
                    CHECK(it != got.end() && it->second <= 16);
                    total += it->second;
                }
                CHECK(total == len);
            }
            CHECK(ph.path_ofs[i] <= ph.path_ofs[i + 1] && (size_t)ph.path_ofs[i + 1] <= ph.path_ids.size());
            for (int p = ph.path_ofs[i]; p < ph.path_ofs[i + 1]; ++p) CHECK(ph.path_ids[p] >= 0 && ph.path_ids[p] < ph.n_partial_rows);
        }
    }
    return 0;
}

// A plan built under other parameters is not carried over: every one of them counts.
static int parameters(int seed) {
    PlanParams a{};
    a.rows_per_thread = 4, a.max_unit_tiles = 512, a.allow_direct = true, a.fuse = true;
    CHECK(a == a);
    int32_t PlanParams::*const numbers[] = {&PlanParams::rows_per_thread, &PlanParams::max_unit_tiles, &PlanParams::matrix_min_rows,
                                            &PlanParams::matrix_min_blocks, &PlanParams::few_units, &PlanParams::few_row_tiles,
                                            &PlanParams::few_again, &PlanParams::few_again_wide, &PlanParams::few_again_narrow, &PlanParams::few_small,
                                            &PlanParams::few_open_cost, &PlanParams::open_cost};
    bool PlanParams::*const flags[] = {&PlanParams::allow_direct, &PlanParams::fuse, &PlanParams::inline_shared};
    static_assert(sizeof(PlanParams) == sizeof numbers / sizeof numbers[0] * 4 + 4, "every parameter is named here (the flags share a word)");
    for (auto m : numbers) {
        PlanParams b = a;
        b.*m += 1;
        CHECK(!(a == b));
    }
    for (auto m : flags) {
        PlanParams b = a;
        b.*m = !(b.*m);
        CHECK(!(a == b));
    }
    return 0;
}

int main(int argc, char** argv) {
    const int first = argc > 1 ? std::atoi(argv[1]) : 0, count = argc > 2 ? std::atoi(argv[2]) : 200;
    if (parameters(-1)) return 1;
    for (int seed = first; seed < first + count; ++seed)
        if (one(seed)) return 1;
    if (count >= 50 && n_few < count / 10) return std::fprintf(stderr, "only %d plans of calls of few units\n", n_few), 1;
    if (count >= 50 && n_packed < count / 20) return std::fprintf(stderr, "only %d of them packed\n", n_packed), 1;
    std::printf("ok: %d forests, %d plans of calls of few units, %d packed\n", count, n_few, n_packed);
    return 0;
}
