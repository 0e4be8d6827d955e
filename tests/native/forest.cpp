// Host test of the merge of a batch: forest DEPTH... builds one game per argument, a chain in which the
// two players move in turn DEPTH times (each move ends the game or goes on), merges them, and checks the
// forest's ids against the games'.
#include <cstdio>
#include <cstdlib>

#include "compiler.hpp"

using namespace cfrx;

#define CHECK(x)                                                    \
    do {                                                            \
        if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } \
    } while (0)

struct Chain {
    std::vector<int8_t> type;
    std::vector<int64_t> begin, kids, key;
    std::vector<int32_t> n;
    std::vector<double> prob, payoff;
    explicit Chain(int depth) {
        std::vector<std::vector<int64_t>> below;
        auto add = [&](int t, int64_t k) {
            type.push_back((int8_t)t); key.push_back(k); payoff.push_back(0.25 * (double)type.size()); below.emplace_back();
            return (int64_t)type.size() - 1;
        };
        int64_t at = add(CFR_NODE_P1, 0);
        for (int d = 1; d < depth; d++) {
            const int64_t stop = add(CFR_NODE_TERMINAL, -1), next = add(d % 2 ? CFR_NODE_P2 : CFR_NODE_P1, d);
            below[(size_t)at] = {stop, next};
            at = next;
        }
        const int64_t a = add(CFR_NODE_TERMINAL, -1), b = add(CFR_NODE_TERMINAL, -1);
        below[(size_t)at] = {a, b};
        for (auto &c : below) {
            begin.push_back((int64_t)kids.size()); n.push_back((int32_t)c.size());
            for (int64_t x : c) { kids.push_back(x); prob.push_back(0.0); }
        }
    }
    cfr_game_desc desc() const {
        cfr_game_desc d{};
        d.num_nodes = (int64_t)type.size(); d.node_type = type.data(); d.child_begin = begin.data();
        d.num_children = n.data(); d.children = kids.data(); d.chance_prob = prob.data(); d.infoset_key = key.data();
        d.payoff = payoff.data(); d.pot = 1.0;
        return d;
    }
};

int main(int argc, char **argv) {
    const int n = argc - 1;
    std::vector<int> depth;
    std::vector<Layout> Ls((size_t)n);
    std::vector<DeviceLayout> Ds((size_t)n);
    std::string err;
    for (int s = 0; s < n; s++) {
        depth.push_back(std::atoi(argv[s + 1]));
        const Chain c(depth.back());
        const cfr_game_desc d = c.desc();
        CHECK(build_layout(&d, Ls[(size_t)s], err) == CFR_OK);
        CHECK(Ls[(size_t)s].max_depth == depth.back());
        CHECK(build_device_layout(Ls[(size_t)s], CFR_LAYOUT_PUBLIC, 2, false, 128, Ds[(size_t)s], err) == CFR_OK);
    }
    const std::vector<DeviceLayout> games = Ds;
    DeviceLayout F;
    CHECK(build_forest(Ls, Ds, F, err) == CFR_OK);
    int md = 0;
    for (int x : depth) md = std::max(md, x);
    CHECK((int)F.depth_off.size() == md + 2);
    // depth by depth the games' nodes in turn, each with its own children and template
    int32_t at = 0;
    for (int d = 0; d <= md; d++) {
        CHECK(F.depth_off[(size_t)d] == at);
        for (int s = 0; s < n; s++) {
            const DeviceLayout &G = games[(size_t)s];
            if (d > depth[(size_t)s]) continue;
            for (int32_t x = G.depth_off[(size_t)d]; x < G.depth_off[(size_t)d + 1]; x++, at++) {
                CHECK(F.tmpl64[(size_t)at] == G.tmpl64[(size_t)x]);
                const int32_t k = G.kid_off[(size_t)x + 1] - G.kid_off[(size_t)x];
                CHECK(F.kid_off[(size_t)at + 1] - F.kid_off[(size_t)at] == k);
                for (int32_t a = 0; a < k; a++) {
                    const int32_t c = F.kid[(size_t)(F.kid_off[(size_t)at] + a)];
                    CHECK(c >= F.depth_off[(size_t)d + 1] && c < F.depth_off[(size_t)d + 2]);
                }
            }
        }
    }
    // a set's own last sequence and its members' opponent sequences lie above it
    for (int d = 0; d <= md; d++)
        for (int32_t i = F.iset_depth_off[(size_t)d]; i < F.iset_depth_off[(size_t)d + 1]; i++) {
            CHECK(F.iset_seq[(size_t)i] < F.slot_off[(size_t)F.iset_depth_off[(size_t)d]]);
            CHECK((F.iset_seq[(size_t)i] >= 0) == (d >= 2));
            for (int32_t m = F.mem_off[(size_t)i]; m < F.mem_off[(size_t)i + 1]; m++) {
                const int32_t x = F.mem_node[(size_t)m] & 0x7fffffff;
                CHECK(x >= F.depth_off[(size_t)d] && x < F.depth_off[(size_t)d + 1]);
                CHECK((F.mem_seq[(size_t)m] >= 0) == (d >= 1));
            }
        }
    // the one-launch schedules' ranges: a game's slots and sets per depth, but for those whose moves all end the
    // game, and parts in which no slot walks more than REACH_WALK slots up, none of them longer than it could be
    const std::vector<int32_t> R = one_launch_ranges(F);
    CHECK(R.size() / DR_FIELDS == F.game_range.size() / GR_FIELDS);
    for (int s = 0; s < n; s++) {
        std::vector<int32_t> starts(1, 0);
        for (int d = 0; d <= depth[(size_t)s]; d++) {
            const int32_t *r = &R[((size_t)s * (md + 1) + d) * DR_FIELDS], *old = &F.game_range[((size_t)s * (md + 1) + d) * GR_FIELDS];
            for (int k = 2; k < GR_FIELDS; k++) CHECK(r[k] == old[k]);
            const int32_t first = F.grp_iset_off[(size_t)r[2]], end = F.grp_iset_off[(size_t)r[3]];
            CHECK(end - first == (d < depth[(size_t)s] ? 1 : 0));
            CHECK(r[8] == first && r[9] == (d < depth[(size_t)s] - 1 ? end : first));
            CHECK(r[0] == F.slot_off[(size_t)r[8]] && (r[1] & ~REACH_CUT) == F.slot_off[(size_t)r[9]]);
            auto longest = [&](int32_t S0) {
                int w = 0;
                for (int32_t i = first; i < end; i++) {
                    int k = 0;
                    for (int32_t p = F.iset_seq[(size_t)i]; p >= S0; k++) {
                        int32_t j = 0;
                        while (F.slot_off[(size_t)j + 1] <= p) j++;
                        p = F.iset_seq[(size_t)j];
                    }
                    w = std::max(w, k);
                }
                return w;
            };
            if (r[1] & REACH_CUT) {
                CHECK(longest(starts.back()) == REACH_WALK + 1);
                starts.push_back(r[0]);
            }
            CHECK(longest(starts.back()) <= REACH_WALK);
        }
        const int moves = (depth[(size_t)s] + 1) / 2;   // of the first player
        CHECK((int)starts.size() == moves / (REACH_WALK + 1) + (moves % (REACH_WALK + 1) > 0));
    }
    std::printf("ok\n");
    return 0;
}
