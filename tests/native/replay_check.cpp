// The contracted walk's two replays on a path of pieces: a tree that is one
// long path (or a random tree), some of its edges toggled in random order
// among inserts between random vertices, against the one-by-one walk on a
// copy.  On a path nearly all removed edges come back at once: walks to the root of
// a path of many pieces are long, so that its runs exceed their budget; those
// of a random tree do not.  Arguments: V, number
// of toggled edges, updates, seed, path (1) or random tree (0); prints
// whether the labelled replay ran.  Built and run by tests/test_replay_host.py
// (host code only, with sanitizers).
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>

#include "contract.hpp"
#include "forest.hpp"

using cupk::Contraction;
using cupk::Forest;

int main(int argc, char **argv)
{
    if (argc != 6) return 3;
    const uint32_t V = atoi(argv[1]), m = atoi(argv[2]), n = atoi(argv[3]);
    std::mt19937 rng(atoi(argv[4]));
    const bool path = atoi(argv[5]) != 0;
    std::vector<uint32_t> la(V), pa(V), lb(V), pb(V);
    Forest A, B;
    A.init(V, la.data(), pa.data());
    B.init(V, lb.data(), pb.data());
    std::vector<std::pair<uint32_t, uint32_t>> tree;
    for (uint32_t i = 1; i < V; i++) {
        const uint32_t p = path ? i - 1 : rng() % i;
        A.link(p, i);
        B.link(p, i);
        tree.push_back({p, i});
    }
    std::set<std::pair<uint32_t, uint32_t>> live(tree.begin(), tree.end());
    for (uint32_t l : A.dirty_labels()) A.clear_dirty(l);
    for (uint32_t l : B.dirty_labels()) B.clear_dirty(l);
    std::vector<std::pair<uint32_t, uint32_t>> pick;
    for (uint32_t i = 0; i < m; i++) pick.push_back(tree[rng() % tree.size()]);
    std::vector<uint64_t> run;
    for (uint32_t i = 0; i < n; i++) {
        std::pair<uint32_t, uint32_t> e = pick[rng() % m];
        if (rng() % (path ? 64 : 4) == 0) {
            e = {rng() % V, rng() % V};
            if (e.first == e.second) continue;
            if (e.first > e.second) std::swap(e.first, e.second);
        }
        const bool del = live.count(e) != 0;
        if (del)
            live.erase(e);
        else
            live.insert(e);
        run.push_back((uint64_t)e.first | (uint64_t)e.second << 32 | (uint64_t)del << 63);
        if (path && del && rng() % 2048) {
            // nearly all back at once, so that the pieces stay one long path
            run.push_back((uint64_t)e.first | (uint64_t)e.second << 32);
            live.insert(e);
        }
    }
    uint64_t l0 = 0, c0 = 0, l1 = 0, c1 = 0;
    for (uint64_t p : run) {
        const uint32_t a = (uint32_t)p, b = (uint32_t)(p >> 32) & 0x7fffffffu;
        if ((p >> 63) == 0) {
            if (A.has_pending()) A.split_pending();
            if (!A.same_tree(a, b)) {
                A.link(a, b);
                l0++;
            }
        } else if (A.is_edge(a, b)) {
            A.remove_edge(a, b);
            c0++;
        }
    }
    A.split_pending();
    Contraction C;
    C.set_budget(64, V);
    bool changed = false;
    if (!C.run(B, run.data(), 0, (uint32_t)run.size(), &l1, &c1, &changed)) return 4;
    if (l0 != l1 || c0 != c1) return fprintf(stderr, "links or cuts\n"), 1;
    std::vector<uint32_t> ua, va, ub, vb;
    A.edges(ua, va);
    B.edges(ub, vb);
    std::set<std::pair<uint32_t, uint32_t>> ea, eb;
    for (size_t i = 0; i < ua.size(); i++) ea.insert({ua[i], va[i]});
    for (size_t i = 0; i < ub.size(); i++) eb.insert({ub[i], vb[i]});
    if (ea != eb || A.n_trees() != B.n_trees()) return fprintf(stderr, "forest edges\n"), 1;
    // trees, their sizes, roots and dirty marks
    std::vector<uint32_t> map(V, cupk::kNone);
    for (uint32_t w = 0; w < V; w++) {
        const uint32_t x = A.label(w), y = B.label(w);
        if (map[x] == cupk::kNone) map[x] = y;
        if (map[x] != y || A.tree_size(x) != B.tree_size(y) || A.is_dirty(x) != B.is_dirty(y) ||
            B.label(B.tree_root(y)) != y || B.parent(B.tree_root(y)) != cupk::kNone)
            return fprintf(stderr, "tree of vertex %u\n", w), 1;
    }
    printf("labelled=%d\n", C.last_labelled ? 1 : 0);
    return 0;
}
