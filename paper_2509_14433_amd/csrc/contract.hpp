// Contracted walk of a run of flagged updates.
//
// Walking a batch's flagged updates one by one on the forest (an insert
// links two different trees, a delete of a forest edge removes it, pieces
// split before the next insert) costs a relabelling of the smaller tree per
// link and a piece search per split.  When the same few edges are linked
// and cut again and again inside one run (bridges between large trees
// toggled many times), most of that work is undone within the run.
//
// The contracted walk gives exactly the same result with work proportional
// to the net change:
//   1. T0 = the forest at the start of the run.  The T0 edges the run
//      deletes are D0; the pieces are the components of T0 - D0.  Every
//      edge of T0 - D0 stays in the forest throughout the run, so each
//      piece stays connected, and two vertices are connected at any moment
//      exactly when their pieces are connected by the forest edges that
//      join different pieces (D0 edges not yet deleted, and edges the run
//      linked).  The piece of a vertex is named by its top vertex: the
//      first vertex at or above it whose parent edge is in D0, or the root.
//      Only the run's endpoints need a piece, found by walking parent
//      pointers up, each vertex once (a walk that would exceed a budget
//      proportional to the run gives up and the caller walks the run one
//      update at a time instead; no edge has been changed then).
//   2. The run is replayed on a small forest over the pieces, starting
//      with the D0 edges: links and removals happen there exactly when they
//      would happen on the whole forest, so the counts of links and cuts
//      are the same.  That forest is parent pointers only: D0 edges hang a
//      piece below the one above its top, a removal clears a pointer, an
//      insert compares the two roots, a link re-roots the endpoint nearer
//      its root.  The run's distinct edges are looked up once and numbered;
//      the replay reads their pieces and whether they are live.  When the
//      walks to the roots exceed a budget (long paths of pieces), the run is
//      replayed from the start on a labelled Forest, whose inserts cost two
//      loads but whose links and splits relabel the smaller side.  40,673
//      updates on 64 pieces: 0.44 ms, 1.75 on a labelled forest with a hash
//      set of the live edges; 6,111 on 6,075 pieces: 0.04 ms, 1.01.
//   3. The net change is applied to the whole forest: D0 edges that ended
//      removed are removed, the pieces split once, and the edges the replay
//      added that were not in T0 are linked (Forest::link_many: each merged
//      tree relabelled once).
//   4. Dirty marks: one by one, a tree ends dirty exactly when it holds an
//      endpoint of an edge removed during the run (each removal makes both
//      sides dirty, marks follow links, and every piece of a split holds
//      such an endpoint) or a vertex of a tree already dirty.  Step 3 sets
//      a subset of those marks; the endpoints of every edge the replay
//      removed mark the rest.
#pragma once

#include <stdint.h>

#include <chrono>
#include <vector>

#include "forest.hpp"

namespace cupk {

class Contraction {
  public:
    // Walk the flagged updates upd[k0, k1) (packed: u in bits 0..31, v in
    // 32..62, delete flag in bit 63) into F.  Pending splits are done first.
    // Returns false, with F's edges untouched, when the piece search
    // exceeds its budget.  *links and *cuts get the links and forest-edge
    // removals of the one-by-one walk; *changed tells whether the forest's
    // edges changed.
    bool run(Forest &F, const uint64_t *upd, uint32_t k0, uint32_t k1, uint64_t *links,
             uint64_t *cuts, bool *changed)
    {
        const uint32_t V = F.V();
        if (cut_.size() != V) {
            cut_.assign(V, 0);
            seen_.assign(V, 0);
            top_.assign(V, 0);
            pid_.assign(V, 0);
            epoch_ = 0;
        }
        if (++epoch_ == 0) {
            std::fill(cut_.begin(), cut_.end(), 0);
            std::fill(seen_.begin(), seen_.end(), 0);
            std::fill(pstamp_.begin(), pstamp_.end(), 0);
            epoch_ = 1;
        }
        const auto t0 = std::chrono::steady_clock::now();
        // labels exact, so that T0 is the current forest
        F.split_pending();
        // the run's distinct edges; D0: the T0 edges it deletes (child
        // endpoint marked)
        const uint32_t K = k1 - k0;
        edges_.clear();
        eid_.resize(K);
        table_.start(K);
        for (uint32_t k = 0; k < K; k++) {
            const uint64_t p = upd[k0 + k];
            Edge e = {};
            ends(p, e.a, e.b);
            const uint32_t i = table_.find(key(e.a, e.b), (uint32_t)edges_.size());
            eid_[k] = i;
            if (i == edges_.size()) {
                e.tree = F.is_edge(e.a, e.b);
                edges_.push_back(e);
            }
            Edge &s = edges_[i];
            if ((p >> 63) && s.tree && !s.d0) {
                s.d0 = s.live = 1;
                cut_[child(F, s)] = epoch_;
            }
        }
        // pieces of the run's endpoints
        size_t budget = budget_per_update_ * K + budget_base_;
        uint32_t P = 0;
        for (Edge &e : edges_) {
            uint32_t q[2];
            for (int s = 0; s < 2; s++) {
                const uint32_t t = find_top(F, s ? e.b : e.a, budget);
                if (t == kNone) return false;
                if (pid_[t] >= P || piece_top_[pid_[t]] != t) {
                    pid_[t] = P++;
                    if (piece_top_.size() < P) piece_top_.resize(P);
                    piece_top_[P - 1] = t;
                }
                q[s] = pid_[t];
            }
            e.pa = q[0];
            e.pb = q[1];
        }
        const auto t1 = std::chrono::steady_clock::now();
        // replay on the piece forest
        ppar_.assign(P, kNone);
        for (const Edge &e : edges_)
            if (e.d0) {
                const bool a_below = child(F, e) == e.a;
                ppar_[a_below ? e.pa : e.pb] = a_below ? e.pb : e.pa;
            }
        uint64_t nl = 0, nc = 0;
        Walked walked{ppar_, budget_per_update_ * K + budget_base_};
        const bool labelled = last_labelled = !replay(walked, upd + k0, K, nl, nc);
        if (labelled) {
            plbl_.resize(P);
            PF_.init(P, plbl_.data(), ppar_.data());
            for (Edge &e : edges_) {
                e.live = e.d0;
                e.cut = 0;
                if (e.d0) PF_.link(e.pa, e.pb);
            }
            nl = nc = 0;
            Labelled lab{PF_};
            replay(lab, upd + k0, K, nl, nc);
        }
        const auto t2 = std::chrono::steady_clock::now();
        // net change on the whole forest: the removals, then every piece of
        // the broken trees (and every tree a net edge joins) settled into its
        // final tree at once, the final trees being the piece forest's
        bool ch = false;
        net_.clear();
        for (const Edge &e : edges_) {
            if (e.d0 && !e.live) {
                F.remove_edge(e.a, e.b);
                ch = true;
            }
            if (e.live && !e.d0) net_.push_back({e.a, e.b});
        }
        const auto t3 = std::chrono::steady_clock::now();
        if (F.has_pending() || !net_.empty()) {
            // final tree of each piece: its root's number, or its label
            if (labelled && PF_.has_pending()) PF_.split_pending();
            auto group = [&](uint32_t q) {
                if (labelled) return PF_.label(q);
                uint32_t r = q;
                while (ppar_[r] != kNone) r = ppar_[r];
                for (uint32_t up; q != r; q = up) {  // shorten the path for the next ones
                    up = ppar_[q];
                    ppar_[q] = r;
                }
                return r;
            };
            if (pstamp_.size() != V) pstamp_.assign(V, 0);
            pieces_.clear();
            uint32_t extra = P;  // group ids past the piece forest's labels
            auto add = [&](uint32_t t) {
                if (pstamp_[t] == epoch_) return;
                pstamp_[t] = epoch_;
                uint32_t g;
                size_t big = (size_t)-1;
                if (seen_[t] == epoch_ || find_top(F, t, big) != kNone) {
                    const uint32_t q = pid_[top_[t]];
                    g = (q < P && piece_top_[q] == top_[t]) ? group(q) : extra++;
                } else {
                    g = extra++;
                }
                pieces_.push_back({t, g});
            };
            for (const auto &pr : F.pending()) {
                add(pr.second);
                add(F.tree_root(pr.first));
            }
            for (const auto &e : net_) {
                add(F.tree_root(F.label(e.first)));
                add(F.tree_root(F.label(e.second)));
            }
            F.settle_regroup(pieces_, net_);
            ch = true;
        }
        for (const Edge &e : edges_)
            if (e.cut) {
                F.set_dirty(F.label(e.a));
                F.set_dirty(F.label(e.b));
            }
        const auto t4 = std::chrono::steady_clock::now();
        auto ms = [](std::chrono::steady_clock::time_point a, std::chrono::steady_clock::time_point b) {
            return std::chrono::duration<double, std::milli>(b - a).count();
        };
        last_ms[0] = ms(t0, t1);  // pending splits, D0, pieces
        last_ms[1] = ms(t1, t2);  // replay on the piece forest
        last_ms[2] = ms(t2, t3);  // removals
        last_ms[3] = ms(t3, t4);  // settling the pieces into their final trees
        last_pieces = P;
        *links += nl;
        *cuts += nc;
        *changed = ch;
        return true;
    }

    // Host time of the last run's phases (ms) and its number of pieces.
    double last_ms[4] = {0, 0, 0, 0};
    uint32_t last_pieces = 0;
    bool last_labelled = false;  // the replay ran out of its walks' budget

    // Parent steps the piece search may take: per update of the run, plus
    // a constant.
    void set_budget(size_t per_update, size_t base)
    {
        budget_per_update_ = per_update;
        budget_base_ = base;
    }

  private:
    static uint64_t key(uint32_t a, uint32_t b) { return (uint64_t)b << 32 | a; }
    static void ends(uint64_t p, uint32_t &a, uint32_t &b)
    {
        a = (uint32_t)p;
        b = (uint32_t)(p >> 32) & 0x7fffffffu;
        if (a > b) std::swap(a, b);
    }
    // A distinct edge of the run: endpoints, their pieces, whether it is in
    // T0, in D0, a forest edge at the moment, and whether it was ever removed.
    struct Edge {
        uint32_t a, b, pa, pb;
        uint8_t tree, d0, live, cut;
    };
    static uint32_t child(const Forest &F, const Edge &e)
    {
        return F.parent(e.a) == e.b ? e.a : e.b;
    }
    // Numbers of keys, in order of first appearance: open addressing, the
    // slots stamped so that a new run starts without clearing them.
    class Table {
      public:
        void start(size_t n)
        {
            size_t cap = 1024;
            while (cap < 2 * n) cap *= 2;
            if (cap > slots_.size()) slots_.assign(cap, Slot{0, 0, 0});
            if (++epoch_ == 0) {
                std::fill(slots_.begin(), slots_.end(), Slot{0, 0, 0});
                epoch_ = 1;
            }
            mask_ = cap - 1;
        }
        // The number of key k; `next` becomes it when k is new.
        uint32_t find(uint64_t k, uint32_t next)
        {
            uint64_t h = k * 0x9E3779B97F4A7C15ull;
            for (size_t i = (h ^ h >> 32) & mask_;; i = (i + 1) & mask_) {
                Slot &s = slots_[i];
                if (s.epoch != epoch_) {
                    s = {k, next, epoch_};
                    return next;
                }
                if (s.key == k) return s.id;
            }
        }

      private:
        struct Slot {
            uint64_t key;
            uint32_t id, epoch;
        };
        std::vector<Slot> slots_;
        size_t mask_ = 0;
        uint32_t epoch_ = 0;
    };
    // The piece forest as parent pointers.  link: 1 if x and y were in
    // different trees and are linked now, 0 if not, -1 out of budget.
    struct Walked {
        std::vector<uint32_t> &par;
        size_t budget;
        int link(uint32_t x, uint32_t y)
        {
            size_t nx = 0, ny = 0;
            uint32_t rx = x, ry = y;
            for (; par[rx] != kNone; rx = par[rx]) nx++;
            for (; par[ry] != kNone; ry = par[ry]) ny++;
            if (nx + ny > budget) return -1;
            budget -= nx + ny;
            if (rx == ry) return 0;
            if (nx > ny) std::swap(x, y);
            for (uint32_t c = x, below = y; c != kNone;) {  // re-root x's tree at x, below y
                const uint32_t up = par[c];
                par[c] = below;
                below = c;
                c = up;
            }
            return 1;
        }
        void cut(uint32_t x, uint32_t y)
        {
            if (par[x] == y)
                par[x] = kNone;
            else
                par[y] = kNone;
        }
    };
    // The same with labels.
    struct Labelled {
        Forest &F;
        int link(uint32_t x, uint32_t y)
        {
            if (F.has_pending()) F.split_pending();
            if (F.same_tree(x, y)) return 0;
            F.link(x, y);
            return 1;
        }
        void cut(uint32_t x, uint32_t y) { F.remove_edge(x, y); }
    };
    // The run's updates in order; false when f is out of budget.
    template <class PieceForest>
    bool replay(PieceForest &f, const uint64_t *upd, uint32_t K, uint64_t &nl, uint64_t &nc)
    {
        for (uint32_t k = 0; k < K; k++) {
            Edge &e = edges_[eid_[k]];
            if ((upd[k] >> 63) == 0) {
                if (e.live || e.pa == e.pb) continue;
                const int r = f.link(e.pa, e.pb);
                if (r < 0) return false;
                if (r) {
                    e.live = 1;
                    nl++;
                }
            } else if (e.live) {
                f.cut(e.pa, e.pb);
                e.live = 0;
                e.cut = 1;
                nc++;
            }
        }
        return true;
    }
    // Top vertex of x's piece; kNone when the budget runs out.  Every
    // vertex on the way up is remembered for this run.
    uint32_t find_top(const Forest &F, uint32_t x, size_t &budget)
    {
        path_.clear();
        uint32_t y = x, t;
        for (;;) {
            if (seen_[y] == epoch_) {
                t = top_[y];
                break;
            }
            path_.push_back(y);
            const uint32_t up = F.parent(y);
            if (up == kNone || cut_[y] == epoch_) {
                t = y;
                break;
            }
            if (budget == 0) return kNone;
            budget--;
            y = up;
        }
        for (uint32_t w : path_) {
            seen_[w] = epoch_;
            top_[w] = t;
        }
        return t;
    }

    std::vector<uint32_t> cut_, seen_, top_, pid_, pstamp_;  // by vertex; stamps are epochs
    std::vector<std::pair<uint32_t, uint32_t>> pieces_;  // (top, final group) to settle
    uint32_t epoch_ = 0;
    size_t budget_per_update_ = 64, budget_base_ = 4096;
    std::vector<uint32_t> piece_top_, path_;
    Table table_;
    std::vector<Edge> edges_;     // the run's distinct edges
    std::vector<uint32_t> eid_;   // by update: its edge
    std::vector<std::pair<uint32_t, uint32_t>> net_;
    std::vector<uint32_t> plbl_, ppar_;
    Forest PF_;
};

}  // namespace cupk
