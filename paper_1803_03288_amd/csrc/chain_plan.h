// Plan of the chain form of TAC (k3_tac_chain.hip): which graphs have it, and its tables.  Host code only.
//
// On model-shaped graphs every recv is introduced by one class of compute ops: with U(c) the union of the dep sets
// of the classes that feed class c, dep(c) \ U(c) is one recv, which c *owns*, or nothing (c joins branches).  When
// every recv has an owner c(r), a recv has P > 0 from the moment pre(r) = U(c(r)) has been transferred ("ready"):
// Q is the set of ready recvs, never empty while recvs are outstanding, and selection is a walk through the partial
// order r' < r iff r' is in pre(r).  (No class can point at a recv other than its own: the first one to do so would
// have had its own recv taken before that recv was ready.)  P of a ready recv is the time of its own class, plus the
// times of the joins of which it is the last recv outstanding.
//
//   direct predecessors of r ("sinks" of pre(r)): the recvs of pre(r) that are in pre of no other recv of pre(r);
//   gate: a set of two or more sinks after which something starts.  It counts its sinks: at zero its successors are
//     ready, at one its join (if it has one) points at the sink that is left;
//   chain: the recvs are covered by chains of the partial order; ready recvs are pairwise incomparable, so there is
//     at most one per chain, which is the slot it is kept in.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace tictac {

constexpr int kChainMaxChains = 8;      // slots of ready recvs in registers
constexpr int kChainAhead = 4;          // how far ahead on its chain the kernel requests the values of a recv
constexpr int kChainMaxGates = 40;      // one LDS word per lane each
constexpr int kChainBlock = 256;        // columns of op_time per block of the class totals

struct ChainRec {                       // per recv, 16 bytes
    int16_t next;                       // the recv that is ready once this one is taken, in the same slot; -1 none
    int16_t gate0, gate1;               // gates of which it is a sink; -1 none
    int16_t more, n_more;               // further recvs that are ready once it is taken: list[more .. more + n_more)
    int16_t slot;                       // its chain
    int16_t total;                      // its class total
    int16_t ahead;                      // the recv kChainAhead places further on its chain; -1 none
};

struct ChainGate {                      // 16 bytes
    int32_t fan_in;                     // number of sinks << 16 | xor of the sinks
    int16_t join;                       // class total of its join; -1 none
    int16_t first, n;                   // successors: list[first .. first + n)
    int16_t unused[3];
};

// The class totals: one row per run of consecutive columns of a set inside a block; the rows of a set are consecutive.
struct ChainColumns {
    std::vector<int32_t> first;         // [D + 1] the first row of every set
    // totals in more than one row, as first row | number of rows << 16: first those in two rows (n_pairs of them)
    std::vector<int32_t> several;
    int n_pairs = 0;
    // op_time columns, block by block of kChainBlock: a bit per column after which a row of the totals is complete
    // (sixteen columns per word), those rows in that order, and where a block starts among them
    std::vector<uint32_t> flush;
    std::vector<int32_t> flush_row, block_first;
};

struct ChainPlan {
    int n_slots = 0;                    // chains
    int32_t empty = -1;                 // total of the ops that depend on no recv
    std::vector<ChainRec> rec;          // [R]
    std::vector<ChainGate> gate;
    std::vector<int16_t> list;          // recvs: the lists above, then those ready at the start at list[start ..)
    int32_t start = 0, n_start = 0;
    std::vector<int16_t> place;         // [R] place of a recv on its chain
    std::vector<int32_t> head;          // the first kChainAhead recvs of every chain: recv | total << 16
    std::vector<int16_t> extra;         // [R] 1-based number among the recvs with a list, 0 for the others
    int n_extra = 0;
    bool second_gates = false;          // some recv is a sink of two gates
    // classes that can attain M+ of a ready recv r: cand[cand_ptr[r] .. cand_ptr[r + 1]), as rows of cls_dep
    std::vector<int32_t> cand_ptr, cand;
};

// Whether as many sets may have the form.
inline bool chain_may_be(int R, int D) { return R >= 1 && R <= 512 && D >= R && D <= R + kChainMaxGates + 1; }

// set_of_col [N]; false: more rows than a record can name
inline bool make_chain_columns(int N, int D, const int32_t *set_of_col, ChainColumns &c)
{
    const int n_blocks = (N + kChainBlock - 1) / kChainBlock;
    std::vector<int32_t> &at = c.first;
    at.assign(D + 1, 0);
    for (int j = 0; j < N; ++j)
        if (j + 1 == N || set_of_col[j + 1] != set_of_col[j] || (j + 1) % kChainBlock == 0) ++at[set_of_col[j] + 1];
    c.several.clear();
    c.n_pairs = 0;
    for (int k = 0; k < D; ++k) {
        const int n = at[k + 1];
        at[k + 1] += at[k];
        if (n > 1) c.several.push_back(at[k] | n << 16);
        c.n_pairs += n == 2;
        if (at[k + 1] > 32767) return false;
    }
    std::stable_partition(c.several.begin(), c.several.end(), [](int32_t v) { return v >> 16 == 2; });
    c.flush.assign((size_t)n_blocks * (kChainBlock / 16), 0);
    c.flush_row.clear();
    c.block_first.assign(1, 0);
    std::vector<int32_t> fill(at.begin(), at.end() - 1);
    for (int j = 0; j < N; ++j) {
        if (j + 1 == N || set_of_col[j + 1] != set_of_col[j] || (j + 1) % kChainBlock == 0) {
            c.flush[j / 16] |= 1u << (j % 16);
            c.flush_row.push_back(fill[set_of_col[j]]++);
        }
        if (j + 1 == N || (j + 1) % kChainBlock == 0) c.block_first.push_back((int32_t)c.flush_row.size());
    }
    return true;
}

// The distinct dep sets of the compute ops, in order of first member, and what they inherit.
struct ChainSets {
    std::vector<const uint64_t *> rows; // [D][W]
    std::vector<int32_t> row_of_set;    // [D] a row of cls_dep that holds the set
    std::vector<uint64_t> U;            // [D][W] the union of the sets of the predecessors
    std::vector<int32_t> par_ptr, par;  // their sets
    std::vector<int32_t> own, owner;    // [D] the recv that a set adds, [R] the set that adds a recv
    std::vector<int32_t> count;         // [D] recvs of a set
    int empty_set = -1;
};

// Whether every recv is added by one set, by itself; without that the graph has not the form.  s.rows and s.row_of_set are given;
// set_of_op [n]: the set of an op, -1 for a recv;  predecessors of op v: col_idx[row_ptr[v] .. row_ptr[v + 1]).
inline bool chain_owners(int R, int W, int n, const int32_t *row_ptr, const int32_t *col_idx, const int32_t *set_of_op, ChainSets &s)
{
    const int D = (int)s.rows.size();
    if (!chain_may_be(R, D)) return false;
    const size_t w8 = (size_t)W;
    std::vector<int32_t> edge_from, edge_into, last(D, -1);
    s.U.assign((size_t)D * w8, 0);
    for (int v = 0; v < n; ++v) {
        const int c = set_of_op[v];
        if (c < 0) continue;
        for (int32_t e = row_ptr[v]; e < row_ptr[v + 1]; ++e) {
            const int u = set_of_op[col_idx[e]];
            if (u < 0 || u == c || last[u] == c) continue;      // (ops of one set tend to follow each other)
            last[u] = c;
            for (int w = 0; w < W; ++w) s.U[c * w8 + w] |= s.rows[u][w];
            edge_from.push_back(u);
            edge_into.push_back(c);
        }
    }
    s.par_ptr.assign(D + 1, 0);
    s.par.resize(edge_from.size());
    for (int32_t c : edge_into) ++s.par_ptr[c + 1];
    for (int c = 0; c < D; ++c) s.par_ptr[c + 1] += s.par_ptr[c];
    {
        std::vector<int32_t> fill(s.par_ptr.begin(), s.par_ptr.end() - 1);
        for (size_t e = 0; e < edge_from.size(); ++e) s.par[fill[edge_into[e]]++] = edge_from[e];
    }
    // owners and joins
    s.own.assign(D, -1);
    s.owner.assign(R, -1);
    s.count.assign(D, 0);
    s.empty_set = -1;
    for (int c = 0; c < D; ++c) {
        int r = -1;
        for (int w = 0; w < W; ++w) {
            s.count[c] += __builtin_popcountll(s.rows[c][w]);
            const uint64_t x = s.rows[c][w] & ~s.U[c * w8 + w];
            if (!x) continue;
            if (r >= 0 || (x & (x - 1))) return false;          // (two recvs at once)
            r = w * 64 + __builtin_ctzll(x);
        }
        if (s.count[c] == 0) { s.empty_set = c; continue; }
        if (r >= 0) {
            if (s.owner[r] >= 0) return false;
            s.owner[r] = c;
            s.own[c] = r;
        }
    }
    for (int r = 0; r < R; ++r)
        if (s.owner[r] < 0) return false;
    return true;
}

// What decides whether a graph has the form: sinks, gates and joins, and a cover by few enough chains.
struct ChainForm {
    std::vector<int32_t> sink_ptr, sink_n, sinks;       // [D] where the sinks of a set start and their number; sinks in rising order
    std::vector<int32_t> by_count;      // [D] the sets, smaller ones first
    std::vector<int32_t> order_r;       // [R] the recvs, smaller sets of their owners first
    std::vector<int32_t> gate_set;      // a set that has the sinks of the gate
    std::vector<int32_t> gate_of;       // [D] the gate of a set with two sinks or more; -1 none
    std::vector<ChainRec> rec;          // [R] gates, slot and next
    int n_slots = 0;
};

// Whether the graph has the form.  s: after chain_owners.  A call asks this before it takes memory or launches anything for the
// form; the lists and candidates of make_chain_plan can be made later.
inline bool chain_form(int R, int W, const ChainSets &s, ChainForm &f)
{
    const int D = (int)s.rows.size();
    const size_t w8 = (size_t)W;
    // sets by their numbers of recvs, and recvs by those of their owners; ties in rising order
    std::vector<int32_t> at(R + 2);
    auto by = [&](auto n_of, int n, std::vector<int32_t> &out) {
        out.resize(n);
        std::fill(at.begin(), at.end(), 0);
        for (int i = 0; i < n; ++i) ++at[n_of(i) + 1];
        for (int i = 0; i <= R; ++i) at[i + 1] += at[i];
        for (int i = 0; i < n; ++i) out[at[n_of(i)]++] = i;
    };
    by([&](int c) { return s.count[c]; }, D, f.by_count);
    by([&](int r) { return s.count[s.owner[r]]; }, R, f.order_r);
    // sinks
    f.sink_ptr.assign(D, 0);
    f.sink_n.assign(D, 0);
    f.sinks.clear();
    f.sinks.reserve(D);
    std::vector<uint64_t> cand(w8), covered(w8);
    for (int c : f.by_count) {
        if (s.count[c] == 0) continue;
        f.sink_ptr[c] = (int32_t)f.sinks.size();
        // (one set before it, as along a chain: what that one adds)
        int u0 = -1;
        bool one = true;
        for (int32_t e = s.par_ptr[c]; e < s.par_ptr[c + 1]; ++e) {
            if (s.count[s.par[e]] == 0) continue;
            one = one && (u0 < 0 || u0 == s.par[e]);
            u0 = s.par[e];
        }
        if (one && u0 >= 0 && s.own[u0] >= 0) {
            if (s.own[c] < 0) return false;
            f.sinks.push_back(s.own[u0]);
            f.sink_n[c] = 1;
            continue;
        }
        std::fill(cand.begin(), cand.end(), 0);
        std::fill(covered.begin(), covered.end(), 0);
        auto take = [&](int r) {
            cand[r >> 6] |= 1ull << (r & 63);
            for (int w = 0; w < W; ++w) covered[w] |= s.U[s.owner[r] * w8 + w];
        };
        for (int32_t e = s.par_ptr[c]; e < s.par_ptr[c + 1]; ++e) {
            const int u = s.par[e];
            if (s.count[u] == 0) continue;
            if (s.own[u] >= 0) take(s.own[u]);
            else for (int i = 0; i < f.sink_n[u]; ++i) take(f.sinks[f.sink_ptr[u] + i]);
        }
        for (int w = 0; w < W; ++w) {
            if ((cand[w] | covered[w]) != s.U[c * w8 + w]) return false;
            for (uint64_t x = cand[w] & ~covered[w]; x; x &= x - 1) f.sinks.push_back(w * 64 + __builtin_ctzll(x));
        }
        f.sink_n[c] = (int32_t)f.sinks.size() - f.sink_ptr[c];
        if (s.own[c] < 0 && f.sink_n[c] < 2) return false;
    }
    // gates
    f.gate_set.clear();
    f.gate_of.assign(D, -1);
    f.rec.assign(R, ChainRec{-1, -1, -1, 0, 0, 0, -1, -1});
    for (int c : f.by_count) {
        const int32_t *const sk = f.sinks.data() + f.sink_ptr[c], n = f.sink_n[c];
        if (n < 2) continue;
        auto same = [&](int u) { return f.sink_n[u] == n && std::equal(sk, sk + n, f.sinks.data() + f.sink_ptr[u]); };
        int g = 0;
        while (g < (int)f.gate_set.size() && !same(f.gate_set[g])) ++g;
        if (g == (int)f.gate_set.size()) {
            if (g == kChainMaxGates) return false;
            f.gate_set.push_back(c);
            for (int i = 0; i < n; ++i) {
                ChainRec &q = f.rec[sk[i]];
                if (q.gate0 < 0) q.gate0 = (int16_t)g;
                else if (q.gate1 < 0) q.gate1 = (int16_t)g;
                else return false;
            }
        }
        f.gate_of[c] = g;
    }
    // chains
    // (a recv goes on from a direct predecessor where it can, else from any recv of pre(r) that ends a chain so far)
    int tail[kChainMaxChains];                      // last recv of every chain
    f.n_slots = 0;
    for (int r : f.order_r) {
        const int c = s.owner[r];
        const int32_t *const sk = f.sinks.data() + f.sink_ptr[c], n = f.sink_n[c];
        int k = -1;
        for (int i = 0; i < n && k < 0; ++i)
            if (tail[f.rec[sk[i]].slot] == sk[i]) k = f.rec[sk[i]].slot;
        for (int i = 0; i < f.n_slots && k < 0; ++i)
            if ((s.U[c * w8 + (tail[i] >> 6)] >> (tail[i] & 63)) & 1ull) k = i;
        if (n == 1 && k >= 0 && tail[k] == sk[0]) f.rec[sk[0]].next = (int16_t)r;
        if (k < 0) {
            if (f.n_slots == kChainMaxChains) return false;
            k = f.n_slots++;
        }
        tail[k] = r;
        f.rec[r].slot = (int16_t)k;
    }
    return true;
}

// Bytes that the tables of make_chain_plan take on the device at most, each from a multiple of 256 on.  (A recv is in one list of another, of a
// gate or of the start, or is the next of one; a set is a candidate of its sinks.)
inline size_t chain_plan_bytes(int R, const ChainForm &f)
{
    const size_t arrays[] = {sizeof(ChainRec) * R, sizeof(ChainGate) * f.gate_set.size(), 2 * (size_t)R, 2 * (size_t)R, 2 * (size_t)R,
                             4 * (size_t)f.n_slots * kChainAhead, 4 * ((size_t)R + 1), 4 * f.sinks.size()};
    size_t bytes = 0;
    for (size_t n : arrays) bytes += (n + 255) & ~(size_t)255;
    return bytes;
}

// The tables of a graph that has the form (f: of chain_form);  at [D + 1]: the first row of totals of every set
inline void make_chain_plan(int R, const ChainSets &s, const ChainForm &f, const std::vector<int32_t> &at, ChainPlan &p)
{
    const int n_gates = (int)f.gate_set.size();
    const std::vector<int32_t> &owner = s.owner, &order_r = f.order_r;
    p.rec = f.rec;
    // gates
    p.gate.clear();
    for (int c : f.gate_set) {
        int32_t v = f.sink_n[c] << 16;
        for (int i = 0; i < f.sink_n[c]; ++i) v ^= f.sinks[f.sink_ptr[c] + i];
        p.gate.push_back(ChainGate{v, -1, 0, 0, {0, 0, 0}});
    }
    std::vector<std::vector<int32_t>> gate_next(n_gates), more(R);
    std::vector<int32_t> gate_join(n_gates, -1), start;
    for (int c : f.by_count) {
        if (f.gate_of[c] < 0) continue;
        if (s.own[c] >= 0) gate_next[f.gate_of[c]].push_back(s.own[c]);
        else gate_join[f.gate_of[c]] = c;
    }
    for (int r : order_r) {
        const int n = f.sink_n[owner[r]], sink = n == 1 ? f.sinks[f.sink_ptr[owner[r]]] : -1;
        if (n == 0) start.push_back(r);
        if (sink >= 0 && p.rec[sink].next != r) more[sink].push_back(r);
    }
    p.n_slots = f.n_slots;
    p.place.assign(R, 0);
    std::vector<std::vector<int32_t>> chain(p.n_slots);
    for (int r : order_r) {
        std::vector<int32_t> &c = chain[p.rec[r].slot];
        p.place[r] = (int16_t)c.size();
        if (c.size() >= (size_t)kChainAhead) p.rec[c[c.size() - kChainAhead]].ahead = (int16_t)r;
        c.push_back(r);
    }
    p.list.clear();
    for (int r = 0; r < R; ++r) {
        p.rec[r].more = (int16_t)p.list.size();
        p.rec[r].n_more = (int16_t)more[r].size();
        p.list.insert(p.list.end(), more[r].begin(), more[r].end());
    }
    for (size_t g = 0; g < p.gate.size(); ++g) {
        p.gate[g].first = (int16_t)p.list.size();
        p.gate[g].n = (int16_t)gate_next[g].size();
        p.list.insert(p.list.end(), gate_next[g].begin(), gate_next[g].end());
    }
    p.extra.assign(R, 0);
    p.n_extra = 0;
    p.second_gates = std::any_of(p.rec.begin(), p.rec.end(), [](const ChainRec &q) { return q.gate1 >= 0; });
    for (int r = 0; r < R; ++r)
        if (p.rec[r].n_more > 0) p.extra[r] = (int16_t)++p.n_extra;
    p.start = (int32_t)p.list.size();
    p.n_start = (int32_t)start.size();
    p.list.insert(p.list.end(), start.begin(), start.end());
    // what can attain M+ of a ready recv: the classes owned by its direct successors and the joins it is a sink of (any
    // other class that holds it and another outstanding recv contains one of these)
    p.cand_ptr.assign(1, 0);
    p.cand.clear();
    for (int r = 0; r < R; ++r) {
        auto add = [&](int set) { p.cand.push_back(s.row_of_set[set]); };
        if (p.rec[r].next >= 0) add(owner[p.rec[r].next]);
        for (int x : more[r]) add(owner[x]);
        for (int g : {(int)p.rec[r].gate0, (int)p.rec[r].gate1})
            if (g >= 0) {
                for (int x : gate_next[g]) add(owner[x]);
                if (gate_join[g] >= 0) add(gate_join[g]);
            }
        p.cand_ptr.push_back((int32_t)p.cand.size());
    }
    p.head.clear();
    for (int r = 0; r < R; ++r) {
        p.rec[r].total = (int16_t)at[owner[r]];
        if (p.place[r] < kChainAhead) p.head.push_back(r | at[owner[r]] << 16);
    }
    for (size_t g = 0; g < p.gate.size(); ++g) p.gate[g].join = (int16_t)(gate_join[g] >= 0 ? at[gate_join[g]] : -1);
    p.empty = s.empty_set >= 0 ? at[s.empty_set] : -1;
}

}  // namespace tictac
