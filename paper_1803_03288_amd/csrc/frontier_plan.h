// Plan of the frontier form of TAC (k3_tac_frontier.hip): the graph of the classes of compute ops.
//
// dep of a class is the union of dep of its inputs: of the classes of the compute ops and of the recvs that precede one
// member none of whose predecessors has the same dep (for a piece of a split set, a member whose predecessors with the same
// dep are of other pieces).  The member of lowest level is such a one, and levels rise along the inputs.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace tictac {

constexpr int32_t kFrontierMaxClasses = (1 << 18) - 1;  // a class shares a word of the kernel's lists with a recv
constexpr int32_t kFrontierMaxRecvs = (1 << 14) - 2;
constexpr int32_t kFrontierMaxQ = 128;                  // members of Q, of the frontier: what the kernel has room for
constexpr int32_t kFrontierMaxFrontier = 448;
constexpr int32_t kFrontierMaxStack = 256;              // classes to be looked at
constexpr int32_t kFrontierMaxInputs = 64;              // of a class: they are looked at again and again

// An output of a class, a class that has it among its inputs: bits 0..17 the class.  Each class keeps the number of its inputs
// (classes) that do not point yet in four bits, those with more than fifteen in a word (bits 0..17 are its number).
constexpr uint32_t kFrontierFill = 1u << 18;            // no class: fills the last four of a list up
constexpr uint32_t kFrontierWide = 1u << 19;            // its counter is a word
constexpr uint32_t kFrontierOnly = 1u << 30;            // no other class is among its inputs
constexpr uint32_t kFrontierLast = 1u << 31;            // of the last four of a list

struct FrontierRow {        // 64 bytes: a class
    int32_t in[4];          // the first inputs: a class, or ~i for recv i, or ~R: none
    uint32_t out[4];        // the first outputs
    int32_t more;           // further inputs: where they start in `inputs` (a multiple of four), times four, and their number of fours
    int32_t rest;           // further outputs: where they start in `outputs`
    int32_t pad[2];
    int32_t n, list;        // number of op_time columns, where they are in cls_cols
    int32_t c0, c1;         // the first two
};

// The kernel keeps the counters of a few thousand consecutive classes in LDS, behind the highest that has been told of an input, and
// names most inputs of a class by how far they are before it.  So the classes are numbered along the graph: as they come, by first
// member, where that does it, by level where one in 32 of a sample of the inputs comes after what it feeds or more than so many before.
// 4 096 samples of 500 x 200 layered ops, as they come and by level: ids that fall along the graph (all inputs) 62.1 and 46.7 ms, at random
// 83.7 and 48.6, in the order of a depth-first walk (one in eleven) 64.1 and 54.9, level by level (none) 46.8 and 47.3; 200 x 100 ops, 1 500
// recvs, depth first (one in fifteen) 14.1 and 13.1, at random along the graph (one in 800) 15.2 and 15.0.
constexpr int32_t kFrontierWindow = 4096;
struct FrontierPlan {
    bool ok = false;
    std::vector<FrontierRow> row;
    bool numbered = false;                  // (else all numbers are the classes)
    std::vector<int32_t> cls_of;            // by number: the class
    std::vector<int32_t> inputs;            // (filled up to fours with ~R)
    std::vector<uint32_t> outputs;
    std::vector<uint32_t> counters;         // before the first round: eight classes per word, then the words of the wide ones
    std::vector<int32_t> wide;              // the wide ones
    std::vector<int32_t> roots;             // classes with recvs but no class among their inputs
    std::vector<int32_t> free_cols;         // columns of the ops that depend on no recv
    std::vector<int32_t> own_ptr, own;      // [R + 1]: the classes with recv i among their inputs
};

// Whether a sample outgrows the kernel's lists by a quarter of one: it is followed as by the kernel, with one unit of time for
// every op and 1/4 to 7/4 of the ops per recv for a recv.  (An estimate, hence the quarter: with 260 classes a level it comes to 131
// members of Q, and samples with exponential times mostly stay within the 128 there is room for.)
inline bool frontier_outgrown(int32_t R, int32_t N, const FrontierPlan &p)
{
    const int32_t C = (int32_t)p.row.size();
    struct Member { int32_t c, low, high; };
    std::vector<int32_t> at(C, 0), open(C), stack(p.roots.rbegin(), p.roots.rend()), Q;     // (at: the recv a class points at)
    std::vector<Member> frontier;
    std::vector<char> gone(R + 1, 0);
    std::vector<float> P(R, 0.0f), t(R);
    gone[R] = 1;
    for (int32_t c = 0; c < C; ++c) open[c] = p.counters[c >> 3] >> (c & 7) * 4 & 15u;
    for (size_t i = 0; i < p.wide.size(); ++i) open[p.wide[i]] = (int32_t)p.counters[(C + 7) / 8 + i];
    uint32_t draw = 1;
    for (float &x : t) {
        draw = draw * 1664525u + 1013904223u;
        x = (float)N / (float)R * (0.25f + 1.5f * (float)(draw >> 8) / (1 << 24));
    }
    const auto over = [](size_t n, int32_t most) { return n * 4 > (size_t)most * 5; };
    for (int32_t step = 0; step < R; ++step) {
        while (!stack.empty()) {
            if (step && over(stack.size(), kFrontierMaxStack)) return true;     // (the first ones come 64 at a time)
            const int32_t c = stack.back();
            const FrontierRow &row = p.row[c];
            stack.pop_back();
            int32_t low = INT32_MAX, high = -1;
            const auto look = [&](const int32_t *in) {
                for (int j = 0; j < 4; ++j) {
                    const int32_t r = in[j] < 0 ? ~in[j] : at[in[j]];
                    if (gone[r]) continue;
                    low = std::min(low, r);
                    high = std::max(high, r);
                }
            };
            look(row.in);
            for (int32_t k = 0; k < (row.more & 15); ++k) look(&p.inputs[(row.more >> 4) * 4 + 4 * k]);
            if (high < 0) continue;
            if (low != high) {
                frontier.push_back({c, low, high});
                if (over(frontier.size(), kFrontierMaxFrontier)) return true;
                continue;
            }
            at[c] = low;
            if (row.n && P[low] == 0.0f) Q.push_back(low);
            P[low] += (float)row.n;
            const uint32_t *out = row.out, *rest = p.outputs.data() + row.rest;
            for (;; out = rest, rest += 4) {
                for (int j = 0; j < 4; ++j) {
                    const int32_t x = (int32_t)(out[j] & 0x3ffffu), o = out[j] & kFrontierWide ? p.wide[x] : x;
                    if (!(out[j] & kFrontierFill) && --open[o] == 0) stack.push_back(o);
                }
                if (out[0] & kFrontierLast) break;
            }
        }
        if (over(Q.size(), kFrontierMaxQ)) return true;
        int32_t best = 0;
        if (!Q.empty()) {
            size_t k = 0;
            for (size_t i = 1; i < Q.size(); ++i)
                if (std::min(P[Q[k]], t[Q[i]]) < std::min(P[Q[i]], t[Q[k]])) k = i;
            best = Q[k];
            Q[k] = Q.back();
            Q.pop_back();
        } else if (!frontier.empty()) {
            const auto M = [&](const Member &m) { return t[m.low] + t[m.high]; };
            best = std::min_element(frontier.begin(), frontier.end(), [&](const Member &a, const Member &b) { return M(a) < M(b); })->low;
        } else {
            while (gone[best]) ++best;
        }
        gone[best] = 1;
        size_t kept = 0;
        for (const Member m : frontier) {
            if (m.low == best || m.high == best) stack.push_back(m.c);
            else frontier[kept++] = m;
        }
        frontier.resize(kept);
    }
    return false;
}

// By op: level, class (-1: a recv), recv (-1: a compute op).  cnt0: |dep| by class.  col_cls: class by column.
inline void make_frontier_plan(int32_t n, int32_t R, int32_t C, const int32_t *row_ptr, const int32_t *col_idx, const int32_t *level,
                               const int32_t *cls_of_op, const int32_t *recv_of_op, const std::vector<int32_t> &cnt0,
                               const std::vector<int32_t> &col_cls, FrontierPlan &p)
{
    if (R < 1 || R > kFrontierMaxRecvs || C < 1 || C > kFrontierMaxClasses) return;
    std::vector<int32_t> rep(C, -1);
    for (int32_t v = 0; v < n; ++v) {
        const int32_t c = cls_of_op[v];
        if (c >= 0 && (rep[c] < 0 || level[v] < level[rep[c]])) rep[c] = v;
    }
    p.cls_of.resize(C);
    std::vector<int32_t> number;                    // of a class (empty: itself)
    for (int32_t c = 0; c < C; ++c) p.cls_of[c] = c;
    int32_t seen = 0, apart = 0;
    for (int32_t c = 0; c < C; c += std::max(1, C / 2048))
        for (int32_t e = row_ptr[rep[c]]; e < row_ptr[rep[c] + 1]; ++e) {
            const int32_t v = cls_of_op[col_idx[e]];
            seen += v >= 0;
            apart += v > c || (v >= 0 && c - v > kFrontierWindow);
        }
    p.numbered = apart * 32 > seen;
    if (p.numbered) {
        std::vector<int32_t> at(1, 0);
        for (int32_t c = 0; c < C; ++c) {
            const size_t l = (size_t)level[rep[c]];
            if (l + 2 > at.size()) at.resize(l + 2, 0);
            ++at[l + 1];
        }
        for (size_t l = 1; l < at.size(); ++l) at[l] += at[l - 1];
        number.resize(C);
        for (int32_t c = 0; c < C; ++c) p.cls_of[number[c] = at[level[rep[c]]]++] = c;
        const std::vector<int32_t> was(rep);
        for (int32_t c = 0; c < C; ++c) rep[c] = was[p.cls_of[c]];
    }
    // (all that follows goes by number, but for cnt0 and the columns)
    const auto num = [&](int32_t c) { return number.empty() ? c : number[c]; };
    const auto recvs = [&](int32_t c) { return cnt0[p.cls_of[c]]; };
    std::vector<int32_t> col_ptr(C + 1, 0), cols(col_cls.size());
    for (int32_t c : col_cls) ++col_ptr[c + 1];
    for (int32_t c = 0; c < C; ++c) col_ptr[c + 1] += col_ptr[c];
    {
        std::vector<int32_t> fill(col_ptr.begin(), col_ptr.end() - 1);
        for (int32_t j = 0; j < (int32_t)col_cls.size(); ++j) cols[fill[col_cls[j]]++] = j;
    }
    // inputs of every class, in_ptr[c] .. in_ptr[c + 1], ascending: recvs (~i) first
    std::vector<int32_t> all_ptr(1, 0), all, in_ptr(1, 0), in, n_open(C, 0), n_out(C, 0), mark(C + R, -1);
    all_ptr.reserve(C + 1);
    all.reserve((size_t)C * 4);
    for (int32_t c = 0; c < C; ++c) {
        const size_t first = all.size();
        if (recvs(c) > 0)
            for (int32_t e = row_ptr[rep[c]]; e < row_ptr[rep[c] + 1]; ++e) {
                const int32_t u = col_idx[e], v = cls_of_op[u] < 0 ? ~recv_of_op[u] : num(cls_of_op[u]);
                if (v >= 0 && recvs(v) == 0) continue;
                size_t k = all.size();
                while (k > first && all[k - 1] > v) --k;
                if (k == first || all[k - 1] != v) all.insert(all.begin() + k, v);
            }
        all_ptr.push_back((int32_t)all.size());
    }
    // without those that are an input of another input: dep of that holds theirs
    p.own_ptr.assign(R + 1, 0);
    in_ptr.reserve(C + 1);
    in.reserve(all.size());
    for (int32_t c = 0; c < C; ++c) {
        for (int32_t k = all_ptr[c]; k < all_ptr[c + 1]; ++k)
            if (const int32_t w = all[k]; w >= 0)
                for (int32_t i = all_ptr[w]; i < all_ptr[w + 1]; ++i) mark[all[i] >= 0 ? all[i] : C + ~all[i]] = c;
        for (int32_t k = all_ptr[c]; k < all_ptr[c + 1]; ++k) {
            const int32_t v = all[k];
            if (mark[v >= 0 ? v : C + ~v] == c) continue;
            in.push_back(v);
            if (v >= 0) { ++n_out[v]; ++n_open[c]; }
            else ++p.own_ptr[~v + 1];
        }
        in_ptr.push_back((int32_t)in.size());
        if (in_ptr[c + 1] - in_ptr[c] > kFrontierMaxInputs) return;
    }
    p.counters.assign(((size_t)C + 7) / 8, 0);
    std::vector<int32_t> place(C, 0);               // (of the wide ones)
    for (int32_t c = 0; c < C; ++c) {
        if (n_open[c] < 16) {
            p.counters[c >> 3] |= (uint32_t)n_open[c] << (c & 7) * 4;
            place[c] = c;
        } else {
            place[c] = (int32_t)p.wide.size();
            p.wide.push_back(c);
        }
    }
    for (int32_t c : p.wide) p.counters.push_back((uint32_t)n_open[c]);
    p.counters.resize((p.counters.size() + 3) / 4 * 4, 0);
    p.row.resize(C);
    std::vector<int32_t> at(C, 0);                  // the output of class c that is next
    int32_t rest = 0;
    for (int32_t c = 0; c < C; ++c) {
        FrontierRow &r = p.row[c];
        const int32_t k = in_ptr[c + 1] - in_ptr[c], *q = in.data() + in_ptr[c];
        for (int32_t j = 0; j < 4; ++j) r.in[j] = j < k ? q[j] : ~R;
        r.more = (int32_t)p.inputs.size() << 2 | std::max(0, (k - 1) / 4);      // (a multiple of four: bits 0..3 are free)
        for (int32_t j = 4; j < (k + 3) / 4 * 4; ++j) p.inputs.push_back(j < k ? q[j] : ~R);
        for (uint32_t &o : r.out) o = kFrontierFill | (n_out[c] <= 4 ? kFrontierLast : 0u);
        r.rest = rest;
        rest += std::max(0, (n_out[c] - 1) / 4 * 4);
        r.pad[0] = r.pad[1] = 0;
        if (!n_open[c] && recvs(c) > 0) p.roots.push_back(c);
        r.list = col_ptr[p.cls_of[c]];
        r.n = col_ptr[p.cls_of[c] + 1] - r.list;
        const int32_t *col = cols.data() + r.list;
        r.c0 = r.n > 0 ? col[0] : 0;
        r.c1 = r.n > 1 ? col[1] : 0;
        if (recvs(c) == 0) p.free_cols.insert(p.free_cols.end(), col, col + r.n);
    }
    p.outputs.assign(rest, kFrontierFill);
    for (int32_t c = 0; c < C; ++c)
        if (n_out[c] > 4)
            for (int32_t j = 0; j < 4; ++j) p.outputs[p.row[c].rest + (n_out[c] - 1) / 4 * 4 - 4 + j] |= kFrontierLast;
    // what is in the kernel's lists before the first round
    {
        std::vector<char> pointed(R, 0);
        int32_t n_q = 0, n_frontier = 0;
        for (int32_t c : p.roots) {
            const int32_t k = in_ptr[c + 1] - in_ptr[c], r = ~in[in_ptr[c]];
            if (k > 1) ++n_frontier;
            else if (!pointed[r]) { pointed[r] = 1; ++n_q; }
        }
        if (n_q > kFrontierMaxQ || n_frontier > kFrontierMaxFrontier) return;
    }
    for (int32_t i = 0; i < R; ++i) p.own_ptr[i + 1] += p.own_ptr[i];
    p.own.resize(p.own_ptr[R]);
    std::vector<int32_t> own_fill(p.own_ptr.begin(), p.own_ptr.end() - 1);
    for (int32_t c = 0; c < C; ++c)
        for (int32_t k = in_ptr[c]; k < in_ptr[c + 1]; ++k) {
            const int32_t v = in[k];
            if (v < 0) {
                p.own[own_fill[~v]++] = c;
                continue;
            }
            const int32_t j = at[v]++;
            uint32_t &o = j < 4 ? p.row[v].out[j] : p.outputs[p.row[v].rest + j - 4];
            o = (o & kFrontierLast) | (uint32_t)place[c] | (n_open[c] == 1 ? kFrontierOnly : n_open[c] > 15 ? kFrontierWide : 0u);
        }
    // What comes later is followed where it may be too long: where a recv or a class holds more classes back than Q has members,
    // or a level has more than twice as many classes (on layered graphs Q grows to about half a level).  Where it outgrows the
    // lists the bit-sliced form takes all of a batch; samples by the frontier form up to there and the bit-sliced one then, against
    // that alone, 4 096 samples: 1 619 classes, one recv in 200 of them, 14.4 and 12.6 ms; 2 270 classes, 900 behind one,
    // 6.6 and 6.6.  (On layered graphs near the line samples still fit: 260 and 280 classes a level, eleven and twelve
    // thousand in all, 9 to 25 ms against 37 to 118.)
    bool follow = false;
    std::vector<int32_t> on_level;
    for (int32_t c = 0; c < C; ++c) {
        const size_t l = (size_t)level[rep[c]];
        if (l >= on_level.size()) on_level.resize(l + 1, 0);
        follow |= n_out[c] > kFrontierMaxQ || ++on_level[l] > 2 * kFrontierMaxQ;
    }
    for (int32_t i = 0; i < R; ++i) follow |= p.own_ptr[i + 1] - p.own_ptr[i] > kFrontierMaxQ;
    p.ok = !follow || !frontier_outgrown(R, (int32_t)col_cls.size(), p);
}

// The plan's rows and outputs as the kernel reads them, one after the other in a table of words.  Lane j of the four that look at a
// class takes words 4 j .. 4 j + 3 of its sixteen at a time: inputs j and 4 + j in sixteen bits each, output j, and
//   j = 0: further inputs: where they start in `inputs` (a multiple of four) times eight, and their number of fours; the first column
//   j = 1: where its further outputs start (bytes from the table's start); the second column (one column: the same again)
//   j = 2: the number of columns, where they are      j = 3: nothing
// An input in sixteen bits is a class, as how far it is before this one, or kInRecv + recv (R: none); where one does not fit all are
// among the further ones, as in FrontierRow.  An output is laid out so that its low five bits are where its counter is in its word.
constexpr uint32_t kOutFill = 1u << 20, kOutWide = 1u << 21, kOutOnly = 1u << 30, kOutLast = 1u << 31;      // bits 2..19: the class, or its number
constexpr uint32_t kOutClass = 0xffffcu;
constexpr uint32_t kInRecv = 0xc000u;

struct FrontierTable {
    std::vector<uint32_t> words;
    std::vector<int32_t> inputs;
};

inline void make_frontier_table(const FrontierPlan &p, FrontierTable &t)
{
    const size_t C = p.row.size();
    const int32_t R = (int32_t)p.own_ptr.size() - 1;
    const auto out = [](uint32_t z) {
        return (z & 0x3ffffu) << 2 | (z & kFrontierFill ? kOutFill : 0u) | (z & kFrontierWide ? kOutWide : 0u) | (z & (kFrontierOnly | kFrontierLast));
    };
    t.words.assign(C * 16 + p.outputs.size(), 0);
    std::vector<int32_t> in;
    for (size_t c = 0; c < C; ++c) {
        const FrontierRow &r = p.row[c];
        const int32_t *more = p.inputs.data() + (r.more >> 4) * 4;
        in.assign(r.in, r.in + 4);
        in.insert(in.end(), more, more + (r.more & 15) * 4);
        while (!in.empty() && in.back() == ~R) in.pop_back();
        bool fits = true;
        for (size_t k = 0; k < std::min<size_t>(8, in.size()); ++k) fits &= in[k] < 0 || (in[k] < (int32_t)c && (int32_t)c - in[k] < (int32_t)kInRecv);
        uint32_t *q = &t.words[c * 16];
        for (int j = 0; j < 4; ++j) {
            for (int h = 0; h < 2; ++h) {
                const size_t k = (size_t)(4 * h + j);
                const uint32_t x = !fits || k >= in.size() ? kInRecv + (uint32_t)R : in[k] < 0 ? kInRecv + (uint32_t)~in[k] : (uint32_t)((int32_t)c - in[k]);
                q[4 * j] |= x << 16 * h;
            }
            q[4 * j + 1] = out(r.out[j]);
        }
        const size_t first = t.inputs.size();
        for (size_t k = fits ? 8 : 0; k < in.size(); ++k) t.inputs.push_back(in[k]);
        t.inputs.resize((t.inputs.size() + 3) / 4 * 4, ~R);
        q[2] = (uint32_t)(first * 8 + (t.inputs.size() - first) / 4);
        q[3] = (uint32_t)r.c0;
        q[6] = (uint32_t)((C * 16 + (size_t)r.rest) * 4);
        q[7] = (uint32_t)(r.n > 1 ? r.c1 : r.c0);
        q[10] = (uint32_t)r.n;
        q[11] = (uint32_t)r.list;
    }
    for (size_t i = 0; i < p.outputs.size(); ++i) t.words[C * 16 + i] = out(p.outputs[i]);
}

}  // namespace tictac
