// Calls into the library's launchers that no entry point reaches in a test (host_lib.py).
#include <stdlib.h>
#include <string.h>

#include "frontier_plan.h"
#include "internal.h"

using namespace tictac;

// the class grouping on the device for N compute ops with rows of W words (nothing is read or written)
extern "C" int host_group_rows(int32_t N, int32_t W)
{
    Dag d;
    d.N = N;
    d.W = W;
    return (int)launch_group_rows(d, nullptr, nullptr, nullptr);
}
extern "C" int64_t host_group_bytes(int32_t N) { return (int64_t)group_workspace_bytes(N); }

// level_records_kernel and level_lists_kernel on the host, node by node
extern "C" void host_run_level_records(const void *params)
{
    const LevelRecordParams &p = *static_cast<const LevelRecordParams *>(params);
    const int32_t zero = p.ring * p.row_bytes;
    *p.used = 0;
    for (int32_t i = 0; i < p.n_levels * p.P; ++i) p.recs[i] = Dag::FastRec{{zero, zero, zero, zero}, {-1, -1}, -1, -1};
    for (int32_t k = 0; k < p.M; ++k) {
        Dag::FastRec &f = p.recs[p.slot[k]];
        const int32_t oldest = (p.slot[k] / p.P + 1) * p.P - p.ring, n = p.ptr[k + 1] - p.ptr[k], *in = p.in + p.ptr[k];
        f.op = p.op[k];
        int32_t nodes = 0, recvs = 0;
        bool fits = true;
        for (int32_t e = 0; e < n && fits; ++e) {
            if (in[e] < 0) fits = recvs < 2;
            else fits = nodes < 4 && p.slot[in[e]] >= oldest;
            if (!fits) break;
            if (in[e] < 0) f.rcv[recvs++] = ~in[e];
            else f.in[nodes++] = (p.slot[in[e]] & (p.ring - 1)) * p.row_bytes;
        }
        if (fits) continue;
        f = Dag::FastRec{{zero, zero, zero, zero}, {-1, -1}, p.op[k], *p.used};
        *p.used += 1 + n;
        if (*p.used > p.room) abort();
        p.lists[f.ovf] = n;
        for (int32_t e = 0; e < n; ++e) p.lists[f.ovf + 1 + e] = in[e] < 0 ? in[e] : p.slot[in[e]];
    }
}

// words per lane and workgroups of the bit-sliced TAC kernel for a graph of C classes and R recvs, B samples: as launched
extern "C" int host_tac_sliced(int32_t C, int32_t R, int32_t B)
{
    Dag d;
    d.C = C; d.R = R; d.W = (R + 63) / 64; d.CW = (C + 63) / 64; d.CWpad = (d.CW + 15) / 16 * 16; d.N = C;
    d.sliced_made = true;
    d.d_colbits = reinterpret_cast<uint64_t *>(&d);             // (only its being there is looked at)
    TacArgs a{};
    a.B = B;
    int32_t *flags = nullptr;
    const int e = (int)launch_tac_sliced(d, a, (size_t)B * 4, (size_t)B * 4, &flags, nullptr);
    (void)hipFree(d.d_work);
    return e;
}

// the plan of the frontier form (frontier_plan.h); NULL: it does not take the graph
extern "C" void *host_frontier_plan(int32_t n, int32_t R, int32_t C, int32_t N, const int32_t *row_ptr, const int32_t *col_idx, const int32_t *level,
                                    const int32_t *cls_of_op, const int32_t *recv_of_op, const int32_t *cnt0, const int32_t *col_cls)
{
    FrontierPlan *p = new FrontierPlan;
    make_frontier_plan(n, R, C, row_ptr, col_idx, level, cls_of_op, recv_of_op, std::vector<int32_t>(cnt0, cnt0 + C),
                       std::vector<int32_t>(col_cls, col_cls + N), *p);
    if (p->ok) return p;
    delete p;
    return nullptr;
}
// the words of one of its arrays
extern "C" int64_t host_frontier_array(const void *plan, const char *name, const void **at)
{
    const FrontierPlan &p = *static_cast<const FrontierPlan *>(plan);
    const struct { const char *name; const void *at; size_t n; } all[] = {
        {"row", p.row.data(), p.row.size() * 16}, {"inputs", p.inputs.data(), p.inputs.size()}, {"outputs", p.outputs.data(), p.outputs.size()},
        {"counters", p.counters.data(), p.counters.size()}, {"wide", p.wide.data(), p.wide.size()}, {"roots", p.roots.data(), p.roots.size()},
        {"free_cols", p.free_cols.data(), p.free_cols.size()}, {"own_ptr", p.own_ptr.data(), p.own_ptr.size()}, {"own", p.own.data(), p.own.size()}, {"cls_of", p.cls_of.data(), p.cls_of.size()}};
    for (const auto &a : all)
        if (!strcmp(a.name, name)) {
            *at = a.at;
            return (int64_t)a.n;
        }
    return -1;
}
// what the kernel reads of it: the words of its table and of the inputs that rows have no room for
extern "C" void *host_frontier_table(const void *plan)
{
    FrontierTable *t = new FrontierTable;
    make_frontier_table(*static_cast<const FrontierPlan *>(plan), *t);
    return t;
}
extern "C" int64_t host_frontier_table_array(const void *table, int32_t inputs, const void **at)
{
    const FrontierTable &t = *static_cast<const FrontierTable *>(table);
    *at = inputs ? static_cast<const void *>(t.inputs.data()) : t.words.data();
    return (int64_t)(inputs ? t.inputs.size() : t.words.size());
}
extern "C" void host_frontier_table_free(void *table) { delete static_cast<FrontierTable *>(table); }
extern "C" void host_frontier_free(void *plan) { delete static_cast<FrontierPlan *>(plan); }
