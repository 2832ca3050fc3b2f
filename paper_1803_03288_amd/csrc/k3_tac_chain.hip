// TAC (Sec. 4.3, Algorithm 3) with the iteration under its order (Sec. 3.2) on graphs that have the chain form of
// chain_plan.h (model-shaped graphs: one class of compute ops introduces each recv), one *lane* per timing sample.
//
// Two kernels:
//   * class_totals_kernel streams op_time once.  A wave takes 64 samples and a range of columns, 256 bytes of a row at a time
//     through LDS, so that lane l adds up the columns of sample l; the columns are the same
//     for all lanes, so which class a column belongs to is a matter of scalar code and no atomics are needed.  Totals and
//     transfer times are written transposed, [row][sample].
//   * tac_chain_kernel walks through the partial order of the recvs.  The ready recvs of a sample (at most one per chain)
//     sit in registers with P and Time; a round is one pass of the comparator over them, and the recv that follows the
//     one taken on its chain is entered from values requested a round earlier.  The time released by a transfer is P of
//     its recv when it is taken, so the makespan is a running maximum.
// What bounds them: the first the bytes of the timing arrays, the second the R dependent rounds of a sample.
// A sample with a transfer time or an owned class total of zero is flagged for the general kernel.
#include <algorithm>

#include "chain_plan.h"
#include "device_utils.h"
#include "internal.h"

namespace tictac {

struct TotalsParams {
    int32_t B, N, R, n_blocks, blocks_per_part, n_parts;
    size_t Bp;                          // samples per row of the outputs, a multiple of 64
    const void *op_time, *recv_time;    // of the first sample
    const uint32_t *flush;
    const int32_t *flush_row, *block_first;
    double *totals;                     // [n_totals][Bp]
    double *t;                          // [R][Bp]
    int32_t *flags;                     // [B] 1 = a transfer time is not positive
};

template <bool PAST>
__device__ __forceinline__ void store_total(double *to, double x)
{
    if constexpr (PAST) __builtin_nontemporal_store(x, to);
    else *to = x;
}

// Per tile 256 bytes of each of the 64 rows: a request of a wave covers four rows.  (128 and 512 bytes: 4 % and 5 % slower
// on inception3's rows, 4 % and 12 % on resnet50's.)  The next tile is requested once the present one is in LDS.
// 65 536 samples take 761 us on inception3 and 198 on resnet50: 4.3 and 3.3 TB/s of rows, but 5.7 and 5.4 of what is read and written,
// the rate of a copy.  The totals and times written are 13 % and 27 % on top of the rows, and lines are read twice: a piece of 256 bytes
// that does not start on a line touches three, and the shared one has left the cache when the next piece comes (3 941 MB read for 3 299 MB
// of rows on inception3, 904 for 661 on resnet50).
// PAST: totals and times are written past the caches, which hold neither all of them (434 MB for inception3) nor then what is
// read meanwhile: inception3 773 -> 761 us and 366 -> 355 for tac_chain_kernel, resnet50 204 -> 198.  (The rows read past the
// caches, whose 128-byte lines two requests share, take 894 us, the orders written so 7 us more.)
template <typename T, bool PAST>
__global__ void __launch_bounds__(64, 2)
class_totals_kernel(const TotalsParams p)
{
    constexpr int VEC = 16 / (int)sizeof(T);            // elements per load
    constexpr int LPR = 16;                             // lanes per row
    constexpr int TC = LPR * VEC;                       // columns per tile
    constexpr int RPI = 64 / LPR, NI = 64 / RPI;        // rows per load, loads per tile
    typedef T Vec __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));
    __shared__ T tile[TC * 65];
    const int lane = threadIdx.x, sub = (lane % LPR) * VEC, lr = lane / LPR;
    const bool recvs = (int)blockIdx.y == p.n_parts;    // the last part transposes the transfer times
    const int width = recvs ? p.R : p.N;
    const int blk = recvs ? 0 : (int)blockIdx.y * p.blocks_per_part;
    const int c_begin = blk * kChainBlock;
    const int c_end = recvs ? width : min(width, c_begin + p.blocks_per_part * kChainBlock);
    const int b0 = blockIdx.x * 64;
    // rows beyond the batch are read as its last one; their outputs are padding
    const T *src = static_cast<const T *>(recvs ? p.recv_time : p.op_time);
    const T *base = src + (size_t)min(b0 + lr, p.B - 1) * width + sub;
    const bool whole = b0 + 64 <= p.B;

    Vec v[NI];
    auto request = [&](int c0) {
        if (whole && c0 + TC <= width) {
#pragma unroll
            for (int i = 0; i < NI; ++i) v[i] = *reinterpret_cast<const Vec *>(base + (size_t)i * RPI * width + c0);
        } else {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const T *q = src + (size_t)min(b0 + i * RPI + lr, p.B - 1) * width + sub;
#pragma unroll
                for (int e = 0; e < VEC; ++e) v[i][e] = c0 + sub + e < width ? q[c0 + e] : T(0);
            }
        }
    };
    auto to_lds = [&]() {
        wave_sync();
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int e = 0; e < VEC; ++e) tile[(sub + e) * 65 + i * RPI + lr] = v[i][e];
        wave_sync();
    };
    if (recvs) {
        double *out = p.t + b0 + lane;
        bool zero_seen = false;
        request(0);
        for (int c0 = 0; c0 < c_end; c0 += TC) {
            to_lds();
            if (c0 + TC < c_end) request(c0 + TC);
            const int n = min(TC, c_end - c0);
            for (int c = 0; c < n; ++c) {
                const double y = (double)tile[c * 65 + lane];
                zero_seen |= !(y > 0.0);
                store_total<PAST>(&out[(size_t)(c0 + c) * p.Bp], y);
            }
        }
        if (b0 + lane < p.B) p.flags[b0 + lane] = zero_seen ? 1 : 0;
        return;
    }
    if (c_begin >= c_end) return;
    double *out = p.totals + b0 + lane;
    double acc = 0.0;
    int run = p.block_first[blk];
    request(c_begin);
    for (int c0 = c_begin; c0 < c_end; c0 += TC) {
        to_lds();
        if (c0 + TC < c_end) request(c0 + TC);
#pragma unroll
        for (int h = 0; h < TC / 16; ++h) {
            const uint32_t mask = c0 + 16 * h < c_end ? p.flush[c0 / 16 + h] : 0u;
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                acc += (double)tile[(16 * h + c) * 65 + lane];
                if ((mask >> c) & 1u) {
                    store_total<PAST>(&out[(size_t)p.flush_row[run++] * p.Bp], acc);
                    acc = 0.0;
                }
            }
        }
    }
}

struct ChainParams {
    int32_t B, R, W, n_gates, start, n_start, n_several, empty;
    size_t Bp;
    const int4 *rec;                    // ChainRec [R]
    const int4 *gate;                   // ChainGate [n_gates]
    const int16_t *list, *place, *extra;
    int32_t n_extra, n_pairs, n_head;
    const int32_t *several, *head;
    const int32_t *cand_ptr, *cand;
    const uint64_t *cls_dep;            // [C][W]
    double *totals;                     // [n_totals][Bp]
    const double *t;                    // [R][Bp]
    int32_t *order, *rank;
    int32_t simulate;
    double *makespan, *eff, *U, *L, *S;
    int32_t *flags;
};

constexpr int kStage = 32;              // rounds whose selections are staged in LDS before they go to memory
constexpr int kStagePad = 66;

static size_t chain_lds_bytes(int NC, const ChainParams &p)
{
    return ((size_t)p.R + NC) * 16 + (size_t)NC * kChainAhead * 64 * 16 + ((size_t)p.n_gates + 1) * 64 * 12 +
           ((size_t)2 * p.W + 1) * 64 * 4 + (size_t)kStage * kStagePad * 2 + ((size_t)p.n_gates + p.n_extra + 1) * NC * 4;
}

// A wave has a SIMD to itself at 65 536 samples, so a round costs its instructions (four cycles each) and every wait that
// nothing covers; a row of totals or times that a wave asks for is used by that wave alone, so it comes from the Infinity
// Cache or from HBM.  Therefore: when a recv is taken, the values of the recv four places further on its chain are
// requested; they land three rounds later in a ring in LDS (per slot and lane), from which a recv that becomes ready is
// entered.  A slot without a ready recv has P < 0 (the P of some recv with its sign set), which precedes nothing and is
// preceded by every ready recv; a recv that is the sink of no gate counts down gate n_gates, which never opens.
//
// The 64 samples of a wave are at different places, so what happens to one recv in thirty happens to some lane in almost
// every round: gates that open and recvs with several successors are on the path of every round.  Therefore what becomes
// ready then is a row of NC packed words, one per slot (successors of one recv do not depend on each other, so they are on
// different chains): one trip to LDS for the row and one for all its recvs.  A round has four dependent trips: the record
// of the recv taken; its ring entry, gates and joins; the row; the recvs of the row.  With the successors one after the
// other, each behind its list, its record and its gate, there were up to nine trips more per successor: 65 536 samples,
// inception3 (four branches) 377 -> 366 us (355 since totals are written past the caches), resnet50 (two) 99 -> 94 us.  What is left, from copies that leave something
// out: 80 and 21 us are the stores of the selections, 40 us and nothing the loads, the rest is a round's 110 vector
// instructions and its trips to LDS.  (A second wave that writes the selections takes the stores off the chain's wave and
// is no faster: 387 and 93 us.)  SECOND: some recv is a sink of two gates.
template <int NC, bool SECOND>
__global__ void __launch_bounds__(64)
tac_chain_kernel(const ChainParams p)
{
    extern __shared__ int4 chain_smem[];
    const int R = p.R, lane = threadIdx.x;
    // record of recv r: x = next | 1-based row of its other successors << 10 | second gate of next << 20 | sign: no next (next =
    // R + slot); y and z = byte offsets of the class total and the times of the recv kChainAhead places further; w = its ring
    // entry | ring entry of next << 5 | its gate << 10 | gate of next << 16 | its second gate << 22
    int4 *rec_l = chain_smem;                                           // [R + NC]
    double2 *ring = reinterpret_cast<double2 *>(rec_l + (R + NC));      // [NC * kChainAhead][64] P, Time
    double *join_l = reinterpret_cast<double *>(ring + NC * kChainAhead * 64);  // [n_gates + 1][64] time of the join
    uint32_t *gcnt = reinterpret_cast<uint32_t *>(join_l + (p.n_gates + 1) * 64);     // [n_gates + 1][64] sinks outstanding << 16 | their xor
    uint32_t *alive = gcnt + (p.n_gates + 1) * 64;                      // [2 W + 1][64] outstanding recvs
    uint16_t *stage = reinterpret_cast<uint16_t *>(alive + (2 * p.W + 1) * 64); // [kStage][kStagePad]
    // [n_gates + n_extra + 1] what is ready once a gate is open or a recv taken, by slot: recv | ring entry << 10 | its gate
    // << 15 | its second gate << 21, ~0 for nothing; the last row is empty
    struct alignas(NC >= 4 ? 16 : 4 * NC) Row { uint32_t e[NC]; };
    Row *rows = reinterpret_cast<Row *>(stage + kStage * kStagePad);
    const int no_row = p.n_gates + p.n_extra;

    const uint32_t row_bytes = (uint32_t)(p.Bp * 8);                    // (all rows together stay below 4 GB)
    const int b0 = blockIdx.x * 64, b = b0 + lane;                      // (rows hold a multiple of 64 samples)
    auto total_at = [&](uint32_t off) __attribute__((always_inline)) -> double & {
        return *reinterpret_cast<double *>(reinterpret_cast<char *>(p.totals) + (off + (uint32_t)b * 8u));
    };
    auto time_at = [&](uint32_t off) __attribute__((always_inline)) {
        return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(p.t) + (off + (uint32_t)b * 8u));
    };
    // totals in several rows are added up into the first, eight loads at a time
    for (int i = 0; i < p.n_pairs; i += 4) {
        double x[4], y[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t off = (uint32_t)(p.several[min(i + j, p.n_pairs - 1)] & 0xffff) * row_bytes;
            x[j] = total_at(off);
            y[j] = total_at(off + row_bytes);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i + j < p.n_pairs) total_at((uint32_t)(p.several[i + j] & 0xffff) * row_bytes) = x[j] + y[j];
    }
    for (int i = p.n_pairs; i < p.n_several; ++i) {
        const uint32_t off = (uint32_t)(p.several[i] & 0xffff) * row_bytes;
        const int n = p.several[i] >> 16;
        double s = 0.0;
        for (int j = 0; j < n; j += 8) {
            double x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = total_at(off + (uint32_t)min(j + e, n - 1) * row_bytes);
#pragma unroll
            for (int e = 0; e < 8; ++e) s += j + e < n ? x[e] : 0.0;
        }
        total_at(off) = s;
    }
    for (int r = lane; r < R; r += 64) {
        const int4 q = p.rec[r];
        const int next = (int)(int16_t)q.x, slot = q.z >> 16, at = p.place[r], extra = p.extra[r];
        const int ahead = (q.w >> 16) >= 0 ? q.w >> 16 : r;             // (at the end of a chain: a value that is never used)
        const int e = slot * kChainAhead, own = e + (at & (kChainAhead - 1)), gate = q.x >> 16, gate1 = (int)(int16_t)q.y;
        const int gate_next = next >= 0 ? p.rec[next].x >> 16 : -1, gate1_next = next >= 0 ? (int)(int16_t)p.rec[next].y : -1;
        rec_l[r] = make_int4((next >= 0 ? next : (R + slot) | (int)0x80000000u) | extra << 10 | (gate1_next >= 0 ? gate1_next : p.n_gates) << 20,
                             (int)((int)(int16_t)p.rec[ahead].w * row_bytes), (int)(ahead * row_bytes),
                             own | (next >= 0 ? e + ((at + 1) & (kChainAhead - 1)) : own) << 5 |
                             (gate >= 0 ? gate : p.n_gates) << 10 | (gate_next >= 0 ? gate_next : p.n_gates) << 16 | (gate1 >= 0 ? gate1 : p.n_gates) << 22);
    }
    if (lane < NC)
        rec_l[R + lane] = make_int4((R + lane) | (int)0x80000000u | p.n_gates << 20, 0, 0, lane * kChainAhead * 0x21 | p.n_gates * 0x410400);
    // (a word of LDS is written by one lane only: a row is its gate's or its recv's)
    auto packed = [&](int r) __attribute__((always_inline)) {
        const int4 q = p.rec[r];
        const int gate = q.x >> 16, gate1 = (int)(int16_t)q.y;
        return (uint32_t)(r | ((q.z >> 16) * kChainAhead + (p.place[r] & (kChainAhead - 1))) << 10 | (gate >= 0 ? gate : p.n_gates) << 15 |
                          (gate1 >= 0 ? gate1 : p.n_gates) << 21);
    };
    auto make_row = [&](int row, int first, int n) __attribute__((always_inline)) {
        Row e;
#pragma unroll
        for (int k = 0; k < NC; ++k) e.e[k] = ~0u;
        for (int i = 0; i < n; ++i) {
            const uint32_t v = packed(p.list[first + i]);
#pragma unroll
            for (int k = 0; k < NC; ++k) e.e[k] = (int)(v >> 10 & 0x1fu) / kChainAhead == k ? v : e.e[k];
        }
        rows[row] = e;
    };
    for (int i = lane; i < p.n_gates; i += 64) {
        const int4 c = p.gate[i];
        make_row(i, c.y >> 16, (int)(int16_t)c.z);
    }
    for (int r = lane; r < R; r += 64)
        if (const int extra = p.extra[r]) {
            const int4 q = p.rec[r];
            make_row(p.n_gates + extra - 1, q.y >> 16, (int)(int16_t)q.z);
        }
    if (lane == 0) make_row(no_row, 0, 0);
    wave_sync();
#pragma unroll 4
    for (int g = 0; g < p.n_gates; ++g) {
        const int4 c = p.gate[g];
        gcnt[g * 64 + lane] = (uint32_t)c.x;
        const int j = (int)(int16_t)c.y;
        const double x = total_at((uint32_t)max(j, 0) * row_bytes);
        join_l[g * 64 + lane] = j >= 0 ? x : 0.0;
    }
    gcnt[p.n_gates * 64 + lane] = 0x40000000u;
    join_l[p.n_gates * 64 + lane] = 0.0;
    // the first recvs of every chain
#pragma unroll 4
    for (int i = 0; i < p.n_head; ++i) {
        const int r = p.head[i] & 0xffff;
        ring[(rec_l[r].w & 0x1f) * 64 + lane] = make_double2(total_at((uint32_t)(p.head[i] >> 16) * row_bytes), time_at(r * row_bytes));
    }
    for (int h = 0; h <= 2 * p.W; ++h) {
        const int nbits = min(32, max(0, R - 32 * h));
        alive[h * 64 + lane] = nbits >= 32 ? 0xffffffffu : ((1u << nbits) - 1u);
    }
    wave_sync();
    bool bad = b < p.B ? p.flags[b] != 0 : true;

    // ---- the ready recvs: slot k holds recv id_k with its P and Time ----
#define TC_EACH(F) F(0) F(1) F(2) F(3) F(4) F(5) F(6) F(7)
#define TC_DECL(k) int id_##k = R + k; double P_##k = -1.0 - k, T_##k = TT_INF;
    TC_EACH(TC_DECL)

    // time of the join of gate g, if a recv that is ready now is the last outstanding sink of it
    auto join_of = [&](int g) __attribute__((always_inline)) {
        const uint32_t left = gcnt[g * 64 + lane];
        const double x = join_l[g * 64 + lane];
        return (left >> 16) == 1u ? x : 0.0;
    };
    // the recvs of a row become ready
    auto enter = [&](const Row &e) __attribute__((always_inline)) {
#define TC_ENTER(k)                                                                       \
        if constexpr (k < NC) {                                                           \
            const double2 v = ring[(k * kChainAhead + ((e.e[k] >> 10) & (kChainAhead - 1))) * 64 + lane]; \
            double pr = v.x + join_of(min((int)((e.e[k] >> 15) & 0x3fu), p.n_gates));     \
            if constexpr (SECOND) pr += join_of(min((int)((e.e[k] >> 21) & 0x3fu), p.n_gates)); \
            const bool here = (int)e.e[k] >= 0;                                           \
            id_##k = here ? (int)(e.e[k] & 0x3ffu) : id_##k;                              \
            P_##k = here ? pr : P_##k;                                                    \
            T_##k = here ? v.y : T_##k;                                                   \
        }
        TC_EACH(TC_ENTER)
    };
    {
        Row e;
#pragma unroll
        for (int k = 0; k < NC; ++k) e.e[k] = ~0u;
        for (int i = 0; i < p.n_start; ++i) {
            const uint32_t v = packed(p.list[p.start + i]);
#pragma unroll
            for (int k = 0; k < NC; ++k) e.e[k] = (int)(v >> 10 & 0x1fu) / kChainAhead == k ? v : e.e[k];
        }
        enter(e);
    }

    // M+ of a ready recv, and the literal ascending scan: only where the comparator ties
    auto m_plus = [&](int r) __attribute__((always_inline)) {
        double best = TT_INF;
        for (int e = p.cand_ptr[r]; e < p.cand_ptr[r + 1]; ++e) {
            const uint64_t *row = p.cls_dep + (size_t)p.cand[e] * p.W;
            int n = 0;
            double s = 0.0;
            for (int w = 0; w < p.W; ++w) {
                uint64_t x = row[w] & ((uint64_t)alive[(2 * w + 1) * 64 + lane] << 32 | alive[2 * w * 64 + lane]);
                n += __builtin_popcountll(x);
                while (x) {
                    s += time_at((w * 64 + __builtin_ctzll(x)) * row_bytes);
                    x &= x - 1;
                }
            }
            if (n >= 2) best = min_f64(best, s);
        }
        return best;
    };
    auto literal_scan = [&]() __attribute__((always_inline)) {
        int best = -1, at = -1, bslot = 0;
        double bP = 0.0, bT = 0.0, mp = -1.0;
        for (;;) {
            int a = R, as = 0;
            double aP = 0.0, aT = 0.0;
#define TC_LOWEST(k)                                                                      \
            if constexpr (k < NC) {                                                       \
                if (id_##k > at && id_##k < a) { a = id_##k; as = k; aP = P_##k; aT = T_##k; } \
            }
            TC_EACH(TC_LOWEST)
            if (a == R) break;
            at = a;
            if (best < 0) { best = a; bslot = as; bP = aP; bT = aT; continue; }
            const double xa = min_f64(bP, aT), ya = min_f64(aP, bT);
            double ma = -1.0;
            bool prec = xa < ya;
            if (xa == ya) {
                ma = m_plus(a);
                if (mp < 0.0) mp = m_plus(best);
                prec = ma < mp;
            }
            if (prec) { best = a; bslot = as; bP = aP; bT = aT; mp = ma; }
        }
        return bslot;
    };

    const double e_time = p.empty >= 0 ? total_at(p.empty * row_bytes) : 0.0;
    double F = 0.0, busy = e_time, sum_c = e_time;
    int32_t *const order_w = p.order + (size_t)b0 * R;
    int32_t *const rank_w = p.rank ? p.rank + (size_t)b0 * R : nullptr;
    // values under way: requested three rounds, two rounds and one round ago, each with the ring entry it goes to
    double2 in_a = ring[lane], in_b = in_a, in_c = in_a;
    int at_a = 0, at_b = 0, at_c = 0;
    // (the first rounds put back what entry 0 holds: nothing else goes there before the fourth round)

    auto round = [&](int step, double2 &in, int &in_at) __attribute__((always_inline)) {
        ring[in_at * 64 + lane] = in;

        // ---- selection.  Without a tie the order in which the ready recvs are compared does not matter: strict
        // precedence is transitive, so the one that is left precedes all others and the ascending scan ends with it too ----
        int slot = 0, best = id_0;
        double bP = P_0, bT = T_0;
        bool tie = false;
#define TC_COMPARE(k)                                                                     \
        if constexpr (k >= 1 && k < NC) {                                                 \
            const double xa = min_f64(bP, T_##k), ya = min_f64(P_##k, bT);                      \
            tie |= xa == ya;                                                              \
            const bool take = xa < ya;                                                    \
            slot = take ? k : slot;                                                       \
            best = take ? id_##k : best;                                                  \
            bP = take ? P_##k : bP;                                                       \
            bT = take ? T_##k : bT;                                                       \
        }
        TC_EACH(TC_COMPARE)
        if (NC > 1 && tie) {
            slot = literal_scan();
#define TC_TAKEN(k) if constexpr (k < NC) { best = slot == k ? id_##k : best; bP = slot == k ? P_##k : bP; bT = slot == k ? T_##k : bT; }
            TC_EACH(TC_TAKEN)
        }
        bad |= !(bP > 0.0);                             // (a time of zero, or nothing ready: left to the general kernel)

        // ---- record it; the iteration ----
        const int4 q = rec_l[best];
        stage[(step & (kStage - 1)) * kStagePad + lane] = (uint16_t)best;
        atomicAnd(&alive[(best >> 5) * 64 + lane], ~(1u << (best & 31)));
        in.x = total_at((uint32_t)q.y);
        in.y = time_at((uint32_t)q.z);
        in_at = q.w & 0x1f;
        const int g = (q.w >> 10) & 0x3f, g1 = (q.w >> 22) & 0x3f;
        const double2 v = ring[((q.w >> 5) & 0x1f) * 64 + lane];
        const double f_join = join_of((q.w >> 16) & 0x3f), f_join1 = SECOND ? join_of((q.x >> 20) & 0x3f) : 0.0;
        const uint32_t c = (gcnt[g * 64 + lane] - 0x10000u) ^ (uint32_t)best;
        const double x = join_l[g * 64 + lane];
        uint32_t c1 = 0x20000u;
        double x1 = 0.0;
        if constexpr (SECOND) {
            c1 = (gcnt[g1 * 64 + lane] - 0x10000u) ^ (uint32_t)best;
            x1 = join_l[g1 * 64 + lane];
        }
        F += bT;
        busy = max_f64(busy, F) + bP;
        sum_c += bP;

        // ---- what is ready now: the next recv on the chain, with the join that points at it already.  (It is no sink of
        // a gate that was counted down: sinks of one gate do not depend on each other.) ----
        const int f = q.x & 0x3ff, extra = (q.x >> 10) & 0x3ff;
        gcnt[g * 64 + lane] = c;
        if constexpr (SECOND) gcnt[g1 * 64 + lane] = c1;
        double fP = __hiloint2double(__double2hiint(v.x) | (q.x & (int)0x80000000u), __double2loint(v.x));
        fP += f_join;
        if constexpr (SECOND) fP += f_join1;
#define TC_NEXT(k)                                                                        \
        if constexpr (k < NC) {                                                           \
            id_##k = slot == k ? f : id_##k;                                              \
            P_##k = slot == k ? fP : P_##k;                                               \
            T_##k = slot == k ? v.y : T_##k;                                              \
        }
        TC_EACH(TC_NEXT)
        // a gate with one sink outstanding: its join points at that sink, if it is ready (else it does once it is)
        auto join_points = [&](uint32_t left, double time) __attribute__((always_inline)) {
            const double y = (left >> 16) == 1u ? time : 0.0;
            const int sink = (int)(left & 0xffffu);
#define TC_JOIN(k) if constexpr (k < NC) { P_##k += id_##k == sink ? y : 0.0; }
            TC_EACH(TC_JOIN)
        };
        if (NC > 1 && c < 0x20000u) join_points(c, x);
        if (SECOND && c1 < 0x20000u) join_points(c1, x1);
        // with none outstanding it opens.  (What it opens, what a second gate opens and the other successors of the recv do
        // not depend on each other either: one word per slot holds them all)
        const bool opens = c < 0x10000u, opens1 = SECOND && c1 < 0x10000u;
        if (NC > 1 && (opens || opens1 || extra != 0)) {
            Row e = rows[opens ? g : no_row];
            const Row e1 = rows[extra != 0 ? p.n_gates + extra - 1 : no_row];
#pragma unroll
            for (int k = 0; k < NC; ++k) e.e[k] = min(e.e[k], e1.e[k]);
            if constexpr (SECOND) {
                const Row e2 = rows[opens1 ? g1 : no_row];
#pragma unroll
                for (int k = 0; k < NC; ++k) e.e[k] = min(e.e[k], e2.e[k]);
            }
            enter(e);
        }

        // ---- selections to memory, kStage rounds at a time: two samples per store, whole lines of the order ----
        if ((step & (kStage - 1)) == kStage - 1 || step == R - 1) {
            wave_sync();
            const int s = (step & ~(kStage - 1)) + (lane & 31), n_b = min(64, p.B - b0);
            if (s <= step)
                for (int j0 = lane >> 5; j0 < 64; j0 += 16) {
                    int r[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) r[i] = min((int)stage[(lane & 31) * kStagePad + j0 + 2 * i], R - 1);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (j0 + 2 * i < n_b) {
                            order_w[(j0 + 2 * i) * R + s] = r[i];
                            if (rank_w) rank_w[(j0 + 2 * i) * R + r[i]] = s;
                        }
                }
            wave_sync();
        }
    };
    int step = 0;
    for (; step + 3 <= R; step += 3) {
        round(step, in_a, at_a);
        round(step + 1, in_b, at_b);
        round(step + 2, in_c, at_c);
    }
    if (step < R) round(step, in_a, at_a);
    if (step + 1 < R) round(step + 1, in_b, at_b);

    if (b < p.B) {
        p.flags[b] = bad ? 1 : 0;
        if (p.simulate && !bad) {
            const double m = busy;                      // (not less than F: the last transfer is in it)
            const double U = sum_c + F;
            const double L = max_f64(sum_c, F);
            if (p.makespan) p.makespan[b] = m;
            if (p.eff) p.eff[b] = (U == L) ? 1.0 : (U - m) / (U - L);
            if (p.U) p.U[b] = U;
            if (p.L) p.L[b] = L;
            if (p.S) p.S[b] = (U == L || L == 0.0) ? 0.0 : (U - L) / L;
        }
    }
}

template <int NC, bool SECOND>
static hipError_t launch_chain_nc(const ChainParams &p, hipStream_t s)
{
    const size_t lds = chain_lds_bytes(NC, p);
    if (lds > 48 * 1024) {
        const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(tac_chain_kernel<NC, SECOND>), lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((tac_chain_kernel<NC, SECOND>), dim3((unsigned)((p.B + 63) / 64)), dim3(64), lds, s, p);
    return hipGetLastError();
}

// Bytes of the workspace that a chunk of samples takes: totals and transposed transfer times.  Where the device has less,
// the chunks are halved, down to 8 192 samples: a chunk takes R rounds whatever its size, and below that the
// register-resident kernel, which needs four bytes per sample, is as fast (launch_tac).
constexpr size_t kChainChunkBytes = (size_t)512 << 20;
constexpr size_t kChainChunkLeast = 8192;
// Bytes read and written by class_totals_kernel up to which totals and times go through the caches: the Infinity Cache (256 MB)
// then still holds enough of them for tac_chain_kernel.  What a pass takes past the caches, against through them (150 to 800 MB in steps of
// 20 to 100; up to 220 MB the same to 3 % more):
//   MB                  300     350     400     420     460     500-520   600     800
//   vgg16     float64   +8 %    +6      +3      +2      +1      +1        -1      -4
//             float32   +7      +3      +5      +4      +1      +1        -4      -4
//   resnet50  float64   -1      +4      +4      +2      +1      +1        +1      -0.5
//             float32   +7      +1      +1      -0.5    -1      -2        -2      -3
//   inception3, both    +1      +1      0       0       0       0         0       -0.5
// So the sides meet between 415 MB (resnet50, float32) and 700 (resnet50, float64), and by then nothing hangs on it.
constexpr size_t kTotalsCached = (size_t)432 << 20;

hipError_t launch_tac_chain(Dag &d, const TacArgs &a, size_t flag_bytes, size_t at_least, int32_t **flags_out, hipStream_t s)
{
    const ChainTables &c = d.chain;
    if (a.sel_P || a.sel_Mplus) return hipErrorNotSupported;
    const size_t per_sample = ((size_t)c.n_totals + d.R) * 8;
    size_t chunk = std::min((size_t)a.B, kChainChunkBytes / per_sample);
    chunk = (chunk + 63) & ~(size_t)63;
    if (std::max(at_least, flag_bytes + chunk * per_sample) > d.work_bytes && being_captured(s)) return hipErrorNotSupported;
    hipError_t e = ensure_workspace(&d, std::max(at_least, flag_bytes + chunk * per_sample));
    while (e == hipErrorOutOfMemory && chunk > kChainChunkLeast) {
        chunk = std::max(kChainChunkLeast, (chunk / 2 + 63) & ~(size_t)63);
        e = ensure_workspace(&d, std::max(at_least, flag_bytes + chunk * per_sample));
    }
    if (e != hipSuccess) return e;
    int32_t *flags = static_cast<int32_t *>(d.d_work);
    double *totals = reinterpret_cast<double *>(static_cast<char *>(d.d_work) + flag_bytes);
    const size_t elem = a.f32 ? 4 : 8;
    const int n_cu = device_cu_count(d.device);
    for (size_t b0 = 0; b0 < (size_t)a.B; b0 += chunk) {
        const int32_t nb = (int32_t)std::min(chunk, (size_t)a.B - b0);
        const int groups = (nb + 63) / 64;
        TotalsParams t{};
        t.B = nb; t.N = d.N; t.R = d.R; t.Bp = chunk;
        t.n_blocks = (d.N + kChainBlock - 1) / kChainBlock;
        // columns are split until there are 32 waves per compute unit, of which LDS holds nine at a time: with no more than
        // those the compute units end at different times and the transfer times come last (65 536 samples, eight and 32 waves:
        // inception3 814 and 763 us, resnet50 204 and 203)
        const int parts = std::max(1, std::min(t.n_blocks, (32 * n_cu + groups - 1) / groups));
        t.blocks_per_part = (t.n_blocks + parts - 1) / parts;
        t.n_parts = (t.n_blocks + t.blocks_per_part - 1) / t.blocks_per_part;
        t.op_time = static_cast<const char *>(a.op_time) + b0 * d.N * elem;
        t.recv_time = static_cast<const char *>(a.recv_time) + b0 * d.R * elem;
        t.flush = c.d_flush; t.flush_row = c.d_flush_row; t.block_first = c.d_block_first;
        t.totals = totals; t.t = totals + (size_t)c.n_totals * chunk; t.flags = flags + b0;
        const dim3 grid((unsigned)groups, (unsigned)t.n_parts + 1);
        const bool past = nb * (((size_t)d.N + d.R) * elem + per_sample) > kTotalsCached;
        void (*const kernel)(TotalsParams) = a.f32 ? (past ? class_totals_kernel<float, true> : class_totals_kernel<float, false>)
                                                   : (past ? class_totals_kernel<double, true> : class_totals_kernel<double, false>);
        hipLaunchKernelGGL(kernel, grid, dim3(64), 0, s, t);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        // (at a handle's first call the tables of the chains are made while the first totals are formed)
        if (b0 == 0) e = ensure_chain_tables(&d);
        if (e != hipSuccess) return e;
        ChainParams p{};
        p.B = nb; p.R = d.R; p.W = d.W; p.Bp = chunk;
        p.n_gates = c.n_gates; p.start = c.start; p.n_start = c.n_start;
        p.n_several = c.n_several; p.empty = c.empty;
        p.rec = c.d_rec; p.gate = c.d_gate; p.list = c.d_list; p.place = c.d_place; p.extra = c.d_extra; p.n_extra = c.n_extra;
        p.n_pairs = c.n_pairs; p.n_head = c.n_head; p.head = c.d_head; p.several = c.d_several;
        p.cand_ptr = c.d_cand_ptr; p.cand = c.d_cand; p.cls_dep = d.d_cls_dep;
        p.totals = totals; p.t = t.t;
        p.order = a.order + b0 * d.R;
        p.rank = a.rank ? a.rank + b0 * d.R : nullptr;
        p.simulate = a.simulate ? 1 : 0;
        p.makespan = a.makespan ? a.makespan + b0 : nullptr;
        p.eff = a.eff ? a.eff + b0 : nullptr;
        p.U = a.U ? a.U + b0 : nullptr;
        p.L = a.L ? a.L + b0 : nullptr;
        p.S = a.S ? a.S + b0 : nullptr;
        p.flags = flags + b0;
        if (c.n_chains <= 1) e = launch_chain_nc<1, false>(p, s);
        else if (c.n_chains <= 2) e = c.second_gates ? launch_chain_nc<2, true>(p, s) : launch_chain_nc<2, false>(p, s);
        else if (c.n_chains <= 4) e = c.second_gates ? launch_chain_nc<4, true>(p, s) : launch_chain_nc<4, false>(p, s);
        else e = c.second_gates ? launch_chain_nc<8, true>(p, s) : launch_chain_nc<8, false>(p, s);
        if (e != hipSuccess) return e;
    }
    *flags_out = flags;
    return hipSuccess;
}

}  // namespace tictac
