// TAC (Sec. 4.3, Algorithm 3) with the iteration under its order (Sec. 3.2): the frontier form, one wave per timing sample.
//
// Algorithm 1 asks, every round, for |dep(c) ∩ R|, the number of outstanding recvs of every class of compute ops.  All the
// selection needs of it is which classes have come down to one outstanding recv (P) and which have the least M among those
// with two or more (M+).  Both can be read off the graph of the classes (frontier_plan.h), since dep of a class is the union
// of dep of its inputs:
//   * a class with one outstanding recv *points* at it.  A class whose inputs all point at a recv (or are recvs) has
//     as outstanding recvs those that are outstanding among these, a handful.  If there is one it points at it; if there
//     are more it belongs to the *frontier*, and it is looked at again when one of two of them (its watches) is transferred;
//   * a class with an input that does not point yet has that input's outstanding recvs, two at least, and its M is no smaller:
//     neither P nor the least M is concerned with it.  It only keeps the number of such inputs, which each input
//     lowers by one when it begins to point.
// So a sample costs one visit per edge of the class graph instead of R rounds over all classes: with 62 837 classes and
// 4 096 recvs 171 000 edges against 1.7 * 10^8 set bits.  The frontier has 40 members on average and 150 at most there, Q (the
// recvs with P > 0) 23 and 79, so one wave keeps both in LDS, and the states of the classes (16 bits each) and the numbers of
// their open inputs (4 bits) are in memory, so that sixteen samples and more share a compute unit.  That is more than the L2
// caches hold (157 KB per sample): 4 096 samples of one of 60 567 classes fetch 48.5 GB and write 25.8, 21 times their times and outputs
// (states, counters, rows, single times of ops: how much of it is whose has not been counted), 1.6 TB/s.  Those of that graph take 49
// ms (bit-sliced: 267 ms, two samples per compute unit), 11.7 us per round and wave, 6.4 us while a wave has the chip to itself: what bounds it is the latency
// of dependent trips to memory,
// for the rows of the classes looked at (0.9 ms in 10 of a sample's time), the states of their inputs (0.7), the counters of
// their outputs (2.5) and the times of the ops released (2.2), and the rest is instructions, 640 vector and 410 scalar ones a
// round.  That is why a class's row is one 64-byte line with its first inputs, outputs and columns, why four lanes look at a
// class side by side, why the outputs after the first four are requested along with the states, and why the times are
// fetched once per round, for all classes that have begun to point in it.  With sixteen-bit counters, in the states, the same
// took 65 ms (the caches hold less), and counters in LDS leave room for seven samples per compute unit.
//   M+ of single recvs is needed only where the comparator ties exactly; it is formed over the classes that hold the recv and
// have no input with two outstanding recvs of which it is one (M of such an input is no larger).
//   P of a recv at its selection is the time of the classes released by it, so the iteration is followed on the way.
//   A sample with a transfer time of zero is flagged for the general kernel (k3_tac.hip).
#include <algorithm>
#include <type_traits>

#include "device_utils.h"
#include "frontier_plan.h"
#include "internal.h"

namespace tictac {

constexpr int kNoRecv = 0x3fff;             // (recvs take 14 bits in the lists)
constexpr int kStack = kFrontierMaxStack, kFrontier = kFrontierMaxFrontier, kLog = 128;      // entries of the lists of a wave
constexpr int kPoints = 0x8000;             // state of a class that points: kPoints | recv; of another: 0

struct FrontierParams {
    int32_t B, R, W, C, N;
    const int4 *row;                // [C][4] FrontierRow
    const int32_t *inputs, *roots, *free_cols, *own_ptr, *own;
    const uint32_t *outputs, *counters;
    const int32_t *wide;
    int32_t n_roots, n_free, n_counters;
    const int32_t *cls_cols;
    const uint64_t *cls_dep;
    const void *op_time, *recv_time;
    int32_t *order, *rank;
    int32_t simulate;
    double *makespan, *eff, *U, *L, *S;
    int32_t *flags;                 // [B] 1: left to the general kernel, 2: to the bit-sliced one (a list was too short)
    char *scratch;                  // per wave: the states of the classes, where LDS does not hold them
    size_t scratch_stride;
};

__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ int rank_below(uint64_t mask)    // set bits below this lane
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}
__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }

// element i of an array in memory, by a 32-bit offset from its (uniform) start
template <typename T>
__device__ __forceinline__ T *at(T *base, uint32_t i)
{
    using Byte = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return reinterpret_cast<T *>(reinterpret_cast<Byte *>(base) + (uint32_t)(i * (uint32_t)sizeof(T)));
}

// over the four lanes of a quad
template <int CTRL>
__device__ __forceinline__ int quad_perm(int v) { return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true); }
__device__ __forceinline__ int quad_min(int v)
{
    v = min(v, quad_perm<0xb1>(v));
    return min(v, quad_perm<0x4e>(v));
}
__device__ __forceinline__ int quad_max(int v)
{
    v = max(v, quad_perm<0xb1>(v));
    return max(v, quad_perm<0x4e>(v));
}

// States of the classes of one sample, 16 bits each, in LDS or in memory: kPoints | recv, or 0.  Only the wave itself reads and
// writes them (plain loads and stores, which the L1 of its compute unit keeps coherent; wait_vmem() between the two).
template <bool LDS>
struct States {
    uint16_t *p;
    __device__ __forceinline__ int get(int c) const
    {
        return LDS ? p[c] : __hip_atomic_load(at(p, (uint32_t)c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    __device__ __forceinline__ void put(int c, int v) const
    {
        if (LDS) p[c] = (uint16_t)v;
        else __hip_atomic_store(at(p, (uint32_t)c), (uint16_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
};
// One less in the counter of an output (frontier_plan.h); the word before.  (A counter is lowered only while it is positive: the
// others of the word are not touched.)
template <bool LDS>
__device__ __forceinline__ uint32_t lower(uint32_t *counters, int n8, uint32_t z)
{
    const uint32_t x = z & 0x3ffffu;
    const bool wide = (z & kFrontierWide) != 0u;
    const uint32_t w = wide ? (uint32_t)n8 + x : x >> 3, by = wide ? 1u : 1u << (x & 7u) * 4u;
    return LDS ? atomicSub(counters + w, by) : __hip_atomic_fetch_sub(at(counters, w), by, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// was it the last?
__device__ __forceinline__ bool lowered(uint32_t z, uint32_t old)
{
    return z & kFrontierWide ? old == 1u : ((old >> (z & 7u) * 4u) & 15u) == 1u;
}

// One sample as the rare parts below see it.  They are functions of their own, so that the code of a round stays together.
template <typename T>
struct Sample {
    const T *rt;
    const uint32_t *alive, *fw, *fc;
    uint32_t *list;                 // the stack, which is empty then 
    const uint16_t *st;
    const int32_t *row, *inputs;
    const uint64_t *cls_dep;
    int nf, C, W;
};

// input number k of class c (more: FrontierRow::more of it)
template <typename T>
__device__ __forceinline__ int frontier_input(const Sample<T> &s, int c, int more, int k)
{
    return k < 4 ? s.row[16 * c + k] : s.inputs[(more >> 4) * 4 + k - 4];
}

// M of class c, formed from its row by the whole wave, and its lowest outstanding recv
template <typename T>
__device__ __forceinline__ double row_M(const Sample<T> &s, int c, int &low)
{
    const int lane = lane_id(), W = s.W;
    double sum = 0.0;
    int l = INT32_MAX;
    for (int w = lane; w < W; w += 64) {
        uint64_t x = s.cls_dep[(size_t)c * W + w] & (s.alive[2 * w] | (uint64_t)s.alive[2 * w + 1] << 32);
        while (x) {
            const int r = w * 64 + __builtin_ctzll(x);
            x &= x - 1;
            sum += (double)s.rt[r];
            l = min(l, r);
        }
    }
    low = wave_min_i32_dpp(l);
    return wave_sum_f64_dpp(sum);
}

// The least M of the members of the frontier, the lowest outstanding recv of those that attain it (INT32_MAX: there is no finite
// one), and the least M of those that hold recv r.
struct FrontierLeast {
    double M, M_of_r;
    int low;
};
template <typename T>
__device__ __forceinline__ FrontierLeast frontier_least(const Sample<T> s, int r)
{
    const int lane = lane_id();
    double gm = TT_INF, gr = TT_INF;
    int gl = INT32_MAX;
    for (int base = 0; base < s.nf; base += 64) {
        const bool in = base + lane < s.nf;
        double M = TT_INF;
        int low = INT32_MAX, n = 0, cls = 0, i = 0, end = 0, more = 0;
        uint32_t w = 0;
        bool holds = false;
        if (in) {
            w = s.fw[base + lane];
            cls = (int)(s.fc[base + lane] >> 14);
            low = (int)(w & kNoRecv);
            const int high = (int)((w >> 14) & kNoRecv);
            holds = low == r || high == r;
            M = (double)s.rt[low] + (double)s.rt[high];
        }
        if (__ballot((w >> 28) != 0u)) {
            // others than these two: the outstanding recvs of the class, ascending (at most eight; more are taken from its row)
            int q[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) q[k] = INT32_MAX;
            if (w >> 28) {
                more = s.row[16 * cls + 8];
                end = 4 + 4 * (more & 15);
            }
            while (__ballot(i < end)) {
                if (i < end) {
                    const int4 u4 = *reinterpret_cast<const int4 *>(i < 4 ? s.row + 16 * cls : s.inputs + (more >> 4) * 4 + i - 4);
                    const int u[4] = {u4.x, u4.y, u4.z, u4.w};
                    i += 4;
                    int x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        x[j] = ~u[j];
                        if (u[j] >= 0) x[j] = s.st[u[j]] & kNoRecv;
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        int v = x[j];
                        bool skip = !((s.alive[v >> 5] >> (v & 31)) & 1u);
                        holds |= !skip && v == r;
#pragma unroll
                        for (int k = 0; k < 8; ++k) skip |= q[k] == v;
                        if (!skip) {
                            ++n;
#pragma unroll
                            for (int k = 0; k < 8; ++k) {
                                const int l = min(q[k], v);
                                v = max(q[k], v);
                                q[k] = l;
                            }
                        }
                    }
                }
            }
            if (end) {
                M = 0.0;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (q[k] != INT32_MAX) M += (double)s.rt[q[k]];
                low = q[0];
            }
            uint64_t many = __ballot(n > 8);
            while (many) {
                const int l = __builtin_ctzll(many);
                many &= many - 1;
                int lw;
                const double m = row_M(s, __builtin_amdgcn_readlane(cls, l), lw);
                if (lane == l) { M = m; low = lw; }
            }
        }
        if (M < gm || (M == gm && low < gl)) { gm = M; gl = low; }
        if (holds) gr = min_f64(gr, M);
    }
    FrontierLeast f;
    f.M = wave_min_f64_dpp(gm);
    f.low = wave_min_i32_dpp(f.M < TT_INF && gm == f.M ? gl : INT32_MAX);
    f.M_of_r = wave_min_f64_dpp(gr);
    return f;
}

// M+ of recv r, given the least M of the members of the frontier that hold it
template <typename T>
__device__ __forceinline__ double frontier_M_plus(const Sample<T> s, const uint32_t *outputs, const int32_t *wide, const int32_t *own_ptr,
                                               const int32_t *own, int r, double best)
{
    const int lane = lane_id(), n8 = (s.C + 7) / 8;
    // Further classes that may attain it: those that do not point and have r, or a class that points at r, among their inputs.
    // The latter are gathered in a list, from eight states per load; first come the former.
    const uint32_t same = (uint32_t)(kPoints | r) * 0x10001u;
    const int o0 = own_ptr[r], o1 = own_ptr[r + 1];
    int ns = 0;
    uint4 q = make_uint4(0, 0, 0, 0);
    if (lane < n8) q = reinterpret_cast<const uint4 *>(s.st)[lane];
    for (int i0 = -((o1 - o0 + 63) / 64 * 64); i0 < n8 + 64; i0 += 64) {            // (the last turn empties the list)
        uint32_t found = 0;
        if (i0 >= 0) {
            const uint32_t x[4] = {q.x ^ same, q.y ^ same, q.z ^ same, q.w ^ same};
#pragma unroll
            for (int j = 0; j < 8; ++j) found |= ((x[j >> 1] >> (j & 1) * 16) & 0xffffu) == 0u ? 1u << j : 0u;
            if (i0 + lane >= n8) found = 0;
            if (i0 + 64 + lane < n8) q = reinterpret_cast<const uint4 *>(s.st)[i0 + 64 + lane];
        }
        bool again = true;
        while (again) {
            uint64_t m;
            while ((m = __ballot(found != 0u)) != 0ull && ns <= 64) {
                if (found) s.list[ns + rank_below(m)] = (uint32_t)((i0 + lane) * 8 + __builtin_ctz(found));
                found &= found - 1;
                ns += __builtin_popcountll(m);
            }
            if (i0 >= 0 && i0 < n8 && ns <= 64) break;
            again = m != 0ull;
            wave_sync();
            // own classes, or the outputs of the sixteen next ones of the list
            for (int base = 0; base < (i0 < 0 ? 1 : ns); base += 16) {
                uint32_t z = kFrontierFill | kFrontierLast;
                int o = 0;
                if (i0 < 0) {
                    const int k = o1 + i0 + lane;
                    if (k >= o0 && k < o1) z = (uint32_t)own[k] | kFrontierLast;
                } else if (base + (lane >> 2) < ns) {
                    const int32_t *row = s.row + 16 * s.list[base + (lane >> 2)];
                    z = (uint32_t)row[4 + (lane & 3)];
                    o = row[9];
                }
                for (;; o += 4) {
                    int y = z & kFrontierFill ? -1 : z & kFrontierWide ? wide[z & 0x3ffffu] : (int)(z & 0x3ffffu);
                    bool ok = y >= 0 && s.st[y < 0 ? 0 : y] == 0;
                    // it does not count if an input has two outstanding recvs or more of which r is one: M of that is no larger
                    if (ok) {
                        const int more = s.row[16 * y + 8];
                        for (int k = 0; k < 4 + 4 * (more & 15) && ok; ++k) {
                            const int u = frontier_input(s, y, more, k);
                            if (u >= 0 && s.st[u] == 0 && ((s.cls_dep[(size_t)u * s.W + (r >> 6)] >> (r & 63)) & 1ull)) ok = false;
                        }
                    }
                    uint64_t c = __ballot(ok);
                    while (c) {
                        const int l = __builtin_ctzll(c);
                        c &= c - 1;
                        int low;
                        best = min_f64(best, row_M(s, __builtin_amdgcn_readlane(y, l), low));
                    }
                    if (!__ballot(!(z & kFrontierLast))) break;
                    z = z & kFrontierLast ? kFrontierFill | kFrontierLast : outputs[o + (lane & 3)];
                }
            }
            wave_sync();
            ns = 0;
        }
    }
    return best;
}

// T: how times are stored; LS: states and counters of the classes in LDS
template <typename T, bool LS>
__global__ void __launch_bounds__(64)
tac_frontier_kernel(const FrontierParams p)
{
    extern __shared__ uint32_t smem[];
    const int lane = threadIdx.x;
    const int R = p.R;
    const int n_alive = (R + 128) / 128 * 4, n8 = (p.C + 7) / 8;

    double *P = reinterpret_cast<double *>(smem);                   // [128] of the members of Q
    uint32_t *stk = smem + 256;                                     // [kStack] classes to be looked at: class << 14 | the recv it points at, kNoRecv: not known
    uint32_t *fw = stk + kStack;                                    // [kFrontier] two outstanding recvs (14 bits each), bit 28: it has more
    uint32_t *fc = fw + kFrontier;                                  // [kFrontier] the class << 14
    uint32_t *lr = fc + kFrontier;                                  // [kLog] of classes that point: recv | number of columns (3: more than two) << 14
    int32_t *l0 = reinterpret_cast<int32_t *>(lr + kLog);           // its columns (more than two: where they are, their number)
    int32_t *l1 = l0 + kLog;
    uint32_t *alive = reinterpret_cast<uint32_t *>(l1 + kLog);      // [n_alive] outstanding recvs (bit R: none)
    uint32_t *counters = LS ? alive + n_alive : reinterpret_cast<uint32_t *>(p.scratch + (size_t)blockIdx.x * p.scratch_stride);
    States<LS> st;
    st.p = reinterpret_cast<uint16_t *>(counters + p.n_counters);
    const int32_t *rows = reinterpret_cast<const int32_t *>(p.row);
    // Parameters that only the rare parts need are read where they are needed: there are not enough scalar registers for all.
    using Arg = const __attribute__((address_space(4))) FrontierParams;
    Arg *args = (Arg *)__builtin_amdgcn_kernarg_segment_ptr();
    const auto rare = [&]() {
        Arg *q;
        asm volatile("" : "=s"(q) : "0"(args));
        return q;
    };

    for (int b = blockIdx.x; b < rare()->B; b += gridDim.x) {
        const T *rt = static_cast<const T *>(rare()->recv_time) + (size_t)b * R;
        const T *ot = static_cast<const T *>(rare()->op_time) + (size_t)b * rare()->N;
        wave_sync();
        bool zero = false;
        for (int r = lane; r < R; r += 64) zero |= !(rt[r] > (T)0);
        if (__ballot(zero)) {                               // left to the general kernel
            if (lane == 0) rare()->flags[b] = 1;
            continue;
        }
        for (int w = lane; w < n_alive; w += 64) alive[w] = R - w * 32 >= 32 ? ~0u : R - w * 32 > 0 ? (1u << (R - w * 32)) - 1u : 0u;
        {
            const uint4 *from = reinterpret_cast<const uint4 *>(rare()->counters);
            const int n = rare()->n_counters / 4;
            for (int i = lane; i < n; i += 64) reinterpret_cast<uint4 *>(counters)[i] = from[i];
        }
        for (int i = lane; i < n8; i += 64) reinterpret_cast<uint4 *>(st.p)[i] = make_uint4(0, 0, 0, 0);
        double s0 = 0.0;
        {
            const int32_t *cols = rare()->free_cols;
            const int n = rare()->n_free;
            for (int i = lane; i < n; i += 64) s0 += (double)ot[cols[i]];
        }
        const double free_time = wave_sum_f64_dpp(s0);
        if (!LS) wait_vmem();
        wave_sync();

        // Q: its members' recv (-1: none) and Time, two per lane; P is in LDS
        int ra = -1, rb = -1;
        double ta = 0.0, tb = 0.0;
        int nf = 0, ns = 0, nl = 0;                         // entries of frontier, stack, log (uniform)
        bool over = false;                                  // a list was too short (uniform)
        // (sums with what was rounded off beside them: one after the other, their error is otherwise twice that of a tree)
        double F = 0.0, busy = free_time, sum_c = free_time, F_lo = 0.0, busy_lo = 0.0, sum_lo = 0.0;
        int mine = 0;                                       // the order, by the lane of step mod 64

        const auto push = [&](bool in, uint32_t v) {
            const uint64_t m = __ballot(in);
            const int k = ns + rank_below(m);
            if (in && k < kStack) stk[k] = v;
            ns += __builtin_popcountll(m);
            if (ns > kStack) { over = true; ns = 0; }
        };

        // (before the first round: the classes that depend on recvs directly, 64 at a time)
        for (int step = -((rare()->n_roots + 63) / 64); step < R && !over; ++step) {
            wave_sync();
            nf = uniform_i32(nf);
            ns = uniform_i32(ns);
            nl = uniform_i32(nl);
            if (step < 0) {
                const int i = (-1 - step) * 64 + lane;
                const bool in = i < rare()->n_roots;
                push(in, in ? (uint32_t)rare()->roots[i] << 14 | kNoRecv : 0u);
            } else {
                // ================= selection =================
                int best;
                double Ps = 0.0, ts;                        // of the recv selected
                const uint64_t qa = __ballot(ra >= 0), qb = __ballot(rb >= 0);
                if ((qa | qb) == 0ull) {
                    // no outstanding recv has P > 0: the recv of lowest index among those of minimal M+
                    const Sample<T> sample = {rt, alive, fw, fc, stk, st.p, rows, rare()->inputs, rare()->cls_dep, nf, rare()->C, rare()->W};
                    const FrontierLeast f = frontier_least(sample, -1);
                    best = uniform_i32(f.low);
                    if (best == INT32_MAX) {
                        // no class with two outstanding recvs: every M+ is infinite, the lowest outstanding recv
                        int l = INT32_MAX;
                        for (int w = lane; w < n_alive; w += 64)
                            if (alive[w]) { l = w * 32 + __builtin_ctz(alive[w]); break; }
                        best = wave_min_i32_dpp(l);
                    }
                    if ((unsigned)best >= (unsigned)R) best = 0;        // (never: keeps indices in range)
                    ts = (double)rt[best];
                } else {
                    int pos;                                // lane, + 64: its second member
                    const bool two = qb != 0ull;
                    const double Pa = P[lane];
                    double Pb = 0.0;
                    if (two) Pb = P[64 + lane];
                    bool sure = true;
                    if (!two && (qa & (qa - 1)) == 0ull) {
                        pos = __builtin_ctzll(qa);
                    } else {
                        // The scan ends at the recv that strictly precedes every other one, if there is one (each pair that
                        // it is in is decided in its favour).  By Johnson's rule that is the one of smallest Time among
                        // those with Time < P, or, where there are none, of largest P.
                        const bool ea = ra >= 0 && ta < Pa, eb = rb >= 0 && tb < Pb;
                        uint64_t ca, cb = 0ull;
                        if (__ballot(ea || eb)) {
                            const double va = ea ? ta : TT_INF;
                            const double m = wave_min_f64_dpp(two && eb ? min_f64(va, tb) : va);
                            ca = __ballot(ea && ta == m);
                            if (two) cb = __ballot(eb && tb == m);
                        } else {
                            const double va = ra >= 0 ? Pa : -TT_INF;
                            const double m = wave_max_f64_dpp(two && rb >= 0 ? max_f64(va, Pb) : va);
                            ca = __ballot(ra >= 0 && Pa == m);
                            if (two) cb = __ballot(rb >= 0 && Pb == m);
                        }
                        pos = ca ? (int)__builtin_ctzll(ca) : cb ? 64 + (int)__builtin_ctzll(cb) : -1;
                        sure = pos >= 0;
                    }
                    if (sure) {
                        if (pos < 64) {
                            Ps = readlane_f64(Pa, pos);
                            ts = readlane_f64(ta, pos);
                        } else {
                            Ps = readlane_f64(Pb, pos - 64);
                            ts = readlane_f64(tb, pos - 64);
                        }
                        // (it does not precede itself)
                        const bool na = ra >= 0 && lane != pos && !(min_f64(Pa, ts) < min_f64(Ps, ta));
                        sure = __ballot(na) == 0ull;
                        if (two) sure = sure && __ballot(rb >= 0 && lane + 64 != pos && !(min_f64(Pb, ts) < min_f64(Ps, tb))) == 0ull;
                    }
                    if (!sure) {
                        // the scan itself, from one recv to the first later one that precedes it or ties with it
                        const Sample<T> sample = {rt, alive, fw, fc, stk, st.p, rows, rare()->inputs, rare()->cls_dep, nf, rare()->C, rare()->W};
                        int cur = -1, at = -1;
                        double lb = -1.0, hb = 0.0;         // bounds of M+ of the best so far (< 0: not formed yet)
                        pos = 0;
                        Ps = ts = 0.0;
                        for (int last = -1;;) {
                            const bool first = cur < 0;
                            const bool ha = ra > last && (first || min_f64(Ps, ta) <= min_f64(Pa, ts));
                            const bool hc = rb > last && (first || min_f64(Ps, tb) <= min_f64(Pb, ts));
                            const int low = wave_min_i32_dpp(min(ha ? ra : INT32_MAX, hc ? rb : INT32_MAX));
                            if (low == INT32_MAX) break;
                            const uint64_t ma = __ballot(ra == low);
                            at = ma ? (int)__builtin_ctzll(ma) : 64 + (int)__builtin_ctzll(__ballot(rb == low));
                            const double P_ = at < 64 ? readlane_f64(Pa, at) : readlane_f64(Pb, at - 64);
                            const double t_ = at < 64 ? readlane_f64(ta, at) : readlane_f64(tb, at - 64);
                            const double xa = min_f64(Ps, t_), ya = min_f64(P_, ts);
                            bool take = first || xa < ya;
                            double la = -1.0, ua = 0.0;
                            if (!first && xa == ya) {
                                // Between bounds first.  A class that holds the recv, is not of the frontier and has no input with two
                                // outstanding recvs of which the recv is one has an input with two others: its M is at
                                // least Time of the recv and the least M of the frontier.
                                for (int k = lb < 0.0 ? 0 : 1; k < 2; ++k) {
                                    const int r = k ? low : cur;
                                    const FrontierLeast f = frontier_least(sample, r);
                                    la = min_f64(f.M_of_r, f.M + (double)rt[r]);
                                    ua = f.M_of_r;
                                    if (!k) { lb = la; hb = ua; }
                                }
                                if (uniform_i32(ua >= lb && la < hb)) {         // (neither sure to be less nor sure not to be)
                                    for (int k = 0; k < 2; ++k) {
                                        if (uniform_i32(k ? !(la < ua) : !(lb < hb))) continue;
                                        const double m = frontier_M_plus(sample, rare()->outputs, rare()->wide, rare()->own_ptr,
                                                                         rare()->own, k ? low : cur, k ? ua : hb);
                                        if (k) la = ua = m;
                                        else lb = hb = m;
                                    }
                                }
                                take = ua < lb;
                            }
                            last = low;
                            if (uniform_i32(take)) { pos = at; cur = low; Ps = P_; ts = t_; lb = la; hb = ua; }
                        }
                    }
                    best = pos < 64 ? __builtin_amdgcn_readlane(ra, pos) : __builtin_amdgcn_readlane(rb, pos - 64);
                    if (lane == pos) ra = -1;
                    if (lane + 64 == pos) rb = -1;
                }
                if (lane == 0) alive[best >> 5] &= ~(1u << (best & 31));
                F = add_exact(F, ts, F_lo);
                if ((F - busy) + (F_lo - busy_lo) > 0.0) { busy = F; busy_lo = F_lo; }
                busy = add_exact(busy, Ps, busy_lo);
                sum_c = add_exact(sum_c, Ps, sum_lo);
                if ((step & 63) == lane) mine = best;
                if ((step & 63) == 63 || step == R - 1) {
                    const int s = (step & ~63) + lane;
                    if (s <= step) {
                        rare()->order[(size_t)b * R + s] = mine;
                        if (int32_t *rank = rare()->rank) rank[(size_t)b * R + mine] = s;
                    }
                }

                // ================= the frontier: classes that watch it =================
                int kept = 0;
                for (int base = 0; base < nf; base += 64) {
                    const bool in = base + lane < nf;
                    const uint32_t w = in ? fw[base + lane] : 0xffffffffu;
                    const int wa = (int)(w & kNoRecv), wb = (int)((w >> 14) & kNoRecv);
                    const bool hit = wa == best || wb == best;
                    const uint64_t hits = __ballot(hit);
                    if (!hits && kept == base) { kept = min(nf, base + 64); continue; }
                    const uint32_t c = in ? fc[base + lane] : 0u;
                    push(hit, c | (uint32_t)(w >> 28 ? kNoRecv : wa == best ? wb : wa));
                    const uint64_t stay = __ballot(in && !hit);
                    wave_sync();
                    if (in && !hit) {
                        const int at = kept + rank_below(stay);
                        fw[at] = w;
                        fc[at] = c;
                    }
                    kept += __builtin_popcountll(stay);
                }
                nf = kept;
            }

            // ================= what follows from it =================
            while ((ns > 0 || nl > 0) && !over) {
                wave_sync();
                nf = uniform_i32(nf);
                ns = uniform_i32(ns);
                nl = uniform_i32(nl);
                if (ns > 0 && nl + 16 <= kLog) {
                    // The classes on the stack, sixteen at a time, four lanes each: a class all of whose inputs point either points as
                    // well, and tells its outputs, or joins the frontier.
                    const int j = lane & 3;
                    const int k = min(ns, 16);
                    ns -= k;
                    const bool in = lane < 4 * k, lead = in && j == 0;
                    const uint32_t e = in ? stk[ns + (lane >> 2)] : 0u;
                    const int y = (int)(e >> 14);
                    int r = (int)(e & kNoRecv);
                    const bool open = in && r == kNoRecv;
                    // (lanes without a class look at class 0)
                    const int32_t *row = at(rows, 16u * (uint32_t)y);
                    const int2 more = *reinterpret_cast<const int2 *>(row + 8);
                    int v = row[j];
                    uint32_t z = (uint32_t)row[4 + j];
                    const int4 c = *reinterpret_cast<const int4 *>(row + 12);
                    if (!LS) wait_vmem();                   // states put by other lanes
                    // (the outputs after the first four on the way, so that both fours tell theirs in one go)
                    uint32_t z1 = kFrontierFill | kFrontierLast;
                    if (!(z & kFrontierLast)) z1 = rare()->outputs[more.y + j];
                    // the least and the greatest outstanding recv among the inputs, and whether there are others
                    if (!open) v = ~R;
                    int x = ~v;
                    if (v >= 0) x = st.get(v) & kNoRecv;
                    bool al = (alive[x >> 5] >> (x & 31)) & 1u;
                    int lo = quad_min(al ? x : INT32_MAX);
                    int hi = quad_max(al && x != lo ? x : -1);
                    int others = al && x != lo && x != hi;
                    if (__ballot(open && (more.x & 15))) {
                        int n = open ? more.x & 15 : 0, at = (more.x >> 4) * 4;
                        while (__ballot(n > 0)) {
                            v = n > 0 ? rare()->inputs[at + j] : ~R;
                            x = ~v;
                            if (v >= 0) x = st.get(v) & kNoRecv;
                            al = (alive[x >> 5] >> (x & 31)) & 1u;
                            const int lo1 = min(lo, quad_min(al ? x : INT32_MAX));
                            int h = al && x != lo1 ? x : -1;
                            if (lo != lo1 && lo != INT32_MAX) h = max(h, lo);
                            const int hi1 = max(hi, quad_max(h));
                            others |= (al && x != lo1 && x != hi1) || (lo != lo1 && lo != hi1 && lo != INT32_MAX) || (hi != hi1 && hi >= 0);
                            lo = lo1;
                            hi = hi1;
                            --n;
                            at += 4;
                        }
                    }
                    const bool front = lead && open && hi >= 0;
                    if (const uint64_t m = __ballot(front)) {
                        others = quad_max(others);
                        const int to = nf + rank_below(m);
                        nf += __builtin_popcountll(m);
                        if (nf > kFrontier) { over = true; break; }
                        if (front) {
                            fw[to] = (uint32_t)lo | (uint32_t)hi << 14 | (uint32_t)others << 28;
                            fc[to] = e & ~(uint32_t)kNoRecv;
                        }
                    }
                    if (open) r = lo;
                    const bool points = in && (!open || (hi < 0 && lo != INT32_MAX));
                    const uint64_t m = __ballot(points && lead);
                    if (!m) continue;
                    if (points && lead) {
                        st.put(y, kPoints | r);
                        const int at = nl + rank_below(m);
                        lr[at] = (uint32_t)r | (uint32_t)min(c.x, 3) << 14;
                        l0[at] = c.x > 2 ? c.y : c.z;
                        l1[at] = c.x > 2 ? c.x : c.w;
                    }
                    nl += __builtin_popcountll(m);
                    if (!points) z = z1 = kFrontierFill | kFrontierLast;
                    for (int o = more.y + 4;; o += 8) {
                        bool act = !(z & kFrontierFill), act1 = !(z1 & kFrontierFill);
                        uint32_t old = 0, old1 = 0;
                        if (!(z & (kFrontierFill | kFrontierOnly))) old = lower<LS>(counters, n8, z);
                        if (!(z1 & (kFrontierFill | kFrontierOnly))) old1 = lower<LS>(counters, n8, z1);
                        const bool last = (z1 & kFrontierLast) != 0u;
                        uint32_t next = kFrontierFill | kFrontierLast, next1 = next;
                        if (!last) next = rare()->outputs[o + j];
                        if (!last && !(next & kFrontierLast)) next1 = rare()->outputs[o + 4 + j];
                        if (!(z & kFrontierOnly)) act = act && lowered(z, old);
                        if (!(z1 & kFrontierOnly)) act1 = act1 && lowered(z1, old1);
                        if (__ballot(act)) {
                            uint32_t of = z & 0x3ffffu;
                            if (act && (z & kFrontierWide)) of = (uint32_t)rare()->wide[of];
                            push(act, of << 14 | kNoRecv);
                        }
                        if (__ballot(act1)) {
                            uint32_t of = z1 & 0x3ffffu;
                            if (act1 && (z1 & kFrontierWide)) of = (uint32_t)rare()->wide[of];
                            push(act1, of << 14 | kNoRecv);
                        }
                        if (!__ballot(!last)) break;
                        z = next;
                        z1 = next1;
                    }
                } else {
                    // P of the recvs that the logged classes point at
                    for (int base = 0; base < nl; base += 64) {
                        const bool in = base + lane < nl;
                        int r = -1;
                        double ct = 0.0, t = 0.0;
                        if (in) {
                            const uint32_t e = lr[base + lane];
                            const int c0 = l0[base + lane], c1 = l1[base + lane];
                            r = (int)(e & kNoRecv);
                            const int n = (int)(e >> 14);
                            t = (double)*at(rt, (uint32_t)r);
                            if (n < 3) {
                                ct = (double)*at(ot, (uint32_t)c0);
                                if (n > 1) ct += (double)*at(ot, (uint32_t)c1);
                            } else {
                                // (four columns at a time, in ascending order)
                                const int32_t *cols = rare()->cls_cols;
                                for (int k = 0; k < c1; k += 4) {
                                    double x[4];
#pragma unroll
                                    for (int i = 0; i < 4; ++i) x[i] = k + i < c1 ? (double)*at(ot, (uint32_t)*at(cols, (uint32_t)(c0 + k + i))) : 0.0;
#pragma unroll
                                    for (int i = 0; i < 4; ++i) ct += x[i];
                                }
                            }
                        }
                        int pos = 0;
                        const bool some = in && !(ct <= 0.0);
                        uint64_t left = __ballot(some);
                        while (left) {
                            const int l = __builtin_ctzll(left);
                            const int r0 = __builtin_amdgcn_readlane(r, l);
                            const bool same = r == r0;
                            left &= ~__ballot(same);
                            uint64_t has = __ballot(ra == r0);
                            int k = 0;
                            if (!has) {
                                has = __ballot(rb == r0);
                                k = 64;
                            }
                            if (!has) {
                                const double t0 = readlane_f64(t, l);
                                has = __ballot(ra < 0);
                                k = 0;
                                if (has) {
                                    if (lane == (int)__builtin_ctzll(has)) { ra = r0; ta = t0; P[lane] = 0.0; }
                                } else {
                                    has = __ballot(rb < 0);
                                    k = 64;
                                    if (!has) { over = true; break; }
                                    if (lane == (int)__builtin_ctzll(has)) { rb = r0; tb = t0; P[64 + lane] = 0.0; }
                                }
                            }
                            k += __builtin_ctzll(has);
                            if (same) pos = k;
                        }
                        wave_sync();
                        // (the lanes of a wave are served in their order)
                        if (some) atomicAdd(&P[pos], ct);
                    }
                    nl = 0;
                }
            }
        }
        if (lane == 0) {
            Arg *q = rare();
            q->flags[b] = over ? 2 : 0;
            if (q->simulate && !over) {
                busy += busy_lo;
                F += F_lo;
                sum_c += sum_lo;
                const double m = max_f64(busy, F), U = sum_c + F, L = max_f64(sum_c, F);
                if (q->makespan) q->makespan[b] = m;
                if (q->eff) q->eff[b] = (U == L) ? 1.0 : (U - m) / (U - L);
                if (q->U) q->U[b] = U;
                if (q->L) q->L[b] = L;
                if (q->S) q->S[b] = (U == L || L == 0.0) ? 0.0 : (U - L) / L;
            }
        }
    }
}

template <typename T, bool LS>
static hipError_t launch_frontier_t(const FrontierParams &p, int grid, size_t lds, hipStream_t s)
{
    const void *k = reinterpret_cast<const void *>(tac_frontier_kernel<T, LS>);
    if (lds > 48 * 1024) {
        const hipError_t e = ensure_dynamic_lds(k, lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((tac_frontier_kernel<T, LS>), dim3(grid), dim3(64), lds, s, p);
    return hipGetLastError();
}

hipError_t launch_tac_frontier(Dag &d, const TacArgs &a, size_t flag_bytes, size_t at_least, int32_t **flags_out, hipStream_t s)
{
    const FrontierTables &f = d.frontier;
    if (!f.ok || a.sel_P || a.sel_Mplus) return hipErrorNotSupported;
    FrontierParams p{};
    p.B = a.B; p.R = d.R; p.W = d.W; p.C = d.C; p.N = d.N;
    p.row = f.d_row; p.inputs = f.d_inputs; p.outputs = f.d_outputs; p.wide = f.d_wide;
    p.counters = f.d_counters; p.n_counters = f.n_counters;
    p.roots = f.d_roots; p.free_cols = f.d_free_cols; p.own_ptr = f.d_own_ptr; p.own = f.d_own;
    p.n_roots = f.n_roots; p.n_free = f.n_free;
    p.cls_cols = d.d_cls_cols; p.cls_dep = d.d_cls_dep;
    p.op_time = a.op_time; p.recv_time = a.recv_time;
    p.order = a.order; p.rank = a.rank; p.simulate = a.simulate ? 1 : 0;
    p.makespan = a.makespan; p.eff = a.eff; p.U = a.U; p.L = a.L; p.S = a.S;

    const size_t state = (size_t)p.n_counters * 4 + ((size_t)d.C + 7) / 8 * 16;
    const bool ls = state <= 4096;
    const size_t lds = 1024 + ((size_t)kStack + 2 * kFrontier + 3 * kLog) * 4 + (size_t)(d.R + 128) / 128 * 16 + (ls ? state : 0);
    if (lds > 150 * 1024) return hipErrorNotSupported;
    const int per_cu = std::min((int)(160 * 1024 / lds), 32);
    const int grid = std::min(a.B, per_cu * device_cu_count(d.device));
    p.scratch_stride = ls ? 0 : (state + 255) & ~(size_t)255;
    const size_t room = std::max(at_least, flag_bytes + p.scratch_stride * grid);
    if (room > d.work_bytes && being_captured(s)) return hipErrorNotSupported;      // (the caller has forms that may do with less)
    const hipError_t e = ensure_workspace(&d, room);
    if (e != hipSuccess) return e;
    p.flags = static_cast<int32_t *>(d.d_work);
    p.scratch = static_cast<char *>(d.d_work) + flag_bytes;
    *flags_out = p.flags;
    if (a.f32) return ls ? launch_frontier_t<float, true>(p, grid, lds, s) : launch_frontier_t<float, false>(p, grid, lds, s);
    return ls ? launch_frontier_t<double, true>(p, grid, lds, s) : launch_frontier_t<double, false>(p, grid, lds, s);
}

}  // namespace tictac
