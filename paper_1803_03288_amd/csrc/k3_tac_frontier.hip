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
// So a sample costs one visit per edge of the class graph instead of R rounds over all classes: on stress, 60 567 classes and
// 4 096 recvs, 193 000 edges against 1.7 * 10^8 set bits.  The frontier has 40 members on average and 150 at most there, Q (the
// recvs with P > 0) 23 and 79, so one wave keeps both in LDS.  The states of the classes (16 bits each) are in memory, and so are the
// numbers of their open inputs (4 bits) but for those of 4 096 classes, which move on with the highest class that has been told of an
// input: classes are numbered along the graph (frontier_plan.h), and what a sample is busy with are a few thousand of them, whose numbers come from the graph when the window reaches them and go to memory
// when it leaves them.  So sixteen samples share a compute unit.
//   A round is a chain of 2.3 goes at up to sixteen classes each.  4 096 samples of stress, cycles per round and wave, sixteen waves
// to a compute unit (all but a tenth of it also while a wave is by itself): the rows of the classes 3 500, the states of their inputs 2 600,
// putting down those that point 1 400, their outputs' counters and the next classes 3 600, and, when all is done, times and P of what points 4 300;
// the selection before 2 800, the frontier 700.  48 GB are fetched: 16 GB of them for the times (with all times read
// from 512 columns 32 GB are left, and the launch takes 38.8 ms instead of 39.1), the rest for what the L2 does not hold of the states and for the
// rows and counters of the classes.  46.1 -> 38.6 ms by the following, each by itself 3 to 8 %: the counters
// in LDS (a trip to the L2 per go; 25.8 GB written -> 8.6); a class's row in one request, sixteen bytes to a lane, with eight inputs, so
// that more than four are no further trip; the sums of the iteration 64 steps at a time, over the lanes; loads and LDS operations by all lanes
// instead of behind branches (640 vector and 370 scalar instructions a round, 800 and 560 before).  Not faster: times
// requested in the go that finds the class (memory operations of a wave come back in order, so the next rows wait for them), times past
// the L2, the selection by the high words of the times with fewer instructions, rare branches out of line.  Sixteen-bit counters beside the states had
// taken 65 ms to 49, and all counters in LDS leave room for seven samples per compute unit.
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
constexpr int kStack = kFrontierMaxStack, kFrontier = kFrontierMaxFrontier, kLog = 127;      // entries of the lists of a wave (and one for lanes that have none)
constexpr int kWindow = kFrontierWindow, kSlide = 256;     // classes whose counters are in LDS, and by how many they move on
constexpr int kPoints = 0x8000;             // state of a class that points: kPoints | recv; of another: 0

struct FrontierParams {
    int32_t B, R, W, C, N;
    const uint32_t *table;          // FrontierTable: [C][16], then the further outputs
    const int32_t *inputs, *roots, *free_cols, *own_ptr, *own;
    const uint32_t *counters;
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

// inclusive prefix sums over the lanes, with what was rounded off beside them
__device__ __forceinline__ void scan_exact(double &v, double &lo)
{
    const auto add = [&](double w, double w_lo) {
        lo += w_lo;
        v = add_exact(v, w, lo);
    };
    add(dpp0_f64<0x111>(v), dpp0_f64<0x111>(lo));
    add(dpp0_f64<0x112>(v), dpp0_f64<0x112>(lo));
    add(dpp0_f64<0x114>(v), dpp0_f64<0x114>(lo));
    add(dpp0_f64<0x118>(v), dpp0_f64<0x118>(lo));
    add(dpp_f64<0x142, 0xa>(0.0, v), dpp_f64<0x142, 0xa>(0.0, lo));
    add(dpp_f64<0x143, 0xc>(0.0, v), dpp_f64<0x143, 0xc>(0.0, lo));
}

// States of the classes of one sample, 16 bits each, in LDS or in memory: kPoints | recv, or 0.  Only the wave itself reads and
// writes them.  A get of what another lane has put needs no wait: the vector memory operations of a wave reach the L1 of its compute unit in
// the order in which they are issued, so what orders the two at the scope of a wavefront (wave_sync(), which lies between any put and the gets of
// the next go, and which the compiler moves neither across) is enough.
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
// One sample as the rare parts below see it.  They are functions of their own, so that the code of a round stays together.
template <typename T>
struct Sample {
    const T *rt;
    const uint32_t *alive, *fw, *fc;
    uint32_t *list;                 // the stack, which is empty then 
    const uint16_t *st;
    const int32_t *row, *inputs;        // (row: the table)
    const uint64_t *cls_dep;
    int nf, C, W, R;
};

// an input in sixteen bits of class c
__device__ __forceinline__ int short_input(uint32_t x, int c) { return x < kInRecv ? c - (int)x : ~(int)(x - kInRecv); }
// input number k of class c, of 8 + 4 * (more % 32) (more: word 2 of its row)
template <typename T>
__device__ __forceinline__ int frontier_input(const Sample<T> &s, int c, int more, int k)
{
    if (k >= 8) return s.inputs[(more >> 5) * 4 + k - 8];
    return short_input((uint32_t)s.row[16 * c + 4 * (k & 3)] >> (k & 4) * 4 & 0xffffu, c);
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
        int low = INT32_MAX, n = 0, cls = 0, end = 0, more = 0;
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
            end = w >> 28 ? 1 : 0;
            int word[4] = {0, 0, 0, 0};                     // of the first eight
            if (end) {
#pragma unroll
                for (int j = 0; j < 4; ++j) word[j] = s.row[16 * cls + 4 * j];
                more = s.row[16 * cls + 2];
                const bool five = (uint32_t)word[0] >> 16 != kInRecv + (uint32_t)s.R;
                end = more & 31 ? 8 + 4 * (more & 31) : five ? 8 : 4;
            }
            for (int i = 0; __ballot(i < end); i += 4) {
                if (i < end) {
                    int u[4];
                    if (i < 8) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) u[j] = short_input((uint32_t)word[j] >> 4 * i & 0xffffu, cls);
                    } else {
                        const int4 u4 = *reinterpret_cast<const int4 *>(s.inputs + (more >> 5) * 4 + i - 8);
                        u[0] = u4.x; u[1] = u4.y; u[2] = u4.z; u[3] = u4.w;
                    }
                    // (requests one after the other, not each behind a branch)
                    int x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = s.st[max(u[j], 0)];
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = u[j] < 0 ? ~u[j] : x[j] & kNoRecv;
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
                double t[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) t[k] = (double)s.rt[q[k] == INT32_MAX ? 0 : q[k]];
                M = 0.0;
#pragma unroll
                for (int k = 0; k < 8; ++k) M += q[k] == INT32_MAX ? 0.0 : t[k];
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
__device__ __forceinline__ double frontier_M_plus(const Sample<T> s, const int32_t *wide, const int32_t *own_ptr,
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
                uint32_t z = kOutFill | kOutLast;
                int o = 0;
                if (i0 < 0) {
                    const int k = o1 + i0 + lane;
                    if (k >= o0 && k < o1) z = (uint32_t)own[k] << 2 | kOutLast;
                } else if (base + (lane >> 2) < ns) {
                    const int32_t *row = s.row + 16 * s.list[base + (lane >> 2)];
                    z = (uint32_t)row[4 * (lane & 3) + 1];
                    o = row[6] >> 2;
                }
                for (;; o += 4) {
                    int y = z & kOutFill ? -1 : z & kOutWide ? wide[(z & kOutClass) >> 2] : (int)((z & kOutClass) >> 2);
                    bool ok = y >= 0 && s.st[y < 0 ? 0 : y] == 0;
                    // it does not count if an input has two outstanding recvs or more of which r is one: M of that is no larger
                    if (ok) {
                        const int more = s.row[16 * y + 2];
                        for (int k = 0; k < 8 + 4 * (more & 31) && ok; ++k) {
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
                    if (!__ballot(!(z & kOutLast))) break;
                    z = z & kOutLast ? kOutFill | kOutLast : (uint32_t)s.row[o + (lane & 3)];
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
__global__ void __launch_bounds__(64, 4)
tac_frontier_kernel(const FrontierParams p)
{
    extern __shared__ uint32_t smem[];
    const int lane = threadIdx.x, j = lane & 3;
    const int R = p.R;
    const int n_alive = (R + 128) / 128 * 4, n8 = (p.C + 7) / 8;

    double *P = reinterpret_cast<double *>(smem);                   // [128] of the members of Q
    uint32_t *stk = smem + 256;                                     // [kStack] classes to be looked at: class << 14 | the recv it points at, kNoRecv: not known
    uint32_t *fw = stk + kStack + 4;                                    // [kFrontier] two outstanding recvs (14 bits each), bit 28: it has more
    uint32_t *fc = fw + kFrontier + 2;                                  // [kFrontier] the class << 14
    uint32_t *lr = fc + kFrontier + 2;                                  // [kLog + 1] of classes that point: recv, bit 14: more than two columns
    int32_t *l0 = reinterpret_cast<int32_t *>(lr + kLog + 1);           // its first two columns (more than two: where they are, their number)
    int32_t *l1 = l0 + kLog + 1;
    uint32_t *alive = reinterpret_cast<uint32_t *>(l1 + kLog + 1);      // [n_alive] outstanding recvs (bit R: none)
    // The counters of classes base .. base + kWindow - 1 are in LDS, those of class c at c mod kWindow; below they are in memory, above
    // they are what they were at the start.
    uint32_t *win = alive + n_alive;                                // LS: of all classes
    uint32_t *counters = LS ? win : reinterpret_cast<uint32_t *>(p.scratch + (size_t)blockIdx.x * p.scratch_stride);
    States<LS> st;
    st.p = reinterpret_cast<uint16_t *>(counters + p.n_counters);
    const int32_t *rows = reinterpret_cast<const int32_t *>(p.table);
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
        int base = 0;
        if (LS) {
            const uint4 *from = reinterpret_cast<const uint4 *>(rare()->counters);
            const int n = rare()->n_counters / 4;
            for (int i = lane; i < n; i += 64) reinterpret_cast<uint4 *>(counters)[i] = from[i];
        } else {
            const uint32_t *from = rare()->counters;
            for (int i = lane; i < min(kWindow / 8, (n8 + 3) / 4 * 4); i += 64) win[i] = i < n8 ? from[i] : 0u;
            for (int i = n8 + lane; i < rare()->n_counters; i += 64) counters[i] = from[i];
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
        // (What is uniform is said to be: the compiler takes a loop whose conditions it cannot see to be for one that lanes leave one by one.)
        int nf = 0, ns = 0, nl = 0;                         // entries of frontier, stack, log
        int over = 0;                                       // a list was too short
        // (sums with what was rounded off beside them: one after the other, their error is otherwise twice that of a tree)
        double F = 0.0, busy = free_time, sum_c = free_time, F_lo = 0.0, busy_lo = 0.0, sum_lo = 0.0;
        // of the last 64 steps, by the lane of step mod 64: the recv, its Time, its P
        int mine = 0;
        double mine_t = 0.0, mine_P = 0.0;

        // moves the window on until classes up to c are in it or below
        const auto slide = [&](int c) {
            while (base + kWindow <= c) {
                wave_sync();
                const int w = base / 8 + (lane & (kSlide / 8 - 1)), next = w + kWindow / 8;
                const uint32_t x = rare()->counters[min(next, n8 - 1)];
                __hip_atomic_store(at(counters, (uint32_t)w), win[w & (kWindow / 8 - 1)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                win[w & (kWindow / 8 - 1)] = next < n8 ? x : 0u;
                base = uniform_i32(base + kSlide);
                wave_sync();
            }
        };
        // (Lanes that have nothing for a list write behind its end: a branch less, and no join at which the compiler would take what
        // is uniform for what lanes have of their own.)
        const auto push = [&](bool in, uint32_t v) {
            const uint64_t m = __ballot(in);
            stk[in ? min(ns + rank_below(m), kStack) : kStack] = v;
            ns = uniform_i32(ns + __builtin_popcountll(m));
            over |= ns > kStack;
            ns = min(ns, kStack);
        };

        // (before the first round: the classes that depend on recvs directly, 64 at a time)
        for (int step = -((rare()->n_roots + 63) / 64); uniform_i32(step < R && !over); ++step) {
            wave_sync();
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
                    const Sample<T> sample = {rt, alive, fw, fc, stk, st.p, rows, rare()->inputs, rare()->cls_dep, nf, rare()->C, rare()->W, R};
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
                        const Sample<T> sample = {rt, alive, fw, fc, stk, st.p, rows, rare()->inputs, rare()->cls_dep, nf, rare()->C, rare()->W, R};
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
                                        const double m = frontier_M_plus(sample, rare()->wide, rare()->own_ptr,
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
                {
                    const bool is = (step & 63) == lane;
                    mine = is ? best : mine;
                    mine_t = is ? ts : mine_t;
                    mine_P = is ? Ps : mine_P;
                }
                if (uniform_i32((step & 63) == 63 || step == R - 1)) {
                    // the order, and the iteration by these steps: the device is busy until the last of them has begun as late as any F_k
                    // makes it, k of these, or from before on, and then for what follows
                    const int s = (step & ~63) + lane;
                    if (s <= step) {
                        rare()->order[(size_t)b * R + s] = mine;
                        if (int32_t *rank = rare()->rank) rank[(size_t)b * R + mine] = s;
                    } else {
                        mine_t = mine_P = 0.0;
                    }
                    double t = mine_t, t_lo = 0.0, q = mine_P, q_lo = 0.0;
                    scan_exact(t, t_lo);
                    scan_exact(q, q_lo);
                    // F_k less the P before it
                    double d_lo = t_lo - q_lo, d = add_exact(t, -q, d_lo);
                    d = add_exact(d, mine_P, d_lo);
                    const double high = d + d_lo;
                    d_lo -= high - d;
                    d = wave_max_f64_dpp(s <= step ? high : -TT_INF);
                    d_lo = wave_max_f64_dpp(s <= step && high == d ? d_lo : -TT_INF);
                    const double all = lane63_f64(q), all_lo = lane63_f64(q_lo);
                    double w_lo = F_lo + d_lo;
                    const double w = add_exact(F, d, w_lo);
                    if ((w - busy) + (w_lo - busy_lo) > 0.0) { busy = w; busy_lo = w_lo; }
                    busy_lo += all_lo;
                    busy = add_exact(busy, all, busy_lo);
                    sum_lo += all_lo;
                    sum_c = add_exact(sum_c, all, sum_lo);
                    F_lo += lane63_f64(t_lo);
                    F = add_exact(F, lane63_f64(t), F_lo);
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
                    const int at = in && !hit ? kept + rank_below(stay) : kFrontier;
                    fw[at] = w;
                    fc[at] = c;
                    kept += __builtin_popcountll(stay);
                }
                nf = kept;
            }

            // ================= what follows from it =================
            for (;;) {
                while (uniform_i32(ns > 0 && nl + 16 <= kLog && !over)) {
                    wave_sync();
                    // The classes on the stack, sixteen at a time, four lanes each: a class all of whose inputs point either points as
                    // well, and tells its outputs, or joins the frontier.  (Loads and LDS operations are made by all lanes, of something in range where
                    // a lane has nothing to do: a branch round each costs as much as ten instructions, and what is under way behind one is
                    // waited for.)
                    const int k = min(ns, 16);
                    ns = uniform_i32(ns - k);
                    const bool in = lane < 4 * k, lead = in && j == 0;
                    uint32_t e = stk[ns + (lane >> 2)];     // (the frontier follows the stack)
                    e = in ? e : 0u;
                    const uint32_t y = e >> 14;
                    int r = (int)(e & kNoRecv);
                    const bool open = in && r == kNoRecv;
                    const uint32_t row_at = y * 64u + (uint32_t)j * 16u;
                    const int4 row = *reinterpret_cast<const int4 *>(reinterpret_cast<const char *>(rows) + row_at);
                    const uint32_t rest = (uint32_t)quad_perm<0x55>(row.z) + 4u * (uint32_t)j;
                    const int n_cols = quad_perm<0xaa>(row.z);
                    uint32_t z = (uint32_t)row.y;
                    // the outputs after the first four, so that both fours are told in one go
                    uint32_t z1 = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(rows) + (z & kOutLast ? row_at + 4u : rest));
                    // the least and the greatest outstanding recv among the inputs, and whether there are others
                    const auto outstanding = [&](int x) -> bool { return (alive[x >> 5] >> (x & 31)) & 1u; };
                    const auto recv_of = [&](int v, int state) { return v < 0 ? ~v : state & kNoRecv; };
                    const uint32_t fifth = (uint32_t)row.x >> 16;
                    const int v = open ? short_input((uint32_t)row.x & 0xffffu, (int)y) : ~R;
                    const bool many = __ballot(open && fifth != kInRecv + (uint32_t)R) != 0ull;
                    const int state = st.get(max(v, 0));
                    int w = ~R, state_w = 0;
                    if (many) {                             // (both requests before either is waited for)
                        w = open ? short_input(fifth, (int)y) : ~R;
                        state_w = st.get(max(w, 0));
                    }
                    int x = recv_of(v, state);
                    const bool al = outstanding(x);
                    int lo = al ? x : INT32_MAX, hi = al ? x : -1;
                    int others;
                    if (many) {
                        w = recv_of(w, state_w);
                        const bool bl = outstanding(w);
                        lo = quad_min(min(lo, bl ? w : INT32_MAX));
                        hi = quad_max(max(hi, bl ? w : -1));
                        others = (int)(al & (x != lo) & (x != hi)) | (int)(bl & (w != lo) & (w != hi));
                    } else {
                        lo = quad_min(lo);
                        hi = quad_max(hi);
                        others = (int)(al & (x != lo) & (x != hi));
                    }
                    if (__ballot(open && j == 0 && (row.z & 31))) {
                        const int more = quad_perm<0>(row.z);
                        int n = open ? more & 31 : 0, from = (more >> 5) * 4 + j;
                        while (__ballot(n > 0)) {
                            const int u = n > 0 ? rare()->inputs[from] : ~R;
                            x = recv_of(u, st.get(max(u, 0)));
                            const bool al = outstanding(x);
                            const int lo1 = min(lo, quad_min(al ? x : INT32_MAX)), hi1 = max(hi, quad_max(al ? x : -1));
                            others |= (al && x != lo1 && x != hi1) || (hi >= 0 && ((lo != lo1 && lo != hi1) || (hi != hi1 && hi != lo1)));
                            lo = lo1;
                            hi = hi1;
                            --n;
                            from += 4;
                        }
                    }
                    const bool front = lead & open & (lo < hi);
                    if (const uint64_t m = __ballot(front)) {
                        others = quad_max(others);
                        const int to = nf + rank_below(m);
                        nf = uniform_i32(nf + __builtin_popcountll(m));
                        over |= nf > kFrontier;
                        nf = min(nf, kFrontier);
                        const int at = front ? min(to, kFrontier) : kFrontier;
                        fw[at] = (uint32_t)lo | (uint32_t)hi << 14 | (uint32_t)others << 28;
                        fc[at] = e & ~(uint32_t)kNoRecv;
                    }
                    r = open ? lo : r;
                    const bool points = in & (!open | (lo == hi));
                    const uint64_t m = __ballot(points && j == 0);
                    if (!m) continue;
                    {
                        const bool two = n_cols <= 2;
                        const int second = quad_perm<0x55>(row.w), list = quad_perm<0xaa>(row.w);
                        const int place = nl + rank_below(m), at = points && j == 0 ? place : kLog;
                        lr[at] = (uint32_t)r | (two ? 0u : 1u << 14);
                        l0[at] = two ? row.w : list;
                        l1[at] = two ? second | (int)(n_cols > 1 ? 0x80000000u : 0u) : n_cols;
                        if (points && j == 0) st.put((int)y, kPoints | r);
                    }
                    nl = uniform_i32(nl + __builtin_popcountll(m));
                    z1 = z & kOutLast ? kOutFill | kOutLast : z1;
                    z = points ? z : kOutFill | kOutLast;
                    z1 = points ? z1 : kOutFill | kOutLast;
                    for (uint32_t o = rest + 16u;; o += 32u) {
                        // One less in the counters of the outputs, unless it is their only input; the words before.  (A counter is lowered only while
                        // it is positive: the others of the word are not touched.)
                        constexpr uint32_t kinds = kOutFill | kOutOnly | kOutWide;
                        const bool on = !(z & kinds), on1 = !(z1 & kinds);
                        uint32_t old, old1;
                        if (LS) {
                            old = atomicSub(counters + ((z & kOutClass) >> 5), on ? 1u << (z & 31u) : 0u);
                            old1 = atomicSub(counters + ((z1 & kOutClass) >> 5), on1 ? 1u << (z1 & 31u) : 0u);
                        } else {
                            const uint32_t top = max(z & kOutClass, z1 & kOutClass);
                            if (__ballot(top >= (uint32_t)(base + kWindow) * 4u)) {
                                slide(wave_max_i32_dpp((int)(top >> 2)));
                                base = uniform_i32(base);
                            }
                            const uint32_t low = (uint32_t)base * 4u;
                            const bool near = on & ((z & kOutClass) >= low), near1 = on1 & ((z1 & kOutClass) >= low);
                            old = atomicSub(win + ((z >> 5) & (kWindow / 8 - 1)), near ? 1u << (z & 31u) : 0u);
                            old1 = atomicSub(win + ((z1 >> 5) & (kWindow / 8 - 1)), near1 ? 1u << (z1 & 31u) : 0u);
                            if (__ballot((on & !near) | (on1 & !near1))) {
                                const auto lower = [&](uint32_t z) {
                                    return __hip_atomic_fetch_sub(at(counters, (z & kOutClass) >> 5), 1u << (z & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                };
                                if (on && !near) old = lower(z);
                                if (on1 && !near1) old1 = lower(z1);
                                __builtin_amdgcn_s_waitcnt(0xf70);          // (here, and not where the two ways meet)
                            }
                        }
                        // those for which it was the last are looked at next
                        // (without short cuts: each would be a branch)
                        bool act = (on & (((old >> (z & 31u)) & 15u) == 1u)) | ((z & kinds) == kOutOnly);
                        bool act1 = (on1 & (((old1 >> (z1 & 31u)) & 15u) == 1u)) | ((z1 & kinds) == kOutOnly);
                        uint32_t of = (z & kOutClass) << 12 | kNoRecv, of1 = (z1 & kOutClass) << 12 | kNoRecv;
                        if (__ballot((z | z1) & kOutWide)) {
                            const auto lower = [&](uint32_t z, bool &act, uint32_t &of) {
                                if (!(z & kOutWide)) return;
                                const uint32_t i = (z & kOutClass) >> 2, w = (uint32_t)n8 + i;
                                const uint32_t before = LS ? atomicSub(counters + w, 1u)
                                                           : __hip_atomic_fetch_sub(at(counters, w), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                act = before == 1u;
                                of = (uint32_t)rare()->wide[i] << 14 | kNoRecv;
                            };
                            lower(z, act, of);
                            lower(z1, act1, of1);
                            __builtin_amdgcn_s_waitcnt(0xf70);
                        }
                        const bool go_on = __ballot(!(z1 & kOutLast)) != 0ull;
                        uint32_t next = kOutFill | kOutLast, next1 = next;
                        if (go_on) {
                            const bool more = !(z1 & kOutLast);
                            next = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(rows) + (more ? o : row_at));
                            next = more ? next : kOutFill | kOutLast;
                            const bool more1 = !(next & kOutLast);
                            next1 = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(rows) + (more1 ? o + 16u : row_at));
                            next1 = more1 ? next1 : kOutFill | kOutLast;
                        }
                        const uint64_t m0 = __ballot(act), m1 = __ballot(act1);
                        if (m0 | m1) {
                            const int n0 = ns + __builtin_popcountll(m0);
                            const int k0 = min(ns + rank_below(m0), kStack), k1 = min(n0 + rank_below(m1), kStack);
                            stk[act ? k0 : kStack] = of;
                            stk[act1 ? k1 : kStack] = of1;
                            ns = uniform_i32(n0 + __builtin_popcountll(m1));
                            over |= ns > kStack;
                            ns = min(ns, kStack);
                        }
                        if (!go_on) break;
                        z = next;
                        z1 = next1;
                    }
                }
                // P of the recvs that the logged classes point at
                wave_sync();
                for (int first = 0; uniform_i32(first < nl && !over); first += 64) {
                    const bool in = first + lane < nl;
                    const int i = in ? first + lane : kLog;
                    const uint32_t e = in ? lr[i] : 0u;
                    const int c0 = l0[i], c1 = l1[i];
                    const int r = in ? (int)(e & kNoRecv) : -1;
                    const bool listed = (e >> 14) != 0u;
                    const double t = (double)*at(rt, in ? (uint32_t)r : 0u);
                    double ct = (double)*at(ot, in && !listed ? (uint32_t)c0 : 0u);
                    const double second = (double)*at(ot, in && !listed ? (uint32_t)c1 & 0x7fffffffu : 0u);
                    __builtin_amdgcn_s_waitcnt(0xf70);      // (all three now: what is left under way would be waited for in the rounds)
                    ct = c1 < 0 ? ct + second : ct;
                    if (__ballot(e >> 14)) {
                        // more than two columns: four at a time, in ascending order
                        const int32_t *cols = rare()->cls_cols;
                        const int n = e >> 14 ? c1 : 0;
                        ct = n ? 0.0 : ct;
                        for (int k = 0; __ballot(k < n); k += 4) {
                            double x[4];
#pragma unroll
                            for (int i = 0; i < 4; ++i) x[i] = k + i < n ? (double)*at(ot, (uint32_t)*at(cols, (uint32_t)(c0 + k + i))) : 0.0;
#pragma unroll
                            for (int i = 0; i < 4; ++i) ct += x[i];
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
                        uint64_t ma = __ballot(ra == r0), mb = __ballot(rb == r0);
                        if (!(ma | mb)) {
                            // a new member of Q (there is no room for it: the sample is given up)
                            const double t0 = readlane_f64(t, l);
                            const uint64_t ea = __ballot(ra < 0), eb = __ballot(rb < 0);
                            over |= !(ea | eb);
                            const int k = ea ? (int)__builtin_ctzll(ea) : (int)__builtin_ctzll(eb | 1ull << 63);
                            const bool to_a = lane == k && ea != 0ull, to_b = lane == k && ea == 0ull;
                            ra = to_a ? r0 : ra;
                            ta = to_a ? t0 : ta;
                            rb = to_b ? r0 : rb;
                            tb = to_b ? t0 : tb;
                            ma = ea ? 1ull << k : 0ull;
                            mb = ea ? 0ull : 1ull << k;
                            P[ea ? k : 64 + k] = 0.0;
                        }
                        pos = same ? (ma ? (int)__builtin_ctzll(ma) : 64 + (int)__builtin_ctzll(mb)) : pos;
                    }
                    wave_sync();
                    // (the lanes of a wave are served in their order)
                    if (some) atomicAdd(&P[pos], ct);
                }
                nl = 0;
                if (uniform_i32(ns <= 0 || over)) break;
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

// rows of W words, row k of `to` from row from_row[k]
__global__ void __launch_bounds__(256)
frontier_rows_kernel(size_t words, int32_t W, const int32_t *__restrict__ from_row, const uint64_t *__restrict__ from, uint64_t *__restrict__ to)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < words) to[i] = from[(size_t)from_row[i / W] * W + i % W];
}

hipError_t launch_frontier_rows(const Dag &d, hipStream_t s)
{
    const size_t words = (size_t)d.C * d.W;
    hipLaunchKernelGGL(frontier_rows_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, words, d.W, d.frontier.d_cls_of,
                       d.d_cls_dep, d.frontier.d_cls_dep);
    return hipGetLastError();
}

hipError_t launch_tac_frontier(Dag &d, const TacArgs &a, size_t flag_bytes, size_t at_least, int32_t **flags_out, hipStream_t s)
{
    const FrontierTables &f = d.frontier;
    if (!f.ok || a.sel_P || a.sel_Mplus) return hipErrorNotSupported;
    FrontierParams p{};
    p.B = a.B; p.R = d.R; p.W = d.W; p.C = d.C; p.N = d.N;
    p.table = f.d_table; p.inputs = f.d_inputs; p.wide = f.d_wide;
    p.counters = f.d_counters; p.n_counters = f.n_counters;
    p.roots = f.d_roots; p.free_cols = f.d_free_cols; p.own_ptr = f.d_own_ptr; p.own = f.d_own;
    p.n_roots = f.n_roots; p.n_free = f.n_free;
    p.cls_cols = d.d_cls_cols; p.cls_dep = f.d_cls_dep ? f.d_cls_dep : d.d_cls_dep;
    p.op_time = a.op_time; p.recv_time = a.recv_time;
    p.order = a.order; p.rank = a.rank; p.simulate = a.simulate ? 1 : 0;
    p.makespan = a.makespan; p.eff = a.eff; p.U = a.U; p.L = a.L; p.S = a.S;

    const size_t state = (size_t)p.n_counters * 4 + ((size_t)d.C + 7) / 8 * 16;
    const bool ls = state <= 4096;
    const size_t lds = 1024 + ((size_t)kStack + 4 + 2 * (kFrontier + 2) + 3 * (kLog + 1)) * 4 + (size_t)(d.R + 128) / 128 * 16 + (ls ? state : std::min(kWindow / 2, (d.C + 31) / 32 * 16));
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
