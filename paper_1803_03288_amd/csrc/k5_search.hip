// Order search with the simulated iteration as its measure.  Finding the best transfer order is
// a job-shop problem and NP-hard (Sec. 3.1), and the comparator of TAC extends a two-recv rule by
// an induction that need not hold in general (Sec. 4.3); climbing from a heuristic order through
// proposed exchanges shows how far it is from a better one.
//
// Per timing sample:  cur = start order, m_cur = makespan(cur); for every move (a, b) in the
// order given: exchange positions a and b of cur, m = makespan of that order; keep the exchange
// when m < m_cur, else undo it.  A move with a == b or a position outside 0 .. R-1 is skipped.
//
// The makespan of an order is the one of the single-channel simulation: F_k = end of the k-th
// transfer (prefix sums over the order), kappa of a class = last position among the recvs of its
// row, A_k = class time released by transfer k, makespan = max_k (F_k + sum_{k' >= k} A_k').
//
// One wave per sample.  The op_time row is read once (class totals); after that a move touches
// registers and LDS only.  A lane owns consecutive classes (their totals and kappa) and consecutive
// positions of the order (the transfer time at that position), so that a sum over positions is a few
// adds per lane and one scan over the lanes, and classes that are released together (neighbours, mostly)
// are added up in the lane before they go to A.  A move changes
// kappa of few classes: when the recv at the earlier position (x) and the one at the later
// position (y) change places, a class with x in its row gets max(kappa, later position); a class
// with y and without x whose kappa was y's position needs its maximum taken again, for which the wave
// looks at 64 positions below at once; every other class keeps its kappa.  Which classes hold a recv is
// one word per slot of classes, in LDS, read by all lanes and used as a scalar.  A and the two scans
// are then formed afresh from the registers, so every makespan is the one a full evaluation of that
// order gives.
//
// Most moves are turned down without that evaluation.  Let k* be a position where the current
// makespan is attained, m_cur = F_k* + S_k* (S_k = class time with kappa >= k).  The makespan after
// the move is at least F'_k* + S'_k*.  Exchanging positions lo < hi leaves F_k and S_k as they are
// for k <= lo and for k > hi + 1, so a move with k* outside lo + 1 .. hi + 1 cannot help, nor does
// one that makes F_k* longer by as much as the classes released at hi + 1, which is the most that S_k*
// can lose (both decided for 64 moves at a time, one per lane; of 1 024 moves on resnet50 162 pass the
// first and 79 both).  Otherwise F_k* changes by Time(y) - Time(x) when k* <= hi, S_k* gains the
// classes with x whose kappa was below k* and loses at most the classes that need their maximum
// taken again; when that sum is not negative the move cannot help either (one wave sum, no LDS
// write).  Only the remaining moves, 63 there, are evaluated; 52 are kept.
//
// Bound by the issue of vector and scalar instructions, five or six waves per SIMD.  resnet50, 16 384 samples, 1 024 moves:
// 1 675 us with positions and classes l, l + 64, ... of a lane and without the second test (41 000 vector instructions per sample,
// 3.4 bank-conflict cycles per LDS instruction), 962 us now (24 000; 1.2).  inception3: 5.59 -> 3.04 ms.
#include <algorithm>

#include "device_utils.h"
#include "internal.h"

namespace tictac {

struct SearchParams {
    int32_t B, R, C, N, W, n_waves, wave_bytes, levels, n_moves, fa_len, rows_bytes;
    const int32_t *col_cls;     // [N] class of every op_time column
    const uint64_t *cls_depT;   // [W][Cpad] class rows, word by word
    int32_t Cpad;
    const int32_t *run_ptr;     // [C+1] runs [run_lo, run_hi) of consecutive recv indices of the class rows
    const int32_t *run_lo, *run_hi;
    const int32_t *order;       // start orders
    int32_t order_stride;
    const int32_t *moves;       // [n_moves][2]
    const double *op_time, *recv_time;
    int32_t *best_order;        // [B][R]
    double *best_makespan;      // [B]
    double *start_makespan;     // [B] or NULL
    int32_t *n_accepted;        // [B] or NULL
};

constexpr int kSearchWaves = 4;
constexpr int kWalk = 32;                // recvs that are tried first where rows have many runs

__device__ __forceinline__ uint64_t uniform_u64(uint64_t x)      // the same in every lane
{
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

#define OS_EACH_T(F) F(1) F(2) F(3) F(4) F(5) F(6) F(7) F(8)
#define OS_EACH(F) F(0) F(1) F(2) F(3) F(4) F(5) F(6) F(7)

// T slots per lane for classes (64 T >= C), and D of consecutive positions (64 D >= R)
template <int T, bool WALK>
__global__ void __launch_bounds__(64 * kSearchWaves)
order_search_kernel(const SearchParams p)
{
    extern __shared__ double smem[];
    constexpr int D = T | 1;                                    // (odd: what lanes read of their positions is in different banks)
    const int R = p.R, C = p.C, N = p.N, W = p.W;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t *holders = reinterpret_cast<uint64_t *>(smem);     // [R][T] the classes with recv r: bit l of word k for (k, l); shared
    char *mine = reinterpret_cast<char *>(smem) + p.rows_bytes + (size_t)wave * p.wave_bytes;
    double *t = reinterpret_cast<double *>(mine);           // [R]   Time(recv)
    double *A = t + R;                                      // [R+1] class time by kappa
    double *Acur = A + (R + 1);                             // [R+1] the same for the order kept
    double *csum = A;                                       // [64 T] class totals while they are summed
    uint16_t *pos = reinterpret_cast<uint16_t *>(A);        // [levels][R] level 0: 1-based position of every recv;
                                                            // level j: maxima over [i, min(i + 2^j, R)) (start order only)
    uint16_t *ordl = reinterpret_cast<uint16_t *>(t + R + p.fa_len);     // [R] the order being tried
    for (int i = wave; i < W * T; i += kSearchWaves) {
        const int w = i / T, k = i % T, c = lane * T + k;
        const uint64_t x = c < C ? p.cls_depT[(size_t)w * p.Cpad + c] : 0ull;
        for (int j = 0; j < 64 && w * 64 + j < R; ++j) {
            const uint64_t has = __ballot((x >> j) & 1ull);
            if (lane == 0) holders[(w * 64 + j) * T + k] = has;
        }
    }
    __syncthreads();

    const int gwave = blockIdx.x * kSearchWaves + wave;
    for (int b = gwave; b < p.B; b += p.n_waves) {
        const double *rt = p.recv_time + (size_t)b * R;
        const double *ot = p.op_time + (size_t)b * N;
        const int32_t *ord = p.order + (size_t)b * p.order_stride;
        wave_sync();                        // LDS of the previous sample is no longer read

        // ---- class totals ----
        for (int c = lane; c < 64 * T; c += 64) csum[c] = 0.0;
        wave_sync();
        class_totals(csum, ot, p.col_cls, N, lane);
        wave_sync();
#define OS_DECL(k) double ct_##k = 0.0; int kap_##k = 0, kn_##k = 0;
        OS_EACH(OS_DECL)
        double xs[D];                           // transfer times at the lane's positions
#define OS_TOTAL(k) if constexpr (k < T) { ct_##k = csum[lane * T + k]; }
        OS_EACH(OS_TOTAL)
        double ct_sum = 0.0;
#define OS_SUM(k) if constexpr (k < T) { ct_sum += ct_##k; }
        OS_EACH(OS_SUM)
        const double sum_c = wave_sum_f64_dpp(ct_sum);
        wave_sync();

        // ---- transfer times, start order, positions ----
        for (int r = lane; r < R; r += 64) {
            t[r] = rt[r];
            pos[r] = 0;
            const int o = ord[r];
            ordl[r] = (uint16_t)((unsigned)o < (unsigned)R ? o : 0);     // an invalid entry is never used as an index
        }
        wave_sync();
        for (int i = lane; i < R; i += 64) pos[ordl[i]] = (uint16_t)(i + 1);
#pragma unroll
        for (int k = 0; k < D; ++k) xs[k] = lane * D + k < R ? t[ordl[lane * D + k]] : 0.0;
        wave_sync();

        // ---- kappa of the start order: range maxima over the runs of every class row ----
        for (int j = 1; j < p.levels; ++j) {
            const uint16_t *prev = pos + (size_t)(j - 1) * R;
            uint16_t *cur = pos + (size_t)j * R;
            const int h = 1 << (j - 1);
            for (int i = lane; i < R; i += 64) cur[i] = max(prev[i], prev[min(i + h, R - 1)]);
            wave_sync();
        }
        // (rows of many runs: most hold one of the recvs that come last)
        if constexpr (WALK) {
            const int last = max(0, R - kWalk);
#pragma unroll 4
            for (int i = R - 1; i >= last; --i) {
                const uint64_t *has = holders + (size_t)ordl[i] * T;
#define OS_LATE(k) if constexpr (k < T) { if (kn_##k == 0 && (has[k] >> lane & 1ull)) kn_##k = i + 1; }
                OS_EACH(OS_LATE)
            }
        }
#define OS_KAPPA0(k)                                                                      \
        if constexpr (k < T) {                                                            \
            const int c = lane * T + k;                                                   \
            if (c < C && (!WALK || kn_##k == 0)) {                                        \
                const int rend = p.run_ptr[c + 1];                                        \
                int m = 0;                                                                \
                for (int q = p.run_ptr[c]; q < rend; ++q) {                               \
                    const int lo = p.run_lo[q], hi = p.run_hi[q];                         \
                    const int j = 31 - __builtin_clz(hi - lo);                            \
                    const uint16_t *lv = pos + (size_t)j * R;                             \
                    m = max(m, max((int)lv[lo], (int)lv[hi - (1 << j)]));                 \
                }                                                                         \
                kn_##k = m;                                                               \
            }                                                                             \
        }
        OS_EACH(OS_KAPPA0)
        wave_sync();                        // (A takes the place of the positions)

        double m_cur = 0.0;
        int n_acc = 0;
        int kstar = 0;                      // a position where the current makespan is attained
        // 64 moves at a time, one per lane: the moves that k* rules out are dropped by one ballot
        int base = -64;                     // first move of the chunk in mv_lo / mv_hi
        int mv_lo = 0, mv_hi = -1;          // lane i: the positions of move base + i; mv_hi < 0: not an exchange
        unsigned long long todo = 0;        // moves of the chunk that are still to be looked at
        // Which of the moves may help, as far as a lane sees it by itself: k* between their positions, and what F and S lose there
        // is more than what F gains (S loses no more than the classes released at the later position).
        const auto worth = [&]() {
            bool ok = mv_hi >= 0 && kstar > mv_lo && kstar <= mv_hi + 1;
            if (ok) ok = (kstar <= mv_hi ? t[ordl[mv_hi]] - t[ordl[mv_lo]] : 0.0) - Acur[mv_hi + 1] < 0.0;
            return __ballot(ok);
        };
        bool first = true;                  // the start order is evaluated before any move
        for (;;) {
            int lo = 0, hi = 0, x = 0, y = 0, cur = 0;
            if (!first) {
                while (todo == 0) {
                    base += 64;
                    if (base >= p.n_moves) break;
                    const int i = base + lane;
                    const int pa = i < p.n_moves ? p.moves[2 * i] : -1;
                    const int pb = i < p.n_moves ? p.moves[2 * i + 1] : -1;
                    const bool ok = (unsigned)pa < (unsigned)R && (unsigned)pb < (unsigned)R && pa != pb;
                    mv_lo = min(pa, pb);
                    mv_hi = ok ? max(pa, pb) : -1;
                    todo = worth();
                }
                if (todo == 0) break;       // no move left
                cur = __builtin_ctzll(todo);
                todo &= todo - 1;
                lo = __builtin_amdgcn_readlane(mv_lo, cur);
                hi = __builtin_amdgcn_readlane(mv_hi, cur);
                x = __builtin_amdgcn_readfirstlane((int)ordl[lo]);      // moves from lo to hi
                y = __builtin_amdgcn_readfirstlane((int)ordl[hi]);      // moves from hi to lo
                const double tx = t[x], ty = t[y];
                // which classes hold x, which hold y: the same words in every lane, so they go to scalar registers, as do
                // the sets of classes that are gained or may be lost
                double dsum = 0.0;          // change of S at k*: classes gained, classes that may be lost
                uint64_t moved = 0ull;
#define OS_HOLD(k)                                                                        \
                uint64_t hx_##k = 0ull, hy_##k = 0ull;                                    \
                if constexpr (k < T) { hx_##k = holders[x * T + k]; hy_##k = holders[y * T + k]; }
                OS_EACH(OS_HOLD)
#define OS_MEMBER(k)                                                                      \
                uint64_t redo_##k = 0ull;                                                 \
                if constexpr (k < T) {                                                    \
                    hx_##k = uniform_u64(hx_##k);                                         \
                    redo_##k = uniform_u64(hy_##k) & ~hx_##k & __ballot(kap_##k == hi + 1); \
                    const uint64_t gain = hx_##k & __ballot(kap_##k < kstar);             \
                    kn_##k = __builtin_amdgcn_inverse_ballot_w64(hx_##k) ? max(kap_##k, hi + 1) : kap_##k; \
                    dsum += __builtin_amdgcn_inverse_ballot_w64(gain) ? ct_##k : 0.0;     \
                    dsum -= __builtin_amdgcn_inverse_ballot_w64(redo_##k) ? ct_##k : 0.0; \
                    moved |= gain | redo_##k;                                             \
                }
                OS_EACH(OS_MEMBER)
                double d = kstar <= hi ? ty - tx : 0.0;
                if (moved != 0ull) d += wave_sum_f64_dpp(dsum);
                // (the comparison is the same in every lane; taking it from the first one tells the compiler so)
                if (__builtin_amdgcn_readfirstlane((int)(d >= 0.0))) continue;     // F'_k* + S'_k* >= m_cur: the move cannot help
                wave_sync();
                if (lane == 0) { ordl[lo] = (uint16_t)y; ordl[hi] = (uint16_t)x; }
                wave_sync();
                // Classes that lose their last recv: the highest position below hi with one of theirs, which is lo (where y
                // is now) at the latest.  64 positions at a time, one per lane, for all such classes of a slot.
#define OS_REDO(k)                                                                        \
                if constexpr (k < T) {                                                    \
                    for (int top = hi - 1; redo_##k != 0ull; top -= 64) {                 \
                        const int at = top - lane;                                        \
                        const uint64_t who = at >= lo ? holders[(int)ordl[at] * T + k] : 0ull; \
                        for (uint64_t left = redo_##k; left != 0ull; left &= left - 1ull) { \
                            const int l = __builtin_ctzll(left);                          \
                            const uint64_t found = __ballot((who >> l) & 1ull);           \
                            if (found != 0ull) {                                          \
                                kn_##k = lane == l ? top - (int)__builtin_ctzll(found) + 1 : kn_##k; \
                                redo_##k &= ~(1ull << l);                                 \
                            }                                                             \
                        }                                                                 \
                        if (top - 63 <= lo) break;      /* (an order with a recv missing) */ \
                    }                                                                     \
                }
                OS_EACH(OS_REDO)
                // the transfer times at the two positions change places
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    xs[k] = lane * D + k == lo ? ty : xs[k];
                    xs[k] = lane * D + k == hi ? tx : xs[k];
                }
            }

            // ---- A by kappa; F; suffix sums of A; makespan ----
            for (int j = lane; j <= R; j += 64) A[j] = 0.0;
            wave_sync();
            // (classes next to each other tend to be released together: those of a lane are added up first, since adds of several
            // lanes to one place are served one after the other)
            double together = ct_0;
#define OS_RELEASE(k)                                                                     \
            if constexpr (k > 0 && k < T) {                                               \
                if (kn_##k != OS_KN(k - 1)) {                                             \
                    atomicAdd(&A[OS_KN(k - 1)], together);                                \
                    together = 0.0;                                                       \
                }                                                                         \
                together += ct_##k;                                                       \
            }
#define OS_KN(k) ((k) == 0 ? kn_0 : (k) == 1 ? kn_1 : (k) == 2 ? kn_2 : (k) == 3 ? kn_3 : (k) == 4 ? kn_4 : (k) == 5 ? kn_5 : (k) == 6 ? kn_6 : kn_7)
            OS_EACH(OS_RELEASE)
            if (lane * T < C) atomicAdd(&A[OS_KN(T - 1)], together);    // (what the last lane has beyond C is nothing, at kappa 0)
            // prefix sums of the transfer times, suffix sums of the class times: over the lane's positions, then over the lanes
            double F[D], S[D];
            F[0] = xs[0];
#pragma unroll
            for (int k = 1; k < D; ++k) F[k] = F[k - 1] + xs[k];
            const double F_before = dpp0_f64<0x138>(wave_incl_scan_f64_dpp(F[D - 1]));
            wave_sync();
#pragma unroll
            for (int k = D - 1; k >= 0; --k) {
                S[k] = lane * D + k < R ? A[lane * D + k + 1] : 0.0;
                if (k < D - 1) S[k] += S[k + 1];
            }
            const double S_incl = wave_incl_scan_f64_dpp(S[0]), S_after = lane63_f64(S_incl) - S_incl;
            double mloc = sum_c;                              // k = 0: F_0 + S_0 = all class time
            int kb = 0;                                       // where this lane's maximum is attained
#pragma unroll
            for (int k = 0; k < D; ++k) {
                const double cand = (F_before + F[k]) + (S_after + S[k]);
                if (lane * D + k < R && cand > mloc) { mloc = cand; kb = lane * D + k + 1; }
            }
            const double m = wave_max_f64_dpp(mloc);

#define OS_KEEP(k) if constexpr (k < T) { kap_##k = kn_##k; }
            if (first || __builtin_amdgcn_readfirstlane((int)(m < m_cur))) {
                m_cur = m;
                const unsigned long long at = __ballot(mloc == m);
                kstar = at ? __builtin_amdgcn_readlane(kb, __builtin_ctzll(at)) : 0;
                OS_EACH(OS_KEEP)
                for (int j = lane; j <= R; j += 64) Acur[j] = A[j];
                if (first) {
                    if (lane == 0 && p.start_makespan) p.start_makespan[b] = m;
                    first = false;
                } else {
                    ++n_acc;
                    // the moves after this one, under the new k*
                    const unsigned long long later = cur == 63 ? 0ull : ~0ull << (cur + 1);
                    wave_sync();
                    todo = worth() & later;
                }
            } else {
                const double tx = t[x], ty = t[y];
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    xs[k] = lane * D + k == lo ? tx : xs[k];
                    xs[k] = lane * D + k == hi ? ty : xs[k];
                }
                wave_sync();
                if (lane == 0) { ordl[lo] = (uint16_t)x; ordl[hi] = (uint16_t)y; }
                wave_sync();
            }
        }

        for (int s = lane; s < R; s += 64) p.best_order[(size_t)b * R + s] = ordl[s];
        if (lane == 0) {
            p.best_makespan[b] = m_cur;
            if (p.n_accepted) p.n_accepted[b] = n_acc;
        }
    }
}

template <int T, bool WALK>
static hipError_t launch_search_t(SearchParams &p, const Dag &d, hipStream_t s)
{
    int levels = 1;
    while ((1 << levels) <= d.R) ++levels;            // floor(log2 R) + 1 levels of the table
    p.levels = levels;
    // (one after the other in the same place: class totals; positions and their maxima; A and what it was)
    const size_t fa = std::max(std::max((size_t)64 * T, ((size_t)levels * d.R * 2 + 7) / 8), (size_t)2 * d.R + 2);
    p.fa_len = (int32_t)fa;
    size_t wave_bytes = ((size_t)d.R + fa) * 8 + ((size_t)d.R + (d.R & 1)) * 2;
    wave_bytes = (wave_bytes + 15) & ~(size_t)15;
    const size_t rows_bytes = (((size_t)d.R * T * 8) + 15) & ~(size_t)15;
    const size_t lds = rows_bytes + wave_bytes * kSearchWaves;
    if (lds > 150 * 1024) return hipErrorNotSupported;     // 160 KB of LDS per compute unit
    p.wave_bytes = (int32_t)wave_bytes;
    p.rows_bytes = (int32_t)rows_bytes;
    hipError_t e;
    if (lds > 48 * 1024) {
        e = ensure_dynamic_lds(reinterpret_cast<const void *>(order_search_kernel<T, WALK>), lds);
        if (e != hipSuccess) return e;
    }
    int per_cu = 0;
    e = cached_blocks_per_cu(&per_cu, reinterpret_cast<const void *>(order_search_kernel<T, WALK>), 64 * kSearchWaves, lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
    const int n_cu = device_cu_count(d.device);
    int grid = per_cu * n_cu;
    const int need = (p.B + kSearchWaves - 1) / kSearchWaves;
    if (grid > need) grid = need;
    p.n_waves = grid * kSearchWaves;
    hipLaunchKernelGGL((order_search_kernel<T, WALK>), dim3(grid), dim3(64 * kSearchWaves), lds, s, p);
    return hipGetLastError();
}

hipError_t launch_order_search(Dag &d, const SearchArgs &a, hipStream_t s)
{
    const int KC = (d.C + 63) / 64, KR = (d.R + 63) / 64;
    const int K = KC > KR ? KC : KR;
    if (d.R == 0 || d.R > 512 || d.C == 0 || K > 8 || !d.d_col_cls || !d.d_cls_depT || !d.d_run_ptr) return hipErrorNotSupported;
    SearchParams p{};
    p.B = a.B; p.R = d.R; p.C = d.C; p.N = d.N; p.W = d.W; p.n_moves = a.n_moves;
    p.col_cls = d.d_col_cls; p.cls_depT = d.d_cls_depT; p.Cpad = d.Cpad;
    p.run_ptr = d.d_run_ptr; p.run_lo = d.d_run_lo; p.run_hi = d.d_run_hi;
    // Trying 32 recvs costs what eight runs or so cost: with seven runs per row (18 x 17 layered ops, 45 recvs) it is neither here nor
    // there, with 17 (12 x 10 and 100) 4 290 samples, 107 moves take 51 us instead of 61, with 42 (24 x 20 and 300) 190 instead of 367.
    const bool walk = d.n_runs > 8 * d.C;
    p.order = a.order; p.order_stride = a.order_stride; p.moves = a.moves;
    p.op_time = a.op_time; p.recv_time = a.recv_time;
    p.best_order = a.best_order; p.best_makespan = a.best_makespan;
    p.start_makespan = a.start_makespan; p.n_accepted = a.n_accepted;
#define OS_LAUNCH(k) if (K <= k) return walk ? launch_search_t<k, true>(p, d, s) : launch_search_t<k, false>(p, d, s);
    OS_EACH_T(OS_LAUNCH)
    return hipErrorNotSupported;
}

}  // namespace tictac
