// One iteration under a transfer order, for a batch of timing samples (Sec. 3.2; channel
// model of Sec. 5.1).  One workgroup per sample.
//
// The channel never waits (recvs are roots and are all requested at t = 0), so the k-th
// transfer of the order ends at F_k = sum of the first k transfer times.  A compute op
// can start once the last of the recvs it depends on has arrived, i.e. after
// kappa = max position of dep[op] in the order (0 if it depends on no recv); ops of a
// class (identical dep) share kappa.  A device that never idles while an op is ready
// finishes the work released up to transfer k at
//     busy_0 = A_0,   busy_k = max(busy_{k-1}, F_k) + A_k,
// A_k = total time of the classes with kappa = k, whatever ready op it picks first
// (a predecessor of a released op was released no later).  makespan = max(busy_R, F_R).
#include <algorithm>

#include "device_utils.h"
#include "internal.h"

namespace tictac {

struct SimKernelParams {
    int32_t B, R, W, C, N;
    const uint64_t *cls_dep;    // [C][W]
    const int32_t *cls_ptr;     // [C+1]
    const int32_t *cls_cols;    // [N]
    const int32_t *order;       // [R] or [B][R]
    int32_t order_stride;
    const int32_t *kappa;       // [C] for a shared order, else NULL
    const void *op_time, *recv_time;    // float64, or float32 when f32 is set
    int32_t f32;
    double *makespan, *eff, *U, *L, *S;
};

// kappa of every class and of every op_time column under an order shared by all samples.  Every workgroup makes the 1-based
// positions for itself (0 for a recv that an invalid order leaves out, so that every position read is in 0 .. R); the first
// one checks the order.  In launches of their own the positions and the check took a third of a call on 1 000 samples of
// resnet50 (33 us).
constexpr int kKappaBlock = 64;             // classes per workgroup, whose columns its 256 threads share
__global__ void __launch_bounds__(256)
kappa_kernel(int32_t R, int32_t W, int32_t C, const uint64_t *__restrict__ cls_dep, const int32_t *__restrict__ order,
             const int32_t *__restrict__ cls_ptr, const int32_t *__restrict__ cls_cols, const int32_t *__restrict__ col_cls,
             int32_t *kappa /*[C]*/, int32_t *kappa_col /*[N] or NULL*/, int32_t *bad_order)
{
    extern __shared__ int32_t pos[];        // [R], then [kKappaBlock] kappa
    int32_t *mine = pos + R;
    for (int k = threadIdx.x; k < R; k += 256) pos[k] = 0;
    __syncthreads();
    for (int k = threadIdx.x; k < R; k += 256)
        if ((unsigned)order[k] < (unsigned)R) pos[order[k]] = k + 1;
    __syncthreads();
    if (blockIdx.x == 0) {
        bool bad = false;
        for (int k = threadIdx.x; k < R; k += 256) bad |= (unsigned)order[k] >= (unsigned)R || pos[order[k]] != k + 1;
        if (bad) atomicOr(bad_order, 1);
    }
    const int c0 = blockIdx.x * kKappaBlock, c = c0 + (threadIdx.x >> 2), part = threadIdx.x & 3;     // four threads per class
    int kap = 0;
    if (c < C) {
        const uint64_t *row = cls_dep + (size_t)c * W;
        for (int w = part; w < W; w += 4) {
            uint64_t x = row[w];
            while (x) {
                kap = max(kap, pos[w * 64 + __builtin_ctzll(x)]);
                x &= x - 1;
            }
        }
    }
    kap = max(kap, __shfl_xor(kap, 1));
    kap = max(kap, __shfl_xor(kap, 2));
    if (c < C && part == 0) {
        kappa[c] = kap;
        mine[c - c0] = kap;
    }
    __syncthreads();
    if (!kappa_col) return;
    const int end = cls_ptr[min(c0 + kKappaBlock, C)];
    for (int m = cls_ptr[c0] + threadIdx.x; m < end; m += 256) {
        const int j = cls_cols[m];
        kappa_col[j] = mine[col_cls[j] - c0];
    }
}

template <int BS>
__global__ void __launch_bounds__(BS)
simulate_kernel(const SimKernelParams p)
{
    extern __shared__ double smem[];
    const int R = p.R, W = p.W, C = p.C, N = p.N;
    const int tid = threadIdx.x;
    double *Fs = smem;                  // [R+1] F_k
    double *A = Fs + (R + 1);           // [R+1] A_k
    double *red = A + (R + 1);          // [16]
    int32_t *pos = reinterpret_cast<int32_t *>(red + 16);   // [R] 1-based position of recv r

    for (int b = blockIdx.x; b < p.B; b += gridDim.x) {
        const TimeRow rt = time_row(p.recv_time, (size_t)b * R, p.f32 != 0);
        const TimeRow ot = time_row(p.op_time, (size_t)b * N, p.f32 != 0);
        const int32_t *ord = p.order + (size_t)b * p.order_stride;
        __syncthreads();
        for (int k = tid; k < R; k += BS) pos[k] = 0;   // (a recv that an invalid order leaves out: position 0)
        __syncthreads();
        for (int k = tid; k < R; k += BS) {
            const int r = ord[k];
            const bool ok = (unsigned)r < (unsigned)R;   // an invalid entry is skipped, never dereferenced
            if (ok) pos[r] = k + 1;
            Fs[k + 1] = ok ? rt[r] : 0.0;   // transfer time of the k-th transfer, summed below
        }
        for (int k = tid; k <= R; k += BS) A[k] = 0.0;
        if (tid == 0) Fs[0] = 0.0;
        __syncthreads();

        double ct_sum = 0.0;
        for (int c0 = 0; c0 < C; c0 += BS) {
            const int c = c0 + tid;
            const bool valid = c < C;
            double s = 0.0;
            int kap = 0;
            if (valid) {
                for (int m = p.cls_ptr[c]; m < p.cls_ptr[c + 1]; ++m) s += ot[p.cls_cols[m]];
                if (p.kappa) {
                    kap = p.kappa[c];
                } else {
                    const uint64_t *row = p.cls_dep + (size_t)c * W;
                    for (int w = 0; w < W; ++w) {
                        uint64_t x = row[w];
                        while (x) {
                            kap = max(kap, pos[w * 64 + __builtin_ctzll(x)]);
                            x &= x - 1;
                        }
                    }
                }
                ct_sum += s;
            }
            lds_scatter_add<BS>(A, kap, s, valid);
        }
        const double sum_c = block_sum_f64<BS>(ct_sum, red);
        __syncthreads();
        if (tid == 0) {
            double F = 0.0, busy = A[0];
            // (fmax: of sums it is one instruction too, and the loop is unrolled, its loads ahead of the chain.  8 192 samples of 4 096
            // recvs, one order: 3.01 ms, with max_f64 7.16)
            for (int k = 1; k <= R; ++k) {
                F += Fs[k];
                busy = fmax(busy, F) + A[k];
            }
            const double m = max_f64(busy, F);
            const double U = sum_c + F;
            const double L = max_f64(sum_c, F);
            p.makespan[b] = m;
            p.eff[b] = (U == L) ? 1.0 : (U - m) / (U - L);
            if (p.U) p.U[b] = U;
            if (p.L) p.L[b] = L;
            if (p.S) p.S[b] = (U == L || L == 0.0) ? 0.0 : (U - L) / L;
        }
    }
}

// The same computation with one wavefront per sample, for graphs with at most 512 recvs.  Lane l owns the classes l, l + 64, ...
// and the positions l, l + 64, ... of the order; a workgroup is four independent waves.  Per sample: the transfer
// times and the order are requested first, into registers, then the op_time row is read once,
// coalesced, every run of columns of one class adding itself to the total of its class in LDS
// (so one trip to memory per sample is waited for, not three); kappa of a class is the maximum of the positions of its recvs,
// taken run by run of consecutive recv indices from a sparse table of range maxima over the position array.  An order of the
// sample's own is checked on the way (resnet50, 65 536 samples: 202 us with a launch for it, 187 without).
//   * When all samples share one order, kappa is a table by column, and the columns are added up by it at once, whatever the
//     number of classes (inception3, 65 536 samples: 650 -> 606 us; 61 x 23 layered ops, 203 recvs, 775 classes, 20 000
//     samples, which went to the kernel above: 917 -> 72 us).
//   * A row of many runs mostly holds one of the recvs that come last: there, and where there are too many classes for the
//     registers (up to the 18 000 or so whose totals LDS holds), those are tried first, from the last one on (61 x 23 ops, an
//     order each: 1 470 -> 222 us).
// Then A by kappa, and
//     makespan = max over k of F_k + (A_k + ... + A_R),   F_0 = 0,
// which is the recurrence above unrolled.
struct SimWaveParams {
    int32_t B, R, C, N, n_waves, wave_bytes, levels;
    const int32_t *col_cls;     // [N] class of every op_time column
    const int32_t *run_ptr;     // [C+1] runs [run_lo, run_hi) of consecutive recv indices of the class rows
    const int32_t *run_lo, *run_hi;
    const int32_t *cls_cnt0;    // [C] recvs of the row
    const uint32_t *depT;       // cls_depT in halves: half h of class c at (h / 2 * Cpad + c) * 2 + h % 2
    int32_t Cpad;
    const int32_t *order;
    int32_t order_stride;
    const int32_t *kappa_col;   // [N] for a shared order, else NULL
    const void *op_time, *recv_time;    // float64, or float32 when f32 is set
    int32_t f32;
    double *makespan, *eff, *U, *L, *S;
    int32_t *bad_order;         // raised when an order is no permutation; not looked at with kappa_col
};

constexpr int kSimWaves = 4;
constexpr int kWalkRecvs = 6, kWalkSteps = 32;

#define SW_EACH_K(F) F(0) F(1) F(2) F(3) F(4) F(5) F(6) F(7)

// Where kappa comes from: a table by column; two runs of most rows, of classes in registers (and memory for the other runs); or
// rows that are read again for every sample, recv by recv, the recvs that come last first.
enum { kKappaTable, kKappaRuns, kKappaLoop, kKappaRunsLong };

// With classes in registers: F, the positions, and from here on (in doubles) the transfer times and A.
__host__ __device__ constexpr int sim_times_at(int R) { return R + (R + 3) / 4; }

// Bytes of a wave.  Times and sums; then the class totals and the positions.  With classes in registers the totals are summed where
// all the others come later, and the range maxima of the positions are in the place of the transfer times, which are known by
// position by then, and of A, which comes after them: 16 KB per wave of inception3 were 10, so that three workgroups instead of
// two share a compute unit.  An order each, 65 536 samples: inception3 842 -> 727 us;
// resnet50, where registers are the bound, 181 -> 171; 3 000 samples of inception3 55 -> 49.  (And with Sums::quads: 678 and 47; as
// float32 974 -> 708.)
static size_t sim_wave_bytes(int KAPPA, int KT, int R, int C, int levels)
{
    size_t n = ((size_t)3 * R + 1) * 8;
    if (KAPPA == kKappaTable) return n;
    if (KAPPA == kKappaLoop) return n + (size_t)C * 8 + (size_t)R * 2;
    n = (size_t)sim_times_at(R) * 8 + ((size_t)2 * R + 1) * 8;
    return std::max(n, std::max((size_t)R * 8 + (size_t)levels * R * 2, (size_t)64 * KT * 8));
}

// Workgroups per compute unit that the registers are to leave room for.  Three share one with up to 168 registers: from five slots
// to seven no more are used without being asked for, and where the compiler is asked it waits for loads earlier (float32, five slots,
// 290 classes with 16 columns each, 65 536 samples: 490 and 558 us; six, 380 classes 599 and 684; seven, inception3 708 and 782; 100
// samples 23.2 and 24.2).  Eight slots would take 186.
constexpr int sim_workgroups(int KT) { return KT <= 3 ? 5 : KT <= 4 ? 4 : KT <= 7 ? 2 : 3; }

template <int KT, int KAPPA>
__global__ void __launch_bounds__(64 * kSimWaves, sim_workgroups(KT))
simulate_wave_kernel(const SimWaveParams p)
{
    extern __shared__ double smem[];
    const int R = p.R, C = p.C, N = p.N;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    char *mine = reinterpret_cast<char *>(smem) + (size_t)wave * p.wave_bytes;
    constexpr bool kInRegs = KAPPA == kKappaRuns || KAPPA == kKappaRunsLong;
    double *F = reinterpret_cast<double *>(mine) + (kInRegs ? 0 : R);       // [R]   F[k-1] = end of the k-th transfer
    double *t = reinterpret_cast<double *>(mine) + (kInRegs ? sim_times_at(R) : 0);     // [R]   Time(recv)
    double *A = (kInRegs ? t : F) + R;                      // [R+1] class time by kappa
    // the class totals while they are summed: by kappa at once; [64 KT] before anything else is there; [C]
    double *csum = KAPPA == kKappaTable ? A : KAPPA == kKappaLoop ? A + (R + 1) : F;
    uint16_t *pos = reinterpret_cast<uint16_t *>(KAPPA == kKappaLoop ? csum + C : F + R);   // [levels][R] range maxima of the 1-based positions

    // Per class slot, fixed for the launch: the first two runs of the class row (lo | hi << 16; longer rows read the rest from
    // memory).
#define SW_RUNS(k)                                                                        \
    [[maybe_unused]] unsigned rn_##k = 0, ra_##k = 0, rc_##k = 0;    /* first run | last + 1 << 16; the first two of them */ \
    if constexpr (k < KT && kInRegs) {                                                    \
        const int c = k * 64 + lane;                                                      \
        if (c < C) {                                                                      \
            const int rb = p.run_ptr[c], re = p.run_ptr[c + 1];                           \
            rn_##k = (unsigned)rb | (unsigned)re << 16;                                   \
            if (re > rb) ra_##k = (unsigned)p.run_lo[rb] | ((unsigned)p.run_hi[rb] << 16);              \
            if (re > rb + 1) rc_##k = (unsigned)p.run_lo[rb + 1] | ((unsigned)p.run_hi[rb + 1] << 16);  \
        }                                                                                 \
    }
    SW_EACH_K(SW_RUNS)

    bool bad = false;
    const int gwave = blockIdx.x * (blockDim.x >> 6) + wave;
    for (int b = gwave; b < p.B; b += p.n_waves) {
        const TimeRow rt = time_row(p.recv_time, (size_t)b * R, p.f32 != 0);
        const TimeRow ot = time_row(p.op_time, (size_t)b * N, p.f32 != 0);
        const int32_t *ord = p.order + (size_t)b * p.order_stride;
        wave_sync();                        // LDS of the previous sample is no longer read

        // ---- everything the sample reads from memory is requested here: the transfer times and
        // the order into registers (position slot q: r = q * 64 + lane), then the op_time row ----
#define SW_REQUEST(q)                                                                     \
        double rt_##q = 0.0;                                                              \
        int or_##q = -1;                                                                  \
        if constexpr (q < KT) {                                                           \
            if (q * 64 + lane < R) { rt_##q = rt[q * 64 + lane]; or_##q = ord[q * 64 + lane]; } \
        }
        SW_EACH_K(SW_REQUEST)
        const int n_totals = KAPPA == kKappaTable ? R + 1 : KAPPA == kKappaLoop ? C : 64 * KT;
        for (int c = lane; c < n_totals; c += 64) csum[c] = 0.0;
        wave_sync();
        constexpr Sums how = KAPPA == kKappaTable ? Sums::rows : KAPPA == kKappaRunsLong ? Sums::quads : kInRegs && KT == 7 ? Sums::plain_together : Sums::plain;
        class_totals<how>(csum, ot, KAPPA == kKappaTable ? p.kappa_col : p.col_cls, N, lane);
        wave_sync();
#define SW_DECL(k) [[maybe_unused]] double ct_##k = 0.0; [[maybe_unused]] int kap_##k = 0;
        SW_EACH_K(SW_DECL)
#define SW_TOTAL(k) if constexpr (k < KT && kInRegs) { ct_##k = csum[k * 64 + lane]; }
        SW_EACH_K(SW_TOTAL)
        if constexpr (kInRegs) wave_sync();
#define SW_TIMES(q)                                                                       \
        if constexpr (q < KT) {                                                           \
            if (q * 64 + lane < R) {                                                      \
                t[q * 64 + lane] = rt_##q;                                                \
                if constexpr (KAPPA != kKappaTable) pos[q * 64 + lane] = 0;               \
            }                                                                             \
        }
        SW_EACH_K(SW_TIMES)
        wave_sync();

        // ---- positions, F ----
        double fc = 0.0;
#define SW_PLACE(q)                                                                       \
        if constexpr (q < KT) {                                                           \
            if (q * 64 < R) {                                                             \
                const int s = q * 64 + lane;                                              \
                const int r = or_##q;                                                     \
                const bool ok = (unsigned)r < (unsigned)R;  /* an invalid entry is skipped, never dereferenced */ \
                if (KAPPA != kKappaTable && ok) pos[r] = (uint16_t)(s + 1);                                       \
                const double x = ok ? t[r] : 0.0;                                         \
                const double inc = wave_incl_scan_f64_dpp(x);                             \
                if (s < R) F[s] = fc + inc;                                               \
                fc += lane63_f64(inc);                                                    \
            }                                                                             \
        }
        SW_EACH_K(SW_PLACE)
        const double Ftot = fc;
        if constexpr (KAPPA == kKappaLoop)
            for (int j = lane; j <= R; j += 64) A[j] = 0.0;
        wave_sync();

        // ---- kappa ----
        double ct_sum = 0.0;
        if constexpr (KAPPA != kKappaTable) {
            // (the check of the order: every recv is at the position that it has been given last)
#define SW_CHECK(q)                                                                       \
            if constexpr (q < KT) {                                                       \
                if (q * 64 + lane < R) bad |= (unsigned)or_##q >= (unsigned)R || pos[or_##q] != q * 64 + lane + 1; \
            }
            SW_EACH_K(SW_CHECK)
            // the recvs that come last, last one first (an invalid entry is skipped)
            [[maybe_unused]] const int late = KAPPA == kKappaLoop && lane < kWalkSteps && lane < R ? ord[R - 1 - lane] : -1;
            [[maybe_unused]] const uint32_t is_late = (uint32_t)__ballot((unsigned)late < (unsigned)R);
            // level j of the table: maximum over [i, min(i + 2^j, R))
            for (int j = 1; KAPPA != kKappaLoop && j < p.levels; ++j) {
                const uint16_t *prev = pos + (size_t)(j - 1) * R;
                uint16_t *cur = pos + (size_t)j * R;
                const int h = 1 << (j - 1);
                for (int i = lane; i < R; i += 64) cur[i] = max(prev[i], prev[min(i + h, R - 1)]);
                wave_sync();
            }
#define SW_RANGE_MAX(lo, hi)                                                              \
                    {                                                                     \
                        const int j_ = 31 - __builtin_clz((hi) - (lo));                   \
                        const uint16_t *lv_ = pos + (size_t)j_ * R;                       \
                        m = max(m, max((int)lv_[lo], (int)lv_[(hi) - (1 << j_)]));        \
                    }
#define SW_KAPPA_RUNS(k)                                                                  \
            if constexpr (k < KT && kInRegs) {                                            \
                if (k * 64 + lane < C) {                                                  \
                    int m = 0;                                                            \
                    const int rb = (int)(rn_##k & 0xffffu), re = (int)(rn_##k >> 16);     \
                    if (re > rb) SW_RANGE_MAX((int)(ra_##k & 0xffffu), (int)(ra_##k >> 16))          \
                    if (re > rb + 1) SW_RANGE_MAX((int)(rc_##k & 0xffffu), (int)(rc_##k >> 16))      \
                    for (int q = rb + 2; q < re; ++q) {                                   \
                        const int lo = p.run_lo[q], hi = p.run_hi[q];                     \
                        SW_RANGE_MAX(lo, hi)                                              \
                    }                                                                     \
                    kap_##k = m;                                                          \
                }                                                                         \
            }
            SW_EACH_K(SW_KAPPA_RUNS)
            if constexpr (KAPPA == kKappaLoop) {
                for (int c0 = 0; c0 < C; c0 += 64) {            // (all lanes take part in the last step)
                    const int c = min(c0 + lane, C - 1);
                    const bool in = c0 + lane < C;
                    const double ct = in ? csum[c] : 0.0;
                    int m = 0, n = 0;
                    if (p.cls_cnt0[c] > kWalkRecvs)
                        for (int i = 0; i < min(R, kWalkSteps) && m == 0; i += 4) {
                            uint32_t w[4];
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const int r = is_late >> (i + j) & 1u ? __builtin_amdgcn_readlane(late, i + j) : 0;
                                w[j] = p.depT[((size_t)(r >> 6) * p.Cpad + c) * 2 + (r >> 5 & 1)] >> (r & 31) & 1u;
                            }
#pragma unroll
                            for (int j = 3; j >= 0; --j)
                                if (w[j] && is_late >> (i + j) & 1u) m = R - (i + j);
                        }
                    for (int h = 0; m == 0 && 32 * h < R; h += 2) {
                        const uint2 row = *reinterpret_cast<const uint2 *>(p.depT + ((size_t)(h >> 1) * p.Cpad + c) * 2);
                        for (uint64_t x = (uint64_t)row.y << 32 | row.x; x != 0ull; x &= x - 1) n = max(n, (int)pos[h * 32 + __builtin_ctzll(x)]);
                    }
                    m = max(m, n);
                    ct_sum += ct;
                    add_by_rows(A, in ? m : -1, ct, lane);
                }
            }
        }

        // ---- A by kappa, suffix sums, makespan ----
        if constexpr (kInRegs) {
            wave_sync();
            for (int j = lane; j <= R; j += 64) A[j] = 0.0;
            wave_sync();
        }
#define SW_RELEASE(k) if constexpr (k < KT && kInRegs) { if (k * 64 + lane < C) atomicAdd(&A[kap_##k], ct_##k); ct_sum += ct_##k; }
        SW_EACH_K(SW_RELEASE)
        wave_sync();
        if constexpr (KAPPA == kKappaTable)
            for (int j = lane; j <= R; j += 64) ct_sum += A[j];
        const double sum_c = wave_sum_f64_dpp(ct_sum);
        double sfx = 0.0, mloc = sum_c;                   // k = 0: F_0 + S_0 = all class time
        for (int base = ((R - 1) / 64) * 64; base >= 0; base -= 64) {
            const int k = base + lane + 1;                // 1 <= k <= R handled here
            const double x = k <= R ? A[k] : 0.0;
            const double inc = wave_incl_scan_f64_dpp(x);
            const double tot = lane63_f64(inc);
            if (k <= R) mloc = max_f64(mloc, F[k - 1] + (sfx + (tot - inc + x)));
            sfx += tot;
        }
        const double m = wave_max_f64_dpp(mloc);
        if (lane == 0) {
            const double U = sum_c + Ftot;
            const double L = max_f64(sum_c, Ftot);
            p.makespan[b] = m;
            p.eff[b] = (U == L) ? 1.0 : (U - m) / (U - L);
            if (p.U) p.U[b] = U;
            if (p.L) p.L[b] = L;
            if (p.S) p.S[b] = (U == L || L == 0.0) ? 0.0 : (U - L) / L;
        }
    }
    if (bad) atomicOr(p.bad_order, 1);
}

template <int KT, int KAPPA>
static hipError_t launch_sim_wave(SimWaveParams &p, const Dag &d, hipStream_t s)
{
    int levels = 1;
    while ((1 << levels) <= d.R) ++levels;            // floor(log2 R) + 1 levels of the table
    p.levels = levels;
    const size_t wave_bytes = (sim_wave_bytes(KAPPA, KT, d.R, d.C, levels) + 15) & ~(size_t)15;
    int waves = kSimWaves;
    while (waves > 1 && wave_bytes * waves > 150 * 1024) waves >>= 1;
    const size_t lds = wave_bytes * waves;
    if (lds > 150 * 1024) return hipErrorNotSupported;     // 160 KB of LDS per compute unit
    p.wave_bytes = (int32_t)wave_bytes;
    hipError_t e;
    if (lds > 48 * 1024) {
        e = ensure_dynamic_lds(reinterpret_cast<const void *>(simulate_wave_kernel<KT, KAPPA>), lds);
        if (e != hipSuccess) return e;
    }
    int per_cu = 0;
    e = cached_blocks_per_cu(&per_cu, reinterpret_cast<const void *>(simulate_wave_kernel<KT, KAPPA>), 64 * waves, lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
    const int n_cu = device_cu_count(d.device);
    int grid = per_cu * n_cu;
    const int need = (p.B + waves - 1) / waves;
    if (grid > need) grid = need;
    p.n_waves = grid * waves;
    hipLaunchKernelGGL((simulate_wave_kernel<KT, KAPPA>), dim3(grid), dim3(64 * waves), lds, s, p);
    return hipGetLastError();
}

// hipErrorNotSupported: the graph is outside what the wave kernel handles
static hipError_t try_simulate_wave(const Dag &d, const SimArgs &a, const int32_t *kappa_col, hipStream_t s)
{
    if (d.R == 0 || d.R > 512 || d.C == 0 || !d.d_col_cls || !d.d_cls_depT || !d.d_bad_order)
        return hipErrorNotSupported;
    SimWaveParams p{};
    p.B = a.B; p.R = d.R; p.C = d.C; p.N = d.N;
    p.col_cls = d.d_col_cls; p.run_ptr = d.d_run_ptr; p.run_lo = d.d_run_lo; p.run_hi = d.d_run_hi;
    p.cls_cnt0 = d.d_cls_cnt0; p.depT = reinterpret_cast<const uint32_t *>(d.d_cls_depT); p.Cpad = d.Cpad; p.bad_order = d.d_bad_order;
    p.order = a.order; p.order_stride = a.order_stride; p.kappa_col = kappa_col;
    p.op_time = a.op_time; p.recv_time = a.recv_time; p.f32 = a.f32 ? 1 : 0;
    p.makespan = a.makespan; p.eff = a.eff; p.U = a.U; p.L = a.L; p.S = a.S;
    // Rows of more than two runs on average, or more classes than the registers of a lane hold: by recv.  65 536 samples, an order
    // each, by run and by recv: 24 x 20 layered ops, 300 recvs 3.59 and 0.58 ms; 21 x 18 and 28, 227 and 107 us; resnet50, less
    // than one run, 171 and 222 us; inception3 678 and 839.
    const int kr = (d.R + 63) / 64, K = std::max((d.C + 63) / 64, kr);      // slots per lane: positions; classes as well
#define SW_LAUNCH_EACH(k, kappa)                                                          \
    SW_LAUNCH(k, 1, kappa) SW_LAUNCH(k, 2, kappa) SW_LAUNCH(k, 3, kappa) SW_LAUNCH(k, 4, kappa)     \
    SW_LAUNCH(k, 5, kappa) SW_LAUNCH(k, 6, kappa) SW_LAUNCH(k, 7, kappa) SW_LAUNCH(k, 8, kappa)
#define SW_LAUNCH(k, n, kappa) if (k <= n) return launch_sim_wave<n, kappa>(p, d, s);
    if (kappa_col) {
        SW_LAUNCH_EACH(kr, kKappaTable)
    } else if (K > 8 || !d.d_run_ptr || d.n_runs > 2 * d.C) {
        SW_LAUNCH_EACH(kr, kKappaLoop)
    } else if (K > 4 && d.long_runs && a.B > kSimWaves * device_cu_count(d.device)) {
        // (by quads, a sample by itself takes longer: up to a workgroup per compute unit, inception3 21.2 and 21.7 us, 300 classes
        // with 64 columns each 26.4 and 29.9)
        SW_LAUNCH(K, 5, kKappaRunsLong) SW_LAUNCH(K, 6, kKappaRunsLong) SW_LAUNCH(K, 7, kKappaRunsLong) SW_LAUNCH(K, 8, kKappaRunsLong)
    } else {
        SW_LAUNCH_EACH(K, kKappaRuns)
    }
    return hipErrorNotSupported;
}

template <int BS>
static hipError_t launch_sim_t(const SimKernelParams &p, int grid, size_t lds, hipStream_t s)
{
    auto kern = simulate_kernel<BS>;
    if (lds > 48 * 1024) {
        hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(grid), dim3(BS), lds, s, p);
    return hipGetLastError();
}

// Several channels (Sec. 4.1: one per parameter server; Sec. 5.1: one transfer at a time per
// channel).  Recv i uses channel chan[i]; every channel serves its recvs back to back from
// t = 0 in the order in which they appear in the given order.  The channels never wait (recvs
// are roots), so recv r arrives at the sum of the transfer times queued up to and including it
// on its channel; a class is released when the last recv of its row has arrived (rho); and a
// device that never idles while an op is ready finishes at
//     max( latest arrival,  max over classes c of  rho_c + sum of the times of the classes with rho >= rho_c ).
// One wave per sample: arrivals by one wave scan per channel, rho by range maxima over the
// arrival array (runs of the class rows), the last step by ranking the
// release dates among the arrivals: on one channel the arrivals increase along the order, so the number of
// arrivals up to rho is one binary search per channel; the class times are added up by that rank and one
// suffix sum over the ranks gives the second term for every class.
struct SimChanParams {
    int32_t B, R, C, N, n_waves, wave_bytes, levels, n_channels, chan_bytes;
    int32_t nb, arr_doubles;    // blocks of four recvs; doubles for the arrivals
    int32_t cls_lane, cls_slot; // class of lane l's k-th slot: l * cls_lane + k * cls_slot
    const uint32_t *depT;       // rows of many runs: cls_depT in halves, as above; else NULL
    int32_t Cpad;
    const int32_t *col_cls, *run_ptr, *run_lo, *run_hi;
    const int32_t *chan;        // [R] channel of every recv, 0 <= chan < n_channels <= 64
    const int32_t *order;
    int32_t order_stride;
    const void *op_time, *recv_time;    // float64, or float32 when f32 is set
    int32_t f32;
    double *makespan, *eff, *U, *L, *S;
    int32_t *bad_order;         // raised when an order is no permutation
};

// D consecutive positions of the order per lane, so that a sum over positions is a few adds per lane and one scan over the lanes.
// The classes of a lane are consecutive too where rows are short: classes that are released together (neighbours, mostly) are
// then added up in the lane.  Where rows have many runs they are l, l + 64, ...: lanes wait for the longest row of a slot, and
// neighbours have rows of similar length.  (More than two runs per row on average; resnet50, less than one, four channels: 257 us
// with consecutive classes, 343 without; 24 x 20 layered ops, 300 recvs, all run by run: 6.9 and 6.2 ms.)
// The order is checked on the way.  65 536 samples, four channels, with the check: inception3 1 188 -> 1 000 us (a scan per channel
// and 64 positions before, 26 % more vector instructions), resnet50 357 -> 257 us.  Waves wait for the op_time row most of
// their time, so what counts is how many there are: the registers (an occupancy bound per KT) and LDS, which holds
// everything but the arrivals in one place, say so.  The first two runs of every class are in LDS, the same for all waves: kept in registers over all samples they
// and what the compiler formed from them ahead of the loop took 45 of 168 and spilled 17 more (seven class slots), and four waves per SIMD
// are possible without them instead of three: inception3, 65 536 samples, one, four and sixteen channels 787 -> 664, 930 -> 732, 1 467 -> 1 113 us; 1 000
// samples 48 -> 40; resnet50 242 -> 224; 22 x 20 layered ops, 380 recvs 1 233 -> 945.  (Two waves per SIMD and nothing spilled: 1 212.)
template <int KT, Sums HOW>
__global__ void __launch_bounds__(256, KT <= 2 ? 6 : KT <= 4 ? 5 : 3)
simulate_channels_kernel(const SimChanParams p)
{
    extern __shared__ double smem[];
    constexpr int D = KT | 1;               // (odd: what lanes read of their positions is in different banks)
    const int R = p.R, C = p.C, N = p.N;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t *chan_l = reinterpret_cast<int32_t *>(smem);    // [R] channel of every recv, shared by the waves
    int32_t *coff = chan_l + R;             // [64] where the arrivals of a channel start in `lists`
    int32_t *clen = coff + 64;              // [64] recvs of a channel
    uint32_t *runs_l = reinterpret_cast<uint32_t *>(clen + 64);         // [2][KT][64] the first two runs of every class
    double *mine = reinterpret_cast<double *>(reinterpret_cast<char *>(smem) + p.chan_bytes + (size_t)wave * p.wave_bytes);
    const int Rp = (R + 3) & ~3, nb = p.nb;
    double *arr = mine;                     // [Rp] arrival of recv r, zero beyond R
    // in one place, one after the other:
    double *csum = arr + p.arr_doubles;     // [64 KT] the class totals while they are summed
    double *t = csum;                       // [R]  Time(recv), until the arrivals are known
    int32_t *place = reinterpret_cast<int32_t *>(t);        // [R] the position of every recv
    double *tab = t;                        // [levels][nb] level j: maxima of the arrivals over the blocks [i, i + 2^j) of four recvs
    double *lists = t;                      // [R] the arrivals channel by channel, in the order's sequence
    const int cls_lane = p.cls_lane, cls_slot = p.cls_slot;
    for (int r = threadIdx.x; r < R; r += blockDim.x) chan_l[r] = p.chan[r];
    __syncthreads();
    if (wave == 0) {
        int n_mine = 0;                     // lane c: recvs of channel c
        for (int r = 0; r < R; ++r) n_mine += chan_l[r] == lane;
        int incl = n_mine;
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        coff[lane] = incl - n_mine;
        clen[lane] = n_mine;
    }
    __syncthreads();
    // the first two runs of every class row (lo | hi << 10) and, above the first, their number; fixed for the launch, as are the
    // further ones, which stay in memory
    for (int i = wave; i < KT; i += blockDim.x >> 6) {
        const int c = lane * cls_lane + i * cls_slot;
        uint32_t ra = 0, rc = 0;
        if (c < C) {
            const int q = p.run_ptr[c], n = p.run_ptr[c + 1] - q;
            if (n > 0) ra = (uint32_t)p.run_lo[q] | (uint32_t)p.run_hi[q] << 10 | (uint32_t)n << 20;
            if (n > 1) rc = (uint32_t)p.run_lo[q + 1] | (uint32_t)p.run_hi[q + 1] << 10;
        }
        runs_l[i * 64 + lane] = ra;
        runs_l[(KT + i) * 64 + lane] = rc;
    }
    __syncthreads();

    bool bad = false;
    const int gwave = blockIdx.x * (blockDim.x >> 6) + wave;
    for (int b = gwave; b < p.B; b += p.n_waves) {
        const TimeRow rt = time_row(p.recv_time, (size_t)b * R, p.f32 != 0);
        const TimeRow ot = time_row(p.op_time, (size_t)b * N, p.f32 != 0);
        const int32_t *ord = p.order + (size_t)b * p.order_stride;
        wave_sync();

        // ---- transfer times and the order are requested first, into registers, then the op_time row ----
        double rt_q[KT];
        int at[D];                          // the recvs at the lane's positions
#pragma unroll
        for (int q = 0; q < KT; ++q) rt_q[q] = q * 64 + lane < R ? rt[q * 64 + lane] : 0.0;
#pragma unroll
        for (int k = 0; k < D; ++k) at[k] = lane * D + k < R ? ord[lane * D + k] : -1;
        for (int c = lane; c < 64 * KT; c += 64) csum[c] = 0.0;
        wave_sync();
        class_totals<HOW>(csum, ot, p.col_cls, N, lane);
        wave_sync();
        double ct[KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) ct[k] = csum[lane * cls_lane + k * cls_slot];
        wave_sync();
#pragma unroll
        for (int q = 0; q < KT; ++q)
            if (q * 64 + lane < R) { t[q * 64 + lane] = rt_q[q]; arr[q * 64 + lane] = 0.0; }
        if (R + lane < Rp) arr[R + lane] = 0.0;
        wave_sync();

        // ---- arrivals: per channel, prefix sums over the positions of the order ----
        double x[D], a[D];
        int of[D];                          // recv | channel << 10 | number among those of the channel << 16, -1: none
        double sum_r = 0.0;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const bool ok = (unsigned)at[k] < (unsigned)R;      // an invalid entry is skipped, never dereferenced
            of[k] = ok ? at[k] | chan_l[at[k]] << 10 : -1;
            x[k] = ok ? t[at[k]] : 0.0;
            a[k] = 0.0;
            sum_r += x[k];
        }
        wave_sync();
        // (the check of the order: every recv is at the place that it has been given last)
#pragma unroll
        for (int k = 0; k < D; ++k)
            if ((unsigned)at[k] < (unsigned)R) place[at[k]] = lane * D + k;
        wave_sync();
#pragma unroll
        for (int k = 0; k < D; ++k)
            if (lane * D + k < R) bad |= (unsigned)at[k] >= (unsigned)R || place[at[k]] != lane * D + k;
        double carry = 0.0;                 // lane c: time queued on channel c
        int queued = 0;                     // lane c: recvs queued on channel c
        for (int c = 0; c < p.n_channels; ++c) {
            double run = 0.0;
            int n = 0;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                run += ((of[k] >> 10) & 63) == c && of[k] >= 0 ? x[k] : 0.0;
                n += ((of[k] >> 10) & 63) == c && of[k] >= 0 ? 1 : 0;
            }
            const double incl = wave_incl_scan_f64_dpp(run);
            const int n_incl = wave_incl_scan_i32_dpp(n);
            if (lane == c) {
                carry = lane63_f64(incl);
                queued = __builtin_amdgcn_readlane(n_incl, 63);
            }
            run = dpp0_f64<0x138>(incl);                        // (what the lanes before have)
            n = dpp0_i32<0x138>(n_incl);
#pragma unroll
            for (int k = 0; k < D; ++k)
                if (((of[k] >> 10) & 63) == c && of[k] >= 0) {
                    run += x[k];
                    a[k] = run;
                    of[k] |= n++ << 16;
                }
        }
#pragma unroll
        for (int k = 0; k < D; ++k)
            if (of[k] >= 0) arr[of[k] & 1023] = a[k];
        sum_r = wave_sum_f64_dpp(sum_r);
        const double last_arrival = wave_max_f64_dpp(lane < p.n_channels ? carry : 0.0);   // = largest channel sum
        wave_sync();

        // ---- rho of every class: maximum arrival over the runs of its row ----
        // A run [lo, hi) is at most three recvs, whole blocks of four, and at most three recvs: the blocks are
        // looked up in a table of maxima over 2^j blocks (two reads), the recvs at the ends are read one by one.
        for (int i = lane; i < nb; i += 64) {
            const double2 u = *reinterpret_cast<const double2 *>(arr + 4 * i), v = *reinterpret_cast<const double2 *>(arr + 4 * i + 2);
            tab[i] = max_f64(max_f64(u.x, u.y), max_f64(v.x, v.y));
        }
        wave_sync();
        for (int j = 1; j < p.levels; ++j) {
            const double *prev = tab + (size_t)(j - 1) * nb;
            double *cur = tab + (size_t)j * nb;
            const int h = 1 << (j - 1);
            for (int i = lane; i < nb; i += 64) cur[i] = max_f64(prev[i], prev[min(i + h, nb - 1)]);
            wave_sync();
        }
        const auto range_max = [&](double m, int lo, int hi) {
            const int b_lo = (lo + 3) >> 2, b_hi = hi >> 2;
            const int e1 = min(4 * b_lo, hi), s2 = max(4 * b_hi, e1);
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                if (lo + u < e1) m = max_f64(m, arr[lo + u]);
                if (s2 + u < hi) m = max_f64(m, arr[s2 + u]);
            }
            if (b_lo < b_hi) {
                const int j = 31 - __builtin_clz(b_hi - b_lo);
                const double *lv = tab + (size_t)j * nb;
                m = max_f64(m, max_f64(lv[b_lo], lv[b_hi - (1 << j)]));
            }
            return m;
        };
        double rho[KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) rho[k] = 0.0;
        if (p.depT) {
            // Rows of many runs: most hold one of the recvs that arrive late.  The maximum over those of them that the row holds
            // is the maximum over the row, whatever the line between late and not.  32 recvs at a time, whose part of the rows is in
            // registers meanwhile.
            const double line = last_arrival * max(0.0, 1.0 - 32.0 / R);
            for (int h = 0; 32 * h < R; ++h) {
                const double x = lane < 32 && 32 * h + lane < R ? arr[32 * h + lane] : -1.0;
                uint32_t late = (uint32_t)__ballot(x >= line);
                if (!late) continue;
                uint32_t row[KT];
#pragma unroll
                for (int k = 0; k < KT; ++k)
                    row[k] = p.depT[((size_t)(h >> 1) * p.Cpad + min(k * 64, p.Cpad - 64) + lane) * 2 + (h & 1)];
                for (; late != 0u; late &= late - 1u) {
                    const int i = __builtin_ctz(late);
                    const double at_r = readlane_f64(x, i);
#pragma unroll
                    for (int k = 0; k < KT; ++k)
                        if ((row[k] >> i & 1u) && at_r > rho[k]) rho[k] = at_r;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            double m = rho[k];
            const uint32_t ra = runs_l[k * 64 + lane], rc = runs_l[(KT + k) * 64 + lane];
            const int n = m > 0.0 ? 0 : (int)(ra >> 20);
            if (n > 0) m = range_max(m, (int)(ra & 1023u), (int)((ra >> 10) & 1023u));
            if (n > 1) m = range_max(m, (int)(rc & 1023u), (int)(rc >> 10));
            if (n > 2) {
                const int q = p.run_ptr[lane * cls_lane + k * cls_slot];
                int lo = p.run_lo[q + 2], hi = p.run_hi[q + 2];
                for (int i = 3;; ++i) {             // (the next run on its way)
                    const int next = q + min(i, n - 1), lo1 = p.run_lo[next], hi1 = p.run_hi[next];
                    m = range_max(m, lo, hi);
                    if (i >= n) break;
                    lo = lo1;
                    hi = hi1;
                }
            }
            rho[k] = m;
            if constexpr (KT > 4) __builtin_amdgcn_sched_barrier(0);        // (slots one after the other: fewer registers)
        }
        wave_sync();

        // ---- the compute device: makespan = max over classes of (release date + time of the classes released
        // then or later) ----
        // the rank of a release date is the number of arrivals up to it, one branch-free binary
        // search per channel (release dates are arrivals, so a later release date has a higher rank and equal
        // ones the same); the class times are added up by rank, a suffix sum over the ranks follows
        double *A = arr;                    // [R + 1] by rank (the arrivals and the table are not read any more)
        for (int j = lane; j <= R; j += 64) A[j] = 0.0;
#pragma unroll
        for (int k = 0; k < D; ++k)         // (an order that is no permutation cannot write past the channel's share)
            if (of[k] >= 0 && of[k] >> 16 < clen[(of[k] >> 10) & 63]) lists[coff[(of[k] >> 10) & 63] + (of[k] >> 16)] = a[k];
        wave_sync();
        int rank[KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) rank[k] = 0;
        for (int c = 0; c < p.n_channels; ++c) {
            const int len = min(__builtin_amdgcn_readlane(queued, c), __builtin_amdgcn_readfirstlane(clen[c]));
            if (len == 0) continue;
            const double *lc = lists + __builtin_amdgcn_readfirstlane(coff[c]);
            // `left` arrivals from pos on may still be up to rho, all before are
            int pos[KT];
#pragma unroll
            for (int k = 0; k < KT; ++k) pos[k] = 0;
            for (int left = len; left > 1;) {
                const int half = left >> 1;
#pragma unroll
                for (int k = 0; k < KT; ++k) pos[k] += lc[pos[k] + half - 1] <= rho[k] ? half : 0;
                left -= half;
            }
#pragma unroll
            for (int k = 0; k < KT; ++k) rank[k] += pos[k] + (lc[pos[k]] <= rho[k] ? 1 : 0);
        }
        wave_sync();
        double ct_sum = 0.0, together = 0.0;
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            ct_sum += ct[k];
            together += ct[k];
            // (a lane without a class in this slot has none in the later ones either; its time is zero)
            if (lane * cls_lane + k * cls_slot < C &&
                (k == KT - 1 || rank[min(k + 1, KT - 1)] != rank[k] || lane * cls_lane + (k + 1) * cls_slot >= C)) {
                atomicAdd(&A[rank[k]], together);
                together = 0.0;
            }
        }
        wave_sync();
        const double sum_c = wave_sum_f64_dpp(ct_sum);
        // ranks 1 .. R; of rank 0 are classes that are there from the start, with all the class time ahead
        double S[D];
#pragma unroll
        for (int k = D - 1; k >= 0; --k) {
            S[k] = lane * D + k < R ? A[lane * D + k + 1] : 0.0;
            if (k < D - 1) S[k] += S[k + 1];
        }
        const double S_incl = wave_incl_scan_f64_dpp(S[0]), S_after = lane63_f64(S_incl) - S_incl;
        if (lane == 0) A[0] = sum_c;
#pragma unroll
        for (int k = 0; k < D; ++k)
            if (lane * D + k < R) A[lane * D + k + 1] = S_after + S[k];         // this rank and every later one
        wave_sync();
        double mloc = last_arrival;
#pragma unroll
        for (int k = 0; k < KT; ++k)
            if (lane * cls_lane + k * cls_slot < C) mloc = max_f64(mloc, rho[k] + A[rank[k]]);
        const double m = wave_max_f64_dpp(mloc);
        if (lane == 0) {
            const double U = sum_c + sum_r;
            const double L = max_f64(sum_c, last_arrival);
            p.makespan[b] = m;
            p.eff[b] = (U == L) ? 1.0 : (U - m) / (U - L);
            if (p.U) p.U[b] = U;
            if (p.L) p.L[b] = L;
            if (p.S) p.S[b] = (U == L || L == 0.0) ? 0.0 : (U - L) / L;
        }
    }
    if (bad) atomicOr(p.bad_order, 1);
}

template <int KT, Sums HOW>
static hipError_t launch_sim_chan(SimChanParams &p, const Dag &d, hipStream_t s)
{
    const int nb = (d.R + 3) / 4;
    int levels = 1;
    while ((1 << levels) <= nb) ++levels;             // floor(log2 nb) + 1 levels of the table of block maxima
    p.levels = levels;
    p.nb = nb;
    // the class totals, the transfer times, the table, the arrivals by channel
    const size_t x_doubles = (std::max(std::max((size_t)64 * KT, (size_t)d.R), (size_t)levels * nb) + 1) & ~(size_t)1;
    const size_t arr_doubles = ((size_t)4 * nb + 2) & ~(size_t)1;             // (sums by rank: one more than there are recvs)
    p.arr_doubles = (int32_t)arr_doubles;
    const size_t wave_bytes = (arr_doubles + x_doubles) * 8;                    // a multiple of 16
    // (more than two runs per row: the late recvs first.  65 536 samples, four channels, an order each, us without and with: three
    // runs (tiny) 100 either way; 4.5 (9 x 17 layered ops, 18 recvs) 190 and 155; seven (18 x 17 and 45) 353 and 234; 57 (24 x 20
    // and 300) 5 622 and 1 699.  The parts of the rows in registers: with a word from memory for every late recv and slot the last
    // took 1 868, and one order that leaves many recvs late, one channel, 11 x 4 ops, 48 recvs, 60 000 samples 172 instead of 119,
    // against 147 run by run)
    const bool many = d.n_runs > 2 * d.C;
    p.depT = many ? reinterpret_cast<const uint32_t *>(d.d_cls_depT) : nullptr;
    p.Cpad = d.Cpad;
    p.cls_lane = many ? 1 : KT;
    p.cls_slot = many ? 64 : 1;
    int waves = 4;
    while (waves > 1 && wave_bytes * waves > 40 * 1024) waves >>= 1;
    const size_t chan_bytes = (((size_t)d.R + 128 + 2 * 64 * KT) * 4 + 15) & ~(size_t)15;
    const size_t lds = chan_bytes + wave_bytes * waves;
    if (lds > 150 * 1024) return hipErrorNotSupported;     // 160 KB of LDS per compute unit
    p.wave_bytes = (int32_t)wave_bytes;
    p.chan_bytes = (int32_t)chan_bytes;
    hipError_t e;
    if (lds > 48 * 1024) {
        e = ensure_dynamic_lds(reinterpret_cast<const void *>(simulate_channels_kernel<KT, HOW>), lds);
        if (e != hipSuccess) return e;
    }
    int per_cu = 0;
    e = cached_blocks_per_cu(&per_cu, reinterpret_cast<const void *>(simulate_channels_kernel<KT, HOW>), 64 * waves, lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
    const int n_cu = device_cu_count(d.device);
    int grid = per_cu * n_cu;
    const int need = (p.B + waves - 1) / waves;
    if (grid > need) grid = need;
    p.n_waves = grid * waves;
    hipLaunchKernelGGL((simulate_channels_kernel<KT, HOW>), dim3(grid), dim3(64 * waves), lds, s, p);
    return hipGetLastError();
}

hipError_t launch_simulate_channels(Dag &d, const SimArgs &a, int32_t n_channels, const int32_t *chan, hipStream_t s)
{
    if (a.B == 0) return hipSuccess;
    const int K = std::max((d.C + 63) / 64, (d.R + 63) / 64);   // slots per lane: classes, and positions of the order
    const int KT = K < 1 ? 1 : K;
    if (d.R == 0 || d.R > 512 || K > 8 || n_channels > 64 || (d.C > 0 && (!d.d_col_cls || !d.d_run_ptr))) return hipErrorNotSupported;
    if (!d.d_bad_order || !a.order) return hipErrorInvalidValue;
    SimChanParams p{};
    p.bad_order = d.d_bad_order;
    p.B = a.B; p.R = d.R; p.C = d.C; p.N = d.N; p.n_channels = n_channels;
    p.col_cls = d.d_col_cls; p.run_ptr = d.d_run_ptr; p.run_lo = d.d_run_lo; p.run_hi = d.d_run_hi;
    p.chan = chan; p.order = a.order; p.order_stride = a.order_stride;
    p.op_time = a.op_time; p.recv_time = a.recv_time; p.f32 = a.f32 ? 1 : 0;
    p.makespan = a.makespan; p.eff = a.eff; p.U = a.U; p.L = a.L; p.S = a.S;
    const bool quads = d.long_runs;
    switch (KT) {
    case 1: return launch_sim_chan<1, Sums::plain>(p, d, s);
    case 2: return launch_sim_chan<2, Sums::plain>(p, d, s);
    case 3: return launch_sim_chan<3, Sums::plain>(p, d, s);
    case 4: return launch_sim_chan<4, Sums::plain>(p, d, s);
    case 5: return quads ? launch_sim_chan<5, Sums::quads>(p, d, s) : launch_sim_chan<5, Sums::plain>(p, d, s);
    case 6: return quads ? launch_sim_chan<6, Sums::quads>(p, d, s) : launch_sim_chan<6, Sums::plain>(p, d, s);
    case 7: return quads ? launch_sim_chan<7, Sums::quads>(p, d, s) : launch_sim_chan<7, Sums::plain>(p, d, s);
    default: return quads ? launch_sim_chan<8, Sums::quads>(p, d, s) : launch_sim_chan<8, Sums::plain>(p, d, s);
    }
}

// Straggler effect of groups of w consecutive samples (Sec. 6): (max - min) / max of their
// makespans.  A group is spread over the lanes of one wave (w > 4) or handled by one thread.
__global__ void __launch_bounds__(256)
straggler_kernel(int32_t n_groups, int32_t w, const double *__restrict__ makespan, double *__restrict__ out)
{
    if (w <= 4) {
        const int g = blockIdx.x * blockDim.x + threadIdx.x;
        if (g >= n_groups) return;
        double mx = makespan[(size_t)g * w], mn = mx;
        for (int i = 1; i < w; ++i) {
            const double m = makespan[(size_t)g * w + i];
            mx = max_f64(mx, m);
            mn = min_f64(mn, m);
        }
        out[g] = mx > 0.0 ? (mx - mn) / mx : 0.0;
        return;
    }
    const int lane = threadIdx.x & 63;
    const int g = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);     // wave-uniform
    if (g >= n_groups) return;
    double mx = -TT_INF, mn = TT_INF;
    for (int i = lane; i < w; i += 64) {
        const double m = makespan[(size_t)g * w + i];
        mx = max_f64(mx, m);
        mn = min_f64(mn, m);
    }
    mx = wave_max_f64_dpp(mx);
    mn = wave_min_f64_dpp(mn);
    if (lane == 0) out[g] = mx > 0.0 ? (mx - mn) / mx : 0.0;
}

hipError_t launch_straggler(int32_t B, int32_t w, const double *makespan, double *out, hipStream_t s)
{
    const int32_t n_groups = B / w;
    if (n_groups == 0) return hipSuccess;
    const int per_block = w <= 4 ? 256 : 4;
    hipLaunchKernelGGL(straggler_kernel, dim3((n_groups + per_block - 1) / per_block), dim3(256), 0, s,
                       n_groups, w, makespan, out);
    return hipGetLastError();
}

// Time oracle estimator (Sec. 5): time[i] = minimum over the measured runs of runs[k][i].
// A streaming kernel: every element is read once per run; two doubles per lane and load.
__global__ void __launch_bounds__(256)
time_oracle_min_kernel(int32_t n_runs, int64_t n, bool pairs_ok, const double *__restrict__ runs,
                       double *__restrict__ time)
{
    const int64_t n2 = n >> 1;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if (pairs_ok) {
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += stride) {
            double2 m = reinterpret_cast<const double2 *>(runs)[i];
            for (int k = 1; k < n_runs; ++k) {
                const double2 x = reinterpret_cast<const double2 *>(runs + (size_t)k * n)[i];
                m.x = min_f64(m.x, x.x);
                m.y = min_f64(m.y, x.y);
            }
            reinterpret_cast<double2 *>(time)[i] = m;
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
            double m = runs[i];
            for (int k = 1; k < n_runs; ++k) m = min_f64(m, runs[(size_t)k * n + i]);
            time[i] = m;
        }
    }
}

hipError_t launch_time_oracle_min(int32_t n_runs, int64_t n, const double *runs, double *time, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    // pairs when every row starts on a 16-byte boundary
    const bool pairs_ok = (n & 1) == 0 && ((reinterpret_cast<uintptr_t>(runs) | reinterpret_cast<uintptr_t>(time)) & 15) == 0;
    const int64_t work = pairs_ok ? n / 2 : n;
    int64_t blocks = (work + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;          // 32 workgroups per compute unit, grid-stride beyond
    hipLaunchKernelGGL(time_oracle_min_kernel, dim3((unsigned)blocks), dim3(256), 0, s, n_runs, n, pairs_ok, runs, time);
    return hipGetLastError();
}

hipError_t launch_simulate(Dag &d, const SimArgs &a, hipStream_t s)
{
    if (a.B == 0) return hipSuccess;
    {
        const hipError_t e = launch_simulate_lanes(d, a, s);
        if (e != hipErrorNotSupported) return e;
    }
    SimKernelParams p{};
    p.B = a.B; p.R = d.R; p.W = d.W; p.C = d.C; p.N = d.N;
    p.cls_dep = d.d_cls_dep; p.cls_ptr = d.d_cls_ptr; p.cls_cols = d.d_cls_cols;
    p.order = a.order; p.order_stride = a.order_stride; p.kappa = nullptr;
    p.op_time = a.op_time; p.recv_time = a.recv_time; p.f32 = a.f32 ? 1 : 0;
    p.makespan = a.makespan; p.eff = a.eff; p.U = a.U; p.L = a.L; p.S = a.S;
    const bool shared = a.order_stride == 0 && d.R > 0 && d.C > 0;
    int32_t *kappa_col = nullptr;
    if (shared) {
        const size_t lds = ((size_t)d.R + kKappaBlock) * 4;
        if (!d.d_bad_order || lds > 48 * 1024) return hipErrorInvalidValue;
        // (where there is no room for a word per column, also on a stream that is being captured: by class, in the last kernel)
        const size_t by_class = (size_t)d.C * sizeof(int32_t), by_col = by_class + (3 + (size_t)d.N) * sizeof(int32_t);
        bool cols = d.R <= 512 && !(by_col > d.work_bytes && being_captured(s));
        hipError_t e = ensure_workspace(&d, cols ? by_col : by_class);
        if (e == hipErrorOutOfMemory && cols) {
            cols = false;
            e = ensure_workspace(&d, by_class);
        }
        if (e != hipSuccess) return e;
        int32_t *kappa = static_cast<int32_t *>(d.d_work);
        if (cols) kappa_col = kappa + ((d.C + 3) & ~3);         // (read four at a time)
        hipLaunchKernelGGL(kappa_kernel, dim3((d.C + kKappaBlock - 1) / kKappaBlock), dim3(256), lds, s, d.R, d.W, d.C, d.d_cls_dep,
                           a.order, d.d_cls_ptr, d.d_cls_cols, d.d_col_cls, kappa, kappa_col, d.d_bad_order);
        p.kappa = kappa;
    }
    // An order each, more than 2 048 classes, no more samples than compute units: sixteen waves per sample rather than one, which
    // walks over the classes by itself.  64 / 256 / 384 samples, us, by sixteen waves and by recv: 3 465 classes, 300 recvs 74 /
    // 79 / 143 and 116 / 126 / 137; 3 815, 128 recvs 89 / 172 / 318 and 183 / 210 / 209; 8 016, 400 recvs 263 / 306 / 572 and 377 /
    // 341 / 379; 13 666, 500 recvs 407 / 417 / 812 and 471 / 478 / 775.  With rows of one word it is by recv at any size: 2 033, 64
    // recvs 105 / 154 / 293 and 92 / 101 / 109.
    const bool wide = !shared && d.C > 2048 && d.W > 1 && a.B <= device_cu_count(d.device);
    if ((!shared && !wide) || kappa_col) {
        const hipError_t e = try_simulate_wave(d, a, kappa_col, s);
        if (e != hipErrorNotSupported) return e;
    }
    if (!shared) {
        const hipError_t e = launch_check_orders(d, a.B, a.order, a.order_stride, s);
        if (e != hipSuccess) return e;
    }
    const size_t lds = ((size_t)(d.R + 1) * 2 + 16) * 8 + (size_t)d.R * 4;
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    if (d.C <= 2048 && lds <= 40 * 1024) {
        const int grid = a.B < 256 * 16 ? a.B : 256 * 16;
        return launch_sim_t<64>(p, grid, lds, s);
    }
    const int grid = a.B < 256 * 2 ? a.B : 256 * 2;
    return launch_sim_t<1024>(p, grid, lds, s);
}

// ---- orders given by the caller ----
// One wave per order: every entry in 0 .. R-1 and none twice (a bit per recv in LDS), else the flag is raised.
// The simulations and the search skip entries out of range themselves; what they return for such a row is unspecified.
__global__ void __launch_bounds__(256)
check_orders_kernel(int32_t R, int32_t rows, const int32_t *__restrict__ order, int32_t stride, int32_t *flag)
{
    extern __shared__ uint32_t seen_all[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, words = (R + 31) >> 5;
    uint32_t *seen = seen_all + (size_t)wave * words;
    bool bad = false;
    for (int b = blockIdx.x * 4 + wave; b < rows; b += gridDim.x * 4) {
        const int32_t *ord = order + (size_t)b * stride;
        for (int i = lane; i < words; i += 64) seen[i] = 0;
        wave_sync();
        for (int k = lane; k < R; k += 64) {
            const int r = ord[k];
            if ((unsigned)r >= (unsigned)R) { bad = true; continue; }
            const uint32_t bit = 1u << (r & 31);
            if (atomicOr(&seen[r >> 5], bit) & bit) bad = true;
        }
        wave_sync();
    }
    if (bad) atomicOr(flag, 1);
}

hipError_t launch_check_orders(Dag &d, int32_t B, const int32_t *order, int32_t order_stride, hipStream_t s)
{
    if (d.R <= 0 || B <= 0 || !order) return hipSuccess;
    if (!d.d_bad_order) return hipErrorInvalidValue;
    const int rows = order_stride == 0 ? 1 : B;
    const size_t lds = (size_t)4 * ((d.R + 31) / 32) * 4;
    if (lds > 48 * 1024) return hipErrorInvalidValue;
    const int blocks = std::min((rows + 3) / 4, 8 * device_cu_count(d.device));
    hipLaunchKernelGGL(check_orders_kernel, dim3(blocks), dim3(256), lds, s, d.R, rows, order, order_stride, d.d_bad_order);
    return hipGetLastError();
}

}  // namespace tictac
