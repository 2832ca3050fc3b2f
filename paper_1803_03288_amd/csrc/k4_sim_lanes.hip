// One iteration under a transfer order (Sec. 3.2; definitions in k4_simulate.hip) for graphs so small that the timing rows
// of 64 samples fit LDS: one *lane* per sample.  A wave per sample, as in k4_simulate.hip, spends hundreds of
// instructions on the few hundred bytes of such a sample; here each instruction serves 64 samples.
//
// A wave takes 64 samples at a time: their rows (consecutive in memory) go to LDS transposed, [column][sample], so that
// lane l reads its own sample without bank conflicts.
//   * One order for all samples: the iteration is one sequence of events, the same for every sample: the columns that
//     depend on no recv, the first transfer, the columns released by it, ...  The wave forms the sequence once, keeps it in
//     registers, and a sample is F += x, busy = max(busy, F) for a transfer and busy += x for a column.
//   * An order per sample: positions per sample in LDS, kappa of a class as the maximum over its row, the class times added
//     up by kappa in LDS, then the same recurrence by position.
// Orders are checked on the way (tictac_dag_check_orders), which saves a launch.
// Bound by the latency of the loads of a tile (few waves fit a compute unit) and, with an order each, by LDS.
#include <algorithm>

#include "device_utils.h"
#include "internal.h"

namespace tictac {

struct SimLanesParams {
    int32_t B, N, R, W, C, n_groups;
    const uint64_t *cls_dep;            // [C][W]
    const int32_t *cls_ptr, *cls_cols, *col_cls;
    const int32_t *order;
    int32_t order_stride;
    const void *op_time, *recv_time;
    double *makespan, *eff, *U, *L, *S;
    int32_t *bad_order;
    int32_t prog_items;
};

constexpr int kLaneCols = 256;          // columns and recvs of a sample at the most: four registers of events

// rows of 64 samples, [width] elements each, into tile[(first + c) * 65 + sample]
template <typename T>
__device__ __forceinline__ void rows_to_lds(T *tile, int first, const T *__restrict__ src, int width, int b0, int B, int lane)
{
    constexpr int VEC = 16 / (int)sizeof(T), LPR = 16, TC = LPR * VEC, RPI = 64 / LPR, NI = 64 / RPI;
    typedef T Vec __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));
    const int sub = (lane % LPR) * VEC, lr = lane / LPR;
    const bool whole = b0 + 64 <= B;
    for (int c0 = 0; c0 < width; c0 += TC) {
        Vec v[NI];
        const int left = width - c0 - sub;              // elements from this lane's first on
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const T *q = src + (size_t)(whole ? b0 + i * RPI + lr : min(b0 + i * RPI + lr, B - 1)) * width + c0 + sub;
            if (left >= VEC) {
                v[i] = *reinterpret_cast<const Vec *>(q);
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) v[i][e] = e < left ? q[e] : T(0);
            }
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (e < left) tile[(first + c0 + sub + e) * 65 + i * RPI + lr] = v[i][e];
    }
}

__device__ __forceinline__ void write_metrics(const SimLanesParams &p, int b, double m, double sum_c, double F)
{
    if (b >= p.B) return;
    const double U = sum_c + F;
    const double L = max_f64(sum_c, F);
    p.makespan[b] = m;
    p.eff[b] = (U == L) ? 1.0 : (U - m) / (U - L);
    if (p.U) p.U[b] = U;
    if (p.L) p.L[b] = L;
    if (p.S) p.S[b] = (U == L || L == 0.0) ? 0.0 : (U - L) / L;
}

// TILES > 0: the rows of the next 64 samples are requested into registers before those in LDS are computed, as TILES pieces
// of 256 bytes of the op_time rows and one of the recv_time rows; 0: longer rows are brought when they are needed.  All waves
// of a compute unit start together, so without that they load together and compute together: vgg16 as above spent 23 us
// loading, 16 computing and 9 before the first sample, 49 in all; now the first rows come while the events are formed and
// the others while samples are computed: 35 us.  All loads are executed without a branch, a lane past the end of a row reads
// its last columns once more.
template <typename T, int TILES>
__global__ void __launch_bounds__(64)
simulate_lanes_shared_kernel(const SimLanesParams p)
{
    extern __shared__ char lanes_smem[];
    const int N = p.N, R = p.R, W = p.W, C = p.C, lane = threadIdx.x;
    constexpr int VEC = 16 / (int)sizeof(T), LPR = 16, TC = LPR * VEC, RPI = 64 / LPR, NI = 64 / RPI;
    typedef T Vec __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));
    const int sub = (lane % LPR) * VEC, lr = lane / LPR;
    Vec ahead[TILES + 1][NI];
    auto request = [&](int g) __attribute__((always_inline)) {
        const int last = min(63, p.B - 1 - g * 64);
        const T *op = static_cast<const T *>(p.op_time) + (size_t)g * 64 * N, *rv = static_cast<const T *>(p.recv_time) + (size_t)g * 64 * R;
#pragma unroll
        for (int t = 0; t <= TILES; ++t)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int row = min(i * RPI + lr, last);
                ahead[t][i] = t < TILES ? *reinterpret_cast<const Vec *>(op + (row * N + min(t * TC + sub, N - VEC)))
                                        : *reinterpret_cast<const Vec *>(rv + (row * R + min(sub, R - VEC)));
            }
    };
    if (TILES > 0) request(blockIdx.x);
    T *tile = reinterpret_cast<T *>(lanes_smem);        // [N + R + 1][65]: columns, recvs, zeros
    // ---- the events, formed in the space of the tile: tile row | 0x8000 for a transfer ----
    int32_t *pos = reinterpret_cast<int32_t *>(lanes_smem);     // [R] 1-based position, 0: left out
    int32_t *off = pos + R;                             // [R + 1] columns by kappa, then where they start
    int32_t *kap = off + R + 1;                         // [C]
    int32_t *seq = kap + C;                             // [N + R, a multiple of 8]
    const int n_ev = N + R, n_pad = (n_ev + 7) & ~7;
    for (int i = lane; i < R; i += 64) pos[i] = 0;
    for (int i = lane; i <= R; i += 64) off[i] = 0;
    for (int i = lane; i < n_pad; i += 64) seq[i] = n_ev;                // (a column of zeros)
    wave_sync();
    bool bad = false;
    for (int k = lane; k < R; k += 64) {
        const int r = p.order[k];
        if ((unsigned)r >= (unsigned)R) bad = true;
        else bad |= atomicExch(&pos[r], k + 1) != 0;
    }
    if (bad && blockIdx.x == 0) atomicOr(p.bad_order, 1);
    wave_sync();
    for (int c = lane; c < C; c += 64) {
        int m = 0;
        for (int w = 0; w < W; ++w)
            for (uint64_t x = p.cls_dep[(size_t)c * W + w]; x; x &= x - 1) m = max(m, pos[w * 64 + __builtin_ctzll(x)]);
        kap[c] = m;
    }
    wave_sync();
    for (int j = lane; j < N; j += 64) atomicAdd(&off[kap[p.col_cls[j]]], 1);
    wave_sync();
    // off[k] = events before the columns of kappa k: the columns of smaller kappa and k transfers
    int carry = 0;
    for (int k0 = 0; k0 <= R; k0 += 64) {
        const int k = k0 + lane, n = k <= R ? off[k] : 0;
        int incl = n;
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(incl, d);
            if (lane >= d) incl += v;
        }
        if (k <= R) off[k] = carry + incl - n + k;
        carry += __builtin_amdgcn_readlane(incl, 63);
    }
    wave_sync();
    for (int k = lane; k < R; k += 64) {
        const int r = p.order[k];
        seq[off[k + 1] - 1] = ((unsigned)r < (unsigned)R ? N + r : n_ev) | 0x8000;
    }
    wave_sync();
    for (int j0 = 0; j0 < N; j0 += 64)
        if (j0 + lane < N) seq[atomicAdd(&off[kap[p.col_cls[j0 + lane]]], 1)] = j0 + lane;
    wave_sync();
    int ev[kLaneCols / 64];
#pragma unroll
    for (int q = 0; q < kLaneCols / 64; ++q) ev[q] = q * 64 + lane < n_pad ? seq[q * 64 + lane] : n_ev;
    wave_sync();
    tile[n_ev * 65 + lane] = T(0);

    for (int g = blockIdx.x; g < p.n_groups; g += gridDim.x) {
        const int b0 = g * 64;
        wave_sync();                                    // the rows of the group before are not read any more
        if constexpr (TILES > 0) {
#pragma unroll
            for (int t = 0; t <= TILES; ++t) {
                const int first = t < TILES ? 0 : N, width = t < TILES ? N : R, c = t < TILES ? t * TC + sub : sub;
                if (c < width) {                        // (the last lane of a row may repeat columns of the one before)
                    T *to = tile + (first + min(c, width - VEC)) * 65 + lr;
#pragma unroll
                    for (int i = 0; i < NI; ++i)
#pragma unroll
                        for (int e = 0; e < VEC; ++e) to[e * 65 + i * RPI] = ahead[t][i][e];
                }
            }
            wave_sync();
            if (g + (int)gridDim.x < p.n_groups) request(g + gridDim.x);
        } else {
            rows_to_lds(tile, 0, static_cast<const T *>(p.op_time), N, b0, p.B, lane);
            rows_to_lds(tile, N, static_cast<const T *>(p.recv_time), R, b0, p.B, lane);
            wave_sync();
        }
        double F = 0.0, busy = 0.0, sum_c = 0.0;
#pragma unroll
        for (int q = 0; q < kLaneCols / 64; ++q) {
            const int n = min(64, n_pad - q * 64);
            for (int i0 = 0; i0 < n; i0 += 8) {
                int e[8];
                double x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    e[i] = __builtin_amdgcn_readlane(ev[q], i0 + i);
                    x[i] = (double)tile[(e[i] & 0x7fff) * 65 + lane];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (e[i] & 0x8000) {
                        F += x[i];
                        busy = max_f64(busy, F);
                    } else {
                        busy += x[i];
                        sum_c += x[i];
                    }
                }
            }
        }
        write_metrics(p, b0 + lane, busy, sum_c, F);
    }
}

// What the samples of an order each have in common is a program over the rows of the tile, formed once per wave and fetched
// 64 items at a time: for every class the positions of its recvs to take the maximum of (those it has beyond the class
// before it, where that one's row is a subset) and the columns to add up.  Positions are kept in the tile, in its type, so
// that eight items can be read from LDS before the first is needed.
enum : int { LN_ROW = 0x3ff, LN_POS = 0x400, LN_FROM_ZERO = 0x800, LN_LAST = 0x1000 };

template <typename T>
__global__ void __launch_bounds__(64)
simulate_lanes_kernel(const SimLanesParams p)
{
    extern __shared__ char lanes_smem[];
    const int N = p.N, R = p.R, W = p.W, C = p.C, lane = threadIdx.x;
    uint16_t *prog = reinterpret_cast<uint16_t *>(lanes_smem);          // [prog_items]
    double *A = reinterpret_cast<double *>(lanes_smem + (size_t)p.prog_items * 2);      // [R + 1][64] class time by kappa
    T *tile = reinterpret_cast<T *>(A + (R + 1) * 64);                  // [N + 2 R][65]: columns, recvs, positions by recv
    int32_t *ord = reinterpret_cast<int32_t *>(A);                      // [R][65] the orders, where A is not in use yet
    int32_t *ord2 = reinterpret_cast<int32_t *>(tile);                  // the same, once the columns are not read any more
    // ---- the program ----
    int n_items = 0;
    for (int c0 = 0; c0 < C; c0 += 64) {
        const int c = c0 + lane;
        int len = 0;
        bool subset = c > 0 && c < C;
        if (c < C) {
            const uint64_t *row = p.cls_dep + (size_t)c * W, *before = row - (subset ? W : 0);
            for (int w = 0; w < W && subset; ++w) subset = (before[w] & ~row[w]) == 0ull;
            for (int w = 0; w < W; ++w) len += __popcll(subset ? row[w] & ~before[w] : row[w]);
            len += p.cls_ptr[c + 1] - p.cls_ptr[c];
        }
        int incl = len;
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(incl, d);
            if (lane >= d) incl += v;
        }
        if (c < C) {
            int at = n_items + incl - len;
            const int first = at;
            const uint64_t *row = p.cls_dep + (size_t)c * W, *before = row - (subset ? W : 0);
            for (int w = 0; w < W; ++w)
                for (uint64_t x = subset ? row[w] & ~before[w] : row[w]; x; x &= x - 1)
                    prog[at++] = (uint16_t)((N + R + w * 64 + __builtin_ctzll(x)) | LN_POS);
            for (int q = p.cls_ptr[c]; q < p.cls_ptr[c + 1]; ++q) prog[at++] = (uint16_t)p.cls_cols[q];
            if (!subset) prog[first] |= LN_FROM_ZERO;
            prog[at - 1] |= LN_LAST;                    // (every class has a column)
        }
        n_items += __builtin_amdgcn_readlane(incl, 63);
    }
    wave_sync();
    bool bad = false;
    for (int g = blockIdx.x; g < p.n_groups; g += gridDim.x) {
        const int b0 = g * 64;
        const int32_t *order = p.order;
        wave_sync();                                    // LDS of the group before is not read any more
        rows_to_lds(ord, 0, order, R, b0, p.B, lane);
        rows_to_lds(tile, 0, static_cast<const T *>(p.op_time), N, b0, p.B, lane);
        rows_to_lds(tile, N, static_cast<const T *>(p.recv_time), R, b0, p.B, lane);
        T *pos = tile + (N + R) * 65 + lane;            // 1-based; 0 for a recv that an invalid order leaves out
        for (int r = 0; r < R; ++r) pos[r * 65] = T(0);
        wave_sync();
        for (int k0 = 0; k0 < R; k0 += 8) {
            int r[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) r[i] = ord[min(k0 + i, R - 1) * 65 + lane];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (k0 + i < R && (unsigned)r[i] < (unsigned)R) pos[r[i] * 65] = T(k0 + i + 1);
        }
        wave_sync();
        // ---- class times by kappa ----
        for (int k = 0; k <= R; ++k) A[k * 64 + lane] = 0.0;
        double sum_c = 0.0, s = 0.0;
        T m = T(0);                                     // kappa of the class (of the one before, at its first item)
        for (int q = 0; q < n_items; q += 64) {
            const int items = q + lane < n_items ? (int)prog[q + lane] : 0;
            const int n = min(64, n_items - q);
            for (int i0 = 0; i0 < n; i0 += 8) {
                int e[8];
                T x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    e[i] = __builtin_amdgcn_readlane(items, i0 + i);
                    x[i] = tile[(e[i] & LN_ROW) * 65 + lane];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (i0 + i >= n) break;
                    if (e[i] & LN_FROM_ZERO) m = T(0);
                    if (e[i] & LN_POS) m = x[i] > m ? x[i] : m;
                    else s += (double)x[i];
                    if (e[i] & LN_LAST) {
                        A[(int)m * 64 + lane] += s;
                        sum_c += s;
                        s = 0.0;
                    }
                }
            }
        }
        // ---- the iteration, position by position, with the check of the order: entry k names a recv whose place is k ----
        wave_sync();
        rows_to_lds(ord2, 0, order, R, b0, p.B, lane);
        wave_sync();
        double F = 0.0, busy = A[lane];
        for (int k0 = 0; k0 < R; k0 += 8) {
            int r[8];
            T x[8], at[8];
            double a[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) r[i] = ord2[min(k0 + i, R - 1) * 65 + lane];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int ri = (unsigned)r[i] < (unsigned)R ? r[i] : 0;
                x[i] = tile[(N + ri) * 65 + lane];
                at[i] = pos[ri * 65];
                a[i] = A[min(k0 + i + 1, R) * 64 + lane];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (k0 + i >= R) break;
                const bool ok = (unsigned)r[i] < (unsigned)R;
                bad |= !ok || at[i] != T(k0 + i + 1);
                F += ok ? (double)x[i] : 0.0;
                busy = max_f64(busy, F) + a[i];
            }
        }
        write_metrics(p, b0 + lane, busy, sum_c, F);
    }
    if (bad) atomicOr(p.bad_order, 1);
}

template <typename T>
static hipError_t launch_lanes_t(SimLanesParams &p, const Dag &d, hipStream_t s)
{
    const bool shared = p.order_stride == 0;
    size_t lds;
    if (shared) {
        const size_t prep = ((size_t)2 * p.R + 1 + p.C + p.N + p.R + 8) * 4;
        lds = std::max((size_t)(p.N + p.R + 1) * 65 * sizeof(T), prep);
    } else {
        // (the program holds at most one item per set bit of the class rows and per column)
        const int64_t items = (d.cls_nnz + p.N + 7) & ~(int64_t)7;
        if (items > 2048 || p.N + 2 * p.R > LN_ROW) return hipErrorNotSupported;
        p.prog_items = (int32_t)items;
        lds = (size_t)items * 2 + (size_t)(p.R + 1) * 64 * 8 + (size_t)(p.N + 2 * p.R) * 65 * sizeof(T);
        if ((size_t)p.R * 4 > (size_t)p.N * sizeof(T)) return hipErrorNotSupported;     // (the orders in the place of the columns)
    }
    lds = (lds + 15) & ~(size_t)15;
    // (two waves per compute unit at the least)
    if (lds > 80 * 1024) return hipErrorNotSupported;
    // The rows of the next 64 samples are requested ahead where they fit registers: three pieces of 64 rows, 192, are what a wave has
    // beside its own at two waves per SIMD.  That is up to 64 columns and 32 recvs in float64, 128 and 64 in float32; wider samples are loaded when
    // the wave comes to them.
    constexpr int VEC = 16 / (int)sizeof(T), TC = 16 * VEC;
    const bool fits = p.N >= VEC && p.R >= VEC && p.N <= 2 * TC && p.R <= TC;
    void (*const kernel)(SimLanesParams) = !shared ? simulate_lanes_kernel<T> : !fits ? simulate_lanes_shared_kernel<T, 0>
                                           : p.N <= TC ? simulate_lanes_shared_kernel<T, 1> : simulate_lanes_shared_kernel<T, 2>;
    const void *kern = reinterpret_cast<const void *>(kernel);
    hipError_t e;
    if (lds > 48 * 1024) {
        e = ensure_dynamic_lds(kern, lds);
        if (e != hipSuccess) return e;
    }
    int per_cu = 0;
    e = cached_blocks_per_cu(&per_cu, kern, 64, lds);
    if (e != hipSuccess) return e;
    const int grid = std::min(p.n_groups, per_cu * device_cu_count(d.device));
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64), lds, s, p);
    return hipGetLastError();
}

// One order for all samples: always, where the rows fit (vgg16, 262 144 samples as float32, with the straggler effect:
// 168 -> 40 us, 105 MB; float64 146 -> 63 us; tiny 570 -> 54 us; with few samples 31 -> 23 us, the checks and kappa are no
// launches of their own).  An order per sample: from 24 576 samples on (vgg16 float32 225 -> 157 us, float64 212 -> 196 us
// for 262 144; tiny 655 -> 221 us, float32 133 us); a smaller batch leaves compute units without a wave of 64 samples, and a
// wave per sample is done sooner (16 384 samples: vgg16 25 against 28 us).
hipError_t launch_simulate_lanes(Dag &d, const SimArgs &a, hipStream_t s)
{
    if (a.order_stride != 0 && a.B < 24 * 1024) return hipErrorNotSupported;
    if (d.R == 0 || d.C == 0 || d.N == 0 || d.N + d.R > kLaneCols || !d.d_col_cls || !d.d_bad_order) return hipErrorNotSupported;
    SimLanesParams p{};
    p.B = a.B; p.N = d.N; p.R = d.R; p.W = d.W; p.C = d.C; p.n_groups = (a.B + 63) / 64;
    p.cls_dep = d.d_cls_dep; p.cls_ptr = d.d_cls_ptr; p.cls_cols = d.d_cls_cols; p.col_cls = d.d_col_cls;
    p.order = a.order; p.order_stride = a.order_stride;
    p.op_time = a.op_time; p.recv_time = a.recv_time;
    p.makespan = a.makespan; p.eff = a.eff; p.U = a.U; p.L = a.L; p.S = a.S;
    p.bad_order = d.d_bad_order;
    return a.f32 ? launch_lanes_t<float>(p, d, s) : launch_lanes_t<double>(p, d, s);
}

}  // namespace tictac
