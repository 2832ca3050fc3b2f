// Wave- and block-level helpers shared by the TAC and simulation kernels (wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tictac {

#define TT_INF (__builtin_huge_val())

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// ordering point for LDS traffic between the lanes of one wave (LDS operations of a wave
// complete in issue order; this only keeps the compiler from moving them across)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a barrier of the workgroup's waves for what they exchange through LDS: memory operations stay under way
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ double wave_min_f64(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
    return v;
}

__device__ __forceinline__ double wave_sum_f64(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

__device__ __forceinline__ double wave_max_f64(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
    return v;
}

// ---- the same reductions and scans through data-parallel-primitive moves (no LDS traffic) ----
// A wave64 is four rows of 16 lanes.  row_shr:n moves a value n lanes up inside a row, row_ror:n rotates a row by n lanes;
// row_bcast:15 hands lane 15 of every row to the whole next row, row_bcast:31 hands lane 31 to rows 2 and 3.  A lane without a
// source gets zero (dpp0) or, also where its row is masked out, keeps `identity` (dpp).  The former needs no instruction
// to set the lanes that keep something: a step is two moves and the operation, not five or six instructions.
template <int CTRL>
__device__ __forceinline__ int dpp0_i32(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}

template <int CTRL>
__device__ __forceinline__ double dpp0_f64(double v)
{
    return __hiloint2double(dpp0_i32<CTRL>(__double2hiint(v)), dpp0_i32<CTRL>(__double2loint(v)));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_i32(int identity, int v)
{
    return __builtin_amdgcn_update_dpp(identity, v, CTRL, ROW_MASK, 0xf, false);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double identity, double v)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(identity), __double2loint(v), CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(identity), __double2hiint(v), CTRL, ROW_MASK, 0xf, false);
    return __hiloint2double(hi, lo);
}

// fmin and fmax of numbers in one instruction: the compiler quiets an operand first that is loaded, selected or moved as two
// integers (half of the minima and maxima of the kernels were that).  Not in a loop that is to be unrolled by a number of turns not
// known before: the compiler takes an asm for convergent and leaves such a loop as it is (simulate_kernel).  With the moves above: order
// search 1 753 -> 1 684 us, sends 109.5 -> 106.7 us, TAC in registers with 14 class slots 1 087 -> 1 068 us, the other cases 0 to
// 1 % faster.
__device__ __forceinline__ double min_f64(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double max_f64(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ double readlane_f64(double v, int l)      // l wave-uniform
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

__device__ __forceinline__ double lane63_f64(double v)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

__device__ __forceinline__ double tt_add_f64(double a, double b) { return a + b; }
__device__ __forceinline__ int tt_add_i32(int a, int b) { return a + b; }
__device__ __forceinline__ int tt_min_i32(int a, int b) { return min(a, b); }
__device__ __forceinline__ int tt_max_i32(int a, int b) { return max(a, b); }

// inclusive prefix sum over the lanes of a wave: four shifts scan the rows, the two broadcasts (to rows 1 and 3, then to rows 2
// and 3) add the totals of the rows before
__device__ __forceinline__ double wave_incl_scan_f64_dpp(double v)
{
    v += dpp0_f64<0x111>(v);
    v += dpp0_f64<0x112>(v);
    v += dpp0_f64<0x114>(v);
    v += dpp0_f64<0x118>(v);
    v += dpp_f64<0x142, 0xa>(0.0, v);
    v += dpp_f64<0x143, 0xc>(0.0, v);
    return v;
}
__device__ __forceinline__ int wave_incl_scan_i32_dpp(int v)
{
    v += dpp0_i32<0x111>(v);
    v += dpp0_i32<0x112>(v);
    v += dpp0_i32<0x114>(v);
    v += dpp0_i32<0x118>(v);
    v += dpp_i32<0x142, 0xa>(0, v);
    v += dpp_i32<0x143, 0xc>(0, v);
    return v;
}
// Reductions are read from lane 63, which sees its own row, the total of row 2 by the first broadcast and that of rows 0 and 1,
// in lane 31 by then, by the second.  (What the broadcasts leave in rows 0 and 2 is not looked at, so no row is masked out.)  Sums
// are added up in the order of the scan above; minima and maxima go round the rows, where every lane has a source.
#define TT_DPP_REDUCE(DPP0, OP, A, B, C, D)                                               \
    v = OP(v, DPP0<A>(v));                                                                \
    v = OP(v, DPP0<B>(v));                                                                \
    v = OP(v, DPP0<C>(v));                                                                \
    v = OP(v, DPP0<D>(v));                                                                \
    v = OP(v, DPP0<0x142>(v));                                                            \
    v = OP(v, DPP0<0x143>(v));
__device__ __forceinline__ double wave_sum_f64_dpp(double v)
{
    TT_DPP_REDUCE(dpp0_f64, tt_add_f64, 0x111, 0x112, 0x114, 0x118)
    return lane63_f64(v);
}
__device__ __forceinline__ double wave_max_f64_dpp(double v)
{
    TT_DPP_REDUCE(dpp0_f64, max_f64, 0x121, 0x122, 0x124, 0x128)
    return lane63_f64(v);
}
__device__ __forceinline__ double wave_min_f64_dpp(double v)
{
    TT_DPP_REDUCE(dpp0_f64, min_f64, 0x121, 0x122, 0x124, 0x128)
    return lane63_f64(v);
}
#undef TT_DPP_REDUCE

// Of whole numbers a move and the operation are one instruction either way.  As a scan with the operation's identity its steps are
// placed among those of a sum that is formed beside it (class_M of the bit-sliced TAC kernel, for which the control wave
// waits); rotations came after the sum, with idle cycles between them: 512 samples of 1 619 classes 5.2 and 5.6 ms, 2 270
// classes 3.55 and 3.75.
template <typename Op>
__device__ __forceinline__ int wave_reduce_i32_dpp(int v, int identity, Op op)
{
    v = op(v, dpp_i32<0x111, 0xf>(identity, v));
    v = op(v, dpp_i32<0x112, 0xf>(identity, v));
    v = op(v, dpp_i32<0x114, 0xf>(identity, v));
    v = op(v, dpp_i32<0x118, 0xf>(identity, v));
    v = op(v, dpp_i32<0x142, 0xa>(identity, v));
    v = op(v, dpp_i32<0x143, 0xc>(identity, v));
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int wave_min_i32_dpp(int v) { return wave_reduce_i32_dpp(v, INT32_MAX, tt_min_i32); }
__device__ __forceinline__ int wave_max_i32_dpp(int v) { return wave_reduce_i32_dpp(v, INT32_MIN, tt_max_i32); }

// A row of a timing array that is stored as float64 or as float32.  A float32 value is converted
// when it is loaded; every sum and comparison is float64.
struct TimeRow {
    const void *p;
    bool f32;
    __device__ __forceinline__ double operator[](int j) const
    {
        return f32 ? (double)static_cast<const float *>(p)[j] : static_cast<const double *>(p)[j];
    }
    __device__ __forceinline__ const float *as_f32() const { return static_cast<const float *>(p); }
    __device__ __forceinline__ const double *as_f64() const { return static_cast<const double *>(p); }
};
__device__ __forceinline__ TimeRow time_row(const void *base, size_t first, bool f32)
{
    return TimeRow{f32 ? static_cast<const void *>(static_cast<const float *>(base) + first)
                       : static_cast<const void *>(static_cast<const double *>(base) + first), f32};
}

// Four consecutive elements with one load (two for float64).  Rows start at any element, so the
// vector types carry the alignment of one element; the class table is read the same way.
typedef float tt_f32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef double tt_f64x2 __attribute__((ext_vector_type(2), aligned(8)));
typedef int tt_i32x4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void load4(const double *__restrict__ q, double (&x)[4])
{
    const tt_f64x2 a = *reinterpret_cast<const tt_f64x2 *>(q), b = *reinterpret_cast<const tt_f64x2 *>(q + 2);
    x[0] = a.x; x[1] = a.y; x[2] = b.x; x[3] = b.y;
}
__device__ __forceinline__ void load4(const float *__restrict__ q, double (&x)[4])
{
    const tt_f32x4 a = *reinterpret_cast<const tt_f32x4 *>(q);
    x[0] = (double)a.x; x[1] = (double)a.y; x[2] = (double)a.z; x[3] = (double)a.w;
}

// a + b; what is rounded off, exactly (Knuth's two-sum), is added to `lost`
__device__ __forceinline__ double add_exact(double a, double b, double &lost)
{
    const double s = a + b, bb = s - a;
    lost += (a - (s - bb)) + (b - bb);
    return s;
}

// x to sums[at] (at < 0: nowhere), a wave with one place, or rows of 16 lanes with one, by one addition for all of them: many
// lanes with the same place would be added one after the other, which takes its time and rounds more.
__device__ __forceinline__ void add_by_rows(double *sums, int at, double x, int lane)
{
    if (__ballot(at == __builtin_amdgcn_readfirstlane(at)) == ~0ull) {
        const double all = wave_sum_f64_dpp(x);
        if (lane == 0 && at >= 0) atomicAdd(&sums[at], all);
        return;
    }
    const uint64_t same = __ballot(at == dpp0_i32<0x111>(at)) | 0x0001000100010001ull;
    const bool whole = ((same >> (lane & 48)) & 0xffffull) == 0xffffull;
    double all = x;
    all += dpp0_f64<0x128>(all);
    all += dpp0_f64<0x124>(all);
    all += dpp0_f64<0x122>(all);
    all += dpp0_f64<0x121>(all);
    if (at >= 0 && (!whole || (lane & 15) == 0)) atomicAdd(&sums[at], whole ? all : x);
}

// x to sums[at] (at < 0: nowhere), four lanes next to each other with one place by one addition; by all lanes of a wave.
__device__ __forceinline__ void add_by_quads(double *sums, int at, double x)
{
    uint64_t quad = __ballot(at == dpp0_i32<0x111>(at)) | 0x1111111111111111ull;    // (the first of four is not compared)
    quad &= quad >> 1;
    quad &= (quad >> 2) & 0x1111111111111111ull;                    // bit 4 q: lanes 4 q to 4 q + 3 have one place
    if (quad != 0ull) {
        double all = x;
        all += dpp0_f64<0xb1>(all);                                 // lanes 1, 0, 3, 2
        all += dpp0_f64<0x4e>(all);                                 // lanes 2, 3, 0, 1
        x = __builtin_amdgcn_inverse_ballot_w64(quad * 15ull) ? all : x;
        at = __builtin_amdgcn_inverse_ballot_w64(quad * 14ull) ? -1 : at;
    }
    if (at >= 0) atomicAdd(&sums[at], x);
}

enum class Sums { plain, quads, rows, plain_together };    // how class_totals adds what lanes next to each other have for one place

// totals[cls_of[j]] += row[j] for j in [0, N), totals in LDS, by one wave.  A lane takes four
// consecutive columns at a time and first adds up runs of equal class in registers: columns of
// one class tend to sit next to each other, and every LDS add of several lanes to one address
// is served one lane after the other.
// Sums::rows: neighbours in the row mostly go to one place (add_by_rows).
// Sums::quads: four lanes with one class make one addition (add_by_quads).  Columns of one class are in runs of 14 on average on
// inception3, a third of them in runs of more than 32: 832 additions one after the other per sample become 280.  Simulation with an
// order each 727 -> 678 us, several channels, 65 536 samples, 987 -> 932.  Where runs are short the test costs 1 to 5 %: those two
// use it by how the columns lie (long_class_runs), with more than four class slots per lane.  TAC in registers uses it from six
// slots to eight; what a round costs leaves nothing to be seen of the sums, but the code of the rounds comes out 2 % faster with
// six to eight and 1.7 % slower with five (a literal scan every round, 290 to 500 recvs).
// Sums::plain_together: as plain, but no lane leaves before the others, which takes up to five registers less and else up to 1 %
// more time.
template <Sums HOW = Sums::plain, typename T>
__device__ __forceinline__ void class_totals(double *totals, const T *__restrict__ row,
                                             const int32_t *__restrict__ cls_of, int N, int lane)
{
    for (int j0 = lane * 4; (HOW == Sums::plain ? j0 : j0 - lane * 4) < N; j0 += 64 * 4 * 2) {   // (rows, quads: lanes leave together)
        // two groups of four in flight per lane
        double x[2][4];
        int c[2][4];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int j = j0 + g * 256;
            if (j + 3 < N) {
                load4(row + j, x[g]);
                const tt_i32x4 q = *reinterpret_cast<const tt_i32x4 *>(cls_of + j);
                c[g][0] = q.x; c[g][1] = q.y; c[g][2] = q.z; c[g][3] = q.w;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    x[g][i] = j + i < N ? (double)row[j + i] : 0.0;
                    c[g][i] = j + i < N ? cls_of[j + i] : -1;
                }
            }
        }
        [[maybe_unused]] double acc0 = 0.0;
        [[maybe_unused]] int cur0 = -1;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            double acc = x[g][0];
            int cur = c[g][0];
#pragma unroll
            for (int i = 1; i < 4; ++i) {
                if (c[g][i] == cur) {
                    acc += x[g][i];
                } else {
                    if (cur >= 0) atomicAdd(&totals[cur], acc);
                    cur = c[g][i];
                    acc = x[g][i];
                }
            }
            if constexpr (HOW == Sums::rows) {
                if (g == 0) {
                    acc0 = acc;
                    cur0 = cur;
                } else if (__ballot(cur == cur0) == ~0ull) {
                    add_by_rows(totals, cur, acc0 + acc, lane);
                } else {
                    add_by_rows(totals, cur0, acc0, lane);
                    add_by_rows(totals, cur, acc, lane);
                }
            } else if constexpr (HOW == Sums::quads) {
                add_by_quads(totals, cur, acc);
            } else if (cur >= 0) {
                atomicAdd(&totals[cur], acc);
            }
        }
    }
}

template <Sums HOW = Sums::plain>
__device__ __forceinline__ void class_totals(double *totals, const TimeRow &row, const int32_t *__restrict__ cls_of,
                                             int N, int lane)
{
    if (row.f32) class_totals<HOW>(totals, row.as_f32(), cls_of, N, lane);
    else class_totals<HOW>(totals, row.as_f64(), cls_of, N, lane);
}

__device__ __forceinline__ int wave_min_i32(int v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off));
    return v;
}

// Block-wide reductions; every thread of the block must call them (uniform control
// flow).  `red` is LDS scratch of at least BS/64 elements of the reduced type; two
// barriers make it reusable right after the call.
template <int BS>
__device__ __forceinline__ double block_min_f64(double v, double *red)
{
    v = wave_min_f64(v);
    if (BS == 64) return v;
    __syncthreads();
    if (lane_id() == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = red[0];
#pragma unroll
    for (int k = 1; k < BS / 64; ++k) r = fmin(r, red[k]);
    return r;
}

template <int BS>
__device__ __forceinline__ double block_sum_f64(double v, double *red)
{
    v = wave_sum_f64(v);
    if (BS == 64) return v;
    __syncthreads();
    if (lane_id() == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = red[0];
#pragma unroll
    for (int k = 1; k < BS / 64; ++k) r += red[k];
    return r;
}

template <int BS>
__device__ __forceinline__ int block_min_i32(int v, double *red)
{
    v = wave_min_i32(v);
    if (BS == 64) return v;
    int *ri = reinterpret_cast<int *>(red);
    __syncthreads();
    if (lane_id() == 0) ri[threadIdx.x >> 6] = v;
    __syncthreads();
    int r = ri[0];
#pragma unroll
    for (int k = 1; k < BS / 64; ++k) r = min(r, ri[k]);
    return r;
}

// arr[idx] += v for the threads with `active`, arr in LDS.  With one wave per block the
// additions are applied one after the other in lane order by lane 0 (a fixed order, so
// the result is reproducible bit for bit); with several waves LDS atomics are used.
// Must be called by all threads of a wave together.
template <int BS>
__device__ __forceinline__ void lds_scatter_add(double *arr, int idx, double v, bool active)
{
    if (BS == 64) {
        unsigned long long m = __ballot(active);
        while (m) {
            const int l = __builtin_ctzll(m);
            m &= m - 1;
            const int i = __shfl(idx, l);
            const double x = __shfl(v, l);
            if (threadIdx.x == 0) arr[i] += x;
        }
    } else {
        if (active) atomicAdd(&arr[idx], v);
    }
}

}  // namespace tictac
