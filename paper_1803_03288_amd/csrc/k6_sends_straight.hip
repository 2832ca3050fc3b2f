// The iteration with send ops (k6_sends.hip) for graphs whose op ids are a topological order, of samples in which the
// compute device runs its ops by ascending id.
//
// The device takes the ready op of lowest id.  With topological ids the lowest op not yet run is always held up by
// recvs alone; as long as those have arrived when the device gets to it, nothing can come before it, and the device goes
// through the columns of op_time one after the other.  An op that has to wait for a recv keeps its place too when no other
// op could run meanwhile, which the graph tells (`alone`: no later op has all its compute predecessors among the ops
// before this one).  A sample in which an op would have to wait and is not alone is given up here and handed to the
// event-driven kernels through a list.  With a deployed order a model's graph has hardly any such sample: the transfers
// run ahead of the ops that need them.
//
// What is left per op is one addition, in an order known beforehand, so the kernel is a stream over op_time.  A workgroup
// takes 64 samples; four of its waves read tiles of 64 columns (512 consecutive bytes of a row) into registers, two tiles
// ahead, sum them along the rows and lay the sums out in LDS by column; the fifth follows the samples, a lane each, and
// looks only at the columns with recvs or sends.  Arrivals (prefix sums over the transfers, laid out by recv) come with the
// tile whose ops need them.  The instant at which a send is requested is the sum after its last predecessor; the sends are
// known in the order of their requests, so the uplink is a second, shorter stream, taken by the four waves in four parts
// (busy -> max(busy + A, B)).
//
// 16 384 samples of the ResNet-50 inference graph with 161 sends (187 MB of times, 38 us at the copy rate): 4.0 ms in the
// event-driven form with a wave per sample, 73 us here (the call 84 us).  Bound by the latencies of a tile, since there is
// one workgroup of 64 samples per compute unit (two of 32 would not fit: a wave has up to 256 registers): waves wait 54 % of their time.  Of
// 75 us, before batches of loads ended with one of eight where eight are enough: 13 us for the arrivals, 43 us for the 18 tiles (18 of them for the fifth wave,
// which is behind the loaders then), 7 us for the uplink.  It was 93 us (18, 55, 20) as long as the loads of a batch hid
// behind branches, each with a wait of its own, the times of transfers and sends were read by a lane per row, and a wait for an
// index in a table was one for the tiles on their way.  With the columns followed one by one the fifth wave took 4 us per
// tile, at the columns that matter 2 us.  On times that are not quantised makespan, U and L are within 4e-16 of sums in long
// double (event-driven form: 3e-15).
#include <algorithm>
#include <type_traits>

#include "device_utils.h"
#include "internal.h"

namespace tictac {

constexpr int kTileCols = 64, kTileChecks = 32, kTilePitch = 65;
constexpr int kRowCols = (2 * kTileCols * kTilePitch + 2 * kTileChecks * 64) / kTilePitch;      // columns of 64 rows that fit the tiles' space
constexpr int kRowsLeast = 16;  // so many and fewer columns are read by lanes, a row each (SMALL)
typedef double Pair __attribute__((ext_vector_type(2), aligned(8)));

// The tables are the same for all lanes: read through the scalar cache, they have a counter of waits of their own.  (By vector
// loads, a wait for the number of a recv was one for the tiles on their way as well.)
typedef int Int2 __attribute__((ext_vector_type(2), aligned(4)));
typedef int Int4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int uniform_int(const int32_t *p) { return *(const __attribute__((address_space(4))) int *)p; }
__device__ __forceinline__ Int2 uniform_int2(const int32_t *p) { return *(const __attribute__((address_space(4))) Int2 *)p; }
__device__ __forceinline__ Int4 uniform_int4(const int4 *p) { return *(const __attribute__((address_space(4))) Int4 *)p; }

struct StraightParams {
    int32_t B, N, R, n_req, n_req0, n_tiles;
    int32_t req_lo, req_span;       // the columns of the sends lie in req_lo .. req_lo + req_span - 1; 0: in more than kRowCols
    const uint32_t *code;           // [n_tiles * 64] see internal.h
    const int32_t *chk;             // recvs, in the order in which the columns need them; 32 zeros after the last
    const int32_t *req_col;         // [n_req] columns of the sends in the order of their requests, the first n_req0 at 0
    const int4 *tiles;              // [n_tiles][2] first column, columns, first entry of chk, entries; see internal.h
    const int32_t *order;
    int32_t order_stride;
    const double *op_time, *recv_time;
    double *makespan, *eff, *U, *L, *S;
    double *arrive;                 // [blocks][R][64]
    double *req_at;                 // [blocks][n_req][64]
    int32_t *list, *count;          // the samples given up
};

// SMALL: at most 64 recvs and sends, a quarter of which is a batch of loads or two.  All loads of a batch are executed, of the last
// place again where there are no more, so that nothing waits between them; 64 lines each where every sample has an order.
// Hence batches of eight, of the recvs four at the end, and the times of at most sixteen recvs or columns of sends by lanes that read their
// rows instead of through LDS.  40 000 samples, an order each, a send behind every op: chains of 8 recvs 33.9 us (51.5 with sixteen at a
// time, through LDS), of 12 36.8 (50.9), of 40 71.4 (74.5), vgg16 59.1 (64.4).  Larger graphs: sixteen at a time, of the recvs eight at the end;
// a chain of 250 recvs 452 us, 528 by eight; resnet50 with one order 221 and 226.
template <bool SMALL>
__global__ void __launch_bounds__(320)
sends_straight_kernel(const StraightParams p)
{
    extern __shared__ double smem[];
    double *xs = smem;                                          // [2][kTileCols * kTilePitch] column by column
    double *as = xs + 2 * kTileCols * kTilePitch;               // [2][kTileChecks * 64]
    double *red = as + 2 * kTileChecks * 64;                    // [2][4][64]
    uint32_t *codes = reinterpret_cast<uint32_t *>(red + 2 * 4 * 64);   // [2][kTileCols]
    int32_t *stop = reinterpret_cast<int32_t *>(codes + 2 * kTileCols); // [2] by turns: a wave may be late to read the last one
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool loader = wave < 4;                               // (the fifth wave follows the samples)
    const int N = p.N, R = p.R;
    double *arrive = p.arrive + (size_t)blockIdx.x * (R + 1) * 64;
    double *req_at = p.req_at + (size_t)blockIdx.x * p.n_req * 64;
    const int groups = (p.B + 63) / 64;
    const int at_row = tid >> 5, at_col = (tid & 31) * 2;       // (of the loaders)
    const bool rows_fit = R > (SMALL ? kRowsLeast : 1) && R <= kRowCols;

    for (int g = blockIdx.x; g < groups; g += gridDim.x) {
        const int b0 = g * 64, here = min(64, p.B - b0);
        const int64_t b = min(b0 + lane, p.B - 1);

        // columns lo .. lo + span - 1 (at most kRowCols) of the 64 rows into the tiles' space, by the four loaders, all loads
        // before the first store
        auto rows_to_lds = [&](const double *src, int width, int lo, int span) __attribute__((always_inline)) {
            Pair v[3][8];
#pragma unroll
            for (int t = 0; t < 3; ++t)
                if (t * 64 < span) {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        v[t][i] = *reinterpret_cast<const Pair *>(src + (int64_t)min(b0 + i * 8 + at_row, p.B - 1) * width +
                                                                  min(lo + t * 64 + at_col, width - 2));
                }
#pragma unroll
            for (int t = 0; t < 3; ++t)
                if (t * 64 < span) {
                    const int c = t * 64 + at_col;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        if (c < span) xs[c * kTilePitch + i * 8 + at_row] = lo + c > width - 2 ? v[t][i].y : v[t][i].x;
                        if (c + 1 < span) xs[(c + 1) * kTilePitch + i * 8 + at_row] = v[t][i].y;
                    }
                }
        };
        // ---- arrivals: each loader takes a quarter of the transfers, twice (sums, then ends); their times from LDS if they
        // fit it (a lane that reads its own row of memory asks for 64 lines per load) ----
        if (rows_fit) {
            if (loader) rows_to_lds(p.recv_time, R, 0, R);
            __syncthreads();
        }
        const int quarter = (R + 3) / 4, k0 = min(R, wave * quarter), k1 = loader ? min(R, k0 + quarter) : k0;
        double sum = 0.0;
        for (int pass = 0; pass < 2; ++pass) {
            if (pass == 1) {
                if (loader) red[wave * 64 + lane] = sum;
                __syncthreads();
                sum = 0.0;
                for (int w = 0; w < wave; ++w) sum += red[w * 64 + lane];
            }
            auto ends = [&](int k, auto loads) __attribute__((always_inline)) {
                constexpr int n = decltype(loads)::value;
                int r[n];
                double x[n];
#pragma unroll
                for (int q = 0; q < n; ++q) r[q] = p.order[b * p.order_stride + min(k + q, k1 - 1)];
                if (rows_fit) {
#pragma unroll
                    for (int q = 0; q < n; ++q) x[q] = xs[min((unsigned)r[q], (unsigned)R - 1u) * kTilePitch + lane];
                } else {
#pragma unroll
                    for (int q = 0; q < n; ++q) x[q] = p.recv_time[b * R + min((unsigned)r[q], (unsigned)R - 1u)];
                }
#pragma unroll
                for (int q = 0; q < n; ++q) {
                    const bool valid = k + q < k1 && (unsigned)r[q] < (unsigned)R;          // (invalid: skipped)
                    sum += valid ? x[q] : 0.0;
                    if (pass == 1) arrive[(size_t)(valid ? r[q] : R) * 64 + lane] = sum;    // (row R is spare)
                }
            };
            int k = k0;
            if constexpr (!SMALL)
                for (; k1 - k > 8; k += 16) ends(k, std::integral_constant<int, 16>());
            if constexpr (SMALL)
                for (; k1 - k > 4; k += 8) ends(k, std::integral_constant<int, 8>());
            if (k < k1) ends(k, std::integral_constant<int, SMALL ? 4 : 8>());
        }
        const double sum_r = wave == 4 ? sum : 0.0;             // (the fifth wave has added up all four quarters)
        if (tid < 2) stop[tid] = 0;
        __syncthreads();

        // ---- the compute device ----
        double base = 0.0, sum_c = 0.0;
        bool off = false, given_up = false;
        if (loader) {
            // Two tiles are on their way while a third is worked on, their registers by turns.  Every load is executed
            // (places outside the tile read something else, which the masks drop), so that the waits can be counted.
            auto load = [&](int t, Pair (&x)[8], Pair (&a)[4], uint32_t &code) {
                const Int4 tile = uniform_int4(p.tiles + 2 * t);
                const int c = tile.x + at_col, from = min(c, N - 2);
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    x[i] = *reinterpret_cast<const Pair *>(p.op_time + (int64_t)min(b0 + i * 8 + at_row, p.B - 1) * N + from);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const Int2 r = uniform_int2(p.chk + tile.z + i * 8 + wave * 2);
                    a[i] = *reinterpret_cast<const Pair *>(arrive + (size_t)((at_row & 1) ? r.y : r.x) * 64 + at_col);
                }
                code = p.code[t * kTileCols + lane];
            };
            // into LDS: the sums of the row's times up to every column (sends count as zeros)
            auto keep = [&](int t, const Pair (&x)[8], const Pair (&a)[4], uint32_t code) {
                const Int4 tile = uniform_int4(p.tiles + 2 * t), mask = uniform_int4(p.tiles + 2 * t + 1);
                const uint64_t run = (uint64_t)(uint32_t)mask.y << 32 | (uint32_t)mask.x;
                const bool run0 = run >> at_col & 1ull, run1 = run >> at_col & 2ull, shifted = tile.x + at_col > N - 2;
                double *xt = xs + (t & 1) * kTileCols * kTilePitch, *at = as + (t & 1) * kTileChecks * 64;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int row = i * 8 + at_row;
                    const double u0 = run0 ? (shifted ? x[i].y : x[i].x) : 0.0, u1 = run1 ? x[i].y : 0.0;
                    double v = u0 + u1;                         // (32 lanes hold a row: the scan stops at half a wave)
                    v += dpp0_f64<0x111>(v);
                    v += dpp0_f64<0x112>(v);
                    v += dpp0_f64<0x114>(v);
                    v += dpp0_f64<0x118>(v);
                    v += dpp_f64<0x142, 0xa>(0.0, v);
                    // (what the lane before has: v less the own two would lose the low bits of a short sum before a long op)
                    const double before = dpp0_f64<0x138>(v);
                    xt[at_col * kTilePitch + row] = (at_col ? before : 0.0) + u0;
                    xt[(at_col + 1) * kTilePitch + row] = v;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    at[(i * 8 + at_row) * 64 + at_col] = a[i].x;
                    at[(i * 8 + at_row) * 64 + at_col + 1] = a[i].y;
                }
                if (wave == 0) codes[(t & 1) * kTileCols + lane] = code;
            };
            Pair x0[8], a0[4], x1[8], a1[4];
            uint32_t c0, c1;
            const int last = p.n_tiles - 1;
            load(0, x0, a0, c0);
            load(min(1, last), x1, a1, c1);
            keep(0, x0, a0, c0);
            __syncthreads();
            // (six tiles per trip: at the head of a loop the compiler waits for all loads on their way)
#define SS_TILE(xa, aa, ca, xb, ab, cb)                                                   \
                load(min(t + 2, last), xa, aa, ca);                                       \
                keep(t + 1, xb, ab, cb);            /* (past the last tile: into the buffer that nobody reads) */ \
                lds_barrier();                                                            \
                if (stop[t & 1]) { given_up = true; break; }                              \
                if (++t > last) break;
            for (int t = 0;;) {
                SS_TILE(x0, a0, c0, x1, a1, c1)
                SS_TILE(x1, a1, c1, x0, a0, c0)
                SS_TILE(x0, a0, c0, x1, a1, c1)
                SS_TILE(x1, a1, c1, x0, a0, c0)
                SS_TILE(x0, a0, c0, x1, a1, c1)
                SS_TILE(x1, a1, c1, x0, a0, c0)
            }
        } else {
            double *req = req_at + (size_t)p.n_req0 * 64 + lane;
            __syncthreads();
            for (int t = 0; t < p.n_tiles; ++t) {
                const Int4 mask = uniform_int4(p.tiles + 2 * t + 1);
                const uint64_t special = (uint64_t)(uint32_t)mask.w << 32 | (uint32_t)mask.z;   // recvs to look at, sends to request
                const uint32_t code = codes[(t & 1) * kTileCols + lane];
                const double *xt = xs + (t & 1) * kTileCols * kTilePitch + lane;
                const double *at = as + (t & 1) * kTileChecks * 64 + lane;
                const double all = xt[(kTileCols - 1) * kTilePitch];
                // only the columns with recvs or sends are looked at, four at a time with their reads from LDS together; the
                // device is at base + the sum up to there
                uint64_t rest = special;
                int at_chk = 0;
                while (rest != 0ull) {
                    uint32_t todo[4];
                    int first_chk[4];
                    double done[4], before[4], arrived[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int c = rest ? __builtin_ctzll(rest) : 0;
                        todo[i] = rest ? (uint32_t)__builtin_amdgcn_readlane((int)code, c) : 0u;
                        rest &= rest - 1ull;                    // (0 stays 0)
                        first_chk[i] = at_chk;
                        at_chk += (int)(todo[i] >> 1 & 0x7fu);
                        done[i] = xt[c * kTilePitch];
                        before[i] = xt[max(c - 1, 0) * kTilePitch];
                        before[i] = c == 0 ? 0.0 : before[i];
                        arrived[i] = at[min(first_chk[i], kTileChecks - 1) * 64];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (const int n_chk = (int)(todo[i] >> 1 & 0x7fu)) {
                            double last = arrived[i];
                            for (int j = 1; j < n_chk; ++j) last = max_f64(last, at[(first_chk[i] + j) * 64]);
                            const bool late = last > base + before[i];
                            off |= !(todo[i] & 0x100u) && late;
                            base = late ? last - before[i] : base;      // (`off`: whatever, the sample is given up)
                        }
                        for (uint32_t j = todo[i] >> 16; j > 0u; --j) { *req = base + done[i]; req += 64; }
                    }
                }
                base += all;
                sum_c += all;
                if (__ballot(!off && lane < here) == 0ull) stop[t & 1] = 1;
                __syncthreads();
                if (stop[t & 1]) { given_up = true; break; }
            }
        }

        // ---- the uplink; its times from LDS too if their columns fit it ----
        if (p.req_span > 0 && !given_up) {                      // (the same for all waves)
            if (loader) rows_to_lds(p.op_time, N, p.req_lo, p.req_span);
            __syncthreads();
        }
        double add = 0.0, least = -TT_INF;
        if (loader && !given_up) {
            const int part = (p.n_req + 3) / 4, q0 = min(p.n_req, wave * part), q1 = min(p.n_req, q0 + part);
            constexpr int n = SMALL ? 8 : 16;
            for (int q = q0; q < q1; q += n) {
                double at[n], y[n];
#pragma unroll
                for (int i = 0; i < n; ++i) at[i] = req_at[(size_t)min(q + i, q1 - 1) * 64 + lane];
                if (p.req_span > 0) {
#pragma unroll
                    for (int i = 0; i < n; ++i) y[i] = xs[(uniform_int(p.req_col + min(q + i, q1 - 1)) - p.req_lo) * kTilePitch + lane];
                } else {
#pragma unroll
                    for (int i = 0; i < n; ++i) y[i] = p.op_time[b * N + uniform_int(p.req_col + min(q + i, q1 - 1))];
                }
#pragma unroll
                for (int i = 0; i < n; ++i)
                    if (q + i < p.n_req0) at[i] = 0.0;          // (requested at the start: not stored)
#pragma unroll
                for (int i = 0; i < n; ++i) {
                    if (q + i < q1) { add += y[i]; least = max_f64(least, at[i]) + y[i]; }
                }
            }
        }
        if (loader) {
            red[wave * 64 + lane] = add;
            red[(4 + wave) * 64 + lane] = least;
        }
        __syncthreads();
        if (!loader) {
            const bool mine = lane < here;
            const uint64_t out = __ballot(mine && (off || given_up));
            if (out) {
                int at = 0;
                if (lane == 0) at = atomicAdd(p.count, (int)__builtin_popcountll(out));
                at = __builtin_amdgcn_readfirstlane(at);
                if (mine && (off || given_up)) p.list[at + __builtin_popcountll(out & ((1ull << lane) - 1ull))] = b0 + lane;
            }
            if (mine && !off && !given_up) {
                double busy = 0.0, sum_s = 0.0;
                for (int w = 0; w < 4; ++w) {
                    busy = max_f64(busy + red[w * 64 + lane], red[(4 + w) * 64 + lane]);
                    sum_s += red[w * 64 + lane];
                }
                const double m = max_f64(max_f64(base, busy), sum_r);
                const double U = sum_c + sum_r + sum_s;
                const double Lb = max_f64(max_f64(sum_c, sum_r), sum_s);
                p.makespan[b] = m;
                p.eff[b] = (U == Lb) ? 1.0 : (U - m) / (U - Lb);
                if (p.U) p.U[b] = U;
                if (p.L) p.L[b] = Lb;
                if (p.S) p.S[b] = (U == Lb || Lb == 0.0) ? 0.0 : (U - Lb) / Lb;
            }
        }
        __syncthreads();
    }
}

// The workspace: the count, the list of up to B samples, and from here on what a kernel needs while it runs (arrivals and
// requests, afterwards the state of the event-driven form).
static size_t rest_offset(int32_t B) { return ((size_t)B * 4 + 4 + 255) & ~(size_t)255; }
void *sends_straight_rest(int32_t *count, int32_t B) { return reinterpret_cast<char *>(count) + rest_offset(B); }

__global__ void clear_count_kernel(int32_t *count) { *count = 0; }

// Runs the kernel above; *list and *count: the samples it gave up.  At least `rest` bytes follow the list.
hipError_t launch_sends_straight(Dag &d, const SimArgs &a, size_t rest, int32_t **list, int32_t **count, hipStream_t s)
{
    const int groups = (int)(((int64_t)a.B + 63) / 64);
    const int grid = std::min(groups, device_cu_count(d.device));
    StraightParams p{};
    p.B = a.B; p.N = d.N; p.R = d.R; p.n_req = (int32_t)d.h_send_ids.size(); p.n_req0 = d.n_send_free; p.n_tiles = d.n_straight_tiles;
    const bool small = d.R <= 64 && p.n_req <= 64;
    p.req_lo = d.straight_req_lo;
    p.req_span = d.straight_req_span > (small ? kRowsLeast : 0) && d.straight_req_span <= kRowCols ? d.straight_req_span : 0;
    p.code = d.d_straight_code; p.chk = d.d_straight_chk; p.req_col = d.d_straight_req; p.tiles = d.d_straight_tiles;
    p.order = a.order; p.order_stride = a.order_stride;
    p.op_time = static_cast<const double *>(a.op_time); p.recv_time = static_cast<const double *>(a.recv_time);
    p.makespan = a.makespan; p.eff = a.eff; p.U = a.U; p.L = a.L; p.S = a.S;
    const size_t arrive = (size_t)grid * (d.R + 1) * 64 * 8, req = (size_t)grid * p.n_req * 64 * 8;
    hipError_t e = ensure_workspace(&d, rest_offset(a.B) + std::max(arrive + req, rest));
    if (e != hipSuccess) return e;
    p.count = static_cast<int32_t *>(d.d_work);
    p.list = p.count + 1;
    p.arrive = static_cast<double *>(sends_straight_rest(p.count, a.B));
    p.req_at = p.arrive + (size_t)grid * (d.R + 1) * 64;
    *list = p.list;
    *count = p.count;
    const size_t lds = (size_t)(2 * kTileCols * kTilePitch + 2 * kTileChecks * 64 + 2 * 4 * 64) * 8 + 2 * kTileCols * 4 + 16;
    void (*const kernel)(StraightParams) = small ? sends_straight_kernel<true> : sends_straight_kernel<false>;
    e = ensure_dynamic_lds(reinterpret_cast<const void *>(kernel), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(clear_count_kernel, dim3(1), dim3(1), 0, s, p.count);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(320), lds, s, p);
    return hipGetLastError();
}

}  // namespace tictac
