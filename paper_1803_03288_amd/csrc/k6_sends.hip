// One iteration with send ops (Sec. 2.2: in the worker's graph the recv ops are roots and the send ops
// leaves), for a batch of timing samples.  Three resources: the channel that serves the recvs back to back
// in the given order (Sec. 5.1), the compute device, and an uplink that carries the sends one at a time,
// first come first served, a send being requested when its last predecessor finishes.
//
// With sends the finish times of single compute ops matter, so the closed form over classes of
// k4_simulate.hip does not apply: the compute device is followed op by op.  It takes, whenever it is
// idle, the ready op of lowest id.  One wavefront per sample:
//   * the downlink needs no events: the k-th transfer ends at F_k, a prefix sum;
//   * the device is a loop over the compute ops in the order in which it runs them.  A step: the lowest set
//     bit of the ready set (a bitmap in LDS, one word per lane and pass), the op's record (successor list,
//     column of its time), finish = start + Time(op); then the transfers that end up to `finish` release
//     their successors, then the op releases its own.  Releasing: one lane per successor decrements its
//     count of unfinished predecessors (LDS, returning atomics); a count that reaches zero sets the ready
//     bit, or, for a send, requests the uplink;
//   * the uplink needs no queue: requests arrive in non-decreasing time (the steps above are taken in
//     time order), and for the requests of one instant only the sum of their times matters, so
//     busy = max(busy, instant) + sum; the last send ends at the final value of busy.
// A step reads from device memory the op's time and its successor list.  Both addresses come with the list entry
// through which the op was released (the lane that released it keeps them), so an op released by the op before it,
// the common case on chains, costs one trip to memory; any other op costs a second one for its record.  The
// per-sample state in LDS is 2 bytes per op plus a bit per op plus 12 bytes per recv.
#include <algorithm>
#include <climits>

#include "device_utils.h"
#include "internal.h"

namespace tictac {

struct SendSimParams {
    int32_t B, n, R, N;
    const int4 *rec;                // [n] per op: successors from succ[x] on (-1: none), column of its time (z; -1 recv), w: 1 = send
    const int4 *succ;               // [E + 64] x: successor op id, top bit set on the last of a list; y, z, w: that op's
                                    // column, start of its successors and send flag (as in rec)
    const uint16_t *indeg;          // [n] number of predecessors
    const uint32_t *ready0;         // [ceil(n / 32)] compute ops (not sends) without predecessors
    const int32_t *send0;           // [n_send0] columns of the sends without predecessors (requested at 0)
    int32_t n_send0;
    const uint8_t *col_kind;        // [N] 1 = the column is a send's
    const int32_t *recv_ids;        // [R]
    const int32_t *order;
    int32_t order_stride;
    const double *op_time, *recv_time;
    double *makespan, *eff, *U, *L, *S;
    int32_t wave_bytes, n_waves;
    const int32_t *list, *count;    // the samples to take (NULL: all of them)
    int32_t most;                   // more samples than this: none
};

__device__ __forceinline__ double uniform(double v)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

__global__ void __launch_bounds__(256)
simulate_sends_kernel(const SendSimParams p)
{
    extern __shared__ double smem[];
    const int n = p.n, R = p.R, N = p.N;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n_words = (n + 31) >> 5;
    char *mine = reinterpret_cast<char *>(smem) + (size_t)wave * p.wave_bytes;
    double *F = reinterpret_cast<double *>(mine);                               // [R] end of the k-th transfer
    int32_t *rop = reinterpret_cast<int32_t *>(F + R);                          // [R] where the successors of the k-th recv start
    uint32_t *rdy = reinterpret_cast<uint32_t *>(rop + R);                      // [n_words]
    uint16_t *waiting = reinterpret_cast<uint16_t *>(rdy + n_words);            // [n] (padded to a multiple of two)

    const int gwave = blockIdx.x * (blockDim.x >> 6) + wave;
    int n_samples = p.list ? *p.count : p.B;
    if (n_samples > p.most) n_samples = 0;                  // (the form with one lane per sample takes that many)
    for (int i = gwave; i < n_samples; i += p.n_waves) {
        const int b = p.list ? p.list[i] : i;
        const double *ot = p.op_time + (size_t)b * N;
        const double *rt = p.recv_time + (size_t)b * R;
        const int32_t *ord = p.order + (size_t)b * p.order_stride;
        wave_sync();

        // ---- the downlink: ends of the transfers in the given order; sums of the three resources ----
        double fc = 0.0;
        for (int base = 0; base < R; base += 64) {
            const int k = base + lane;
            int r = k < R ? ord[k] : 0;
            const bool ok = k < R && (unsigned)r < (unsigned)R;     // an invalid entry is skipped, never dereferenced
            if (!ok) r = 0;
            const double x = ok ? rt[r] : 0.0;
            const double inc = wave_incl_scan_f64_dpp(x);
            if (k < R) { F[k] = fc + inc; rop[k] = ok ? p.rec[p.recv_ids[r]].x : -1; }
            fc += lane63_f64(inc);
        }
        const double sum_r = fc;
        double sc = 0.0, ss = 0.0;
        for (int j = lane; j < N; j += 64) {
            const double x = ot[j];
            if (p.col_kind[j]) ss += x; else sc += x;
        }
        const double sum_c = wave_sum_f64_dpp(sc), sum_s = wave_sum_f64_dpp(ss);

        // ---- state of the sample ----
        for (int w = lane; w < n_words; w += 64) rdy[w] = p.ready0[w];
        for (int v = lane; v < n; v += 64) waiting[v] = p.indeg[v];
        double up_busy = 0.0, m = 0.0;
        {
            double s0 = 0.0;                                        // sends without predecessors: requested at 0
            for (int i = lane; i < p.n_send0; i += 64) s0 += ot[p.send0[i]];
            s0 = wave_sum_f64_dpp(s0);
            if (p.n_send0 > 0) { up_busy = s0; m = s0; }
        }
        wave_sync();

        // What the lane knows of the op it released last: id, column of its time, start of its successors.
        int held_op = -1, held_col = 0, held_beg = 0;
        // the successors listed from succ[beg] on are released at time `at`
        auto release = [&](int beg, double at) {
            if (beg < 0) return;
            double sent = 0.0;
            bool any_send = false;
            for (int base = beg;; base += 64) {
                const int4 se = p.succ[base + lane];
                const uint64_t ends = __ballot(se.x < 0);
                const int n_here = ends ? __builtin_ctzll(ends) + 1 : 64;   // entries of this list among the 64 read
                if (lane < n_here) {
                    const int s2 = se.x & 0x7fffffff;
                    // (16-bit counters: the atomic works on the 32-bit word that holds the counter)
                    uint32_t *word = reinterpret_cast<uint32_t *>(waiting) + (s2 >> 1);
                    const int sh = (s2 & 1) * 16;
                    const uint32_t old = atomicSub(word, 1u << sh);
                    if (((old >> sh) & 0xffffu) == 1u) {
                        if (se.w) { sent += ot[se.y]; any_send = true; }
                        else {
                            atomicOr(&rdy[s2 >> 5], 1u << (s2 & 31));
                            held_op = s2; held_col = se.y; held_beg = se.z;
                        }
                    }
                }
                if (ends) break;
            }
            if (__ballot(any_send) != 0ull) {
                up_busy = fmax(up_busy, at) + wave_sum_f64_dpp(sent);
                m = fmax(m, up_busy);
            }
        };

        // ---- the compute device, op by op ----
        double t_dev = 0.0;
        int k = 0;                                                  // transfers released so far
        for (;;) {
            wave_sync();
            int v = -1;
            for (int w0 = 0; w0 < n_words; w0 += 64) {
                const uint32_t x = w0 + lane < n_words ? rdy[w0 + lane] : 0u;
                const uint64_t has = __ballot(x != 0u);
                if (has != 0ull) {
                    const int l = __builtin_ctzll(has);
                    const uint32_t xw = (uint32_t)__builtin_amdgcn_readlane((int)x, l);
                    v = ((w0 + l) << 5) + __builtin_ctz(xw);
                    break;
                }
            }
            if (v < 0) {
                if (k >= R) break;                                  // nothing ready and no transfer left
                // the device idles until the next transfer ends
                const double at = uniform(F[k]);
                t_dev = fmax(t_dev, at);
                do {
                    release(__builtin_amdgcn_readfirstlane(rop[k]), uniform(F[k]));
                    ++k;
                } while (k < R && uniform(F[k]) <= t_dev);
                continue;
            }
            int v_col, v_beg;
            const uint64_t holders = __ballot(held_op == v);
            if (holders) {
                const int l = __builtin_ctzll(holders);
                v_col = __builtin_amdgcn_readlane(held_col, l);
                v_beg = __builtin_amdgcn_readlane(held_beg, l);
            } else {
                const int4 rv = p.rec[v];
                v_col = __builtin_amdgcn_readfirstlane(rv.z);
                v_beg = __builtin_amdgcn_readfirstlane(rv.x);
            }
            const double finish = t_dev + uniform(ot[v_col]);
            if (lane == 0) rdy[v >> 5] &= ~(1u << (v & 31));
            // transfers that end while the op runs release their successors first (requests to the uplink
            // are served in the order of their instants)
            while (k < R && uniform(F[k]) <= finish) {
                release(__builtin_amdgcn_readfirstlane(rop[k]), uniform(F[k]));
                ++k;
            }
            release(v_beg, finish);
            t_dev = finish;
            m = fmax(m, finish);
        }
        if (R > 0) m = fmax(m, uniform(F[R - 1]));

        if (lane == 0) {
            const double U = sum_c + sum_r + sum_s;
            const double L = fmax(fmax(sum_c, sum_r), sum_s);
            p.makespan[b] = m;
            p.eff[b] = (U == L) ? 1.0 : (U - m) / (U - L);
            if (p.U) p.U[b] = U;
            if (p.L) p.L[b] = L;
            if (p.S) p.S[b] = (U == L || L == 0.0) ? 0.0 : (U - L) / L;
        }
    }
}

// ---- one lane per sample ----
// The loop above keeps a wave for a sample and is bound by its instructions: some hundred per op, nearly all on one
// lane's behalf.  Here every lane follows a sample of its own, with the state in LDS next to those of its neighbours
// (a bit per op, half a byte or a byte per op of several predecessors) and the graph in LDS too, once per workgroup:
//   * ops go by the columns of their times, which ascend with their ids.  rec[v]: the first successor, and where the
//     others start.  An op of one predecessor has no counter: its release needs no memory at all, and the op found ready
//     last stays in a register (`cand`).  The first successor's record and time are read before its release;
//   * `low`, the lowest op in the bitmap, is kept too; the bitmap is read only when an op is taken out of it;
//   * the ends of the transfers are laid out in the order of the samples before the loop (all lanes of the wave, a
//     sample at a time), with the first successor of each recv beside them, and read one ahead;
//   * the rows of op times are read ahead by one more wave of the workgroup, which follows the columns that the lanes
//     announce and touches the lines after them; a lane that waited for its own miss would hold up all the others;
//   * a send leaves its instant and its id in a list in memory, nothing waits for that; after the loop the wave goes
//     through the lists of its samples: the last send ends at the largest instant + times of the sends from there on.
// A step is a chain of latencies (LDS, memory, the sum), so the lanes of a compute unit are spread over up to eight
// waves: more of them, each with fewer lanes, hide each other's waits until their instructions fill the unit.
// 16 384 samples of the ResNet-50 inference graph with 161 sends: 4.06 ms with a wave per sample; 1.07 ms here without the
// wave that reads ahead, 0.86 ms with it, 0.81 ms with the record and time of the expected op read early.
// An entry: column of the op (13 bits), 1 << 13 for a send, (counter + 1) << 14, kNoEntry for none, 1 << 31 last of a list.
constexpr uint32_t kNoEntry = 1u << 30;

constexpr int kLinesAhead = 2;          // (lines of 128 bytes)

struct SendTransfer {                           // 16 bytes
    double end;
    uint32_t entry, more;
};

struct SendLaneParams {
    int32_t B, R, N, n_send, n_send0;
    const uint2 *rec;               // [N] first successor; index of the others + 1 (0: none)
    const uint2 *recv_rec;          // [R] first successor, index of the others + 1
    const uint32_t *succ;           // [n_succ] the other successors
    int32_t n_succ;
    const uint32_t *cnt0;           // [cnt_stride / 4] the counters at the start
    int32_t cnt_stride, half;       // half: two counters in a byte
    const uint64_t *ready0;         // [n_words]
    int32_t n_words, words;         // (words: n_words made odd, the rows of the lanes start in different banks)
    const int32_t *send0;           // [n_send0] columns of the sends without predecessors
    const int32_t *order;
    int32_t order_stride;
    const double *op_time, *recv_time;
    double *makespan, *eff, *U, *L, *S;
    SendTransfer *tr;               // [waves][lanes][R]
    double *req_at;                 // [waves][lanes][n_send]
    uint16_t *req_op;
    int32_t lanes, n_waves;         // samples per wave, waves of the grid
    const int32_t *list, *count;    // the samples to take (NULL: all of them)
    int32_t least;                  // fewer samples than this: none
};

__global__ void __launch_bounds__(576)
simulate_sends_lanes_kernel(const SendLaneParams p)
{
    extern __shared__ double smem[];
    const int R = p.R, N = p.N, L = p.lanes;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = (blockDim.x >> 6) - 1;
    uint2 *rec = reinterpret_cast<uint2 *>(smem);                               // [N]
    uint64_t *rdy_all = reinterpret_cast<uint64_t *>(rec + N);                  // [waves][L][words]
    uint32_t *succ = reinterpret_cast<uint32_t *>(rdy_all + (size_t)waves * L * p.words);
    int32_t *first = reinterpret_cast<int32_t *>(succ + p.n_succ);              // [waves] first sample; -1 not yet, -2 done
    int32_t *col_now = first + waves;                                           // [waves][L] column of the lane's op
    uint8_t *cnt_all = reinterpret_cast<uint8_t *>(col_now + waves * L);        // [waves][L][cnt_stride]
    const int n_samples = p.list ? *p.count : p.B;
    if (n_samples < p.least) return;                        // (the form with one wave per sample takes them)
    const int used = min(L, (n_samples + p.n_waves - 1) / p.n_waves);           // lanes of a wave with a sample
    if (threadIdx.x < waves) first[threadIdx.x] = -1;
    for (int i = threadIdx.x; i < N; i += blockDim.x) rec[i] = p.rec[i];
    for (int i = threadIdx.x; i < p.n_succ; i += blockDim.x) succ[i] = p.succ[i];
    for (int i = threadIdx.x; i < waves * L; i += blockDim.x) col_now[i] = 0;
    __syncthreads();

    auto sample = [&](int i) { return p.list ? p.list[i] : i; };
    if (wave == waves) {
        // reads ahead until every other wave has ended; addresses come from `first` and `col_now` and are kept inside the
        // arrays, so what is read there while it changes can only make a touch useless
        for (;;) {
            bool some = false;
            for (int i0 = 0; i0 < waves * L; i0 += 64) {
                const int i = i0 + lane;
                const int b = i < waves * L ? __hip_atomic_load(first + i / L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : -2;
                some |= b != -2;
                if (b >= 0 && i % L < used && b + i % L < n_samples) {
                    const double *ot = p.op_time + (int64_t)sample(b + i % L) * N;
                    const int c = __hip_atomic_load(col_now + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
                    for (int ahead = 1; ahead <= kLinesAhead; ++ahead) {
                        const double x = ot[min(c + 16 * ahead, N - 1)];
                        asm volatile("" :: "v"(x));
                    }
                }
            }
            if (__ballot(some) == 0ull) return;
            __builtin_amdgcn_s_sleep(1);
        }
    }
    uint64_t *rdy = rdy_all + (wave * L + lane) * p.words;                      // (lane < L)
    uint8_t *cnt = cnt_all + (wave * L + lane) * p.cnt_stride;
    const bool half = p.half != 0;
    const int gwave = wave * gridDim.x + blockIdx.x;        // (few samples: one per compute unit)
    SendTransfer *tr_all = p.tr + (size_t)gwave * L * R;
    const size_t req_base = (size_t)gwave * L * p.n_send;
    uint64_t sum0_start = 0ull, sum1_start = 0ull;
    int low_start = INT_MAX;
    for (int w = p.n_words - 1; w >= 0; --w)
        if (const uint64_t x = p.ready0[w]) {
            if (w < 64) sum0_start |= 1ull << w; else sum1_start |= 1ull << (w - 64);
            low_start = w * 64 + __builtin_ctzll(x);
        }

    for (int64_t i0 = (int64_t)gwave * used; i0 < n_samples; i0 += (int64_t)p.n_waves * used) {
        const int here = min(used, (int)(n_samples - i0));
        const int64_t b = sample((int)i0 + min(lane, here - 1));                 // of the lane
        if (lane < L) col_now[wave * L + lane] = 0;
        if (lane == 0) __hip_atomic_store(first + wave, (int32_t)i0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        // ---- the downlink, a sample at a time; the state of the samples ----
        double sum_r = 0.0;
        for (int j0 = 0; j0 < here; j0 += 4) {
            double fc[4] = {0.0, 0.0, 0.0, 0.0};
            int64_t at[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) at[q] = sample((int)i0 + min(j0 + q, here - 1));
            for (int base = 0; base < R; base += 64) {
                const int k = base + lane;
                int r[4];
                double x[4];
                uint2 e[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) r[q] = k < R && j0 + q < here ? p.order[at[q] * p.order_stride + k] : -1;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // an invalid entry is skipped, never dereferenced
                    const bool ok = (unsigned)r[q] < (unsigned)R;
                    x[q] = 0.0;
                    e[q] = make_uint2(kNoEntry, 0u);
                    if (ok) { x[q] = p.recv_time[at[q] * R + r[q]]; e[q] = p.recv_rec[r[q]]; }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double inc = wave_incl_scan_f64_dpp(x[q]);
                    if (k < R && j0 + q < here) {
                        SendTransfer t;
                        t.end = fc[q] + inc;
                        t.entry = e[q].x;
                        t.more = e[q].y;
                        tr_all[(size_t)(j0 + q) * R + k] = t;
                    }
                    fc[q] += lane63_f64(inc);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) sum_r = lane == j0 + q ? fc[q] : sum_r;
        }
        for (int i = lane; i < p.n_words; i += 64) {
            const uint64_t x = p.ready0[i];
            for (int j = 0; j < here; ++j) rdy_all[(wave * L + j) * p.words + i] = x;
        }
        for (int i = lane; i < p.cnt_stride / 4; i += 64) {
            const uint32_t x = p.cnt0[i];
            for (int j = 0; j < here; ++j) reinterpret_cast<uint32_t *>(cnt_all + (wave * L + j) * p.cnt_stride)[i] = x;
        }
        __threadfence_block();
        wave_sync();

        double m = 0.0, sum_c = 0.0;
        int n_req = 0;
        if (lane < here) {
            const double *ot = p.op_time + b * N;
            const SendTransfer *tr = tr_all + (size_t)lane * R;
            double *req_at = p.req_at + req_base + (size_t)lane * p.n_send;
            uint16_t *req_op = p.req_op + req_base + (size_t)lane * p.n_send;
            for (int i = 0; i < p.n_send0; ++i) { req_at[i] = 0.0; req_op[i] = (uint16_t)p.send0[i]; }
            n_req = p.n_send0;
            uint64_t sum0 = sum0_start, sum1 = sum1_start;
            int low = low_start, cand = INT_MAX;
            double t_dev = 0.0;
            int k = 0;
            SendTransfer cur, next;
            cur.end = TT_INF; cur.entry = kNoEntry; cur.more = 0u;
            next = cur;
            if (R > 0) { cur = tr[0]; next = tr[min(1, R - 1)]; }

            // the successors in `entry` and succ[more - 1 ..] are released at `at`
            auto release = [&](uint32_t entry, uint32_t more, double at) {
                while (!(entry & kNoEntry)) {
                    const uint32_t c = (entry >> 14) & 0xffffu;
                    bool free = true;
                    if (c != 0u) {
                        const uint32_t i = c - 1u, sh = half ? (i & 1u) * 4u : 0u, mask = half ? 15u : 255u;
                        uint8_t *q = cnt + (half ? i >> 1 : i);
                        const uint32_t x = *q, left = (x >> sh) & mask;
                        if (left != 0u) *q = (uint8_t)(x - (1u << sh));
                        free = left == 1u;
                    }
                    const int u = (int)(entry & 0x1fffu);
                    if (free && (entry & 0x2000u)) {
                        if (n_req < p.n_send) { req_at[n_req] = at; req_op[n_req] = (uint16_t)u; ++n_req; }
                    } else if (free) {
                        // the lower of the two stays in the register, the other goes into the bitmap
                        const int put = max(cand, u);
                        cand = min(cand, u);
                        if (put != INT_MAX) {
                            atomicOr(reinterpret_cast<uint32_t *>(rdy) + (put >> 5), 1u << (put & 31));
                            const int w = put >> 6;
                            const uint64_t bit = 1ull << (w & 63);
                            sum0 |= w < 64 ? bit : 0ull;
                            sum1 |= w < 64 ? 0ull : bit;
                            low = min(low, put);
                        }
                    }
                    entry = kNoEntry;
                    if (more != 0u) {
                        const uint32_t e = succ[more - 1u];
                        more = (e >> 31) ? 0u : more + 1u;
                        entry = e & 0x7fffffffu;
                    }
                }
            };
            // the op expected next (the first successor of the one that runs), its record and its time
            int ahead = INT_MAX;
            uint2 ahead_rec = make_uint2(kNoEntry, 0u);
            double ahead_x = 0.0;
            for (;;) {
                const int v = min(cand, low);
                bool idle = v == INT_MAX;
                if (idle && k >= R) break;                  // nothing ready and no transfer left
                uint2 rv = make_uint2(kNoEntry, 0u);
                if (idle) {
                    t_dev = fmax(t_dev, cur.end);           // the device idles until the next transfer ends
                } else {
                    if (v != ahead) { ahead_rec = rec[v]; ahead_x = ot[v]; }
                    rv = ahead_rec;
                    t_dev += ahead_x;
                    sum_c += ahead_x;
                    m = fmax(m, t_dev);
                    // (a send is not run: its time is not touched here)
                    ahead = (rv.x & (0x2000u | kNoEntry)) ? v : (int)(rv.x & 0x1fffu);
                    ahead_rec = rec[ahead];
                    ahead_x = ot[ahead];
                    __hip_atomic_store(col_now + wave * L + lane, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (v == cand) {
                        cand = INT_MAX;
                    } else {
                        int w = v >> 6;
                        uint64_t y = rdy[w];
                        y &= y - 1ull;
                        rdy[w] = y;
                        if (y == 0ull) {
                            const uint64_t bit = 1ull << (w & 63);
                            sum0 &= w < 64 ? ~bit : ~0ull;
                            sum1 &= w < 64 ? ~0ull : ~bit;
                            w = sum0 != 0ull ? __builtin_ctzll(sum0) : (sum1 != 0ull ? 64 + __builtin_ctzll(sum1) : w);
                            y = rdy[w];
                        }
                        low = y != 0ull ? (w << 6) + __builtin_ctzll(y) : INT_MAX;
                    }
                }
                // transfers that end up to then release their successors first (requests to the uplink are served in
                // the order of their instants); `idle`: the first of them whatever it compares to
                while (k < R && (idle || cur.end <= t_dev)) {
                    idle = false;
                    release(cur.entry, cur.more, cur.end);
                    cur = next;
                    ++k;
                    next = tr[min(k + 1, R - 1)];
                }
                release(rv.x, rv.y, t_dev);
            }
            m = fmax(m, sum_r);
        }
        __threadfence_block();
        wave_sync();

        // ---- the uplink, a sample at a time: entries from the last one down ----
        double sum_s = 0.0;
        for (int j0 = 0; j0 < here; j0 += 4) {
            double acc[4] = {0.0, 0.0, 0.0, 0.0}, last[4] = {0.0, 0.0, 0.0, 0.0};
            int count[4], most = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                count[q] = j0 + q < here ? __builtin_amdgcn_readlane(n_req, j0 + q) : 0;
                most = max(most, count[q]);
            }
            for (int down = 0; down < most; down += 64) {
                double x[4], at[4];
                int op[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = count[q] - 1 - down - lane;
                    const size_t slot = req_base + (size_t)(j0 + q) * p.n_send + i;
                    op[q] = -1;
                    at[q] = 0.0;
                    if (i >= 0) { op[q] = p.req_op[slot]; at[q] = p.req_at[slot]; }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x[q] = 0.0;
                    if (op[q] >= 0) x[q] = p.op_time[(int64_t)sample((int)i0 + j0 + q) * N + op[q]];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double inc = wave_incl_scan_f64_dpp(x[q]);
                    if (op[q] >= 0) last[q] = fmax(last[q], at[q] + (acc[q] + inc));
                    acc[q] += lane63_f64(inc);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double end = wave_max_f64_dpp(last[q]);
                m = lane == j0 + q ? fmax(m, end) : m;
                sum_s = lane == j0 + q ? acc[q] : sum_s;
            }
        }

        if (lane < here) {
            const double U = sum_c + sum_r + sum_s;
            const double Lb = fmax(fmax(sum_c, sum_r), sum_s);
            p.makespan[b] = m;
            p.eff[b] = (U == Lb) ? 1.0 : (U - m) / (U - Lb);
            if (p.U) p.U[b] = U;
            if (p.L) p.L[b] = Lb;
            if (p.S) p.S[b] = (U == Lb || Lb == 0.0) ? 0.0 : (U - Lb) / Lb;
        }
        wave_sync();
    }
    if (lane == 0) __hip_atomic_store(first + wave, -2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

struct LanesShape {
    int waves = 0, lanes = 0, grid = 0;             // waves == 0: the graph does not suit the form
    size_t lds = 0, tr_bytes = 0, at_bytes = 0, bytes = 0;
};

static LanesShape lanes_shape(const Dag &d, int B, int wave_form_resident)
{
    LanesShape f;
    if (!d.d_lane_rec || d.N < 1) return f;
    const int cus = device_cu_count(d.device);
    const size_t words = (((size_t)d.N + 63) / 64) | 1, tables = (size_t)d.N * 8 + (size_t)d.n_lane_succ * 4 + 64;
    const size_t state = words * 8 + (size_t)d.lane_cnt_bytes + 4, budget = 158 * 1024;
    if (tables >= budget) return f;
    const int cap = (int)std::min<size_t>((budget - tables) / state, 512);
    const int want = (int)std::min<int64_t>(((int64_t)B + cus - 1) / cus, 512);     // samples of a compute unit
    if (cap < 1 || (cap < want && cap <= wave_form_resident)) return f;
    const int per_cu = std::max(1, std::min(cap, want));
    f.waves = std::min(8, per_cu);
    f.lanes = std::min(64, per_cu / f.waves);
    const int64_t groups = ((int64_t)B + f.lanes - 1) / f.lanes;
    f.grid = (int)std::min<int64_t>((groups + f.waves - 1) / f.waves, cus);
    f.lds = tables + state * f.waves * f.lanes;
    const size_t slots = (size_t)f.grid * f.waves * f.lanes;
    f.tr_bytes = slots * d.R * sizeof(SendTransfer);
    f.at_bytes = slots * d.h_send_ids.size() * 8;
    f.bytes = f.tr_bytes + f.at_bytes + slots * d.h_send_ids.size() * 2 + 64;
    return f;
}

static hipError_t launch_sends_lanes(Dag &d, const SimArgs &a, const LanesShape &f, void *work, const int32_t *list,
                                     const int32_t *count, int least, hipStream_t s)
{
    SendLaneParams p{};
    p.least = std::max(1, least);
    p.B = a.B; p.R = d.R; p.N = d.N; p.n_send = (int32_t)d.h_send_ids.size(); p.n_send0 = d.n_send_free;
    p.rec = d.d_lane_rec; p.recv_rec = d.d_lane_recv_rec; p.succ = d.d_lane_succ; p.n_succ = d.n_lane_succ;
    p.cnt0 = reinterpret_cast<const uint32_t *>(d.d_lane_cnt0); p.cnt_stride = d.lane_cnt_bytes; p.half = d.lane_half;
    p.ready0 = d.d_lane_ready0; p.n_words = (d.N + 63) / 64; p.words = p.n_words | 1;
    p.send0 = d.d_send_free;
    p.order = a.order; p.order_stride = a.order_stride;
    p.op_time = static_cast<const double *>(a.op_time); p.recv_time = static_cast<const double *>(a.recv_time);
    p.makespan = a.makespan; p.eff = a.eff; p.U = a.U; p.L = a.L; p.S = a.S;
    p.lanes = f.lanes; p.n_waves = f.grid * f.waves;
    p.list = list; p.count = count;
    p.tr = static_cast<SendTransfer *>(work);
    p.req_at = reinterpret_cast<double *>(static_cast<char *>(work) + f.tr_bytes);
    p.req_op = reinterpret_cast<uint16_t *>(static_cast<char *>(work) + f.tr_bytes + f.at_bytes);
    if (f.lds > 48 * 1024) {
        const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(simulate_sends_lanes_kernel), f.lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(simulate_sends_lanes_kernel, dim3(f.grid), dim3(64 * (f.waves + 1)), f.lds, s, p);
    return hipGetLastError();
}

hipError_t launch_simulate_sends(Dag &d, const SimArgs &a, hipStream_t s)
{
    if (a.B == 0) return hipSuccess;
    if (!d.d_send_rec || d.n > 65535 * 2) return hipErrorNotSupported;
    SendSimParams p{};
    p.B = a.B; p.n = d.n; p.R = d.R; p.N = d.N;
    p.rec = d.d_send_rec; p.succ = d.d_send_succ; p.indeg = d.d_send_indeg; p.ready0 = d.d_send_ready0;
    p.send0 = d.d_send_free; p.n_send0 = d.n_send_free; p.col_kind = d.d_send_col_kind;
    p.recv_ids = d.d_send_recv_ids;
    p.order = a.order; p.order_stride = a.order_stride;
    p.op_time = static_cast<const double *>(a.op_time); p.recv_time = static_cast<const double *>(a.recv_time);
    p.makespan = a.makespan; p.eff = a.eff; p.U = a.U; p.L = a.L; p.S = a.S;
    const size_t n_words = ((size_t)d.n + 31) / 32;
    size_t per_wave = (size_t)d.R * 12 + n_words * 4 + (((size_t)d.n + 1) & ~(size_t)1) * 2;
    per_wave = (per_wave + 15) & ~(size_t)15;
    int waves = 4;
    while (waves > 1 && per_wave * waves > 150 * 1024) --waves;
    const bool wave_form = per_wave * waves <= 150 * 1024;
    const size_t lds = per_wave * waves;
    int per_cu = 0;
    hipError_t e = hipSuccess;
    if (wave_form) {
        p.wave_bytes = (int32_t)per_wave;
        if (lds > 48 * 1024) {
            e = ensure_dynamic_lds(reinterpret_cast<const void *>(simulate_sends_kernel), lds);
            if (e != hipSuccess) return e;
        }
        e = cached_blocks_per_cu(&per_cu, reinterpret_cast<const void *>(simulate_sends_kernel), 64 * waves, lds);
        if (e != hipSuccess) return e;
        if (per_cu < 1) per_cu = 1;
    }
    const int resident = per_cu * waves * device_cu_count(d.device);
    const LanesShape f = lanes_shape(d, a.B, per_cu * waves);
    if (!wave_form && f.waves == 0) return hipErrorNotSupported;
    int32_t *list = nullptr, *count = nullptr;
    if (d.d_straight_tiles) {
        e = launch_sends_straight(d, a, f.bytes, &list, &count, s);
        if (e != hipSuccess) return e;
    }
    // Samples that the wave-per-sample form holds all at once are its own where lists of successors are long: it releases a
    // list in one step, a lane entry by entry (layered graphs, 2.5 successors per op: a lane takes 1.4 times as long; model
    // graphs, 1.0 to 1.5: 0.6 to 0.75 times), and on graphs so small that what comes before and after the ops counts.
    const bool wave_first = wave_form && (f.waves == 0 || d.n < 192 || (int64_t)d.E * 10 > (int64_t)d.n * 16);
    p.list = list; p.count = count;
    p.most = f.waves == 0 ? a.B : resident;
    if (f.waves > 0 && (!wave_first || a.B > resident)) {
        if (!list) {
            e = ensure_workspace(&d, f.bytes);
            if (e != hipSuccess) return e;
        }
        e = launch_sends_lanes(d, a, f, list ? sends_straight_rest(count, a.B) : d.d_work, list, count,
                               wave_first ? resident + 1 : 1, s);
        if (e != hipSuccess || !wave_first || !list) return e;
    }
    int grid = per_cu * device_cu_count(d.device);
    const int need = (a.B + waves - 1) / waves;
    if (grid > need) grid = need;
    p.n_waves = grid * waves;
    hipLaunchKernelGGL(simulate_sends_kernel, dim3(grid), dim3(64 * waves), lds, s, p);
    return hipGetLastError();
}

}  // namespace tictac
