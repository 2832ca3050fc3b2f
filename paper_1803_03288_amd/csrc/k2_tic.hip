// TIC (Sec. 4.2, Algorithm 2): with every recv outstanding and the General Time Oracle
// (recv = 1, others = 0), op.M = |op.dep|, every P is 0 and
//   priority(recv i) = M+ = min{ |dep[v]| : v a compute op, i in dep[v], |dep[v]| > 1 }.
// Integer arithmetic throughout, so the result does not depend on the order of the
// min-updates.
#include <algorithm>

#include "internal.h"

namespace tictac {

__global__ void fill_i32(int32_t *p, size_t n, int32_t value)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

// One wave per row at a time: popcount of the row, then a min-update of every recv in it.
// USE_LDS: the block keeps its own copy of prio in LDS and merges it at the end.
template <bool USE_LDS>
__global__ void __launch_bounds__(256)
tic_min_kernel(int32_t n, int32_t R, int32_t W, const uint64_t *__restrict__ dep,
               const int32_t *__restrict__ recv_of_op, int32_t rows_per_block, int32_t *prio)
{
    extern __shared__ int32_t prio_l[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    if (USE_LDS) {
        for (int32_t i = threadIdx.x; i < R; i += blockDim.x) prio_l[i] = TICTAC_PRIO_INF;
        __syncthreads();
    }
    int32_t *target = USE_LDS ? prio_l : prio;
    const int32_t v0 = blockIdx.x * rows_per_block;
    const int32_t v1 = min(n, v0 + rows_per_block);
    for (int32_t v = v0 + wave; v < v1; v += n_waves) {
        if (recv_of_op[v] >= 0) continue;                 // wave-uniform
        const uint64_t *row = dep + (size_t)v * W;
        int32_t cnt = 0;
        for (int32_t w = lane; w < W; w += 64) cnt += __popcll(row[w]);
        for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
        if (cnt <= 1) continue;                           // wave-uniform
        for (int32_t w = lane; w < W; w += 64) {
            uint64_t x = row[w];
            while (x) {
                const int b = __builtin_ctzll(x);
                x &= x - 1;
                atomicMin(&target[w * 64 + b], cnt);
            }
        }
    }
    if (USE_LDS) {
        __syncthreads();
        for (int32_t i = threadIdx.x; i < R; i += blockDim.x)
            if (prio_l[i] != TICTAC_PRIO_INF) atomicMin(&prio[i], prio_l[i]);
    }
}

// rank[i] = number of recvs j with (prio[j], j) < (prio[i], i); order[rank[i]] = i.
__global__ void __launch_bounds__(256)
tic_rank_kernel(int32_t R, const int32_t *__restrict__ prio, int32_t *order, int32_t *rank)
{
    __shared__ int32_t tile[1024];
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t pi = (i < R) ? prio[i] : 0;
    int32_t r = 0;
    for (int32_t j0 = 0; j0 < R; j0 += 1024) {
        const int32_t m = min(1024, R - j0);
        __syncthreads();
        for (int32_t j = threadIdx.x; j < m; j += blockDim.x) tile[j] = prio[j0 + j];
        __syncthreads();
        if (i < R)
            for (int32_t j = 0; j < m; ++j) {
                const int32_t pj = tile[j];
                r += (pj < pi) || (pj == pi && (j0 + j) < i);
            }
    }
    if (i < R) {
        if (rank) rank[i] = r;
        if (order) order[r] = i;
    }
}

// Small graphs in one launch of one workgroup: the minimum of |dep| over the classes (compute ops with identical rows)
// whose row holds the recv, then its rank by counting.  depT is the transposed class table [W][Cpad].  When the table and
// the class sizes fit (lds_words > 0: W * Cpad words, then C counts), the workgroup first copies them to LDS with all its
// threads, so that the loop over the classes does not wait on memory.  Each recv has `parts` threads, a wave apart
// (thread q * Rpad + i, Rpad the recvs rounded up to whole waves), each with a share of the classes and then of the other
// recvs: one thread per recv took 14 us for 161 recvs and 166 classes, nearly all of it the two loops.
__global__ void __launch_bounds__(1024)
tic_small_kernel(int32_t R, int32_t C, int32_t Cpad, int32_t lds_words, int32_t Rpad, int32_t parts,
                 const uint64_t *__restrict__ depT, const int32_t *__restrict__ cnt0, int32_t *prio, int32_t *order, int32_t *rank)
{
    extern __shared__ uint64_t tic_table[];         // [lds_words] depT, then [C] counts
    __shared__ int32_t tile[1024], below[1024];
    const int32_t t = threadIdx.x;
    const int32_t q = t / Rpad, i = t - q * Rpad;
    int32_t *cnt_l = reinterpret_cast<int32_t *>(tic_table + lds_words);
    if (lds_words > 0) {
        for (int32_t x = t; x < lds_words; x += blockDim.x) tic_table[x] = depT[x];
        for (int32_t c = t; c < C; c += blockDim.x) cnt_l[c] = cnt0[c];
    }
    if (t < Rpad) { tile[t] = TICTAC_PRIO_INF; below[t] = 0; }
    __syncthreads();
    if (q < parts && i < R) {
        const int32_t share = (C + parts - 1) / parts, c0 = q * share, c1 = min(C, c0 + share);
        const int sh = i & 63;
        int32_t m = TICTAC_PRIO_INF;
        if (lds_words > 0) {
            const uint64_t *col = tic_table + (size_t)(i >> 6) * Cpad;
#pragma unroll 8
            for (int32_t c = c0; c < c1; ++c) {
                const int32_t k = cnt_l[c];
                if (((col[c] >> sh) & 1ull) && k > 1) m = min(m, k);
            }
        } else {
            const uint64_t *col = depT + (size_t)(i >> 6) * Cpad;   // the same word for the 64 lanes of a wave
#pragma unroll 8
            for (int32_t c = c0; c < c1; ++c) {
                const int32_t k = cnt0[c];
                if (((col[c] >> sh) & 1ull) && k > 1) m = min(m, k);
            }
        }
        atomicMin(&tile[i], m);
    }
    __syncthreads();
    if (q < parts && i < R && (order || rank)) {
        const int32_t share = (R + parts - 1) / parts, j0 = q * share, j1 = min(R, j0 + share);
        const int32_t m = tile[i];
        int32_t r = 0;
#pragma unroll 8
        for (int32_t j = j0; j < j1; ++j) {
            const int32_t pj = tile[j];
            r += (pj < m) || (pj == m && j < i);
        }
        atomicAdd(&below[i], r);
    }
    __syncthreads();
    if (t < R) {
        prio[t] = tile[t];
        if (rank) rank[t] = below[t];
        if (order) order[below[t]] = t;
    }
}

hipError_t launch_tic(const Dag &d, int32_t *prio, int32_t *order, int32_t *rank, int32_t *, hipStream_t s)
{
    const int32_t R = d.R;
    if (R == 0) return hipSuccess;
    if (R <= 1024 && d.C <= 8192 && d.d_cls_depT && d.d_cls_cnt0) {
        const int Rpad = (R + 63) / 64 * 64;
        // (parts that save less than a few steps of the loops are not worth their atomics)
        const int parts = std::max(1, std::min(1024 / Rpad, (std::max(R, d.C) + 15) / 16));
        const size_t words = (size_t)d.W * d.Cpad;
        const size_t lds = words * 8 + (size_t)d.C * 4;
        const bool in_lds = lds <= 40 * 1024;
        int threads = Rpad * parts;
        if (in_lds && threads < 256) threads = 256;     // more threads for the copy
        hipLaunchKernelGGL(tic_small_kernel, dim3(1), dim3(threads), in_lds ? lds : 0, s, R, d.C, d.Cpad,
                           in_lds ? (int32_t)words : 0, Rpad, parts, d.d_cls_depT, d.d_cls_cnt0, prio, order, rank);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(fill_i32, dim3((R + 255) / 256), dim3(256), 0, s, prio, (size_t)R, (int32_t)TICTAC_PRIO_INF);
    if (d.n > 0) {
        const int32_t rows_per_block = d.n <= 4096 ? 32 : 128;
        const int blocks = (d.n + rows_per_block - 1) / rows_per_block;
        const size_t lds = (size_t)R * sizeof(int32_t);
        if (lds <= 48 * 1024)
            hipLaunchKernelGGL(tic_min_kernel<true>, dim3(blocks), dim3(256), lds, s, d.n, R, d.W, d.d_dep,
                               d.d_recv_of_op, rows_per_block, prio);
        else
            hipLaunchKernelGGL(tic_min_kernel<false>, dim3(blocks), dim3(256), 0, s, d.n, R, d.W, d.d_dep,
                               d.d_recv_of_op, rows_per_block, prio);
    }
    if (order || rank)
        hipLaunchKernelGGL(tic_rank_kernel, dim3((R + 255) / 256), dim3(256), 0, s, R, prio, order, rank);
    return hipGetLastError();
}

// ---- class grouping on the device (see internal.h) ----
__device__ __forceinline__ uint64_t mix64(uint64_t h, uint64_t x, uint64_t k)
{
    h ^= x + k + (h << 6) + (h >> 2);
    return h * 0xFF51AFD7ED558CCDull;
}

// one wave per compute op: lanes take words lane, lane + 64, ...; the two hashes mix the words in index order, so
// they are formed by lane 0 from the words gathered through LDS-free cross-lane reads, 64 words at a time
__global__ void __launch_bounds__(256)
row_digest_kernel(int32_t N, int32_t W, const int32_t *__restrict__ op_of_col, const uint64_t *__restrict__ dep,
                  int32_t *__restrict__ digest)
{
    const int lane = threadIdx.x & 63;
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= N) return;
    const uint64_t *row = dep + (size_t)op_of_col[j] * W;
    uint64_t h0 = 0x9E3779B97F4A7C15ull, h1 = 0xC2B2AE3D27D4EB4Full;
    int cnt = 0, lowest = -1;
    for (int w0 = 0; w0 < W; w0 += 64) {
        const uint64_t x = w0 + lane < W ? row[w0 + lane] : 0ull;
        cnt += __builtin_popcountll(x);
        const uint64_t has = __ballot(x != 0ull);
        if (lowest < 0 && has != 0ull) {
            const int l = __builtin_ctzll(has);
            const uint64_t xl = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), l) << 32) |
                                (uint32_t)__builtin_amdgcn_readlane((int)x, l);
            lowest = (w0 + l) * 64 + __builtin_ctzll(xl);
        }
        // position-dependent contribution of every word, combined by a sum: independent of the order of the lanes
        const uint64_t k = (uint64_t)(w0 + lane) * 0x9E3779B97F4A7C15ull;
        uint64_t a = mix64(0x243F6A8885A308D3ull ^ k, x, 0x9E3779B97F4A7C15ull);
        uint64_t b = mix64(0x13198A2E03707344ull + k, x ^ (x >> 29), 0xA4093822299F31D0ull);
        a ^= a >> 32; b ^= b >> 31;
        if (x == 0ull) { a = 0; b = 0; }            // (rows are sparse; an absent word adds nothing)
        for (int off = 32; off > 0; off >>= 1) {
            a += ((uint64_t)(uint32_t)__shfl_xor((int)(a >> 32), off) << 32) | (uint32_t)__shfl_xor((int)a, off);
            b += ((uint64_t)(uint32_t)__shfl_xor((int)(b >> 32), off) << 32) | (uint32_t)__shfl_xor((int)b, off);
        }
        h0 = mix64(h0, a, 0x9E3779B97F4A7C15ull);
        h1 = mix64(h1, b, 0x452821E638D01377ull);
    }
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
    if (lane == 0) {
        int32_t *o = digest + (size_t)j * 8;
        o[0] = (int32_t)h0; o[1] = (int32_t)(h0 >> 32); o[2] = (int32_t)h1; o[3] = (int32_t)(h1 >> 32);
        o[4] = cnt; o[5] = lowest; o[6] = 0; o[7] = 0;
    }
}

// Ops of equal digests find each other through a table of at least twice as many slots, probed one after the other: the
// first to take a slot lends it its digest, the lowest op of the slot becomes the representative of all of them.
__global__ void __launch_bounds__(256)
group_insert_kernel(int32_t N, uint32_t mask, const int4 *__restrict__ digest, int32_t *slot, uint32_t *lowest, uint32_t *where)
{
    const int32_t j = blockIdx.x * 256 + threadIdx.x;
    if (j >= N) return;
    const int4 g = digest[2 * (size_t)j];
    const int cnt = digest[2 * (size_t)j + 1].x;
    uint32_t q = ((uint32_t)g.x ^ (uint32_t)g.y * 0x9E3779B1u ^ (uint32_t)g.w) & mask;
    for (uint32_t tries = 0; tries <= mask; ++tries) {
        const int32_t held = atomicCAS(&slot[q], -1, j);
        const int32_t leader = held < 0 ? j : held;
        const int4 l = digest[2 * (size_t)leader];
        if (l.x == g.x && l.y == g.y && l.z == g.z && l.w == g.w && digest[2 * (size_t)leader + 1].x == cnt) break;
        q = (q + 1) & mask;
    }
    atomicMin(&lowest[q], (uint32_t)j);
    where[j] = q;
}

// out: [N] the representative of every op, [N] the set bits of its row, [N] the lowest one
__global__ void __launch_bounds__(256)
group_out_kernel(int32_t N, const int4 *__restrict__ digest, const uint32_t *__restrict__ lowest, const uint32_t *__restrict__ where,
                 int32_t *out)
{
    const int32_t j = blockIdx.x * 256 + threadIdx.x;
    if (j >= N) return;
    const int4 d = digest[2 * (size_t)j + 1];
    out[j] = (int32_t)lowest[where[j]];
    out[N + (size_t)j] = d.x;
    out[2 * (size_t)N + j] = d.y;
}

// workspace: the result [3][N] first (see group_out_kernel), then digests [N][8], slots, lowest members and the op's slot
// (N is bounded by group_on_device, so the places of the table are counted in 32 bits)
static uint32_t group_slots(int32_t N)
{
    uint32_t cap = 64;
    while (cap < 2 * (uint32_t)N) cap *= 2;
    return cap;
}
static size_t group_digest_offset(int32_t N) { return ((size_t)N * 12 + 255) & ~(size_t)255; }
size_t group_workspace_bytes(int32_t N) { return group_digest_offset(N) + (size_t)N * 36 + (size_t)group_slots(N) * 8; }

// The digests take a wave per op and the check of the rows a thread per word; a grid counts its threads in 32 bits.
bool group_on_device(int32_t N, int32_t W) { return N <= 1 << 25 && (int64_t)N * W <= (int64_t)1 << 31; }

hipError_t launch_group_rows(const Dag &d, const int32_t *op_of_col, void *work, hipStream_t s)
{
    const int32_t N = d.N;
    if (N == 0) return hipSuccess;
    if (!group_on_device(N, d.W)) return hipErrorInvalidValue;
    const uint32_t cap = group_slots(N);
    int32_t *digest = reinterpret_cast<int32_t *>(static_cast<char *>(work) + group_digest_offset(N));
    int32_t *slot = digest + (size_t)N * 8;
    uint32_t *lowest = reinterpret_cast<uint32_t *>(slot + cap), *where = lowest + cap;
    const int4 *dg = reinterpret_cast<const int4 *>(digest);
    const dim3 per_op((N + 255) / 256);
    hipLaunchKernelGGL(row_digest_kernel, dim3((N + 3) / 4), dim3(256), 0, s, N, d.W, op_of_col, d.d_dep, digest);
    hipLaunchKernelGGL(fill_i32, dim3((2 * cap + 255) / 256), dim3(256), 0, s, slot, (size_t)2 * cap, -1);
    hipLaunchKernelGGL(group_insert_kernel, per_op, dim3(256), 0, s, N, cap - 1, dg, slot, lowest, where);
    hipLaunchKernelGGL(group_out_kernel, per_op, dim3(256), 0, s, N, dg, lowest, where, static_cast<int32_t *>(work));
    return hipGetLastError();
}

// thread per (class, word): the class's row from its first op, into cls_dep and cls_depT
__global__ void __launch_bounds__(256)
class_rows_kernel(int32_t C, int32_t Cpad, int32_t W, const int32_t *__restrict__ first_op,
                  const uint64_t *__restrict__ dep, uint64_t *__restrict__ cls_dep, uint64_t *__restrict__ cls_depT)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)Cpad * W) return;
    const int c = (int)(idx / W), w = (int)(idx % W);
    const uint64_t x = c < C ? dep[(size_t)first_op[c] * W + w] : 0ull;
    if (c < C) cls_dep[idx] = x;
    cls_depT[(size_t)w * Cpad + c] = x;
}

// thread per (compute op, word): the op's row against the row of its class
__global__ void __launch_bounds__(256)
class_check_kernel(int32_t N, int32_t W, const int32_t *__restrict__ op_of_col, const int32_t *__restrict__ col_cls,
                   const uint64_t *__restrict__ dep, const uint64_t *__restrict__ cls_dep, int32_t *mismatch)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)N * W) return;
    const int j = (int)(idx / W), w = (int)(idx % W);
    if (dep[(size_t)op_of_col[j] * W + w] != cls_dep[(size_t)col_cls[j] * W + w]) atomicOr(mismatch, 1);
}

hipError_t launch_class_rows(const Dag &d, const int32_t *op_of_col, const int32_t *first_op, int32_t *mismatch,
                             hipStream_t s)
{
    if (d.C == 0 || d.W == 0) return hipSuccess;
    const size_t total = (size_t)d.Cpad * d.W;
    hipLaunchKernelGGL(class_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, d.C, d.Cpad, d.W,
                       first_op, d.d_dep, d.d_cls_dep, d.d_cls_depT);
    const size_t all = (size_t)d.N * d.W;
    hipLaunchKernelGGL(class_check_kernel, dim3((unsigned)((all + 255) / 256)), dim3(256), 0, s, d.N, d.W, op_of_col,
                       d.d_col_cls, d.d_dep, d.d_cls_dep, mismatch);
    return hipGetLastError();
}

}  // namespace tictac
