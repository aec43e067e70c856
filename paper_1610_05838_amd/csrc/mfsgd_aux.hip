// mfsgd_aux.hip -- storage-type independent kernels: RMSE final reduction,
// index checks, ticket reset and the wavefront-update planner.
#include <algorithm>

#include "mfsgd_device.hpp"
#include "mfsgd_launch.hpp"

namespace mfsgd {

// Pass 2 of the test RMSE: one workgroup adds the kRmseWaves partial sums in
// a fixed order (strided per thread, then a fixed tree), so the result does
// not depend on timing.
__global__ __launch_bounds__(256) void k_rmse_final(const double* __restrict__ partial, int64_t ntest,
                                                    double* __restrict__ out)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < kRmseWaves; i += 256)
        acc += partial[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        out[0] = ntest > 0 ? sqrt(red[0] / (double)ntest) : 0.0;
}

hipError_t rmse_final(const double* partial, int64_t ntest, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_rmse_final, dim3(1), dim3(256), 0, st, partial, ntest, out);
    return hipGetLastError();
}

// Index check, bound by reading the samples (99 M: 0.17 ms, 6.9 TB/s with part
// of them in the Infinity Cache).
__global__ void k_check(const Sample* __restrict__ S, int64_t nnz, int64_t m, int64_t n, int* bad, int* too,
                        uint32_t* prio)
{
    int found = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * blockDim.x) {
        const int u = __builtin_nontemporal_load(&S[i].u);
        const int v = __builtin_nontemporal_load(&S[i].v);
        found |= (u < 0) | (u >= m) | (v < 0) | (v >= n);
    }
    if (found) {
        atomicOr(bad, 1);
        if (too)
            atomicOr(too, 1);
    }
    if (prio && blockIdx.x == 0 && threadIdx.x == 0) {
        const int64_t units = (nnz + 63) / 64;
        *prio = units > 0xffffffffll ? 0xffffffffu : (uint32_t)units;
    }
}

hipError_t check_indices(const Sample* S, int64_t nnz, int64_t m, int64_t n, int* bad, hipStream_t st)
{
    if (nnz <= 0)
        return hipSuccess;
    const int64_t blocks = std::min<int64_t>((nnz + 255) / 256, 8192);
    hipLaunchKernelGGL(k_check, dim3((unsigned)blocks), dim3(256), 0, st, S, nnz, m, n, bad, (int*)nullptr,
                       (uint32_t*)nullptr);
    return hipGetLastError();
}

hipError_t check_one_block(const Sample* S, int64_t nnz, int64_t m, int64_t n, int* gate, int* err, uint32_t* prio,
                           hipStream_t st)
{
    const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((nnz + 255) / 256, 8192));
    hipLaunchKernelGGL(k_check, dim3((unsigned)blocks), dim3(256), 0, st, S, nnz, m, n, gate, err, prio);
    return hipGetLastError();
}

__global__ void k_reset_tickets(uint32_t* tickets, uint32_t* sched, int64_t* one, int64_t nnz)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMaxGrid)
        tickets[i] = 0u;
    if (i < kSchedWords)
        sched[i] = 0u;
    if (one && i < 2)
        one[i] = i ? nnz : 0;
}

hipError_t reset_tickets(uint32_t* tickets, uint32_t* sched, int64_t* one, int64_t nnz, hipStream_t st)
{
    hipLaunchKernelGGL(k_reset_tickets, dim3((kSchedWords + 255) / 256), dim3(256), 0, st, tickets, sched, one, nnz);
    return hipGetLastError();
}

// Critical-path priorities of a block-scheduled epoch.  Block (t, w) is team
// t's block of wave w, column C[(t + O[w]) mod s]; it must be exhausted
// before the same team's block of wave w+1 can be claimed, and completed
// before the column's block of wave w+1 (team (t + O[w] - O[w+1]) mod s)
// opens.  prio[t*s + w] = the largest number of 64-sample units on a chain
// of such successors from (t, w) to the end of the epoch, its own included:
// the work that still has to follow this block one step at a time.  One
// workgroup, lane t for team t, waves from the last to the first.
__global__ __launch_bounds__(kMaxGrid) void k_block_priority(const int64_t* __restrict__ bstart, int s,
                                                            uint64_t sigma_c, uint64_t sigma_o,
                                                            uint32_t* __restrict__ prio)
{
    __shared__ int Cperm[kMaxGrid], Ooff[kMaxGrid];
    __shared__ uint64_t chain[kMaxGrid];
    const int t = threadIdx.x;
    if (t == 0) {
        shuffle_perm(sigma_c, s, Cperm);
        shuffle_perm(sigma_o, s, Ooff);
    }
    chain[t] = 0;
    __syncthreads();
    for (int w = s - 1; w >= 0; --w) {
        uint64_t v = 0;
        if (t < s) {
            const int64_t b = (int64_t)t * s + Cperm[(t + Ooff[w]) % s];
            v = (uint64_t)((bstart[b + 1] - bstart[b] + 63) / 64);
            if (w + 1 < s) {
                const int tc = ((t + Ooff[w] - Ooff[w + 1]) % s + s) % s;
                v += chain[t] > chain[tc] ? chain[t] : chain[tc];
            }
        }
        __syncthreads();
        if (t < s) {
            chain[t] = v;
            prio[(int64_t)t * s + w] = v > 0xffffffffull ? 0xffffffffu : (uint32_t)v;
        }
        __syncthreads();
    }
}

hipError_t block_priority(const int64_t* bstart, int s, uint64_t sigma_c, uint64_t sigma_o, uint32_t* prio,
                          hipStream_t st)
{
    hipLaunchKernelGGL(k_block_priority, dim3(1), dim3(kMaxGrid), 0, st, bstart, s, sigma_c, sigma_o, prio);
    return hipGetLastError();
}

// Which XCD (accelerator complex die) runs each workgroup: the hardware
// register XCC_ID of gfx94x/gfx950.
__global__ void k_probe_xcc(int* out)
{
    unsigned xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    if (threadIdx.x == 0)
        out[blockIdx.x] = (int)(xcc & 0xf);
}

hipError_t probe_xcc(int* out, int n, hipStream_t st)
{
    hipLaunchKernelGGL(k_probe_xcc, dim3(n), dim3(64), 0, st, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Planner: a stable counting sort of the samples by block id
// (row block floor(u*s/m)) * s + (column block floor(v*s/n)).
//   1. each of `chunks` workgroups counts its contiguous chunk per block (and
//      flags indices out of range);
//   2. per block, an exclusive scan over the chunks;
//   3. an exclusive scan over the blocks gives the block starts;
//   4. one wavefront per chunk walks it in order, 64 samples at a time, ranks
//      the samples of equal blocks by lane and scatters them.
// Chunks, steps and lanes are all taken in array order, so every block keeps
// its samples in array order.
// ---------------------------------------------------------------------------
// Block cut: the first index of every range, rb[0..s] and cb[0..s] (rb[s] = m,
// cb[s] = n; index i is in the last range whose first index is <= i), and for
// equal index ranges (floor(i*s/N)) the scale s/N (0: ranges of other sizes).
struct Cut {
    int rb[kMaxGrid + 1];
    int cb[kMaxGrid + 1];
};

__device__ __forceinline__ void load_cut(Cut& c, const int64_t* __restrict__ rbnd, const int64_t* __restrict__ cbnd,
                                         int s)
{
    for (int i = threadIdx.x; i <= s; i += blockDim.x) {
        c.rb[i] = (int)rbnd[i];
        c.cb[i] = (int)cbnd[i];
    }
}

// The range of index i.  Equal ranges: i * (s/N) in binary32 is off by less
// than one range (i, s and N are each rounded once, s <= 64), so one look at
// the guessed range's two ends settles it; the 64-bit division this replaces
// took most of the counting kernel's instructions.  Other cuts: bisection.
__device__ __forceinline__ int range_of(int i, const int* b, int s, float scale)
{
    if (scale > 0.f) {
        int q = (int)((float)i * scale);
        q = q < s ? q : s - 1;
        return q - (i < b[q] ? 1 : 0) + (i >= b[q + 1] ? 1 : 0);
    }
    int lo = 0, hi = s - 1; // largest k in [0, s-1] with b[k] <= i
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (b[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int block_of(int u, int v, int s, float su, float sv, const Cut& c)
{
    return range_of(u, c.rb, s, su) * s + range_of(v, c.cb, s, sv);
}

// Per-index sample counts (users and items) for the balanced cut and the
// hot-row/column measures; indices out of range are skipped and flagged.
// A workgroup counts a tile of kDegTile samples into open-addressed LDS
// tables (kDegSlots slots each, so at most half full: every probe sequence
// ends), then adds each distinct index's count to global memory once.  Under
// Zipf-like popularity one index can hold several percent of all samples;
// per-sample global atomics on its counter would serialise.
constexpr int kDegTile = 2048;
constexpr int kDegSlots = 4096;
static_assert(kDegSlots >= 2 * kDegTile, "degree tables must stay at most half full");

__device__ __forceinline__ void deg_insert(int* keys, unsigned* cnt, int key)
{
    unsigned h = ((unsigned)key * 2654435761u) >> 20; // 12 bits: kDegSlots = 4096
    for (;;) {
        const int old = atomicCAS(&keys[h], -1, key);
        if (old == -1 || old == key) {
            atomicAdd(&cnt[h], 1u);
            return;
        }
        h = (h + 1) & (kDegSlots - 1);
    }
}

// One position of each of `picks` equal cells of the array, at a place of its
// own inside the cell (hashed, so no regular order of the array can hide an
// index from the picks); every position when picks == nnz.
__device__ __forceinline__ int64_t pick_position(int64_t i, int64_t picks, int64_t nnz)
{
    if (picks == nnz)
        return i;
    const int64_t lo = i * nnz / picks, hi = (i + 1) * nnz / picks; // picks <= 2^20 here: no overflow
    return lo + (int64_t)(((sm64_at(0, (uint64_t)i) >> 32) * (uint64_t)(hi - lo)) >> 32);
}

// MARKED: only the indices whose bit is set in the marks (one bit per hash
// value: a marked index's samples are all counted, an unmarked one's never or
// all, by chance of its hash).  Indices out of range are flagged either way.
constexpr int kMarkBits = 17; // 16 KB of LDS per side
constexpr int kMarkWords = 1 << (kMarkBits - 5);

__device__ __forceinline__ unsigned mark_hash(int i) { return ((unsigned)i * 2246822519u) >> (32 - kMarkBits); }

template <bool MARKED>
__global__ __launch_bounds__(MARKED ? 512 : 256) void k_degrees(const Sample* __restrict__ S, int64_t nnz,
                                                               int64_t picks, int64_t m, int64_t n,
                                                               const uint32_t* __restrict__ marks,
                                                               unsigned long long* __restrict__ du,
                                                               unsigned long long* __restrict__ dv, int* bad)
{
    __shared__ int ku[kDegSlots], kv[kDegSlots];
    __shared__ unsigned cu[kDegSlots], cv[kDegSlots];
    __shared__ uint32_t mu[MARKED ? kMarkWords : 1], mv[MARKED ? kMarkWords : 1];
    __shared__ int dirty; // whether the tile put anything into the tables
    for (int j = threadIdx.x; j < kDegSlots; j += blockDim.x) {
        ku[j] = kv[j] = -1;
        cu[j] = cv[j] = 0u;
    }
    if constexpr (MARKED)
        for (int j = threadIdx.x; j < kMarkWords; j += blockDim.x) {
            mu[j] = marks[j];
            mv[j] = marks[kMarkWords + j];
        }
    if (threadIdx.x == 0)
        dirty = 0;
    __syncthreads();
    auto marked = [](const uint32_t* w, int i) {
        const unsigned h = mark_hash(i);
        return ((w[h >> 5] >> (h & 31)) & 1u) != 0;
    };
    int found = 0;
    const int64_t tiles = (picks + kDegTile - 1) / kDegTile;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t lo = t * kDegTile;
        const int64_t hi = lo + kDegTile < picks ? lo + kDegTile : picks;
        for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) {
            const Sample* x = S + pick_position(i, picks, nnz);
            const int u = __builtin_nontemporal_load(&x->u);
            const int v = __builtin_nontemporal_load(&x->v);
            if (u < 0 || u >= m || v < 0 || v >= n) {
                found = 1;
                continue;
            }
            if (!MARKED || marked(mu, u)) {
                deg_insert(ku, cu, u);
                dirty = 1;
            }
            if (!MARKED || marked(mv, v)) {
                deg_insert(kv, cv, v);
                dirty = 1;
            }
        }
        __syncthreads();
        if (dirty)
            for (int j = threadIdx.x; j < kDegSlots; j += blockDim.x) {
                if (ku[j] >= 0) {
                    atomicAdd(du + ku[j], (unsigned long long)cu[j]);
                    ku[j] = -1;
                    cu[j] = 0u;
                }
                if (kv[j] >= 0) {
                    atomicAdd(dv + kv[j], (unsigned long long)cv[j]);
                    kv[j] = -1;
                    cv[j] = 0u;
                }
            }
        __syncthreads();
        if (threadIdx.x == 0)
            dirty = 0;
        __syncthreads();
    }
    if (found)
        atomicOr(bad, 1);
}

// Marks every index counted at least `least` times and clears the counts.
__global__ void k_mark(unsigned long long* __restrict__ deg, int64_t rows, unsigned long long least,
                       uint32_t* __restrict__ marks)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < rows; i += (int64_t)gridDim.x * blockDim.x) {
        const unsigned long long d = deg[i];
        if (d >= least) {
            const unsigned h = mark_hash((int)i);
            atomicOr(marks + (h >> 5), 1u << (h & 31));
        }
        if (d)
            deg[i] = 0;
    }
}

// Samples of every row block and column block, and the most any one index of
// it holds: workgroup j < s takes row block j (users bnd[j] .. bnd[j+1]-1),
// workgroup s + j column block j; out[2 j] = samples, out[2 j + 1] = largest.
__global__ __launch_bounds__(1024) void k_block_tops(const unsigned long long* __restrict__ du,
                                                     const unsigned long long* __restrict__ dv,
                                                     const int64_t* __restrict__ rbnd, const int64_t* __restrict__ cbnd,
                                                     int s, unsigned long long* __restrict__ out)
{
    const bool col = (int)blockIdx.x >= s;
    const int j = col ? (int)blockIdx.x - s : (int)blockIdx.x;
    const unsigned long long* d = col ? dv : du;
    const int64_t* bnd = col ? cbnd : rbnd;
    unsigned long long sum = 0, top = 0;
    for (int64_t i = bnd[j] + threadIdx.x; i < bnd[j + 1]; i += blockDim.x) {
        const unsigned long long x = d[i];
        sum += x;
        top = x > top ? x : top;
    }
    for (int o = 32; o > 0; o >>= 1) {
        sum += __shfl_xor(sum, o);
        const unsigned long long y = __shfl_xor(top, o);
        top = y > top ? y : top;
    }
    __shared__ unsigned long long ws[16], wt[16];
    if ((threadIdx.x & 63) == 0) {
        ws[threadIdx.x >> 6] = sum;
        wt[threadIdx.x >> 6] = top;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) {
            sum += ws[w];
            top = wt[w] > top ? wt[w] : top;
        }
        out[2 * blockIdx.x] = sum;
        out[2 * blockIdx.x + 1] = top;
    }
}

hipError_t block_tops(const unsigned long long* du, const unsigned long long* dv, const int64_t* rbnd,
                      const int64_t* cbnd, int s, unsigned long long* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_block_tops, dim3(2 * s), dim3(1024), 0, st, du, dv, rbnd, cbnd, s, out);
    return hipGetLastError();
}

// One thread per 32 rows: no atomics, every word written once.
__global__ void k_hot_bits(const unsigned long long* __restrict__ deg, int64_t rows, unsigned long long thr,
                           uint32_t* __restrict__ bits)
{
    const int64_t words = (rows + 31) / 32;
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < words; w += (int64_t)gridDim.x * blockDim.x) {
        uint32_t b = 0;
        for (int i = 0; i < 32; ++i) {
            const int64_t r = w * 32 + i;
            if (r < rows && deg[r] >= thr)
                b |= 1u << i;
        }
        bits[w] = b;
    }
}

hipError_t hot_bits(const unsigned long long* deg, int64_t rows, unsigned long long thr, uint32_t* bits,
                    hipStream_t st)
{
    const int64_t words = (rows + 31) / 32;
    if (words == 0)
        return hipSuccess;
    int64_t blocks = (words + 255) / 256;
    if (blocks > 4096)
        blocks = 4096;
    hipLaunchKernelGGL(k_hot_bits, dim3((unsigned)blocks), dim3(256), 0, st, deg, rows, thr, bits);
    return hipGetLastError();
}

// Largest entry of deg[0 .. rows-1], atomically folded into *out (which the
// caller zeroes).
__global__ void k_max_u64(const unsigned long long* __restrict__ deg, int64_t rows, unsigned long long* out)
{
    unsigned long long mx = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < rows; i += (int64_t)gridDim.x * blockDim.x)
        mx = deg[i] > mx ? deg[i] : mx;
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long y = __shfl_xor(mx, o);
        mx = y > mx ? y : mx;
    }
    if ((threadIdx.x & 63) == 0 && mx > 0)
        atomicMax(out, mx);
}

hipError_t max_degree(const unsigned long long* deg, int64_t rows, unsigned long long* out, hipStream_t st)
{
    if (rows <= 0)
        return hipSuccess;
    int64_t blocks = (rows + 255) / 256;
    if (blocks > 1024)
        blocks = 1024;
    hipLaunchKernelGGL(k_max_u64, dim3((unsigned)blocks), dim3(256), 0, st, deg, rows, out);
    return hipGetLastError();
}

hipError_t plan_degrees(const Sample* S, int64_t nnz, int64_t picks, int64_t m, int64_t n, unsigned long long* du,
                        unsigned long long* dv, int* bad, hipStream_t st)
{
    if (nnz <= 0)
        return hipSuccess;
    if (picks > nnz)
        picks = nnz;
    int64_t blocks = (picks + kDegTile - 1) / kDegTile;
    if (blocks > 2048)
        blocks = 2048;
    hipLaunchKernelGGL(k_degrees<false>, dim3((unsigned)blocks), dim3(256), 0, st, S, nnz, picks, m, n,
                       (const uint32_t*)nullptr, du, dv, bad);
    return hipGetLastError();
}

hipError_t top_degrees(const Sample* S, int64_t nnz, int64_t picks, int64_t least, int64_t m, int64_t n,
                       unsigned long long* du, unsigned long long* dv, uint32_t* marks, int* bad, hipStream_t st)
{
    static_assert(2 * kMarkWords == kTopMarkWords, "marks of users, then of items");
    hipError_t e = plan_degrees(S, nnz, picks, m, n, du, dv, bad, st);
    if (e != hipSuccess || picks >= nnz)
        return e;
    const int64_t blocks = std::min<int64_t>((nnz + kDegTile - 1) / kDegTile, 2048);
    hipLaunchKernelGGL(k_mark, dim3((unsigned)std::min<int64_t>((m + 255) / 256, 2048)), dim3(256), 0, st, du, m,
                       (unsigned long long)least, marks);
    hipLaunchKernelGGL(k_mark, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 2048)), dim3(256), 0, st, dv, n,
                       (unsigned long long)least, marks + kMarkWords);
    hipLaunchKernelGGL(k_degrees<true>, dim3((unsigned)blocks), dim3(512), 0, st, S, nnz, nnz, m, n,
                       (const uint32_t*)marks, du, dv, bad);
    return hipGetLastError();
}

// Sixteen wavefronts share a chunk's histogram (up to 16 KB of LDS), two
// workgroups fill a CU; bound by reading the samples (384 M: 3.84 ms with one
// wavefront per workgroup and 64-bit divisions, 0.78 ms so, 5.9 TB/s; 3.07 G:
// 6.2 ms).
__global__ __launch_bounds__(1024) void k_plan_count(const Sample* __restrict__ S, int64_t nnz, int m, int n, int s,
                                                    float su, float sv, const int64_t* __restrict__ rbnd,
                                                    const int64_t* __restrict__ cbnd, int64_t* __restrict__ counts,
                                                    int chunks, int* bad)
{
    __shared__ Cut cut;
    extern __shared__ int hist[]; // s*s
    const int nb = s * s;
    for (int i = threadIdx.x; i < nb; i += blockDim.x)
        hist[i] = 0;
    load_cut(cut, rbnd, cbnd, s);
    __syncthreads();
    const int64_t cs = (nnz + chunks - 1) / chunks;
    const int64_t lo = (int64_t)blockIdx.x * cs;
    const int64_t hi = lo + cs < nnz ? lo + cs : nnz;
    int found = 0;
    for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += 4 * (int64_t)blockDim.x) {
        int u[4], v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t i = i0 + r * (int64_t)blockDim.x;
            u[r] = v[r] = 0;
            if (i < hi) {
                u[r] = __builtin_nontemporal_load(&S[i].u);
                v[r] = __builtin_nontemporal_load(&S[i].v);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (i0 + r * (int64_t)blockDim.x >= hi)
                break;
            if ((unsigned)u[r] >= (unsigned)m || (unsigned)v[r] >= (unsigned)n) {
                found = 1;
                continue;
            }
            atomicAdd(&hist[block_of(u[r], v[r], s, su, sv, cut)], 1);
        }
    }
    if (found)
        atomicOr(bad, 1);
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
        counts[(int64_t)b * chunks + blockIdx.x] = hist[b];
}

// exclusive scan of counts[b][0..chunks) in place, total to totals[b]
// (chunks is a multiple of 256; thread j scans chunks j*per .. j*per+per-1)
__global__ __launch_bounds__(256) void k_plan_scan_chunks(int64_t* __restrict__ counts, int chunks,
                                                          int64_t* __restrict__ totals)
{
    const int per = chunks / 256;
    __shared__ int64_t part[256];
    int64_t* row = counts + (int64_t)blockIdx.x * chunks + (int64_t)threadIdx.x * per;
    int64_t acc = 0;
    for (int i = 0; i < per; ++i)
        acc += row[i];
    part[threadIdx.x] = acc;
    __syncthreads();
    // inclusive Hillis-Steele scan of the 256 thread sums
    for (int off = 1; off < 256; off <<= 1) {
        int64_t add = (int)threadIdx.x >= off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    int64_t run = threadIdx.x > 0 ? part[threadIdx.x - 1] : 0;
    for (int i = 0; i < per; ++i) {
        const int64_t x = row[i];
        row[i] = run;
        run += x;
    }
    if (threadIdx.x == 255)
        totals[blockIdx.x] = part[255];
}

// exclusive scan of the block totals: bstart[0..nb]
__global__ __launch_bounds__(1024) void k_plan_scan_blocks(const int64_t* __restrict__ totals, int nb,
                                                           int64_t* __restrict__ bstart)
{
    constexpr int per = (kMaxGrid * kMaxGrid) / 1024;
    __shared__ int64_t part[1024];
    int64_t local[per];
    int64_t acc = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        const int b = threadIdx.x * per + i;
        local[i] = b < nb ? totals[b] : 0;
        acc += local[i];
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        int64_t add = (int)threadIdx.x >= off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    int64_t run = threadIdx.x > 0 ? part[threadIdx.x - 1] : 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        const int b = threadIdx.x * per + i;
        if (b < nb)
            bstart[b] = run;
        run += local[i];
    }
    if (threadIdx.x == 1023)
        bstart[nb] = part[1023];
}

// Orders the LDS accesses of a wavefront's lanes with each other.  The hardware
// completes them in order, so this costs no instruction: it keeps the compiler
// from moving one lane's read past another lane's write.
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// One workgroup of NW wavefronts per chunk, in tiles of NW * kPlanRounds * 64
// samples, wavefront w taking the w-th part of the tile.
//   * Within 64 samples the ones of one block find each other with one ballot
//     per bit of the block id (BITS bits): a lane keeps the lanes that agree
//     with it on every bit; its rank is the number of those below it plus the
//     wavefront's count of the block so far, which the first of them moves on.
//     A fixed number of instructions, where taking a step's distinct blocks
//     one after the other needs up to 64 rounds.
//   * Per tile the wavefronts' counts are turned into prefix sums, block by
//     block, which puts the wavefronts' parts in array order.
// What bounds it is the scattered 12-byte write: at s = 64 a chunk has 4096
// lines open, an XCD's 32 chunks more than its L2 holds, and a line leaves the
// L2 in pieces, 36 B per sample where 12 would do (WRITE_SIZE; 3.07 G samples:
// 52.4 ms, 2.8 TB/s past the L2s with the 12 B read).  The fewer chunks are in
// flight, the longer a line stays, so it is one chunk per CU at a time.  384 M
// samples at s = 64: 51.8 ms taking the distinct blocks one by one, 14.1 ms with
// the ballots and a chunk per wavefront (2560 in flight), 6.2 ms so; 99 M
// samples at s = 32: 11.9 ms to 1.1 ms.
// OFF: the positions' type, 32 bits where nnz fits them.
constexpr int kPlanRounds = 8;

template <int BITS, typename OFF, int NW>
__global__ __launch_bounds__(64 * NW) void k_plan_scatter(const Sample* __restrict__ S, int64_t nnz, int m, int n,
                                                          int s, float su, float sv,
                                                          const int64_t* __restrict__ rbnd,
                                                          const int64_t* __restrict__ cbnd,
                                                          const int64_t* __restrict__ counts, int chunks,
                                                          const int64_t* __restrict__ bstart,
                                                          Sample* __restrict__ Sp, int64_t* __restrict__ orig)
{
    constexpr int kBins = 1 << BITS;
    constexpr int kThreads = 64 * NW;
    constexpr int kPer = (kBins + kThreads - 1) / kThreads; // bins per thread
    __shared__ OFF base[kBins];
    __shared__ __align__(16) uint16_t cnt[NW][kBins]; // at most 64 * kPlanRounds per wavefront and tile
    __shared__ Cut cut;
    const int nb = s * s;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int b = threadIdx.x; b < nb; b += kThreads)
        base[b] = (OFF)(bstart[b] + counts[(int64_t)b * chunks + blockIdx.x]);
    load_cut(cut, rbnd, cbnd, s);
    const int64_t cs = (nnz + chunks - 1) / chunks;
    const int64_t lo = (int64_t)blockIdx.x * cs;
    const int64_t hi = lo + cs < nnz ? lo + cs : nnz;
    for (int64_t t0 = lo; t0 < hi; t0 += (int64_t)kThreads * kPlanRounds) {
        Sample x[kPlanRounds];
        int at[kPlanRounds], bin[kPlanRounds];
        const int64_t i0 = t0 + (int64_t)w * (64 * kPlanRounds) + lane;
#pragma unroll
        for (int r = 0; r < kPlanRounds; ++r) {
            x[r] = Sample{-1, -1, 0.f};
            if (i0 + 64 * r < hi) {
                x[r].u = __builtin_nontemporal_load(&S[i0 + 64 * r].u);
                x[r].v = __builtin_nontemporal_load(&S[i0 + 64 * r].v);
                x[r].r = __builtin_nontemporal_load(&S[i0 + 64 * r].r);
            }
        }
        for (int j = threadIdx.x; j < NW * kBins / 8; j += kThreads)
            reinterpret_cast<uint4*>(&cnt[0][0])[j] = uint4{0u, 0u, 0u, 0u};
        __syncthreads(); // counts cleared; base and cut in place
#pragma unroll
        for (int r = 0; r < kPlanRounds; ++r) {
            // the host never scatters a plan with bad indices; a lane past the
            // chunk's end holds -1
            const bool valid = (unsigned)x[r].u < (unsigned)m && (unsigned)x[r].v < (unsigned)n;
            const int b = valid ? block_of(x[r].u, x[r].v, s, su, sv, cut) : 0;
            const uint64_t same = __ballot(valid);
            uint32_t lo32 = (uint32_t)same, hi32 = (uint32_t)(same >> 32);
#pragma unroll
            for (int k = 0; k < BITS; ++k) {
                const bool one = ((b >> k) & 1) != 0;
                const uint64_t ones = __ballot(one);
                const uint32_t flip = one ? 0u : ~0u;
                lo32 &= (uint32_t)ones ^ flip;
                hi32 &= (uint32_t)(ones >> 32) ^ flip;
            }
            const int rank = (int)__builtin_amdgcn_mbcnt_hi(hi32, __builtin_amdgcn_mbcnt_lo(lo32, 0u));
            bin[r] = valid ? b : -1;
            const int have = cnt[w][b];
            at[r] = have + rank;
            wave_order(); // every lane has read the count ...
            if (valid && rank == 0)
                cnt[w][b] = (uint16_t)(have + __popc(lo32) + __popc(hi32));
            wave_order(); // ... before the block's first lane moves it on, for the next 64 to read
        }
        __syncthreads();
        uint32_t total[kPer];
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            const int b = threadIdx.x + p * kThreads;
            uint32_t run = 0;
            if (b < kBins) {
#pragma unroll
                for (int v = 0; v < NW; ++v) {
                    const uint32_t c = cnt[v][b];
                    cnt[v][b] = (uint16_t)run;
                    run += c;
                }
            }
            total[p] = run;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kPlanRounds; ++r)
            if (bin[r] >= 0) {
                const int64_t dest = (int64_t)base[bin[r]] + cnt[w][bin[r]] + at[r];
                Sp[dest] = x[r];
                if (orig)
                    orig[dest] = i0 + 64 * r;
            }
        __syncthreads(); // every position read before the blocks' bases move on
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            const int b = threadIdx.x + p * kThreads;
            if (b < kBins)
                base[b] += (OFF)total[p];
        }
    }
}

static float cut_scale(int64_t N, int s, bool equal) { return equal ? (float)s / (float)N : 0.f; }

hipError_t plan_build(const Sample* S, int64_t nnz, int64_t m, int64_t n, int s, const PlanBuffers& b,
                      hipStream_t st)
{
    const int nb = s * s;
    if (b.chunks < 256 || b.chunks % 256 != 0)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_plan_count, dim3(b.chunks), dim3(1024), sizeof(int) * (size_t)nb, st, S, nnz, (int)m, (int)n,
                       s, cut_scale(m, s, b.equal), cut_scale(n, s, b.equal), b.rbnd, b.cbnd, b.counts, b.chunks,
                       b.bad);
    hipLaunchKernelGGL(k_plan_scan_chunks, dim3(nb), dim3(256), 0, st, b.counts, b.chunks, b.totals);
    hipLaunchKernelGGL(k_plan_scan_blocks, dim3(1), dim3(1024), 0, st, b.totals, nb, b.bstart);
    return hipGetLastError();
}

template <int BITS>
static void launch_scatter(const Sample* S, int64_t nnz, int64_t m, int64_t n, int s, const PlanBuffers& b,
                           hipStream_t st)
{
    const float su = cut_scale(m, s, b.equal), sv = cut_scale(n, s, b.equal);
    if (nnz <= 0xffffffffll)
        hipLaunchKernelGGL((k_plan_scatter<BITS, uint32_t, 16>), dim3(b.chunks), dim3(1024), 0, st, S, nnz, (int)m, (int)n,
                           s, su, sv, b.rbnd, b.cbnd, b.counts, b.chunks, b.bstart, b.Sp, b.orig);
    else
        hipLaunchKernelGGL((k_plan_scatter<BITS, uint64_t, 8>), dim3(b.chunks), dim3(512), 0, st, S, nnz, (int)m, (int)n,
                           s, su, sv, b.rbnd, b.cbnd, b.counts, b.chunks, b.bstart, b.Sp, b.orig);
}

hipError_t plan_scatter(const Sample* S, int64_t nnz, int64_t m, int64_t n, int s, const PlanBuffers& b,
                        hipStream_t st)
{
    if (s <= 4)
        launch_scatter<4>(S, nnz, m, n, s, b, st);
    else if (s <= 8)
        launch_scatter<6>(S, nnz, m, n, s, b, st);
    else if (s <= 16)
        launch_scatter<8>(S, nnz, m, n, s, b, st);
    else if (s <= 32)
        launch_scatter<10>(S, nnz, m, n, s, b, st);
    else
        launch_scatter<12>(S, nnz, m, n, s, b, st);
    return hipGetLastError();
}

} // namespace mfsgd
