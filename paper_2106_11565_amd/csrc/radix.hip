// Device-wide exclusive scan and a batched stable LSD radix sort of (key,
// index) pairs, used by the index build and by inserts: points by bucket code
// for all tables at once, points by group for all repetitions at once.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "flinng_internal.h"

namespace flinng {

namespace {

// Exclusive scan of a workgroup's per-thread totals; returns this thread's
// exclusive prefix, and the workgroup total in *total.
template <class T>
__device__ inline T block_exclusive_scan(T v, T *lds, T *total) {
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    T inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    T wpre = 0, tot = 0;
    for (int w = 0; w < (int)(blockDim.x / 64); ++w) {
        const T c = lds[w];
        if (w < wave) wpre += c;
        tot += c;
    }
    __syncthreads();
    *total = tot;
    return wpre + inc - v;
}

// ---------------------------------------------------------------------------
// Scan in three launches: tile sums, one workgroup over the tile sums (64-bit:
// the total may pass 2^32 and is checked by the caller), then the prefixes.
constexpr int SC_T = 256, SC_I = 16, SC_TILE = SC_T * SC_I;

__global__ __launch_bounds__(SC_T) void scan_sums_kernel(const uint32_t *__restrict__ in, uint64_t n,
                                                         uint64_t *__restrict__ sums) {
    __shared__ uint64_t lds[SC_T / 64];
    const uint64_t b = (uint64_t)blockIdx.x * SC_TILE;
    uint64_t s = 0;
#pragma unroll
    for (int i = 0; i < SC_I; ++i) {
        const uint64_t p = b + (uint64_t)i * SC_T + threadIdx.x;
        if (p < n) s += in[p];
    }
    uint64_t tot;
    block_exclusive_scan<uint64_t>(s, lds, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// sums -> exclusive prefixes plus base, in place; *total = base + their sum.
constexpr int SB_T = 1024, SB_I = 8;
__global__ __launch_bounds__(SB_T) void scan_bases_kernel(uint64_t *__restrict__ sums, uint64_t nt,
                                                          uint64_t base,
                                                          uint64_t *__restrict__ total) {
    __shared__ uint64_t lds[SB_T / 64];
    uint64_t carry = base;
    for (uint64_t b = 0; b < nt; b += (uint64_t)SB_T * SB_I) {
        const uint64_t p = b + (uint64_t)threadIdx.x * SB_I;
        uint64_t v[SB_I], s = 0;
#pragma unroll
        for (int i = 0; i < SB_I; ++i) {
            v[i] = p + i < nt ? sums[p + i] : 0ull;
            s += v[i];
        }
        uint64_t tot;
        uint64_t pre = carry + block_exclusive_scan<uint64_t>(s, lds, &tot);
#pragma unroll
        for (int i = 0; i < SB_I; ++i) {
            if (p + i < nt) sums[p + i] = pre;
            pre += v[i];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) *total = carry;
}

// data -> exclusive prefix (base included), in place.
__global__ __launch_bounds__(SC_T) void scan_apply_kernel(uint32_t *__restrict__ data, uint64_t n,
                                                          const uint64_t *__restrict__ sums) {
    __shared__ uint32_t st[SC_TILE + SC_TILE / 32];  // one pad word per 32
    __shared__ uint32_t lds[SC_T / 64];
    const uint64_t b = (uint64_t)blockIdx.x * SC_TILE;
    auto at = [](uint32_t j) { return j + (j >> 5); };
#pragma unroll
    for (int i = 0; i < SC_I; ++i) {
        const uint32_t j = (uint32_t)i * SC_T + threadIdx.x;
        st[at(j)] = b + j < n ? data[b + j] : 0u;
    }
    __syncthreads();
    uint32_t v[SC_I], s = 0;
#pragma unroll
    for (int i = 0; i < SC_I; ++i) {
        v[i] = st[at(threadIdx.x * SC_I + i)];
        s += v[i];
    }
    uint32_t tot;
    uint32_t pre = (uint32_t)sums[blockIdx.x] + block_exclusive_scan<uint32_t>(s, lds, &tot);
#pragma unroll
    for (int i = 0; i < SC_I; ++i) {
        st[at(threadIdx.x * SC_I + i)] = pre;
        pre += v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SC_I; ++i) {
        const uint32_t j = (uint32_t)i * SC_T + threadIdx.x;
        if (b + j < n) data[b + j] = st[at(j)];
    }
}

}  // namespace

size_t scan_scratch_bytes(uint64_t n) { return (n + SC_TILE - 1) / SC_TILE * 8 + 8; }

void device_exclusive_scan_u32(uint32_t *data, uint64_t n, uint64_t base, uint64_t *total,
                               void *scratch, hipStream_t s) {
    uint64_t *sums = static_cast<uint64_t *>(scratch);
    const uint64_t nt = (n + SC_TILE - 1) / SC_TILE;
    if (nt) {
        hipLaunchKernelGGL(scan_sums_kernel, dim3((unsigned)nt), dim3(SC_T), 0, s, data, n, sums);
        FL_CHECK_LAUNCH();
    }
    hipLaunchKernelGGL(scan_bases_kernel, dim3(1), dim3(SB_T), 0, s, sums, nt, base, total);
    FL_CHECK_LAUNCH();
    if (nt) {
        hipLaunchKernelGGL(scan_apply_kernel, dim3((unsigned)nt), dim3(SC_T), 0, s, data, n, sums);
        FL_CHECK_LAUNCH();
    }
}

// ---------------------------------------------------------------------------
// Batched pair sort: `count` independent sorts of n keys each (blockIdx.y),
// the keys of sort t at keys[t*n ..], each below 2^bits.  The result pairs
// are key << 32 | index, ascending by key and, within a key, by index.  LSD
// digits of at most 8 bits, evenly split over the passes; the first pass
// reads the 4-byte keys and makes the pairs.  Per pass: tile histograms, an
// exclusive scan of each digit's row over the tiles, and the scatter (which
// adds the digits' starts from their totals): three launches for the whole
// batch.  Memory bound: 8 bytes in and out per pair and pass, plus the
// histogram's read.  10M pairs (two URL tables) scatter in 41 us, 3.9 TB/s of
// read plus write, and are counted in 20 us.
constexpr int PS_T = 256, PS_I = 16, PS_TILE = PS_T * PS_I, PS_W = PS_T / 64;

namespace {

template <bool FIRST>
__device__ inline uint32_t ps_key(const uint32_t *k32, const uint64_t *k64, uint64_t p) {
    return FIRST ? k32[p] : (uint32_t)(k64[p] >> 32);
}

// hist[(t*256 + digit)*nb + tile]
template <bool FIRST>
__global__ __launch_bounds__(PS_T) void ps_hist_kernel(const uint32_t *__restrict__ k32,
                                                       const uint64_t *__restrict__ k64, uint64_t n,
                                                       int shift, uint32_t mask, uint64_t nb,
                                                       uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * PS_TILE, o = (uint64_t)blockIdx.y * n;
#pragma unroll
    for (int i = 0; i < PS_I; ++i) {
        const uint64_t p = base + (uint64_t)i * PS_T + threadIdx.x;
        if (p < n) atomicAdd(&h[(ps_key<FIRST>(k32, k64, o + p) >> shift) & mask], 1u);
    }
    __syncthreads();
    if (threadIdx.x <= mask)
        hist[((uint64_t)blockIdx.y * 256 + threadIdx.x) * nb + blockIdx.x] = h[threadIdx.x];
}

// Exclusive scan of one digit's row over the tiles, in place; its total.
__global__ __launch_bounds__(PS_T) void ps_rows_kernel(uint32_t *__restrict__ hist, uint64_t nb,
                                                       uint32_t *__restrict__ tot) {
    __shared__ uint32_t lds[PS_T / 64];
    const uint64_t r = (uint64_t)blockIdx.y * 256 + blockIdx.x;
    uint32_t *row = hist + r * nb;
    uint32_t carry = 0;
    for (uint64_t b = 0; b < nb; b += PS_T) {
        const uint64_t p = b + threadIdx.x;
        const uint32_t v = p < nb ? row[p] : 0u;
        uint32_t t;
        const uint32_t pre = block_exclusive_scan<uint32_t>(v, lds, &t);
        if (p < nb) row[p] = carry + pre;
        carry += t;
    }
    if (threadIdx.x == 0) tot[r] = carry;
}

// Stable scatter.  Wavefront w of the tile takes its keys base + 1024 w + 64 i
// + lane in order of i: a key's rank among the wavefront's equal digits is
// the count of earlier rounds (a counter row of its own in LDS, so no barrier
// between rounds) plus its place in the round's digit-match mask (a ballot
// per digit bit).  The wavefronts' counts then give each digit's start in the
// tile, the tile is ordered by digit in LDS, and consecutive threads store
// consecutive addresses of a digit's run.
template <bool FIRST>
__global__ __launch_bounds__(PS_T) void ps_scatter_kernel(
    const uint32_t *__restrict__ k32, const uint64_t *__restrict__ k64, uint64_t n, int shift,
    int dbits, uint64_t nb, const uint32_t *__restrict__ hist, const uint32_t *__restrict__ tot,
    uint64_t *__restrict__ out) {
    __shared__ uint32_t wc[PS_W][256];
    __shared__ uint32_t gdel[256];  // global start minus local start, per digit
    __shared__ uint32_t sl[PS_W];
    __shared__ uint64_t tk[PS_TILE];
    const int t = threadIdx.x, lane = t % 64, wave = t / 64;
    const uint32_t mask = (1u << dbits) - 1u;
#pragma unroll
    for (int w = 0; w < PS_W; ++w) wc[w][t] = 0;
    const uint64_t base = (uint64_t)blockIdx.x * PS_TILE, o = (uint64_t)blockIdx.y * n;
    const uint64_t wb = base + (uint64_t)wave * (64 * PS_I);
    uint64_t key[PS_I];
    uint32_t rank[PS_I];
#pragma unroll
    for (int i = 0; i < PS_I; ++i) {
        const uint64_t p = wb + 64 * i + lane;
        key[i] = ~0ull;
        if (p < n) key[i] = FIRST ? ((uint64_t)k32[o + p] << 32) | (uint32_t)p : k64[o + p];
    }
    __syncthreads();
    const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < PS_I; ++i) {
        const bool valid = wb + 64 * i + lane < n;
        const uint32_t dgt = (uint32_t)(key[i] >> (32 + shift)) & mask;
        unsigned long long peers = __ballot(valid);
        for (int b = 0; b < dbits; ++b) {
            const bool bit = (dgt >> b) & 1u;
            const unsigned long long m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t before = (uint32_t)__popcll(peers & lt);
        uint32_t c = 0;
        if (valid) c = wc[wave][dgt];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) wc[wave][dgt] = c + (uint32_t)__popcll(peers);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        rank[i] = c + before;
    }
    __syncthreads();
    {
        // digit t: its keys in the tile, their start there and in the output
        uint32_t cnt = 0, w0[PS_W], total;
#pragma unroll
        for (int w = 0; w < PS_W; ++w) {
            w0[w] = cnt;
            cnt += wc[w][t];
        }
        const uint32_t ls = block_exclusive_scan<uint32_t>(cnt, sl, &total);
        const uint64_t r = (uint64_t)blockIdx.y * 256 + t;
        const bool used = (uint32_t)t <= mask;
        const uint32_t gs = block_exclusive_scan<uint32_t>(used ? tot[r] : 0u, sl, &total);
        gdel[t] = used ? gs + hist[r * nb + blockIdx.x] - ls : 0u;
#pragma unroll
        for (int w = 0; w < PS_W; ++w) wc[w][t] = ls + w0[w];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PS_I; ++i) {
        if (wb + 64 * i + lane < n)
            tk[wc[wave][(uint32_t)(key[i] >> (32 + shift)) & mask] + rank[i]] = key[i];
    }
    __syncthreads();
    const uint32_t m = n - base < (uint64_t)PS_TILE ? (uint32_t)(n - base) : (uint32_t)PS_TILE;
    uint64_t *dst = out + o;
#pragma unroll 4
    for (uint32_t j = t; j < m; j += PS_T) {
        const uint64_t k = tk[j];
        const uint32_t gp = gdel[(uint32_t)(k >> (32 + shift)) & mask] + j;
        dst[gp] = k;
    }
}

inline int ps_passes(int bits) { return std::max(1, (bits + 7) / 8); }

}  // namespace

size_t pair_sort_scratch_bytes(uint64_t n, uint32_t count) {
    const uint64_t nb = (n + PS_TILE - 1) / PS_TILE;
    return ((size_t)256 * nb + 256) * count * 4;
}

void pair_sort(const uint32_t *keys, uint64_t n, uint32_t count, int bits, uint64_t *out,
               uint64_t *tmp, void *scratch, hipStream_t s) {
    if (n == 0 || count == 0) return;
    const uint64_t nb = (n + PS_TILE - 1) / PS_TILE;
    uint32_t *hist = static_cast<uint32_t *>(scratch);
    uint32_t *tot = hist + (size_t)256 * nb * count;
    const int passes = ps_passes(bits);
    // the last pass writes `out`
    uint64_t *dst = passes % 2 ? out : tmp, *src = passes % 2 ? tmp : out;
    const dim3 grid((unsigned)nb, count);
    int shift = 0;
    for (int p = 0; p < passes; ++p) {
        const int db = std::max(1, (bits - shift + passes - p - 1) / (passes - p));
        const uint32_t mask = (1u << db) - 1u;
        if (p == 0)
            hipLaunchKernelGGL(ps_hist_kernel<true>, grid, dim3(PS_T), 0, s, keys,
                               (const uint64_t *)nullptr, n, shift, mask, nb, hist);
        else
            hipLaunchKernelGGL(ps_hist_kernel<false>, grid, dim3(PS_T), 0, s,
                               (const uint32_t *)nullptr, src, n, shift, mask, nb, hist);
        FL_CHECK_LAUNCH();
        hipLaunchKernelGGL(ps_rows_kernel, dim3(mask + 1, count), dim3(PS_T), 0, s, hist, nb, tot);
        FL_CHECK_LAUNCH();
        if (p == 0)
            hipLaunchKernelGGL(ps_scatter_kernel<true>, grid, dim3(PS_T), 0, s, keys,
                               (const uint64_t *)nullptr, n, shift, db, nb, hist, tot, dst);
        else
            hipLaunchKernelGGL(ps_scatter_kernel<false>, grid, dim3(PS_T), 0, s,
                               (const uint32_t *)nullptr, src, n, shift, db, nb, hist, tot, dst);
        FL_CHECK_LAUNCH();
        std::swap(src, dst);
        shift += db;
    }
}

}  // namespace flinng
