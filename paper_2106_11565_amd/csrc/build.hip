// One-pass index build on gfx950 (Algorithm 1 and the reverse index of
// Section 6, Implementation).
//
// Groups: repetition r permutes the points with a keyed bijection P_r of
// [0, N) and point x joins group P_r(x) mod B (Algorithm 1: a random
// permutation, then blocks by modulo), so group b holds exactly
// floor(N/B) + [b < N mod B] points.  P_r is a 4-round balanced Feistel
// network on [0, 2^nb) (nb the smallest even width >= 2 covering N) with
// round function F_i(v) = splitmix_finalize(v XOR k_{r,i}) mod 2^(nb/2) and
// keys k_{r,i} = sm64(sm64(seed, GROUP), 4r + i), restricted to [0, N) by
// cycle walking (Black and Rogaway 2002).
//
// The reverse index is built in lists.hip.
//
// Points arriving after the build (ids N0, N0+1, ...): the arrivals are cut
// into blocks of B; within block j the point at position u joins group
// pi_{r,j}(u) of repetition r, pi_{r,j} a 4-round balanced Feistel network
// on [0, 2^nb) (nb the smallest even width >= 2 covering B) restricted to
// [0, B) by cycle walking, round keys sm64(sm64(seed, STREAM), 4(16j + r) + i).
// Every complete block adds one point to each group, so group sizes stay
// within two of each other.  An insert merges the new points' cells into the
// lists, and appends the new members (ascending id is preserved: new ids
// exceed every old one) into copies of the member arrays, growing their
// per-cell stride when a cell outgrows it.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "flinng_internal.h"

namespace flinng {

__device__ inline uint64_t feistel(uint64_t v, uint32_t half, const uint64_t *keys) {
    const uint64_t mask = (1ull << half) - 1ull;
    uint64_t hi = v >> half, lo = v & mask;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint64_t f = splitmix_finalize(lo ^ keys[i]) & mask;
        const uint64_t nlo = hi ^ f;
        hi = lo;
        lo = nlo;
    }
    return (hi << half) | lo;
}

struct GroupKeys {
    uint64_t k[16][4];
};

// grp[x*Rp + r] = P_r(x) mod B; the padding repetitions R..Rp-1 repeat
// repetition R-1's group, so a reader may take the minimum over all Rp
// entries (a repeated cell changes neither the minimum nor its cell).
__global__ void groups_kernel(uint64_t N, uint32_t R, uint32_t Rp, uint32_t B, uint32_t half,
                              GroupKeys gk, uint16_t *__restrict__ grp) {
    const uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= N) return;
    for (uint32_t r = 0; r < R; ++r) {
        uint64_t y = feistel(x, half, gk.k[r]);
        while (y >= N) y = feistel(y, half, gk.k[r]);
        grp[x * Rp + r] = (uint16_t)(y % B);
    }
    for (uint32_t r = R; r < Rp; ++r) grp[x * Rp + r] = grp[x * Rp + R - 1];
}

// keys[q*n + i] = group of point x0 + i in repetition r0 + q
__global__ void member_keys_kernel(const uint16_t *__restrict__ grp, uint64_t x0, uint64_t n,
                                   uint32_t Rp, uint32_t r0, uint32_t *__restrict__ keys) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys[(uint64_t)blockIdx.y * n + i] = grp[(x0 + i) * Rp + r0 + blockIdx.y];
}

// sorted position p of group b = pairs[p] >> 32 sits at run offset
// p - (b*floor(N/B) + min(b, N mod B)); its id goes to slot b*mstride + that.
__global__ void member_slots_kernel(const uint64_t *__restrict__ pairs, uint64_t N, uint32_t B,
                                    uint32_t mstride, uint32_t *__restrict__ mem) {
    const uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const uint64_t b = pairs[p] >> 32;
    const uint64_t q0 = N / B, rem = N % B;
    const uint64_t run = b * q0 + (b < rem ? b : rem);
    mem[b * mstride + (p - run)] = (uint32_t)pairs[p];
}

// The inverse of feistel.
__device__ inline uint64_t feistel_inverse(uint64_t v, uint32_t half, const uint64_t *keys) {
    const uint64_t mask = (1ull << half) - 1ull;
    uint64_t hi = v >> half, lo = v & mask;
#pragma unroll
    for (int i = 3; i >= 0; --i) {
        const uint64_t plo = hi;  // the round's input: (lo XOR F(plo), plo)
        hi = lo ^ (splitmix_finalize(plo ^ keys[i]) & mask);
        lo = plo;
    }
    return (hi << half) | lo;
}

// A group row (RP uint16) by vector loads and stores.
template <int RP>
struct GroupRow {
    uint32_t w[(RP + 1) / 2];
    __device__ void load(const uint16_t *p) {
        if constexpr (RP == 1) w[0] = *p;
        else if constexpr (RP == 2) w[0] = *reinterpret_cast<const uint32_t *>(p);
        else if constexpr (RP == 4) *reinterpret_cast<uint2 *>(w) = *reinterpret_cast<const uint2 *>(p);
        else
#pragma unroll
            for (int i = 0; i < RP / 8; ++i)
                reinterpret_cast<uint4 *>(w)[i] = reinterpret_cast<const uint4 *>(p)[i];
    }
    __device__ void store(uint16_t *p) const {
        if constexpr (RP == 1) *p = (uint16_t)w[0];
        else if constexpr (RP == 2) *reinterpret_cast<uint32_t *>(p) = w[0];
        else if constexpr (RP == 4) *reinterpret_cast<uint2 *>(p) = *reinterpret_cast<const uint2 *>(w);
        else
#pragma unroll
            for (int i = 0; i < RP / 8; ++i)
                reinterpret_cast<uint4 *>(p)[i] = reinterpret_cast<const uint4 *>(w)[i];
    }
};

// One cell (r, b) per workgroup: its members are P_r^-1(b + j*B) for j below
// its size, found by running the permutation backwards and sorted in LDS
// (cap: a power of two at least mstride), with their group rows and filter
// words.  A one-wavefront workgroup for cells of up to 512 members: no barrier
// waits, and enough of them to fill the chip.  Replaces a stable sort of all
// ids by group per repetition, and two gather passes: 5M points in 131,072
// cells 6.5 -> 1.8 ms, 1M in 65,536 1.3 -> 0.2 ms.
constexpr uint32_t CELL_CAP = 8192;
template <int RP, int T>
__global__ __launch_bounds__(T) void cells_kernel(uint64_t N, uint32_t R, uint32_t B, uint32_t half,
                                                  GroupKeys gk, uint32_t mstride, uint32_t cap,
                                                  const uint16_t *__restrict__ grp,
                                                  uint32_t *__restrict__ mem, uint16_t *__restrict__ cmg,
                                                  uint32_t *__restrict__ cfl,
                                                  uint32_t *__restrict__ gsize) {
    extern __shared__ uint32_t ids[];
    const uint32_t b = blockIdx.x, r = blockIdx.y, tid = threadIdx.x;
    const uint32_t size = (uint32_t)(N / B + (b < N % B ? 1 : 0));
    for (uint32_t j = tid; j < cap; j += T) {
        uint32_t id = 0xFFFFFFFFu;
        if (j < size) {
            uint64_t x = feistel_inverse(b + (uint64_t)j * B, half, gk.k[r]);
            while (x >= N) x = feistel_inverse(x, half, gk.k[r]);
            id = (uint32_t)x;
        }
        ids[j] = id;
    }
    __syncthreads();
    for (uint32_t run = 2; run <= cap; run <<= 1) {
        for (uint32_t d = run >> 1; d; d >>= 1) {
            for (uint32_t i = tid; i < cap / 2; i += T) {
                const uint32_t lo = 2 * i - (i & (d - 1)), hi = lo + d;
                const uint32_t p = ids[lo], q = ids[hi];
                if ((p > q) == ((lo & run) == 0)) {
                    ids[lo] = q;
                    ids[hi] = p;
                }
            }
            __syncthreads();
        }
    }
    const uint64_t slot0 = ((uint64_t)r * B + b) * mstride;
    const uint32_t r1 = (r + 1) % R, r2 = (r + 2) % R;
    for (uint32_t j = tid; j < mstride; j += T) {
        const uint32_t x = ids[j];
        GroupRow<RP> row{};
        uint32_t f = 0;
        if (x != 0xFFFFFFFFu) {
            const uint16_t *g = grp + (uint64_t)x * RP;
            row.load(g);
            f = (uint32_t)g[r1] | ((uint32_t)g[r2] << 16);
        }
        mem[slot0 + j] = x;
        row.store(cmg + (slot0 + j) * RP);
        cfl[slot0 + j] = f;
    }
    if (tid == 0) gsize[(uint64_t)r * B + b] = size;
}

template <int RP>
static void launch_cells(const Index &ix, uint32_t half, const GroupKeys &gk, uint32_t cap, hipStream_t s) {
    const dim3 grid(ix.p.B, ix.p.R);
    if (cap <= 512)
        hipLaunchKernelGGL((cells_kernel<RP, 64>), grid, dim3(64), cap * 4, s, ix.N, ix.p.R, ix.p.B, half,
                           gk, ix.mstride, cap, ix.grp, ix.mem, ix.cmg, ix.cfl, ix.gsize);
    else
        hipLaunchKernelGGL((cells_kernel<RP, 256>), grid, dim3(256), cap * 4, s, ix.N, ix.p.R, ix.p.B, half,
                           gk, ix.mstride, cap, ix.grp, ix.mem, ix.cmg, ix.cfl, ix.gsize);
    FL_CHECK_LAUNCH();
}

// cmg[slot][r] = group in repetition r of the member stored in mem[slot]
// (zeros for the padding slots).
__global__ void cell_groups_kernel(const uint32_t *__restrict__ mem, const uint16_t *__restrict__ grp,
                                   uint64_t nslots, uint32_t Rp, uint16_t *__restrict__ cmg) {
    const uint64_t sl = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (sl >= nslots) return;
    const uint32_t x = mem[sl];
    for (uint32_t r = 0; r < Rp; ++r)
        cmg[sl * Rp + r] = (x == 0xFFFFFFFFu) ? (uint16_t)0 : grp[(uint64_t)x * Rp + r];
}

// cfl[r][b][j] = the groups, in repetitions r+1 and r+2 (mod R), of the
// member in slot j of cell (r, b): low and high 16 bits (zero for padding
// slots).  One launch per repetition r.
__global__ void filter_groups_kernel(const uint32_t *__restrict__ mem_r,
                                     const uint16_t *__restrict__ grp, uint64_t nslots, uint32_t Rp,
                                     uint32_t r1, uint32_t r2, uint32_t *__restrict__ cfl_r) {
    const uint64_t sl = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (sl >= nslots) return;
    const uint32_t x = mem_r[sl];
    cfl_r[sl] = (x == 0xFFFFFFFFu)
                    ? 0u
                    : (uint32_t)grp[(uint64_t)x * Rp + r1] | ((uint32_t)grp[(uint64_t)x * Rp + r2] << 16);
}

void build_filter(const Index &ix, const uint32_t *mem, const uint16_t *grp, uint32_t mstride,
                  uint32_t *cfl, hipStream_t s) {
    const uint32_t R = ix.p.R, B = ix.p.B;
    const uint64_t per = (uint64_t)B * mstride;
    for (uint32_t r = 0; r < R; ++r) {
        hipLaunchKernelGGL(filter_groups_kernel, dim3((unsigned)((per + 255) / 256)), dim3(256), 0, s,
                           mem + r * per, grp, per, ix.Rp, (r + 1) % R, (r + 2) % R, cfl + r * per);
        FL_CHECK_LAUNCH();
    }
}

void build_groups(Index &ix, hipStream_t s) {
    const uint64_t N = ix.N;
    const uint32_t R = ix.p.R, B = ix.p.B;
    uint32_t nb = 2;
    while (nb < 64 && (1ull << nb) < N) nb += 2;
    GroupKeys gk{};
    const uint64_t key = sm64(ix.p.seed, TAG_GROUP);
    for (uint32_t r = 0; r < R; ++r)
        for (int i = 0; i < 4; ++i) gk.k[r][i] = sm64(key, (uint64_t)r * 4 + i);
    const unsigned grid = (unsigned)((N + 255) / 256);
    hipLaunchKernelGGL(groups_kernel, dim3(grid), dim3(256), 0, s, N, R, ix.Rp, B, nb / 2, gk,
                       ix.grp);
    FL_CHECK_LAUNCH();
    // cell sizes (Algorithm 1's balanced design), the host's copy
    ix.gsize_host.assign((size_t)R * B, 0);
    for (uint32_t r = 0; r < R; ++r)
        for (uint32_t b = 0; b < B; ++b)
            ix.gsize_host[(size_t)r * B + b] = (uint32_t)(N / B + (b < N % B ? 1 : 0));
    ix.gmax = (uint32_t)((N + B - 1) / B);
    // cells whose members fit a workgroup's LDS are made one per workgroup
    uint32_t cap = 2;
    while (cap < ix.mstride) cap <<= 1;
    if (ix.mstride <= CELL_CAP) {
        switch (ix.Rp) {
            case 1: launch_cells<1>(ix, nb / 2, gk, cap, s); break;
            case 2: launch_cells<2>(ix, nb / 2, gk, cap, s); break;
            case 4: launch_cells<4>(ix, nb / 2, gk, cap, s); break;
            case 8: launch_cells<8>(ix, nb / 2, gk, cap, s); break;
            default: launch_cells<16>(ix, nb / 2, gk, cap, s); break;
        }
        return;
    }
    // larger cells: stable sort of ids by group, then each group's run (at
    // b*floor(N/B) + min(b, N mod B)) moves to its 16-byte aligned slot
    // b*mstride; unused slot tails hold 0xFFFFFFFF
    DevBuf keys = DevBuf::pooled(N * 4, s), pairs = DevBuf::pooled(N * 8, s),
           tmp = DevBuf::pooled(N * 8, s), ps = DevBuf::pooled(pair_sort_scratch_bytes(N, 1), s);
    int gbits = 1;
    while ((1u << gbits) < B) ++gbits;
    FL_HIP(hipMemsetAsync(ix.mem, 0xFF, (size_t)R * B * ix.mstride * 4, s));
    for (uint32_t r = 0; r < R; ++r) {
        hipLaunchKernelGGL(member_keys_kernel, dim3(grid), dim3(256), 0, s, ix.grp, (uint64_t)0, N,
                           ix.Rp, r, keys.as<uint32_t>());
        FL_CHECK_LAUNCH();
        pair_sort(keys.as<uint32_t>(), N, 1, gbits, pairs.as<uint64_t>(), tmp.as<uint64_t>(), ps.ptr, s);
        hipLaunchKernelGGL(member_slots_kernel, dim3(grid), dim3(256), 0, s, pairs.as<uint64_t>(), N, B,
                           ix.mstride, ix.mem + (uint64_t)r * B * ix.mstride);
        FL_CHECK_LAUNCH();
    }
    const uint64_t nslots = (uint64_t)R * B * ix.mstride;
    hipLaunchKernelGGL(cell_groups_kernel, dim3((unsigned)((nslots + 255) / 256)), dim3(256), 0, s,
                       ix.mem, ix.grp, nslots, ix.Rp, ix.cmg);
    FL_CHECK_LAUNCH();
    build_filter(ix, ix.mem, ix.grp, ix.mstride, ix.cfl, s);
    FL_HIP(hipMemcpyAsync(ix.gsize, ix.gsize_host.data(), (size_t)R * B * 4, hipMemcpyHostToDevice, s));
    FL_HIP(hipStreamSynchronize(s));  // the host vector is the copy's source
}

void build_lists(Index &ix, const uint32_t *codes, hipStream_t s) {
    Lists l = make_lists(ix, codes, ix.grp, ix.N, s);
    ix.offsets = l.offsets;
    ix.cells = l.cells;
    ix.list_entries = l.entries;
    ix.mean_entries = l.mean_entries;
}

// ---------------------------------------------------------------------------
// inserts

// Groups of the arrivals x0 .. x0+n-1 (the build had N0 points).
__global__ void stream_groups_kernel(uint64_t x0, uint64_t n, uint64_t N0, uint32_t R, uint32_t Rp,
                                     uint32_t B, uint32_t half, uint64_t skey,
                                     uint16_t *__restrict__ grp) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t x = x0 + i, a = x - N0;
    const uint64_t j = a / B, u = a % B;
    for (uint32_t r = 0; r < R; ++r) {
        uint64_t keys[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) keys[k] = sm64(skey, 4 * (16 * j + r) + (uint64_t)k);
        uint64_t y = feistel(u, half, keys);
        while (y >= B) y = feistel(y, half, keys);
        grp[x * Rp + r] = (uint16_t)y;
    }
    for (uint32_t r = R; r < Rp; ++r) grp[x * Rp + r] = grp[x * Rp + R - 1];
}

// Where each group's run starts and ends in the arrivals sorted by group (one
// repetition per blockIdx.y).
__global__ void run_bounds_kernel(const uint64_t *__restrict__ pairs, uint64_t n, uint32_t B,
                                  uint32_t *__restrict__ start, uint32_t *__restrict__ end) {
    const uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint64_t *v = pairs + (uint64_t)blockIdx.y * n;
    const uint64_t b = v[p] >> 32, o = (uint64_t)blockIdx.y * B + b;
    if (p == 0 || v[p - 1] >> 32 != b) start[o] = (uint32_t)p;
    if (p == n - 1 || v[p + 1] >> 32 != b) end[o] = (uint32_t)(p + 1);
}

__global__ void run_counts_kernel(const uint32_t *__restrict__ start, const uint32_t *__restrict__ end,
                                  uint32_t B, uint32_t *__restrict__ cnt) {
    const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) cnt[b] = end[b] - start[b];
}

// Copy each cell's member ids and group rows into arrays of a larger stride.
__global__ void restride_kernel(const uint32_t *__restrict__ mem, const uint16_t *__restrict__ cmg,
                                uint64_t ncells, uint32_t s0, uint32_t s1, uint32_t Rp,
                                uint32_t *__restrict__ mem1, uint16_t *__restrict__ cmg1) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ncells * s0) return;
    const uint64_t c = i / s0, j = i % s0;
    mem1[c * s1 + j] = mem[i];
    for (uint32_t r = 0; r < Rp; ++r) cmg1[(c * s1 + j) * Rp + r] = cmg[i * Rp + r];
}

// The sorted arrivals of a repetition (blockIdx.y) join their cells after the
// members already there: member id x0 + index and its group row.
__global__ void place_members_kernel(const uint64_t *__restrict__ pairs, uint64_t n, uint64_t x0,
                                     const uint32_t *__restrict__ start,
                                     const uint32_t *__restrict__ gsize, uint32_t B, uint32_t mstride,
                                     const uint16_t *__restrict__ grp, uint32_t Rp,
                                     uint32_t *__restrict__ mem, uint16_t *__restrict__ cmg) {
    const uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint64_t v = pairs[(uint64_t)blockIdx.y * n + p];
    const uint64_t c = (uint64_t)blockIdx.y * B + (v >> 32);  // cell (r, b)
    const uint64_t slot = c * mstride + gsize[c] + (p - start[c]);
    const uint64_t x = x0 + (uint32_t)v;
    mem[slot] = (uint32_t)x;
    for (uint32_t r = 0; r < Rp; ++r) cmg[slot * Rp + r] = grp[x * Rp + r];
}

__global__ void add_u32_kernel(const uint32_t *__restrict__ a, const uint32_t *__restrict__ b,
                               uint64_t n, uint32_t *__restrict__ out) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = a[i] + b[i];
}

void insert_points(Index &ix, const uint32_t *codes, uint64_t n, hipStream_t s) {
    if (n == 0) return;
    const uint64_t x0 = ix.N;
    if (x0 + n > 0xFFFFFFFEull) fail(FLINNG_EINVAL, "at most 2^32-2 points");
    const uint32_t R = ix.p.R, B = ix.p.B, Rp = ix.Rp;
    const uint64_t ncells = (uint64_t)R * B;
    // arrays of the new version (freed on failure)
    uint16_t *grp1 = nullptr;
    char *slab = nullptr;
    Lists lists;
    try {
        // 1. group rows of the arrivals (grp is not read by queries; a larger
        //    copy replaces it under the lock below)
        uint16_t *grp = ix.grp;
        if (x0 + n > ix.grp_cap) {
            const uint64_t cap = std::max<uint64_t>(x0 + n, ix.grp_cap + ix.grp_cap / 2);
            grp1 = static_cast<uint16_t *>(pool_malloc(cap * Rp * 2, s));
            FL_HIP(hipMemcpyAsync(grp1, ix.grp, x0 * Rp * 2, hipMemcpyDeviceToDevice, s));
            grp = grp1;
        }
        uint32_t nb = 2;
        while (nb < 64 && (1ull << nb) < B) nb += 2;
        const unsigned gn = (unsigned)((n + 255) / 256);
        hipLaunchKernelGGL(stream_groups_kernel, dim3(gn), dim3(256), 0, s, x0, n, ix.N0, R, Rp, B,
                           nb / 2, sm64(ix.p.seed, TAG_STREAM), grp);
        FL_CHECK_LAUNCH();
        // 2. arrivals sorted by group, per repetition; new cell sizes
        int gbits = 1;
        while ((1u << gbits) < B) ++gbits;
        Pieces pc;
        const size_t o_keys = pc.add(n * R * 4), o_pairs = pc.add(n * R * 8), o_tmp = pc.add(n * R * 8),
                     o_ps = pc.add(pair_sort_scratch_bytes(n, R)), o_starts = pc.add(ncells * 4),
                     o_ends = pc.add(ncells * 4), o_cnt = pc.add(ncells * 4);
        DevBuf ws = DevBuf::pooled(pc.total, s);
        char *w = ws.as<char>();
        uint32_t *skeys = reinterpret_cast<uint32_t *>(w + o_keys);
        uint64_t *pairs = reinterpret_cast<uint64_t *>(w + o_pairs);
        uint32_t *starts = reinterpret_cast<uint32_t *>(w + o_starts);
        uint32_t *ends = reinterpret_cast<uint32_t *>(w + o_ends);
        uint32_t *cnt = reinterpret_cast<uint32_t *>(w + o_cnt);
        FL_HIP(hipMemsetAsync(starts, 0, ncells * 4, s));
        FL_HIP(hipMemsetAsync(ends, 0, ncells * 4, s));
        hipLaunchKernelGGL(member_keys_kernel, dim3(gn, R), dim3(256), 0, s, grp, x0, n, Rp, 0u,
                           skeys);
        FL_CHECK_LAUNCH();
        pair_sort(skeys, n, R, gbits, pairs, reinterpret_cast<uint64_t *>(w + o_tmp), w + o_ps, s);
        hipLaunchKernelGGL(run_bounds_kernel, dim3(gn, R), dim3(256), 0, s, pairs, n, B,
                           starts, ends);
        FL_CHECK_LAUNCH();
        hipLaunchKernelGGL(run_counts_kernel, dim3((unsigned)((ncells + 255) / 256)), dim3(256), 0, s,
                           starts, ends, (uint32_t)ncells,
                           cnt);
        FL_CHECK_LAUNCH();
        std::vector<uint32_t> add(ncells);
        FL_HIP(hipMemcpyAsync(add.data(), cnt, ncells * 4, hipMemcpyDeviceToHost, s));
        FL_HIP(hipStreamSynchronize(s));
        std::vector<uint32_t> gs1(ix.gsize_host);
        uint32_t gmax1 = 0;
        for (uint64_t c = 0; c < ncells; ++c) {
            gs1[c] += add[c];
            gmax1 = std::max(gmax1, gs1[c]);
        }
        // 3. member arrays of the new version: a copy, at a larger stride when
        //    a cell outgrows the old one, then the arrivals appended
        uint32_t ms1 = ix.mstride;
        if (gmax1 > ms1) ms1 = (uint32_t)((std::max<uint64_t>(gmax1, ms1 + ms1 / 2) + 3) & ~3ull);
        const MemberLayout ml(ncells, ms1, Rp);
        slab = static_cast<char *>(pool_malloc(ml.total, s));
        uint32_t *mem1 = reinterpret_cast<uint32_t *>(slab);
        uint16_t *cmg1 = reinterpret_cast<uint16_t *>(slab + ml.cmg);
        uint32_t *cfl1 = reinterpret_cast<uint32_t *>(slab + ml.cfl);
        uint32_t *gsize1 = reinterpret_cast<uint32_t *>(slab + ml.gsize);
        if (ms1 == ix.mstride) {
            FL_HIP(hipMemcpyAsync(mem1, ix.mem, ncells * ms1 * 4, hipMemcpyDeviceToDevice, s));
            FL_HIP(hipMemcpyAsync(cmg1, ix.cmg, ncells * ms1 * Rp * 2, hipMemcpyDeviceToDevice, s));
        } else {
            FL_HIP(hipMemsetAsync(mem1, 0xFF, ncells * ms1 * 4, s));
            FL_HIP(hipMemsetAsync(cmg1, 0, ncells * ms1 * Rp * 2, s));
            const uint64_t tot = ncells * ix.mstride;
            hipLaunchKernelGGL(restride_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s,
                               ix.mem, ix.cmg, ncells, ix.mstride, ms1, Rp, mem1, cmg1);
            FL_CHECK_LAUNCH();
        }
        hipLaunchKernelGGL(place_members_kernel, dim3(gn, R), dim3(256), 0, s, pairs, n,
                           x0, starts, ix.gsize, B, ms1, grp, Rp, mem1, cmg1);
        FL_CHECK_LAUNCH();
        build_filter(ix, mem1, grp, ms1, cfl1, s);
        hipLaunchKernelGGL(add_u32_kernel, dim3((unsigned)((ncells + 255) / 256)), dim3(256), 0, s,
                           ix.gsize, cnt, ncells, gsize1);
        FL_CHECK_LAUNCH();
        // 4. reverse index: the arrivals' cells merged into the old lists
        lists = merge_lists(ix, codes, grp + x0 * Rp, n, s);
        FL_HIP(hipStreamSynchronize(s));
        // 5. swap the new version in while no query is being enqueued, and
        //    free the old one once the device has finished all work using it
        std::unique_lock<std::shared_mutex> lk(ix.rw);
        void *old[4] = {ix.offsets, ix.cells, ix.mem, grp1 ? ix.grp : nullptr};
        ix.offsets = lists.offsets;
        ix.cells = lists.cells;
        // (kept as it was, scaled: it only chooses between query kernels)
        ix.mean_entries *= (double)lists.entries / (double)std::max<uint64_t>(ix.list_entries, 1);
        ix.list_entries = lists.entries;
        ix.mem = mem1;
        ix.cmg = cmg1;
        ix.cfl = cfl1;
        ix.gsize = gsize1;
        if (grp1) {
            ix.grp = grp1;
            ix.grp_cap = std::max<uint64_t>(x0 + n, ix.grp_cap + ix.grp_cap / 2);
        }
        ix.mstride = ms1;
        ix.gsize_host = std::move(gs1);
        ix.gmax = gmax1;
        ix.N = x0 + n;
        ix.device_bytes = index_device_bytes(ix);
        lists = Lists();
        slab = nullptr;
        grp1 = nullptr;
        FL_HIP(hipDeviceSynchronize());
        for (void *p : old) pool_free(p);
    } catch (...) {
        (void)hipDeviceSynchronize();
        pool_free(grp1);
        pool_free(slab);
        free_lists(lists);
        throw;
    }
}

}  // namespace flinng
