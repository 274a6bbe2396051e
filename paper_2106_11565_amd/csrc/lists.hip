// The reverse index on gfx950 (Section 6, Implementation): for every table
// and bucket the ascending distinct cells r*Bp + g_r(x) over the points x of
// the bucket (a filter bit is set once).
//
// The points, not the (bucket, cell) pairs, are sorted: R times fewer keys
// and only the bucket's bits to sort by.  Per batch of tables:
//   1. the codes are transposed to one run per table, and the tables' points
//      sorted by code together (pair_sort: code << 32 | point);
//   2. each bucket's points are then one run of the sorted array, and its
//      list needs only the run's group rows.  Runs of at most RUN_SHORT
//      points are handled a thread per point: the run's rows are in LDS and a
//      point finds by comparison with its run which of its cells come first
//      and how many smaller distinct cells each has before it.  Longer runs
//      take a workgroup each: a bit per cell of the grid in LDS, set by the
//      run's points and read back in order.
//   3. lists are sized first (a count per run, an exclusive scan over all
//      tables), so the cells are written once, into an allocation of their
//      exact size; the offsets of all 2^bits buckets come from a merge of the
//      bucket numbers with the sorted codes.
//
// Inserts build the lists of the new points the same way and merge them into
// the old ones: an added cell's place in its old list is found by binary
// search, and the new cells array is one merge-path copy.
//
// What bounds it: bytes.  Per table, N points and R repetitions: about
// (8 + 16 ceil(bits/8)) N for the sort, two gathers of 2 Rp bytes per point
// from the group rows (cache resident up to some 10 M points), 12 N for
// counts and scan, R N cell ids and 2^bits offsets written.  Measured, kernel
// time of all lists: 5M URL strings (48 tables of 2^22 buckets, R = 8, 1.9 G
// entries) 157 -> 20 ms against sorting and compacting every (bucket, cell)
// pair table by table; 1M embeddings (12 tables of 2^24 buckets, R = 8)
// 8.3 -> 3.7 ms; an insert of 10,000 reads into 900,000 (12 tables, R = 4)
// 4.5 -> 0.7 ms.  Of the 20 ms the run kernels take 9.2 and the offsets 3.0.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <memory>
#include <utility>
#include <vector>

#include "flinng_internal.h"

namespace flinng {

namespace {

// ---------------------------------------------------------------------------
// out[t*n + x] = codes[x*L + t0 + t] for t < nt: 32 x 64 tiles through LDS, so
// that both sides move whole lines.
constexpr int TR_P = 64, TR_T = 32;
__global__ __launch_bounds__(256) void transpose_codes_kernel(const uint32_t *__restrict__ codes,
                                                              uint64_t n, uint32_t L, uint32_t t0,
                                                              uint32_t nt, uint32_t *__restrict__ out) {
    __shared__ uint32_t tile[TR_P][TR_T + 1];
    const uint64_t x0 = (uint64_t)blockIdx.x * TR_P;
    const uint32_t tb = blockIdx.y * TR_T;
    for (uint32_t j = threadIdx.x; j < TR_P * TR_T; j += 256) {
        const uint32_t i = j / TR_T, t = j % TR_T;
        if (x0 + i < n && tb + t < nt) tile[i][t] = codes[(x0 + i) * L + t0 + tb + t];
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < TR_P * TR_T; j += 256) {
        const uint32_t t = j / TR_P, i = j % TR_P;
        if (x0 + i < n && tb + t < nt) out[(uint64_t)(tb + t) * n + x0 + i] = tile[i][t];
    }
}

// ---------------------------------------------------------------------------
// Short runs.  A workgroup owns the runs that start in its RUN_TILE sorted
// points and loads RUN_SHORT more, so a short run is whole in LDS.  The rows
// of points in long runs are not gathered.  RUN_SHORT = 32: a point of a run
// of n costs about 4 R n instructions here, while a long run costs its
// workgroup a pass over R*B bits.
constexpr uint32_t RUN_TILE = 1024, RUN_SHORT = 32, RUN_LOAD = RUN_TILE + RUN_SHORT;
constexpr uint32_t WORK_SAMPLE = 8;

template <int RP>
struct RowWords {
    static constexpr int W = (RP + 1) / 2;
};

template <int RP>
__device__ inline void load_group_row(const uint16_t *__restrict__ grp, uint64_t x, uint32_t *o) {
    if constexpr (RP == 1) {
        o[0] = grp[x];
    } else if constexpr (RP == 2) {
        o[0] = reinterpret_cast<const uint32_t *>(grp)[x];
    } else if constexpr (RP == 4) {
        const uint2 v = reinterpret_cast<const uint2 *>(grp)[x];
        o[0] = v.x;
        o[1] = v.y;
    } else {
#pragma unroll
        for (int i = 0; i < RP / 8; ++i) {
            const uint4 v = reinterpret_cast<const uint4 *>(grp)[x * (RP / 8) + i];
            o[4 * i] = v.x;
            o[4 * i + 1] = v.y;
            o[4 * i + 2] = v.z;
            o[4 * i + 3] = v.w;
        }
    }
}

template <int W>
__device__ inline uint32_t row_half(const uint32_t (&w)[W], int r) {
    return (w[r >> 1] >> (16 * (r & 1))) & 0xFFFFu;
}

// COUNT: cnt[i] = list length of the run that starts at sorted point i (0
// where none starts, and for now where a long one does), the long runs' starts
// appended to `longs`, and list lengths times run lengths added to `work`.  Otherwise: the cells of the short runs, the
// list of the run that starts at i beginning at cells[pos[i]].
template <typename CellT, int RP, bool COUNT>
__global__ __launch_bounds__(256) void short_runs_kernel(
    const uint64_t *__restrict__ pairs, uint64_t n, const uint16_t *__restrict__ grp, uint32_t R,
    uint32_t Bp, uint32_t *__restrict__ cnt, uint64_t *__restrict__ longs,
    unsigned int *__restrict__ nlong, unsigned long long *__restrict__ work,
    CellT *__restrict__ cells) {
    constexpr int W = RowWords<RP>::W;
    constexpr int PER = (RUN_LOAD + 255) / 256;
    __shared__ uint32_t sc[RUN_LOAD + 1];  // sc[j + 1]: code of point base + j
    __shared__ __align__(16) uint32_t rows[RUN_LOAD][W];
    __shared__ uint32_t aux[COUNT ? RUN_TILE : RUN_LOAD];  // counts, or first-occurrence masks
    const int tid = threadIdx.x;
    const uint64_t base = (uint64_t)blockIdx.x * RUN_TILE, o = (uint64_t)blockIdx.y * n;
    uint32_t xid[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const uint32_t j = tid + 256 * p;
        xid[p] = 0;
        if (j < RUN_LOAD) {
            // past the end: a code no table has (codes stay below 2^24)
            const uint64_t v = base + j < n ? pairs[o + base + j] : ~0ull;
            sc[j + 1] = (uint32_t)(v >> 32);
            xid[p] = (uint32_t)v;
            if (COUNT && j < RUN_TILE) aux[j] = 0;
        }
    }
    if (tid == 0) sc[0] = base ? (uint32_t)(pairs[o + base - 1] >> 32) : 0xFFFFFFFEu;
    __syncthreads();
    // the run of each point: its start, or none of this workgroup's short runs
    uint32_t st[PER], own[PER][W];
    bool act[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const uint32_t j = tid + 256 * p;
        act[p] = false;
        st[p] = 0;
        if (j < RUN_LOAD && base + j < n) {
            const uint32_t c = sc[j + 1];
            uint32_t s = j;
            while (s > 0 && j - s < RUN_SHORT && sc[s] == c) --s;
            // s = 0 with the point before it in the same run: not ours
            const bool mine = s < RUN_TILE && sc[s] != c;
            const bool is_long = mine && sc[s + RUN_SHORT + 1] == c;
            if (COUNT && is_long && j == s) longs[atomicAdd(nlong, 1u)] = o + base + s;
            act[p] = mine && !is_long;
            st[p] = s;
            if (act[p]) {
                load_group_row<RP>(grp, xid[p], own[p]);
#pragma unroll
                for (int w = 0; w < W; ++w) rows[j][w] = own[p][w];
            }
        }
    }
    __syncthreads();
    const uint32_t rmask = (1u << R) - 1u;
    uint32_t dup[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const uint32_t j = tid + 256 * p;
        dup[p] = 0;
        if (act[p]) {
            for (uint32_t i = st[p]; i < j; ++i) {
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const uint32_t x = rows[i][w] ^ own[p][w];
                    if ((x & 0xFFFFu) == 0) dup[p] |= 1u << (2 * w);
                    if ((x >> 16) == 0) dup[p] |= 2u << (2 * w);
                }
            }
            const uint32_t first = rmask & ~dup[p];
            if (COUNT) atomicAdd(&aux[st[p]], (uint32_t)__popc(first));
            else aux[j] = first;
        }
    }
    __syncthreads();
    if constexpr (COUNT) {
#pragma unroll
        for (int p = 0; p < (int)(RUN_TILE / 256); ++p) {
            const uint32_t j = tid + 256 * p;
            if (base + j < n) cnt[o + base + j] = aux[j];
        }
        // list entries met by the runs' points as queries: from one tile in
        // WORK_SAMPLE (an estimate is all that is needed, and a counter that
        // every tile added to would cost as much as the tiles)
        if ((blockIdx.x + blockIdx.y) % WORK_SAMPLE == 0) {
            uint32_t sum = 0;
#pragma unroll
            for (int p = 0; p < PER; ++p) sum += act[p] ? aux[st[p]] : 0u;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
            if (tid % 64 == 0 && sum) atomicAdd(work, (unsigned long long)sum * WORK_SAMPLE);
        }
    } else {
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const uint32_t j = tid + 256 * p;
            if (!act[p]) continue;
            const uint32_t c = sc[j + 1];
            // rank[r]: distinct cells of repetition r in the run below mine;
            // uniq[r]: distinct cells of repetition r
            uint32_t rank[RP], uniq[RP];
#pragma unroll
            for (int r = 0; r < RP; ++r) rank[r] = uniq[r] = 0;
            for (uint32_t i = st[p]; i < RUN_LOAD && sc[i + 1] == c; ++i) {
                const uint32_t f = aux[i];
                uint32_t w[W];
#pragma unroll
                for (int q = 0; q < W; ++q) w[q] = rows[i][q];
#pragma unroll
                for (int r = 0; r < RP; ++r) {
                    const uint32_t b = (f >> r) & 1u;
                    uniq[r] += b;
                    rank[r] += row_half<W>(w, r) < row_half<W>(own[p], r) ? b : 0u;
                }
            }
            uint32_t at = cnt[o + base + st[p]];
            const uint32_t first = aux[j];
#pragma unroll
            for (int r = 0; r < RP; ++r) {
                if ((first >> r) & 1u)
                    cells[(uint64_t)at + rank[r]] = (CellT)((uint32_t)r * Bp + row_half<W>(own[p], r));
                at += uniq[r];
            }
        }
    }
}

// Long runs: a persistent grid over the list of their starts.  The points of
// a run set bits of an LDS bitmap over the R*Bp cells (each wavefront walks
// its own 64-point pieces until the run ends); COUNT counts the bits,
// otherwise the cells are written in order.
template <typename CellT, int RP, bool COUNT>
__global__ __launch_bounds__(256) void long_runs_kernel(const uint64_t *__restrict__ pairs, uint64_t n,
                                                        const uint16_t *__restrict__ grp, uint32_t R,
                                                        uint32_t Bp, uint32_t nwords,
                                                        const uint64_t *__restrict__ longs,
                                                        const unsigned int *__restrict__ nlong,
                                                        uint32_t *__restrict__ cnt,
                                                        unsigned long long *__restrict__ work,
                                                        CellT *__restrict__ cells) {
    constexpr int W = RowWords<RP>::W;
    extern __shared__ uint32_t bits[];
    __shared__ uint32_t wsum[4];
    __shared__ uint32_t npts;
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const unsigned int total = *nlong;
    for (unsigned int q = blockIdx.x; q < total; q += gridDim.x) {
        const uint64_t f = longs[q];
        const uint64_t end = f / n * n + n;  // of its table
        const uint32_t c = (uint32_t)(pairs[f] >> 32);
        for (uint32_t w = tid; w < nwords; w += 256) bits[w] = 0;
        if (COUNT && tid == 0) npts = 0;
        __syncthreads();
        uint32_t mine_pts = 0;
        for (uint64_t p = f + 64 * wave;; p += 256) {
            const uint64_t v = p + lane < end ? pairs[p + lane] : ~0ull;
            const bool in = (uint32_t)(v >> 32) == c;
            if (in) {
                uint32_t w[W];
                load_group_row<RP>(grp, (uint32_t)v, w);
#pragma unroll
                for (int r = 0; r < RP; ++r) {
                    if ((uint32_t)r < R) {
                        const uint32_t cell = (uint32_t)r * Bp + row_half<W>(w, r);
                        atomicOr(&bits[cell >> 5], 1u << (cell & 31));
                    }
                }
            }
            mine_pts += (uint32_t)__popcll(__ballot(in));
            if (__ballot(!in)) break;  // the run ends inside this piece
        }
        if (COUNT && lane == 0) atomicAdd(&npts, mine_pts);
        __syncthreads();
        if constexpr (COUNT) {
            uint32_t s = 0;
            for (uint32_t w = tid; w < nwords; w += 256) s += (uint32_t)__popc(bits[w]);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
            if (lane == 0) wsum[wave] = s;
            __syncthreads();
            if (tid == 0) {
                const uint32_t len = wsum[0] + wsum[1] + wsum[2] + wsum[3];
                cnt[f] = len;
                atomicAdd(work, (unsigned long long)len * npts);
            }
        } else {
            uint32_t at = cnt[f];
            for (uint32_t w0 = 0; w0 < nwords; w0 += 256) {
                uint32_t v = w0 + tid < nwords ? bits[w0 + tid] : 0u;
                uint32_t inc = (uint32_t)__popc(v);
                const uint32_t mine = inc;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t y = __shfl_up(inc, off, 64);
                    if (lane >= off) inc += y;
                }
                if (lane == 63) wsum[wave] = inc;
                __syncthreads();
                uint32_t pre = inc - mine, all = 0;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    pre += w < wave ? wsum[w] : 0u;
                    all += wsum[w];
                }
                uint64_t d = (uint64_t)at + pre;
                for (; v; v &= v - 1) cells[d++] = (CellT)((w0 + tid) * 32 + __ffs(v) - 1);
                at += all;
                __syncthreads();
            }
        }
        __syncthreads();
    }
}

// tstart[t] = where table t's entries start: the prefix at its first point,
// and the total after the last table.
__global__ void table_starts_kernel(const uint32_t *__restrict__ pos, uint64_t n, uint32_t nt,
                                    const uint64_t *__restrict__ total, uint64_t *__restrict__ tstart) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t <= nt) tstart[t] = t < nt ? pos[(uint64_t)t * n] : *total;
}

// ---------------------------------------------------------------------------
// Bucket offsets without atomics, as a merge of two sorted sequences: the
// bucket numbers 0 .. nbk and the codes of a table's n sorted points, where
// bucket b goes before the points of buckets >= b.  The offset of bucket b is
// the list start of the first such point (a run's first).  Each thread takes
// OB_ITEMS consecutive items of the merged order: a binary search on its
// diagonal finds how many points precede its first item, then it walks its
// items, consuming a point or writing one offset per step.  The work per
// thread is bounded however the points crowd into few buckets (SRP codes of
// clustered data leave gaps of millions of empty buckets).  A workgroup's
// offsets form one contiguous run of at most OB_BLOCK buckets: gathered in
// LDS and written with whole-line stores.
constexpr uint32_t OB_ITEMS = 32;
constexpr uint64_t OB_BLOCK = 256ull * OB_ITEMS;       // merged items per workgroup
constexpr uint32_t OB_LDS = OB_BLOCK + OB_BLOCK / 32;  // one pad word per 32
__device__ inline uint32_t ob_pad(uint64_t j) { return (uint32_t)(j + (j >> 5)); }

// Where the merge path crosses diagonal d: the first point index i in [lo, hi)
// that does not go before bucket d-1-i.
__device__ inline uint64_t ob_cross(const uint64_t *__restrict__ pairs, uint64_t d, uint64_t lo,
                                    uint64_t hi) {
    while (lo < hi) {
        const uint64_t m = (lo + hi) / 2;
        if ((pairs[m] >> 32) + 1 + m < d) lo = m + 1;  // bucket(m) < d-1-m
        else hi = m;
    }
    return lo;
}

// The crossings of the workgroups' first diagonals (one thread each): the
// crossing only grows along the path, so a thread of bucket_offsets_kernel
// then searches its workgroup's stretch of at most OB_BLOCK points, mostly in
// cache, instead of the whole table.
__global__ void bucket_blocks_kernel(const uint64_t *__restrict__ pairs, uint64_t n, uint64_t nbk,
                                     uint64_t nblk, uint64_t *__restrict__ blo) {
    const uint64_t b = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b > nblk) return;
    const uint64_t total = nbk + 1 + n;
    const uint64_t d = b * OB_BLOCK < total ? b * OB_BLOCK : total;
    blo[blockIdx.y * (nblk + 1) + b] = ob_cross(pairs + blockIdx.y * n, d,
                                                d > nbk + 1 ? d - (nbk + 1) : 0, d < n ? d : n);
}

__global__ __launch_bounds__(256) void bucket_offsets_kernel(
    const uint64_t *__restrict__ pairs_all, const uint32_t *__restrict__ pos_all, uint64_t n,
    uint64_t nbk, const uint64_t *__restrict__ blo_all, uint64_t nblk,
    const uint64_t *__restrict__ tstart, uint32_t *__restrict__ off) {
    __shared__ uint32_t run[OB_LDS];
    const uint64_t total = nbk + 1 + n;
    const uint32_t t = blockIdx.y;
    const uint64_t *pairs = pairs_all + (uint64_t)t * n;
    const uint32_t *pos = pos_all + (uint64_t)t * n;
    const uint64_t *blo = blo_all + (uint64_t)t * (nblk + 1);
    // the workgroup's diagonals [d0, d1) emit the buckets [b0, b1)
    const uint64_t d0 = (uint64_t)blockIdx.x * OB_BLOCK;
    const uint64_t d1 = d0 + OB_BLOCK < total ? d0 + OB_BLOCK : total;
    const uint64_t c0 = blo[blockIdx.x], c1 = blo[blockIdx.x + 1];
    const uint64_t b0 = d0 - c0, b1 = d1 - c1;
    const uint64_t d = d0 + (uint64_t)threadIdx.x * OB_ITEMS;
    if (d < total) {
        // the crossing of d lies between those of the workgroup's diagonals
        uint64_t lo = d > nbk + 1 ? d - (nbk + 1) : 0, hi = d < n ? d : n;
        lo = lo > c0 ? lo : c0;
        hi = hi < c1 ? hi : c1;
        uint64_t i = ob_cross(pairs, d, lo, hi), b = d - i;
        const uint32_t last = (uint32_t)tstart[t + 1];
        const uint64_t end = d + OB_ITEMS < total ? d + OB_ITEMS : total;
        uint64_t kb = i < n ? pairs[i] >> 32 : 0;  // bucket of point i
        uint32_t pv = 0;                           // its list start, once read
        bool have = false;
        for (uint64_t e = d; e < end; ++e) {
            if (i < n && (b > nbk || kb < b)) {
                ++i;
                if (i < n) kb = pairs[i] >> 32;
                have = false;
            } else {
                if (!have) {
                    pv = i < n ? pos[i] : last;
                    have = true;
                }
                run[ob_pad(b - b0)] = pv;
                ++b;
            }
        }
    }
    __syncthreads();
    uint32_t *o = off + (uint64_t)t * (nbk + 1) + b0;
    for (uint64_t j = threadIdx.x; j < b1 - b0; j += blockDim.x) o[j] = run[ob_pad(j)];
}

// ---------------------------------------------------------------------------
// merging the lists of new points into the old ones

// Entry e of the new points' lists: whether its cell is missing from the old
// list of its bucket (add[e]), and the old entry it goes before (before[e]).
// The table comes from the tables' starts, the bucket by binary search over
// the table's offsets.
template <typename CellT>
__global__ void added_cells_kernel(const uint32_t *__restrict__ doff, const CellT *__restrict__ dcells,
                                   uint64_t n, const uint32_t *__restrict__ ooff,
                                   const CellT *__restrict__ ocells, uint32_t L, uint64_t nbk,
                                   uint32_t *__restrict__ add, uint32_t *__restrict__ before) {
    const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    uint32_t tl = 0, th = L;  // the last table that starts at or before e
    while (th - tl > 1) {
        const uint32_t m = (tl + th) / 2;
        if (doff[(uint64_t)m * (nbk + 1)] <= e) tl = m; else th = m;
    }
    const uint64_t to = (uint64_t)tl * (nbk + 1);
    uint64_t lo = 0, hi = nbk;  // doff[to + lo] <= e < doff[to + hi]
    while (hi - lo > 1) {
        const uint64_t m = (lo + hi) / 2;
        if (doff[to + m] <= e) lo = m; else hi = m;
    }
    const CellT c = dcells[e];
    uint32_t a = ooff[to + lo];
    const uint32_t end = ooff[to + lo + 1];
    uint32_t b = end;
    while (a < b) {  // the first old entry >= c
        const uint32_t m = a + (b - a) / 2;
        if (ocells[m] < c) a = m + 1; else b = m;
    }
    add[e] = (a < end && ocells[a] == c) ? 0u : 1u;
    before[e] = a;
}

// The added cells packed: cell, and the new position of each (the old entries
// before it plus the added ones).  rank: prefix of `add`, from `base` (the cells
// added to the tables before) to *nadd.
template <typename CellT>
__global__ void pack_added_kernel(const CellT *__restrict__ dcells, const uint32_t *__restrict__ before,
                                  const uint32_t *__restrict__ rank, uint64_t n, uint64_t base,
                                  const uint64_t *__restrict__ nadd, uint32_t *__restrict__ at,
                                  CellT *__restrict__ ac) {
    const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const uint32_t r = rank[e], nx = e + 1 < n ? rank[e + 1] : (uint32_t)*nadd;
    if (nx == r) return;
    at[r - (uint32_t)base] = before[e] + r;
    ac[r - (uint32_t)base] = dcells[e];
}

// How many of the ascending values v[0, n) lie below x.
__device__ inline uint64_t count_below(const uint32_t *__restrict__ v, uint64_t n, uint64_t x) {
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        const uint64_t m = (lo + hi) / 2;
        if (v[m] < x) lo = m + 1; else hi = m;
    }
    return lo;
}

// New entries [first, end), those of some tables: entry p is the a-th added cell
// where at[a] = p, else old entry p minus the added cells before it (`base` of
// them in earlier tables).  A workgroup writes 2048 consecutive entries: the first
// of its added cells by one binary search, the rest counted from them.
constexpr uint32_t MG_TILE = 2048;
template <typename CellT>
__global__ __launch_bounds__(256) void merge_cells_kernel(const CellT *__restrict__ ocells,
                                                          const uint32_t *__restrict__ at,
                                                          const CellT *__restrict__ ac, uint64_t nadd,
                                                          uint64_t base, uint64_t first, uint64_t end,
                                                          CellT *__restrict__ out) {
    __shared__ uint64_t range[2];
    __shared__ uint32_t sat[MG_TILE];
    const uint64_t p0 = first + (uint64_t)blockIdx.x * MG_TILE;
    const uint64_t p1 = p0 + MG_TILE < end ? p0 + MG_TILE : end;
    if (threadIdx.x < 2) range[threadIdx.x] = count_below(at, nadd, threadIdx.x ? p1 : p0);
    __syncthreads();
    const uint64_t a0 = range[0];
    const uint32_t na = (uint32_t)(range[1] - a0);  // at most one per new entry
    for (uint32_t i = threadIdx.x; i < na; i += 256) sat[i] = at[a0 + i];
    __syncthreads();
    for (uint64_t p = p0 + threadIdx.x; p < p1; p += 256) {
        uint32_t lo = 0, hi = na;
        while (lo < hi) {
            const uint32_t m = (lo + hi) / 2;
            if (sat[m] < p) lo = m + 1; else hi = m;
        }
        out[p] = (lo < na && sat[lo] == p) ? ac[a0 + lo] : ocells[p - (base + a0 + lo)];
    }
}

// New offset = old offset + the added cells of all earlier lists (rank counts
// those of the tables before too).
__global__ void merge_offsets_kernel(const uint32_t *__restrict__ ooff,
                                     const uint32_t *__restrict__ doff,
                                     const uint32_t *__restrict__ rank, uint64_t nd,
                                     const uint64_t *__restrict__ nadd, uint64_t n,
                                     uint32_t *__restrict__ out) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t d = doff[i];
    out[i] = ooff[i] + (d < nd ? rank[d] : (uint32_t)*nadd);
}

unsigned blocks_for(uint64_t n, uint32_t per) { return (unsigned)((n + per - 1) / per); }

// An index array in the making: freed, once the device is idle, unless
// released.
struct MemFree {
    void operator()(void *p) const {
        (void)hipDeviceSynchronize();
        pool_free(p);
    }
};
using HipMem = std::unique_ptr<void, MemFree>;

HipMem hip_mem(size_t bytes, hipStream_t s) { return HipMem(pool_malloc(std::max<size_t>(bytes, 1), s)); }

// What one batch of tables runs on.
struct Batch {
    uint64_t *pairs;   // [nt][n] sorted
    uint32_t *pos;     // [nt][n] counts, then list starts
    uint64_t *longs;
    unsigned int *nlong;
    uint64_t *tstart;  // [nt + 1]
    uint64_t *total;   // entries so far, and the work of the runs
    uint64_t *blo;
};

template <typename CellT, int RP, bool COUNT>
void launch_runs(const Index &ix, const Batch &b, uint64_t n, uint32_t nt, const uint16_t *grp,
                 CellT *cells, hipStream_t s) {
    const uint32_t Bp = (ix.p.B + 3) & ~3u;
    hipLaunchKernelGGL((short_runs_kernel<CellT, RP, COUNT>), dim3(blocks_for(n, RUN_TILE), nt),
                       dim3(256), 0, s, b.pairs, n, grp, ix.p.R, Bp, b.pos, b.longs, b.nlong,
                       reinterpret_cast<unsigned long long *>(b.total + 1), cells);
    FL_CHECK_LAUNCH();
    if (n > RUN_SHORT) {
        const uint32_t nwords = (ix.p.R * Bp + 31) / 32;  // at most 128 KiB (R <= 16, B <= 65536)
        static const bool attr_ok = [] {
            FL_HIP(hipFuncSetAttribute(
                reinterpret_cast<const void *>(&long_runs_kernel<CellT, RP, COUNT>),
                hipFuncAttributeMaxDynamicSharedMemorySize, 16 * 65536 / 8));
            return true;
        }();
        (void)attr_ok;
        // enough workgroups to fill the chip at any bitmap size; a run's
        // workgroup leaves once the list is drained
        const uint64_t most = n * nt / (RUN_SHORT + 1) + 1;
        hipLaunchKernelGGL((long_runs_kernel<CellT, RP, COUNT>),
                           dim3((unsigned)std::min<uint64_t>(most, 2048)), dim3(256), nwords * 4, s,
                           b.pairs, n, grp, ix.p.R, Bp, nwords, b.longs, b.nlong, b.pos,
                           reinterpret_cast<unsigned long long *>(b.total + 1), cells);
        FL_CHECK_LAUNCH();
    }
}

template <typename CellT, bool COUNT>
void runs(const Index &ix, const Batch &b, uint64_t n, uint32_t nt, const uint16_t *grp, void *cells,
          hipStream_t s) {
    CellT *c = static_cast<CellT *>(cells);
    switch (ix.Rp) {
        case 1: launch_runs<CellT, 1, COUNT>(ix, b, n, nt, grp, c, s); break;
        case 2: launch_runs<CellT, 2, COUNT>(ix, b, n, nt, grp, c, s); break;
        case 4: launch_runs<CellT, 4, COUNT>(ix, b, n, nt, grp, c, s); break;
        case 8: launch_runs<CellT, 8, COUNT>(ix, b, n, nt, grp, c, s); break;
        default: launch_runs<CellT, 16, COUNT>(ix, b, n, nt, grp, c, s); break;
    }
}

// the last bytes of a cells array, zeroed with a kernel
__global__ void zero_tail_kernel(unsigned char *p, uint64_t a, uint64_t b) {
    for (uint64_t i = a + threadIdx.x; i < b; i += blockDim.x) p[i] = 0;
}

HipMem cells_with_tail(uint64_t entries, size_t csz, hipStream_t s) {
    HipMem m = hip_mem(cells_alloc_bytes(entries, csz), s);
    hipLaunchKernelGGL(zero_tail_kernel, dim3(1), dim3(64), 0, s,
                       static_cast<unsigned char *>(m.get()), entries * csz,
                       (uint64_t)cells_alloc_bytes(entries, csz));
    FL_CHECK_LAUNCH();
    return m;
}

}  // namespace

void free_lists(Lists &l) {
    if (l.offsets || l.cells) (void)hipDeviceSynchronize();
    pool_free(l.offsets);
    pool_free(l.cells);
    l = Lists();
}

// Scratch of a batch of tables, at most this much for more than one table:
// the workloads' indexes take one batch (URL strings, 5M points, 48 tables:
// 4.8 GB), whose cells are then written straight into their final array.
constexpr uint64_t LISTS_SCRATCH = 6ull << 30;
// tables sorted together: the sort's second buffer at most this large, which
// keeps both sides of a pass in the 256 MB last-level cache
constexpr uint64_t SORT_TMP = 96ull << 20;

// The lists of tables tb .. tb+L-1; their offsets ([L][nbuckets + 1]) go to
// `off`, the entries counted from the first.
static Lists make_tables(const Index &ix, const uint32_t *codes, const uint16_t *grp, uint64_t n,
                         uint32_t tb, uint32_t L, uint32_t *off, hipStream_t s) {
    const uint64_t nbk = nbuckets(ix);
    const size_t csz = ix.cell_bytes;
    const uint64_t per_table = 8 * n + 4 * n + 8 * (n / (RUN_SHORT + 1) + 2);
    const uint32_t bt = (uint32_t)std::min<uint64_t>(L, std::max<uint64_t>(1, LISTS_SCRATCH / per_table));
    const uint32_t stn = (uint32_t)std::min<uint64_t>(bt, std::max<uint64_t>(1, SORT_TMP / (8 * n)));
    const uint64_t nblk = (nbk + 1 + n + OB_BLOCK - 1) / OB_BLOCK;

    Lists out;
    std::vector<std::pair<HipMem, uint64_t>> parts;  // the batches' cells
    Pieces pc;
    auto piece = [&](size_t bytes) { return pc.add(bytes); };
    const size_t o_pairs = piece((size_t)bt * n * 8), o_tmp = piece((size_t)stn * n * 8);
    const size_t o_pos = piece((size_t)bt * n * 4);
    const size_t o_longs = piece((size_t)bt * (n / (RUN_SHORT + 1) + 1) * 8);
    const size_t o_nlong = piece(4), o_ts = piece((bt + 1) * 8), o_total = piece(16);
    const size_t o_blo = piece((size_t)bt * (nblk + 1) * 8);
    const size_t o_ps = piece(pair_sort_scratch_bytes(n, stn));
    const size_t o_scan = piece(scan_scratch_bytes((uint64_t)bt * n));
    DevBuf ws = DevBuf::pooled(pc.total, s);
    char *w = ws.as<char>();
    const Batch b{reinterpret_cast<uint64_t *>(w + o_pairs), reinterpret_cast<uint32_t *>(w + o_pos),
                  reinterpret_cast<uint64_t *>(w + o_longs), reinterpret_cast<unsigned int *>(w + o_nlong),
                  reinterpret_cast<uint64_t *>(w + o_ts), reinterpret_cast<uint64_t *>(w + o_total),
                  reinterpret_cast<uint64_t *>(w + o_blo)};
    uint64_t *tmp = reinterpret_cast<uint64_t *>(w + o_tmp);
    hipLaunchKernelGGL(zero_tail_kernel, dim3(1), dim3(64), 0, s,
                       reinterpret_cast<unsigned char *>(b.total), 0ull, 16ull);
    FL_CHECK_LAUNCH();
    for (uint32_t t0 = 0; t0 < L; t0 += bt) {
        const uint32_t nt = std::min(bt, L - t0);
        // codes by table (in the counts' place), sorted points
        hipLaunchKernelGGL(transpose_codes_kernel, dim3(blocks_for(n, TR_P), blocks_for(nt, TR_T)),
                           dim3(256), 0, s, codes, n, ix.p.L, tb + t0, nt, b.pos);
        FL_CHECK_LAUNCH();
        for (uint32_t q = 0; q < nt; q += stn)
            pair_sort(b.pos + (uint64_t)q * n, n, std::min(stn, nt - q), (int)ix.nbits,
                      b.pairs + (uint64_t)q * n, tmp, w + o_ps, s);
        // list sizes and starts
        hipLaunchKernelGGL(zero_tail_kernel, dim3(1), dim3(64), 0, s,
                           reinterpret_cast<unsigned char *>(b.nlong), 0ull, 4ull);
        FL_CHECK_LAUNCH();
        runs<uint16_t, true>(ix, b, n, nt, grp, nullptr, s);
        device_exclusive_scan_u32(b.pos, (uint64_t)nt * n, out.entries, b.total, w + o_scan, s);
        uint64_t got[2] = {0, 0};
        FL_HIP(hipMemcpyAsync(got, b.total, 16, hipMemcpyDeviceToHost, s));
        // offsets (queued before the total is waited for)
        hipLaunchKernelGGL(table_starts_kernel, dim3(blocks_for(nt + 1, 64)), dim3(64), 0, s, b.pos, n,
                           nt, b.total, b.tstart);
        FL_CHECK_LAUNCH();
        hipLaunchKernelGGL(bucket_blocks_kernel, dim3(blocks_for(nblk + 1, 256), nt), dim3(256), 0, s,
                           b.pairs, n, nbk, nblk, b.blo);
        FL_CHECK_LAUNCH();
        hipLaunchKernelGGL(bucket_offsets_kernel, dim3((unsigned)nblk, nt), dim3(256), 0, s, b.pairs,
                           b.pos, n, nbk, b.blo, nblk, b.tstart,
                           off + (uint64_t)t0 * (nbk + 1));
        FL_CHECK_LAUNCH();
        FL_HIP(hipStreamSynchronize(s));
        const uint64_t total = got[0];
        out.mean_entries = (double)got[1] / (double)n;
        if (total > 0xFFFFFFFFull) fail(FLINNG_EINVAL, "reverse index exceeds 2^32 entries");
        const uint64_t here = total - out.entries;
        parts.emplace_back(cells_with_tail(here, csz, s), here);
        // list starts are absolute; this batch's cells begin at out.entries
        char *c0 = static_cast<char *>(parts.back().first.get()) - out.entries * csz;
        if (csz == 2) runs<uint16_t, false>(ix, b, n, nt, grp, c0, s);
        else runs<uint32_t, false>(ix, b, n, nt, grp, c0, s);
        out.entries = total;
    }
    if (parts.size() > 1) {
        HipMem all = cells_with_tail(out.entries, csz, s);
        uint64_t at = 0;
        for (auto &p : parts) {
            if (p.second)
                FL_HIP(hipMemcpyAsync(static_cast<char *>(all.get()) + at * csz, p.first.get(),
                                      p.second * csz, hipMemcpyDeviceToDevice, s));
            at += p.second;
        }
        FL_HIP(hipStreamSynchronize(s));
        parts.clear();
        parts.emplace_back(std::move(all), out.entries);
    }
    out.cells = parts[0].first.release();
    return out;
}

Lists make_lists(const Index &ix, const uint32_t *codes, const uint16_t *grp, uint64_t n,
                 hipStream_t s) {
    HipMem offsets = hip_mem((size_t)ix.p.L * (nbuckets(ix) + 1) * 4, s);
    Lists out = make_tables(ix, codes, grp, n, 0, ix.p.L, static_cast<uint32_t *>(offsets.get()), s);
    out.offsets = static_cast<uint32_t *>(offsets.release());
    return out;
}

// Offsets of the arrivals' own lists, at most this much for more than one table:
// an insert works through the tables in batches, so that what it needs beside the
// new version stays bounded where the offsets are most of an index (255 tables of
// 2^24 buckets: 17 GB of them).  The workloads' indexes take one batch (URL
// strings, 48 tables of 2^22: 0.8 GB).
constexpr uint64_t MERGE_OFFSETS = 1ull << 30;

namespace {

// The cells that the arrivals add to a batch of tables.
struct Added {
    HipMem list;            // the arrivals' own cells
    DevBuf ws;
    uint32_t *at = nullptr; // new position of each
    void *cells = nullptr;
    uint64_t n = 0;
    uint64_t before = 0;    // cells added to the tables before
    uint64_t first = 0;     // old entries of the tables before
};

// Tables tb .. tb+nt-1: the new offsets from the old ones, and the cells to add.
template <typename CellT>
Added merge_tables(const Index &ix, const uint32_t *codes, const uint16_t *grp_rows, uint64_t n,
                   uint32_t tb, uint32_t nt, uint64_t before, uint32_t *doff, HipMem &offsets,
                   hipStream_t s) {
    const uint64_t nbk = nbuckets(ix), no = (uint64_t)nt * (nbk + 1);
    const Lists d = make_tables(ix, codes, grp_rows, n, tb, nt, doff, s);
    Added out;
    out.list.reset(d.cells);
    out.before = before;
    const uint64_t nd = d.entries;  // every point has a cell in every table
    const CellT *dc = static_cast<const CellT *>(d.cells);
    const CellT *oc = static_cast<const CellT *>(ix.cells);
    const uint32_t *ooff = ix.offsets + (uint64_t)tb * (nbk + 1);
    Pieces pc;
    const size_t o_rank = pc.add(nd * 4), o_below = pc.add(nd * 4), o_at = pc.add(nd * 4),
                 o_ac = pc.add(nd * sizeof(CellT)), o_total = pc.add(8),
                 o_sc = pc.add(scan_scratch_bytes(nd));
    out.ws = DevBuf::pooled(pc.total, s);
    char *w = out.ws.as<char>();
    uint32_t *rk = reinterpret_cast<uint32_t *>(w + o_rank), *below = reinterpret_cast<uint32_t *>(w + o_below);
    out.at = reinterpret_cast<uint32_t *>(w + o_at);
    out.cells = w + o_ac;
    uint64_t *total = reinterpret_cast<uint64_t *>(w + o_total);
    hipLaunchKernelGGL(added_cells_kernel<CellT>, dim3(blocks_for(nd, 256)), dim3(256), 0, s, doff, dc, nd,
                       ooff, oc, nt, nbk, rk, below);
    FL_CHECK_LAUNCH();
    device_exclusive_scan_u32(rk, nd, before, total, w + o_sc, s);
    hipLaunchKernelGGL(pack_added_kernel<CellT>, dim3(blocks_for(nd, 256)), dim3(256), 0, s, dc, below, rk,
                       nd, before, total, out.at, static_cast<CellT *>(out.cells));
    FL_CHECK_LAUNCH();
    uint64_t after = 0;
    uint32_t first = 0;
    FL_HIP(hipMemcpyAsync(&after, total, 8, hipMemcpyDeviceToHost, s));
    if (tb) FL_HIP(hipMemcpyAsync(&first, ooff, 4, hipMemcpyDeviceToHost, s));
    if (!offsets) offsets = hip_mem(ix.p.L * (nbk + 1) * 4, s);
    hipLaunchKernelGGL(merge_offsets_kernel, dim3(blocks_for(no, 256)), dim3(256), 0, s, ooff, doff, rk, nd,
                       total, no, static_cast<uint32_t *>(offsets.get()) + (uint64_t)tb * (nbk + 1));
    FL_CHECK_LAUNCH();
    FL_HIP(hipStreamSynchronize(s));
    out.n = after - before;
    out.first = first;
    return out;
}

template <typename CellT>
Lists merge_into(const Index &ix, const uint32_t *codes, const uint16_t *grp_rows, uint64_t n,
                 hipStream_t s) {
    const uint32_t L = ix.p.L;
    const uint64_t row = nbuckets(ix) + 1;
    const uint32_t bt = (uint32_t)std::min<uint64_t>(L, std::max<uint64_t>(1, MERGE_OFFSETS / (row * 4)));
    std::vector<Added> added;
    uint64_t nadd = 0;
    HipMem doff = hip_mem(bt * row * 4, s);  // of one batch at a time
    HipMem offsets;
    for (uint32_t tb = 0; tb < L; tb += bt) {
        added.push_back(merge_tables<CellT>(ix, codes, grp_rows, n, tb, std::min(bt, L - tb), nadd,
                                            static_cast<uint32_t *>(doff.get()), offsets, s));
        nadd += added.back().n;
    }
    Lists out;
    out.entries = ix.list_entries + nadd;
    if (out.entries > 0xFFFFFFFFull) fail(FLINNG_EINVAL, "reverse index exceeds 2^32 entries");
    HipMem cells = cells_with_tail(out.entries, sizeof(CellT), s);
    for (size_t i = 0; i < added.size(); ++i) {
        const Added &a = added[i];
        const uint64_t p0 = a.first + a.before;
        const uint64_t p1 = i + 1 < added.size() ? added[i + 1].first + added[i + 1].before : out.entries;
        hipLaunchKernelGGL(merge_cells_kernel<CellT>, dim3(blocks_for(p1 - p0, MG_TILE)), dim3(256), 0, s,
                           static_cast<const CellT *>(ix.cells), a.at, static_cast<const CellT *>(a.cells),
                           a.n, a.before, p0, p1, static_cast<CellT *>(cells.get()));
        FL_CHECK_LAUNCH();
    }
    FL_HIP(hipStreamSynchronize(s));
    out.offsets = static_cast<uint32_t *>(offsets.release());
    out.cells = cells.release();
    return out;
}

}  // namespace

Lists merge_lists(const Index &ix, const uint32_t *codes, const uint16_t *grp_rows, uint64_t n,
                  hipStream_t s) {
    return ix.cell_bytes == 2 ? merge_into<uint16_t>(ix, codes, grp_rows, n, s)
                              : merge_into<uint32_t>(ix, codes, grp_rows, n, s);
}

}  // namespace flinng
