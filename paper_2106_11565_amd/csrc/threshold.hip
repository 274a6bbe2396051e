// Fixed-threshold query (Algorithm 2) on gfx950.
//
// Algorithm 2 marks a cell positive when its group test fires -- its count
// of colliding tables reaches the threshold t (positive means count >= t) --
// takes in each repetition the union of the positive cells' points and
// reports the intersection of those unions over the R repetitions.  A point
// x is therefore reported iff m(x) = min_r C[r, g_r(x)] >= t, and every
// reported point lies in a positive cell of any single repetition.
//
// One workgroup per query:
//   1. the L list ranges (a thread per table) and their entries as one
//      sequence, counted into the B*R cell counters: bytes in LDS, 4 per dword
//      (Section 6, Implementation).  The entry that takes a cell to t notes the
//      cell as positive, so no scan of the counters is needed;
//   2. the repetition with the fewest positive cells is enumerated (ties: the
//      lowest), in order (cells ascending, members by ascending id).  The cells'
//      filter words (the members' groups in the two next repetitions) come
//      first; only members whose cells there are positive have their row looked
//      up.  Few positive cells: a wavefront takes four at a time and the
//      answer's slots are ranked in LDS.  Many, or an answer that passes the
//      list: T * 4 slots of the cells at a time, with an ordered compaction.
// Bound by the latency of a query's chain of reads and barriers, eight
// workgroups to a compute unit.  A whole call against walking ids and rows, a
// member per thread, with the tables counted one after another: 10,000 reads (12
// tables, t = 6) 102 -> 50 us, of them the kernel 88 -> 35; 532 ReLU rows 164 ->
// 89; 3,000 URLs 387 -> 137; 3,000 points in 400 cells per repetition, a quarter
// of them positive, 218 -> 136.
// Up to max_out ids are written per query; counts[q] receives the size of the
// answer even when it is larger.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "flinng_internal.h"

namespace flinng {

namespace {

struct TArgs {
    const uint32_t *codes;
    uint64_t nq;
    const uint32_t *offsets;
    const void *cells;
    const uint32_t *mem;
    const uint16_t *cmg;
    const uint32_t *cfl;
    uint32_t L, R, Rp, B, Bp, nbits, t, max_out;
    uint32_t mstride, cnt_words;
    bool small_slots;       // a repetition's member slots fit 32 bits
    uint32_t *ids;
    uint32_t *counts;
};

// misc slots after the counters
enum { T_TOTAL = 0, T_NL, T_NP, T_SCAN, T_NPOS = T_SCAN + 16 };  // T_NPOS: R words
// positive cells and answer slots that the fast path holds
constexpr uint32_t T_LIST = 256;
// Up to FEW positive cells, or one in FEW, are taken cell by cell: the filter
// then rejects nearly all members and the ordered walk would scan B cells for
// little (the first three calls above: 50, 89, 137 us by cell, 72, 130, 245 us in
// order).  With more, members pass by the dozen and a cell of 125 leaves half of
// a wavefront idle (the last call: 324 us by cell, 136 in order).
constexpr uint32_t FEW = 16;

// LDS words of the lists (no more than the T of one round where T = 1024, the
// workgroup size of grids whose counters fill the LDS).
__host__ __device__ constexpr uint32_t list_words(int T, uint32_t L) {
    return 2 * T_LIST + 2 * L > (uint32_t)T ? 2 * T_LIST + 2 * L : (uint32_t)T;
}

template <int T>
__device__ inline uint32_t block_scan_excl(uint32_t v, uint32_t *scr, uint32_t *total) {
    constexpr int TW = T / 64;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) scr[wave] = inc;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < TW; ++w) {
        const uint32_t c = scr[w];
        pre += (w < wave) ? c : 0u;
        tot += c;
    }
    __syncthreads();
    *total = tot;
    return pre + inc - v;
}

__device__ inline uint32_t count_of(const uint32_t *cnt32, uint32_t c) {
    return (cnt32[c >> 2] >> (8 * (c & 3))) & 255u;
}

template <typename CellT, int T>
__global__ __launch_bounds__(T) void threshold_kernel(TArgs A) {
    extern __shared__ __align__(16) uint32_t tl[];
    uint32_t *cnt32 = tl;
    uint32_t *misc = tl + A.cnt_words;
    uint32_t *npos = misc + T_NPOS;
    // list_words(): up to T positive cells of one round; before that, in the
    // fast path, its T_LIST cells, T_LIST positive cells of all repetitions
    // (then slots of the answer), and the tables' list ranges
    uint32_t *lb = npos + 16;
    uint32_t *plist = lb + T_LIST;
    uint32_t *pree = plist + T_LIST, *lst = pree + A.L;
    const int tid = threadIdx.x;
    const uint64_t q = blockIdx.x;
    if (q >= A.nq) return;
    const uint32_t L = A.L, R = A.R, B = A.B, Bp = A.Bp, t = A.t;
    const uint64_t nbk1 = (1ull << A.nbits) + 1;
    const CellT *cells = static_cast<const CellT *>(A.cells);

    // 1. list ranges, issued before the counters are cleared (a code outside the
    // table matches no bucket)
    uint32_t st = 0, en = 0;
    if ((uint32_t)tid < L) {
        const uint32_t h = A.codes[q * L + tid];
        if ((uint64_t)h + 1 < nbk1) {
            const uint32_t *o = A.offsets + (uint64_t)tid * nbk1 + h;
            st = o[0];
            en = o[1];
        }
    }
    for (uint32_t w = tid; w < A.cnt_words; w += T) cnt32[w] = 0u;
    if (tid < 16) npos[tid] = 0u;
    if (tid == 0) misc[T_TOTAL] = misc[T_NP] = misc[T_NL] = 0u;
    uint32_t nent;
    const uint32_t ex = block_scan_excl<T>(en - st, misc + T_SCAN, &nent);
    if ((uint32_t)tid < L) {
        pree[tid] = ex;
        lst[tid] = st - ex;
    }
    __syncthreads();
    auto count = [&](uint32_t c) {  // and note the cell when it becomes positive
        const uint32_t sh = 8 * (c & 3);
        const uint32_t n = ((atomicAdd(&cnt32[c >> 2], 1u << sh) >> sh) & 255u) + 1;
        if (n == t) {
            atomicAdd(&npos[c / Bp], 1u);
            const uint32_t at = atomicAdd(&misc[T_NP], 1u);
            if (at < T_LIST) plist[at] = c;
        }
    };
    // positive cells per repetition from the counters (a counter word holds four
    // cells of one repetition: Bp is a multiple of 4)
    auto count_positive = [&] {
        for (uint32_t w = tid; w < A.cnt_words; w += T) {
            const uint32_t v = cnt32[w];
            const uint32_t r = (4 * w) / Bp;
            if (r >= R) continue;
            uint32_t n = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t b = 4 * w + j - r * Bp;
                n += (b < B && ((v >> (8 * j)) & 255u) >= t) ? 1u : 0u;
            }
            if (n) atomicAdd(&npos[r], n);
        }
        __syncthreads();
    };
    const bool longl = nent >= L * (T / 4);
    if (longl) {
        // long lists: a table at a time, four loads in flight per thread, and the
        // positive cells from the counters afterwards (returning atomics on the
        // few cells of such a grid would wait for each other)
        for (uint32_t tb = 0; tb < L; ++tb) {
            const uint32_t j1 = tb + 1 < L ? pree[tb + 1] : nent;
            for (uint32_t j0 = pree[tb] + tid; j0 < j1; j0 += 4 * T) {
                uint32_t c[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) c[e] = j0 + e * T < j1 ? (uint32_t)cells[lst[tb] + j0 + e * T] : ~0u;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c[e] != ~0u) atomicAdd(&cnt32[c[e] >> 2], 1u << (8 * (c[e] & 3)));
            }
        }
    } else {
        for (uint32_t j0 = tid; j0 < nent; j0 += 4 * T) {
            uint32_t c[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t j = j0 + e * T;
                c[e] = ~0u;
                if (j < nent) {
                    uint32_t lo = 0, hi = L;  // the last table whose entries start at or before j
                    while (hi - lo > 1) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (pree[mid] <= j) lo = mid; else hi = mid;
                    }
                    c[e] = cells[lst[lo] + j];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c[e] != ~0u) count(c[e]);
        }
    }
    __syncthreads();
    if (longl || t == 0) count_positive();  // (at t = 0 the untouched cells too)
    uint32_t *out = A.ids + q * (uint64_t)A.max_out;
    const uint64_t rstride = (uint64_t)B * A.mstride;

    // 2. fast path: the positive cells of the repetition with the fewest fit the
    // list; they come from the noted ones if all were, else from its counters
    uint32_t rep = 0;
    for (uint32_t r = 1; r < R; ++r)
        if (npos[r] < npos[rep]) rep = r;
    // a member's groups beyond the enumerated repetition and the two of its filter
    // word (where the members' rows are read by the dozen, each group of one costs a
    // load over 16 cache lines: reading all R, 12,000 queries with every cell of 4 x
    // 100 positive took 1,742 us, the one that is left 519)
    auto others_positive = [&](const uint16_t *row) {
        bool ok = true;
        for (uint32_t i = 3, r = (rep + 3) % R; i < R; ++i, r = r + 1 < R ? r + 1 : 0)
            ok &= count_of(cnt32, r * Bp + row[r]) >= t;
        return ok;
    };
    // (with one repetition every member of a positive cell is reported: only if
    // they fit the answer's list, or all would be walked twice; 12,000 queries, 5
    // cells of 100, 164 us, 107 in order alone)
    if (t >= 1 && npos[rep] <= T_LIST && (npos[rep] <= FEW || npos[rep] * FEW <= B) &&
        A.small_slots && (R > 1 || npos[rep] * (uint64_t)A.mstride <= T_LIST)) {
        const uint32_t np = misc[T_NP];
        if (!longl && np <= T_LIST) {
            for (uint32_t i = tid; i < np; i += T) {
                const uint32_t b = plist[i] - rep * Bp;
                if (b < B) lb[atomicAdd(&misc[T_NL], 1u)] = b;
            }
        } else {
            for (uint32_t w = tid; w < Bp / 4; w += T) {
                const uint32_t v = cnt32[rep * (Bp / 4) + w];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (4 * w + j < B && ((v >> (8 * j)) & 255u) >= t)
                        lb[atomicAdd(&misc[T_NL], 1u)] = 4 * w + j;
            }
        }
        __syncthreads();
        const uint32_t nl = misc[T_NL];
        const uint32_t *memr = A.mem + rep * rstride, *cflr = A.cfl + rep * rstride;
        const uint16_t *cmgr = A.cmg + rep * rstride * A.Rp;
        const uint32_t f1b = ((rep + 1) % R) * Bp, f2b = ((rep + 2) % R) * Bp;
        // four cells in flight per wavefront, 256 member slots of each at a time
        for (uint32_t c0 = tid / 64 * 4; c0 < nl; c0 += T / 64 * 4) {
            for (uint32_t j0 = 0; j0 < A.mstride; j0 += 256) {
                const uint32_t j = j0 + 4 * (tid % 64);
                uint4 v[4];
                uint32_t s0[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool in = c0 + i < nl && j < A.mstride;
                    s0[i] = in ? lb[c0 + i] * A.mstride + j : ~0u;
                    v[i] = in ? *reinterpret_cast<const uint4 *>(cflr + s0[i]) : make_uint4(0, 0, 0, 0);
                }
                // members that pass the filter, then looked up one per lane and
                // round (bit 4i + e: member e of cell i)
                uint32_t pend = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t fw[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool pass = R < 2 || (count_of(cnt32, f1b + (fw[e] & 0xFFFFu)) >= t &&
                                                    count_of(cnt32, f2b + (fw[e] >> 16)) >= t);
                        if (pass && s0[i] != ~0u) pend |= 1u << (4 * i + e);
                    }
                }
                while (pend) {
                    const uint32_t m = (uint32_t)__builtin_ctz(pend);
                    pend &= pend - 1;
                    uint32_t sl = s0[0];
#pragma unroll
                    for (int i = 1; i < 4; ++i) sl = (m >> 2) == (uint32_t)i ? s0[i] : sl;
                    sl += m & 3u;
                    const uint16_t *row = cmgr + (uint64_t)sl * A.Rp;
                    bool in = memr[sl] != 0xFFFFFFFFu;  // not the cell's padding
                    in &= others_positive(row);
                    if (in) {
                        const uint32_t at = atomicAdd(&misc[T_TOTAL], 1u);
                        if (at < T_LIST) plist[at] = sl;  // the cells are in lb by now
                    }
                }
            }
        }
        __syncthreads();
        const uint32_t ns = misc[T_TOTAL];
        if (ns <= T_LIST) {
            for (uint32_t i = tid; i < ns; i += T) {
                const uint32_t sl = plist[i];
                uint32_t rank = 0;
                for (uint32_t j = 0; j < ns; ++j) rank += plist[j] < sl ? 1u : 0u;
                if (rank < A.max_out) out[rank] = memr[sl];
            }
            for (uint32_t j = ns + tid; j < A.max_out; j += T) out[j] = 0xFFFFFFFFu;
            if (tid == 0) A.counts[q] = ns;
            return;
        }
    }

    // the ordered walk over all cells of the repetition, four member slots per
    // thread (mstride is a multiple of four) and T threads at a time
    __syncthreads();
    const uint32_t *memr = A.mem + rep * rstride, *cflr = A.cfl + rep * rstride;
    const uint16_t *cmgr = A.cmg + rep * rstride * A.Rp;
    const uint32_t f1b = ((rep + 1) % R) * Bp, f2b = ((rep + 2) % R) * Bp;
    const uint32_t quads = A.mstride / 4;  // B * quads < 2^31: ids are 32 bits
    uint32_t total = 0;
    if (npos[rep] != 0) {
        for (uint32_t b0 = 0; b0 < B; b0 += T) {
            const uint32_t b = b0 + tid;
            const bool pos = b < B && count_of(cnt32, rep * Bp + b) >= t;
            uint32_t nl;
            const uint32_t at = block_scan_excl<T>(pos ? 1u : 0u, misc + T_SCAN, &nl);
            if (pos) lb[at] = b;
            __syncthreads();
            const uint32_t items = nl * quads;
            for (uint32_t i0 = 0; i0 < items; i0 += T) {
                const uint32_t i = i0 + tid;
                uint32_t x[4], in = 0;
                if (i < items) {
                    const uint32_t ci = i / quads;
                    const uint64_t slot = (uint64_t)lb[ci] * A.mstride + 4 * (i - ci * quads);
                    const uint4 m = *reinterpret_cast<const uint4 *>(memr + slot);
                    const uint4 v = *reinterpret_cast<const uint4 *>(cflr + slot);
                    const uint32_t fw[4] = {v.x, v.y, v.z, v.w};
                    x[0] = m.x, x[1] = m.y, x[2] = m.z, x[3] = m.w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        bool ok = x[e] != 0xFFFFFFFFu &&  // not the cell's padding
                                  (R < 2 || (count_of(cnt32, f1b + (fw[e] & 0xFFFFu)) >= t &&
                                             count_of(cnt32, f2b + (fw[e] >> 16)) >= t));
                        if (ok && R > 3) ok = others_positive(cmgr + (slot + e) * A.Rp);
                        in |= ok ? 1u << e : 0u;
                    }
                }
                uint32_t nnew;
                uint32_t p = total + block_scan_excl<T>((uint32_t)__popc(in), misc + T_SCAN, &nnew);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (in >> e & 1u) {
                        if (p < A.max_out) out[p] = x[e];
                        ++p;
                    }
                total += nnew;
            }
        }
    }
    for (uint32_t j = total + tid; j < A.max_out; j += T) out[j] = 0xFFFFFFFFu;
    if (tid == 0) A.counts[q] = total;
}

}  // namespace

size_t threshold_lds_bytes(const Index &ix, int T) {
    const uint32_t Bp = (ix.p.B + 3) & ~3u;
    const size_t cnt_words = ((size_t)ix.p.R * Bp / 4 + 3) & ~(size_t)3;
    return (cnt_words + T_NPOS + 16 + list_words(T, ix.p.L)) * 4;
}

void threshold_launch(const Index &ix, const uint32_t *codes_dev, uint64_t nq, uint32_t t,
                      uint32_t max_out, uint32_t *ids_dev, uint32_t *counts_dev, hipStream_t s) {
    if (nq == 0) return;
    if (nq > 0x7FFFFFFFull) fail(FLINNG_EINVAL, "query batch too large for one launch");
    TArgs a{};
    a.codes = codes_dev;
    a.nq = nq;
    a.offsets = ix.offsets;
    a.cells = ix.cells;
    a.mem = ix.mem;
    a.cmg = ix.cmg;
    a.cfl = ix.cfl;
    a.small_slots = (uint64_t)ix.p.B * ix.mstride < (1ull << 32);
    a.L = ix.p.L;
    a.R = ix.p.R;
    a.Rp = ix.Rp;
    a.B = ix.p.B;
    a.Bp = (ix.p.B + 3) & ~3u;
    a.nbits = ix.nbits;
    a.t = t;
    a.max_out = max_out;
    a.mstride = ix.mstride;
    a.cnt_words = (uint32_t)((((size_t)a.R * a.Bp) / 4 + 3) & ~(size_t)3);
    a.ids = ids_dev;
    a.counts = counts_dev;
    int dev = 0;
    FL_HIP(hipGetDevice(&dev));
    int max_lds = 0;
    FL_HIP(hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    const bool big = threshold_lds_bytes(ix, 256) > 32 * 1024;
    const size_t lds = threshold_lds_bytes(ix, big ? 1024 : 256);
    if (lds > (size_t)max_lds)
        fail(FLINNG_EINVAL, "per-query counters (" + std::to_string(lds) +
                                " bytes) exceed the workgroup LDS limit; reduce B*R");
    auto go = [&](auto kern, int T) {
        FL_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, max_lds));
        hipLaunchKernelGGL(kern, dim3((unsigned)nq), dim3(T), lds, s, a);
        FL_CHECK_LAUNCH();
    };
    if (ix.cell_bytes == 2) {
        if (big) go(threshold_kernel<uint16_t, 1024>, 1024);
        else go(threshold_kernel<uint16_t, 256>, 256);
    } else {
        if (big) go(threshold_kernel<uint32_t, 1024>, 1024);
        else go(threshold_kernel<uint32_t, 256>, 256);
    }
}

}  // namespace flinng
