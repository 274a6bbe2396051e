// The query kernel for queries that touch few of the grid's cells.
//
// The general kernel (query.hip) keeps a byte of LDS per cell of the grid:
// 64 KiB to 128 KiB for grids of 2^16 and 2^17 cells, hence one workgroup per
// compute unit, which waits out every dependent read of its one query.  A
// query that meets a few thousand list entries can only touch that many
// cells, so here its counters are a bit per cell (touched or not), a running
// count of the touched cells per 32-cell word, and one byte per touched cell,
// found at the word's running count plus the set bits below the cell's:
// exact, without collisions, in a sixth of the space.  Several workgroups then
// share a compute unit and hide each other's waits.  Everything else is the
// general kernel's: the same levels, passes, keys and results.
//
//   1. the L list ranges; a query with more than T*E entries is left to the
//      general kernel (its first id is set to DEFERRED);
//   2. up to E entries per thread, kept in registers: set their cells' bits;
//   3. running counts of the set bits;
//   4. the entries again: count in the touched cells' bytes, and add to the
//      count-at-least histogram of the cell's repetition;
//   5. level and decode passes.  A pass lists its repetition's cells of count
//      >= level from the bitmap, and walks their members' filter words in
//      items of 4 << ils slots, 1 << ils lanes each, ils fitted to the cell
//      size, one round of loads ahead (a cell's padding slots hold no id and
//      drop out with the filter's other rejects, so no size is read).  A
//      member passes when its cells in repetitions r+1 and r+2 are touched:
//      two bit tests, which reject nearly as many members as their counts
//      would.  The few that pass go to a queue of the wavefront in LDS and are
//      looked up 64 at a time, whatever lanes and rounds they came from;
//   6. the wavefronts' nonempty top-k entries are packed together: at most 64
//      in nearly every query, sorted and written out by one wavefront.
//
// What bounds it: vector instructions and the chain of dependent reads; for
// 10,000 ReLU queries the vector units are busy 72% of 357 us (803 us in the
// general kernel), the LDS 38%.  Held to 64 registers for eight wavefronts per
// SIMD, it spills 20, 56 and 144 bytes per lane at Rp = 4, 8 and 16 (none at 1
// and 2): of the 1.45 GB that those queries move (4 TB/s), 0.26 GB are such
// stores and 0.66 GB what the kernel asks for.  10,000 URL queries, 8 x 16,384
// cells: 416 us (general 1,138) and 1.5 GB.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "query_common.h"

namespace flinng {

namespace {

// listed cells per pass (a pass with more goes to the general kernel): no more
// than the query's entries, and at most 2048
constexpr uint32_t sp_list(int T, int E) { return T * E < 2048 ? T * E : 2048u; }

struct SLayout {
    uint32_t wp;      // 32-cell words of one repetition
    uint32_t rep_mul; // cell position / (32 wp) = umulhi(position, rep_mul) >> 4
    uint32_t words;   // of all repetitions, rounded up to a multiple of 4
    uint32_t off_pf, off_cn, off_hist, off_pree, off_lst, off_ms, off_lb, off_wl, off_wq, off_misc, total;
};

SLayout sp_layout(uint32_t L, uint32_t R, uint32_t Bp, uint32_t k, int T, int E) {
    SLayout l;
    l.wp = (Bp + 31) / 32;
    // ceil(2^36 / (32 wp)) < 2^32; exact for positions below 2^18 >= 32 wp
    l.rep_mul = (uint32_t)(((1ull << 36) + 32ull * l.wp - 1) / (32ull * l.wp));
    l.words = (R * l.wp + 3) / 4 * 4;
    uint32_t o = l.words * 4;
    auto piece = [&](uint32_t bytes) { const uint32_t at = o; o += (bytes + 15) & ~15u; return at; };
    l.off_pf = piece(l.words * 2);
    l.off_cn = piece((uint32_t)T * E + 4);
    l.off_hist = piece(R * (L + 1) * 4);
    l.off_pree = piece((L + 1) * 4);
    l.off_lst = piece(L * 4);
    l.off_ms = piece((L + 1) * 4);
    l.off_lb = piece(sp_list(T, E) * 2);
    l.off_wl = piece((1 + (uint32_t)T / 64) * k * 8);
    l.off_wq = piece((uint32_t)T / 64 * WALK_QUEUE * 4);
    l.off_misc = piece(64 * 4);
    l.total = o;
    return l;
}

template <typename CellT, int RP, int T, int E>
__global__ __launch_bounds__(T, 8) void sparse_query_kernel(QArgs A, SLayout lay) {
    constexpr int QW = T / 64;
    constexpr int U = 2;  // filter items in flight per lane
    extern __shared__ __align__(16) unsigned char lds[];
    uint32_t *bm = reinterpret_cast<uint32_t *>(lds);
    uint16_t *pf = reinterpret_cast<uint16_t *>(lds + lay.off_pf);
    uint32_t *cn32 = reinterpret_cast<uint32_t *>(lds + lay.off_cn);
    const uint8_t *cn8 = lds + lay.off_cn;
    uint32_t *hist = reinterpret_cast<uint32_t *>(lds + lay.off_hist);
    uint32_t *pree = reinterpret_cast<uint32_t *>(lds + lay.off_pree);
    uint32_t *lst = reinterpret_cast<uint32_t *>(lds + lay.off_lst);
    uint32_t *ms = reinterpret_cast<uint32_t *>(lds + lay.off_ms);
    uint16_t *lb = reinterpret_cast<uint16_t *>(lds + lay.off_lb);
    uint64_t *buf = reinterpret_cast<uint64_t *>(lds + lay.off_wl);
    uint32_t *wq = reinterpret_cast<uint32_t *>(lds + lay.off_wq) + threadIdx.x / 64 * WALK_QUEUE;
    uint32_t *misc = reinterpret_cast<uint32_t *>(lds + lay.off_misc);
    uint32_t *scr = misc + M_SCAN0;

    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const uint32_t L = A.L, R = A.R, B = A.B, Bp = A.Bp, k = A.k;
    const uint64_t q = blockIdx.x;
    uint32_t *oid = A.ids + q * (uint64_t)k;
    uint32_t *osc = A.scores ? A.scores + q * (uint64_t)k : nullptr;

    // ---- 1. list ranges (issued first, in flight while the state is cleared)
    uint32_t st = 0, en = 0;
    if ((uint32_t)tid < L) {
        // a code outside the table (caller-supplied codes) matches no bucket
        const uint64_t nbk1 = (1ull << A.nbits) + 1;
        const uint32_t h = A.codes[q * L + tid];
        if ((uint64_t)h + 1 < nbk1) {
            const uint32_t *o = A.offsets + (uint64_t)tid * nbk1 + h;
            st = o[0];
            en = o[1];
        }
    }
    {
        const uint4 z = make_uint4(0u, 0u, 0u, 0u);
        uint4 *b4 = reinterpret_cast<uint4 *>(bm), *c4 = reinterpret_cast<uint4 *>(cn32);
        for (uint32_t w = tid; w < lay.words / 4; w += T) b4[w] = z;
        for (uint32_t w = tid; w < (T * E + 19) / 16; w += T) c4[w] = z;
        for (uint32_t w = tid; w < R * (L + 1); w += T) hist[w] = 0u;
    }
    if (tid == 0) {
        misc[M_THI] = 0;
        misc[M_NEXT] = 0;
        misc[M_ST_ALL] = 0;
        misc[M_ST_PASSES] = 0;
    }
    const uint32_t ne = en - st;
    if (L <= 64) {
        if (wave == 0) {
            uint32_t inc = ne;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = (uint32_t)__shfl_up((int)inc, o, 64);
                if (lane >= o) inc += y;
            }
            if ((uint32_t)lane < L) {
                pree[lane] = inc - ne;
                lst[lane] = st - (inc - ne);
            }
            if (lane == 63) pree[L] = inc;  // lanes past L add nothing
        }
    } else {
        uint32_t total;
        const uint32_t ex = wg_excl_scan<T>(ne, scr, &total);
        if ((uint32_t)tid < L) {
            pree[tid] = ex;
            lst[tid] = st - ex;
        }
        if (tid == 0) pree[L] = total;
    }
    __syncthreads();
    const uint32_t nent = __builtin_amdgcn_readfirstlane(pree[L]);
    if (nent > T * E) {
        if (tid == 0) oid[0] = DEFERRED;
        return;
    }

    // ---- 2. entries: entry j = e*T + tid lies in the last table with
    // pree[t] <= j (the searches of a thread's entries run side by side)
    uint32_t c[E];
    {
        uint32_t lo[E];
#pragma unroll
        for (int e = 0; e < E; ++e) lo[e] = 0;
        for (uint32_t step = A.lstep; step; step >>= 1) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if (e * T < nent) {
                    const uint32_t m = lo[e] + step;
                    if (m < L && pree[m] <= (uint32_t)(e * T + tid)) lo[e] = m;
                }
            }
        }
        const CellT *cells = static_cast<const CellT *>(A.cells);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            c[e] = ~0u;
            if (e * T < nent) {
                const uint32_t j = e * T + tid;
                if (j < nent) c[e] = cells[lst[lo[e]] + j];
            }
        }
    }
    // cell (r, b)'s position in the bitmap: 32 wp r + b (each repetition starts
    // a word, so that a group id alone gives the bit)
    const uint32_t rbits = 32 * lay.wp, rpad = rbits - Bp;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e * T < nent && c[e] != ~0u) {
            if (rpad) c[e] += div_small(c[e], Bp, A.inv_bp) * rpad;
            atomicOr(&bm[c[e] >> 5], 1u << (c[e] & 31));
        }
    }
    __syncthreads();

    // ---- 3. running counts of the touched cells per word
    {
        const uint32_t n4 = lay.words / 4, per = (n4 + T - 1) / T;
        const uint4 *b4 = reinterpret_cast<const uint4 *>(bm);
        uint32_t s = 0;
        for (uint32_t i = 0; i < per; ++i) {
            const uint32_t w = tid * per + i;
            if (w < n4) {
                const uint4 v = b4[w];
                s += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
            }
        }
        uint32_t total;
        uint32_t at = wg_excl_scan<T>(s, scr, &total);
        for (uint32_t i = 0; i < per; ++i) {
            const uint32_t w = tid * per + i;
            if (w < n4) {
                const uint4 v = b4[w];
                const uint32_t a1 = at + __popc(v.x), a2 = a1 + __popc(v.y), a3 = a2 + __popc(v.z);
                reinterpret_cast<uint2 *>(pf)[w] = make_uint2(at | (a1 << 16), a2 | (a3 << 16));
                at = a3 + __popc(v.w);
            }
        }
    }
    __syncthreads();

    // ---- 4. counts and count-at-least histograms
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e * T < nent && c[e] != ~0u) {
            const uint32_t w = c[e] >> 5;
            const uint32_t i = pf[w] + __popc(bm[w] & ((1u << (c[e] & 31)) - 1u));
            const uint32_t sh = 8 * (i & 3);
            const uint32_t ob = (atomicAdd(&cn32[i >> 2], 1u << sh) >> sh) & 255u;
            const uint32_t r = __umulhi(c[e], lay.rep_mul) >> 4;
            atomicAdd(&hist[r * (L + 1) + ob + 1], 1u);
        }
    }
    __syncthreads();
    // ---- 5. level (as in the general kernel): ms[t] = the fewest cells of
    // count >= t over the repetitions; level t belongs to thread t - 1
    {
        const uint32_t t = 1 + tid;
        uint64_t sz = 0;
        if (t <= L) {
            uint32_t mn = 0xFFFFFFFFu;
            for (uint32_t r = 0; r < R; ++r) {
                const uint32_t n = hist[r * (L + 1) + t];
                mn = n < mn ? n : mn;
            }
            ms[t] = mn;
            sz = (uint64_t)mn * A.gmax;
        }
        const unsigned long long mh = __ballot(t <= L && sz >= k);
        const unsigned long long ml = __ballot(t <= L && sz <= A.budget);
        uint32_t thi, tlo;
        if (L <= 64) {
            thi = (uint32_t)__popcll(mh);  // every level is in wavefront 0
            tlo = L + 1 - (uint32_t)__popcll(ml);
        } else {
            if (lane == 0 && (uint32_t)wave * 64 < L) {
                atomicAdd(&misc[M_THI], (uint32_t)__popcll(mh));
                atomicAdd(&misc[M_NEXT], (uint32_t)__popcll(ml));
            }
            __syncthreads();
            thi = misc[M_THI];
            tlo = L + 1 - misc[M_NEXT];
        }
        if (tid == 0) misc[M_LEVEL] = (thi == 0) ? 0u : (tlo <= thi ? tlo : thi);
    }

    const uint64_t rstride = (uint64_t)B * A.mstride;  // below 2^32 (the launcher checks)
    for (;;) {
        if (tid == 0) {
            uint32_t level = misc[M_LEVEL], rep = R - 1, keep = 1;
            if (level == 0) {
                level = 1;
            } else {
                uint32_t best = 0xFFFFFFFFu;
                for (uint32_t r = 0; r < R; ++r) {
                    const uint32_t n = hist[r * (L + 1) + level];
                    if (n < best) {
                        best = n;
                        rep = r;
                    }
                }
                // R = 1: one pass keeping every key serves both outcomes
                keep = level == 1 && R < 2 && (uint64_t)best * A.gmax <= 2ull * A.budget;
            }
            misc[M_LEVEL] = level;
            misc[M_REP] = rep;
            misc[M_KEEPALL] = keep;
            misc[M_BUFN] = 0;
            misc[M_NGE] = 0;
            misc[M_NALL] = 0;
            misc[M_LCNT] = 0;
            misc[M_MEMB] = 0;
            misc[M_GATH] = 0;
        }
        __syncthreads();
        const uint32_t level = __builtin_amdgcn_readfirstlane(misc[M_LEVEL]);
        const uint32_t rep = __builtin_amdgcn_readfirstlane(misc[M_REP]);
        const bool keep = __builtin_amdgcn_readfirstlane(misc[M_KEEPALL]) != 0;
        const uint32_t nl = __builtin_amdgcn_readfirstlane(hist[rep * (L + 1) + level]);
        if (nl > sp_list(T, E)) {
            if (tid == 0) oid[0] = DEFERRED;
            return;
        }
        for (uint32_t w = tid; w < lay.wp; w += T) {
            const uint32_t v = bm[rep * lay.wp + w];
            for (uint32_t m = v; m; m &= m - 1) {
                const uint32_t b = (uint32_t)__builtin_ctz(m);
                if (level > 1 && cn8[pf[rep * lay.wp + w] + __popc(v & ((1u << b) - 1u))] < level) continue;
                lb[atomicAdd(&misc[M_LCNT], 1u)] = (uint16_t)(32 * w + b);
            }
        }
        __syncthreads();

        // ---- walk
        WaveState ws{~0ull, ~0ull, 0u, 0u, 0u, 0u};
        {
            const uint32_t *memr = A.mem + rep * rstride;
            const uint16_t *cmgr = A.cmg + rep * rstride * RP;
            const uint32_t *cflr = A.cfl + rep * rstride;
            const uint32_t *bm1 = bm + ((rep + 1) % R) * lay.wp, *bm2 = bm + ((rep + 2) % R) * lay.wp;
            const bool filt = !keep && R >= 2;
            walk_items<RP, QW, U>(
                lb, nl, memr, cmgr, filt ? cflr : nullptr, R, Bp, A, level, keep, wq, lane, wave, ws,
                [&](uint32_t w) {
                    // the shifts are by a group id's low five bits, its bit in
                    // its repetition's words
                    const uint32_t g2 = w >> 16;
                    return ((bm1[(w & 0xFFFFu) >> 5] >> (w & 31)) & (bm2[g2 >> 5] >> (g2 & 31)) & 1u) != 0;
                },
                [&](uint32_t r, uint32_t b) {
                    const uint32_t w = r * lay.wp + (b >> 5), v = bm[w];
                    const uint32_t n = cn8[pf[w] + __popc(v & ((1u << (b & 31)) - 1u))];
                    return (v >> (b & 31)) & 1u ? 255u - n : 255u;
                });
        }
        if (A.stats) {  // members of the listed cells
            uint32_t n = 0;
            for (uint32_t i = tid; i < nl; i += T) n += A.gsize[rep * B + lb[i]];
            atomicAdd(&misc[M_MEMB], n);
        }

        // ---- 6. the wavefronts' kept keys, packed
        uint64_t *wlist = buf + k;
        const unsigned long long have = __ballot(ws.wl != ~0ull);  // lanes 0 .. n-1
        uint32_t at = 0;
        if (lane == 0) {
            if (have) at = atomicAdd(&misc[M_BUFN], (uint32_t)__popcll(have));
            if (ws.n_ge) atomicAdd(&misc[M_NGE], ws.n_ge);
            if (ws.n_all) atomicAdd(&misc[M_NALL], ws.n_all);
            if (A.stats) atomicAdd(&misc[M_GATH], ws.gathered);
        }
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        if (ws.wl != ~0ull) wlist[at + lane] = ws.wl;
        __syncthreads();
        const uint32_t nge = misc[M_NGE], nall = misc[M_NALL], nk = misc[M_BUFN];
        if (tid == 0) {
            misc[M_ST_ALL] += misc[M_MEMB];
            misc[M_ST_PASSES] += 1;
        }
        if (nge >= k || keep) {
            const uint32_t nres = nall < k ? nall : k;
            if (nk <= 64) {
                if (wave != 0) return;
                const uint64_t v = wave_sort64((uint32_t)lane < nk ? wlist[lane] : ~0ull, lane);
                if ((uint32_t)lane < nres) {
                    oid[lane] = (uint32_t)v;
                    if (osc) osc[lane] = 255u - (uint32_t)(v >> 56);
                }
            } else {
                // rank = the keys below this one (keys are distinct)
                for (uint32_t i = tid; i < nk; i += T) {
                    const uint64_t key = wlist[i];
                    uint32_t rank = 0;
                    for (uint32_t j = 0; j < nk; ++j) rank += wlist[j] < key ? 1u : 0u;
                    if (rank < nres) {
                        oid[rank] = (uint32_t)key;
                        if (osc) osc[rank] = 255u - (uint32_t)(key >> 56);
                    }
                }
                if (wave != 0) return;
            }
            if (nge < k && nres < k) {
                // zero fill from repetition R-1, cells ascending, ids ascending
                uint32_t need = k - nres, outp = nres;
                const uint32_t *memz = A.mem + (R - 1) * rstride;
                for (uint32_t b0 = 0; b0 < B && need; b0 += 64) {
                    const uint32_t b = b0 + lane;
                    const bool z = b < B && !((bm[(R - 1) * lay.wp + (b >> 5)] >> (b & 31)) & 1u);
                    unsigned long long zm = __ballot(z);
                    while (zm && need) {
                        const uint32_t bb = b0 + (uint32_t)(__ffsll((long long)zm) - 1);
                        zm &= zm - 1;
                        const uint32_t sz = A.gsize[(R - 1) * B + bb];
                        const uint32_t takeN = sz < need ? sz : need;
                        const uint64_t mo = (uint64_t)bb * A.mstride;
                        for (uint32_t j = lane; j < takeN; j += 64) {
                            oid[outp + j] = memz[mo + j];
                            if (osc) osc[outp + j] = 0u;
                        }
                        outp += takeN;
                        need -= takeN;
                    }
                }
                for (uint32_t j = outp + lane; j < k; j += 64) {
                    oid[j] = 0xFFFFFFFFu;
                    if (osc) osc[j] = 0u;
                }
            }
            if (A.stats && tid == 0) {
                atomicAdd(&A.stats[0], (unsigned long long)nent);
                atomicAdd(&A.stats[1], (unsigned long long)misc[M_ST_ALL]);
                atomicAdd(&A.stats[2], (unsigned long long)misc[M_MEMB]);
                atomicAdd(&A.stats[3], (unsigned long long)misc[M_ST_PASSES]);
                atomicAdd(&A.stats[4], (unsigned long long)misc[M_GATH]);
            }
            return;
        }
        // lower the level: the lowest level whose cheapest enumeration stays
        // within 8x the larger of the budget and this pass
        const uint32_t lv = misc[M_LEVEL];
        const uint64_t lim = 8ull * (A.budget > nall ? A.budget : nall);
        __syncthreads();
        if (tid == 0) misc[M_NEXT] = 0;
        __syncthreads();
        {
            const uint32_t t = 1 + tid;
            const unsigned long long ml = __ballot(t <= L && (uint64_t)ms[t] * A.gmax <= lim);
            if (lane == 0 && (uint32_t)wave * 64 < L) atomicAdd(&misc[M_NEXT], (uint32_t)__popcll(ml));
        }
        __syncthreads();
        if (tid == 0) {
            const uint32_t t1 = L + 1 - misc[M_NEXT];
            misc[M_LEVEL] = (t1 < lv) ? t1 : lv - 1;  // 0 selects the fill path
        }
        __syncthreads();
    }
}

template <typename CellT, int RP, int T, int E>
void launch_one(const QArgs &a, const SLayout &l, hipStream_t s) {
    hipLaunchKernelGGL((sparse_query_kernel<CellT, RP, T, E>), dim3((unsigned)a.nq), dim3(T), l.total, s,
                       a, l);
    FL_CHECK_LAUNCH();
}

template <typename CellT, int T, int E>
void launch_rp(const QArgs &a, const SLayout &l, hipStream_t s) {
    switch (a.Rp) {
        case 1: launch_one<CellT, 1, T, E>(a, l, s); break;
        case 2: launch_one<CellT, 2, T, E>(a, l, s); break;
        case 4: launch_one<CellT, 4, T, E>(a, l, s); break;
        case 8: launch_one<CellT, 8, T, E>(a, l, s); break;
        default: launch_one<CellT, 16, T, E>(a, l, s); break;
    }
}

template <int T, int E>
void launch_te(QArgs &a, uint32_t cell_bytes, hipStream_t s) {
    const SLayout l = sp_layout(a.L, a.R, a.Bp, a.k, T, E);
    if (cell_bytes == 2) launch_rp<uint16_t, T, E>(a, l, s);
    else launch_rp<uint32_t, T, E>(a, l, s);
}

}  // namespace

// Which variant serves an index, by the list entries that a query distributed
// like its points meets: a workgroup of T threads takes queries of up to T*E
// entries, so the mean is kept below 0.4 of that (few queries pass it; 0.6 for
// the largest, where the general kernel is the alternative).  The smallest that
// does is the fastest: 10,000 reads with 74 entries each take 86 us in 128
// threads, 89 in 64, 109 in 256, and 92 in the general kernel; URL strings with
// 1,193 entries 411 us in 256 threads, 455 in 512, general 1,138; ReLU
// embeddings with 3,227 entries 368 us in 512 threads, 560 in 256 (a sixth of
// the queries deferred), general 803.  Not for
//   - general k (k > 64), or L beyond the workgroup;
//   - grids whose general kernel has 256 threads (its counters are small) and
//     queries that touch a good part of them: 4,096 cells at 8,901 entries
//     take 92 us in the general kernel and were twice that here; nor where they
//     touch more than an eighth of them (10,000 queries, k = 10, 192 entries in
//     400 cells 146 us general, 161 here; 5,000, 180 in 900 cells, 65 and 77;
//     180 in 2,000 cells 66 and 52);
//   - batches that the general kernel takes in one or two rounds of workgroups
//     (eight on a compute unit of 256 threads, one of 1024): the slowest query
//     is then most of what there is to wait for, and the second launch (5-6 us to
//     find nothing deferred) only adds to it;
//   - batches whose launch, a workgroup per query, would have 2^32 threads: the
//     runtime refuses such a grid, the persistent one takes any batch.
int sparse_variant(const Index &ix, const QArgs &a) {
    if (a.k > 64 || (uint64_t)a.B * a.mstride >= (1ull << 32) || a.gmax > 65536) return 0;
    if (a.nq < (a.threads == 1024 ? 384 : 4096)) return 0;
    const double m = ix.mean_entries;
    auto fits = [&](int threads) { return a.nq * threads < (1ull << 32); };
    if (a.threads != 1024 && m * 8 > (double)a.R * a.B) return 0;
    if (m <= 0.4 * 1024 && a.L <= 128) return fits(128) ? 1 : 0;
    if (a.threads != 1024) return 0;
    if (m <= 0.4 * 4096) return fits(256) ? 2 : 0;
    if (m <= 0.6 * 8192) return fits(512) ? 3 : 0;
    return 0;
}

void sparse_query_launch(const Index &ix, int variant, QArgs a, hipStream_t s) {
    a.lstep = 1;
    while (a.lstep * 2 < a.L) a.lstep *= 2;
    switch (variant) {
        case 1: launch_te<128, 8>(a, ix.cell_bytes, s); break;
        case 2: launch_te<256, 16>(a, ix.cell_bytes, s); break;
        default: launch_te<512, 16>(a, ix.cell_bytes, s); break;
    }
}

}  // namespace flinng
