// Wavefront helpers shared by the query kernels: scans, sorts, and the
// register top-k list.
#pragma once
#include <hip/hip_runtime.h>

#include "flinng_internal.h"

namespace flinng {

struct QArgs {
    const uint32_t *codes;
    uint64_t nq;
    const uint32_t *offsets;
    const void *cells;
    const uint32_t *mem;   // [R][B][mstride] member ids
    const uint16_t *cmg;   // [R][B][mstride][Rp] member group rows
    const uint32_t *cfl;   // [R][B][mstride] groups in repetitions r+1, r+2
    uint64_t N;
    const uint32_t *gsize; // [R][B] members of each cell
    uint32_t gmax;         // the largest cell
    uint32_t L, R, Rp, B, Bp, nbits, k, cap;
    uint32_t mstride;      // member slots per cell (multiple of 4)
    uint32_t threads;      // workgroup size the kernel is launched with
    uint32_t hc;           // histogram copies (a power of two)
    float inv_bp;          // 1 / Bp, for cell id -> repetition
    uint32_t *ids;
    uint32_t *scores;
    uint8_t *counts_out;   // debug: write counters and skip decode
    uint32_t *work;        // persistent grid: next query counter
    bool deferred;         // persistent grid: take the queries that the sparse
                           // kernel passed on instead (DEFERRED in ids[q*k])
    uint32_t budget;
    unsigned long long *stats;  // optional per-launch totals: list entries read,
                                // members read (all passes), members read in
                                // final passes, passes, group rows read in
                                // final passes
    // walk items of 4 << ils members, cpc of them per cell (walk_items)
    uint32_t ils, cpc, cpc_mul;
    uint32_t lstep;  // the largest power of two below L (1 for L = 1)
};

// In the first id of a query: the sparse kernel left it to the general one, and
// a workgroup of that has taken it (no point has these ids, and the first id of
// an answered query is a point's).
constexpr uint32_t DEFERRED = 0xFFFFFFFFu, CLAIMED = 0xFFFFFFFEu;

// misc slots
enum { M_Q = 0, M_BUFN, M_NGE, M_NALL, M_LEVEL, M_REP, M_KEEPALL, M_NEXT, M_LCNT, M_MEMB,
       M_THI, M_ST_ALL, M_ST_FINAL, M_ST_PASSES, M_NT, M_GATH,
       M_ST_GATH, M_SCAN0 };

// c / d for c < 2^24 and d >= 1, from the float quotient (within one of the
// true quotient: c is exact in float and the two roundings of c * (1/d)
// perturb it by less than one for d >= 2; d = 1 is exact) and one correction.
// A copy of a lane-dependent value that the compiler cannot merge with the
// original: an LDS address derived from it is then recomputed where it is
// used instead of being kept live (and spilled) across the whole query.
__device__ inline uint32_t fresh_copy(uint32_t x) {
    uint32_t y;
    asm volatile("v_mov_b32 %0, %1" : "=v"(y) : "v"(x));
    return y;
}

__device__ inline uint32_t div_small(uint32_t c, uint32_t d, float inv) {
    uint32_t q = (uint32_t)((float)c * inv);
    const int32_t rr = (int32_t)(c - q * d);
    return rr < 0 ? q - 1 : (rr >= (int32_t)d ? q + 1 : q);
}

template <int T>
__device__ inline uint32_t wg_excl_scan(uint32_t v, uint32_t *scr, uint32_t *total) {
    constexpr int TW = T / 64;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) scr[wave] = inc;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < TW; ++w) {
        uint32_t c = scr[w];
        pre += (w < wave) ? c : 0u;
        tot += c;
    }
    __syncthreads();
    *total = tot;
    return pre + inc - v;
}

__device__ inline uint64_t shfl64(uint64_t v, int src) {
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src, 64);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src, 64);
    return ((uint64_t)hi << 32) | lo;
}
__device__ inline uint64_t shfl64_up1(uint64_t v) {
    const uint32_t lo = (uint32_t)__shfl_up((int)(uint32_t)v, 1, 64);
    const uint32_t hi = (uint32_t)__shfl_up((int)(uint32_t)(v >> 32), 1, 64);
    return ((uint64_t)hi << 32) | lo;
}

// Per-wavefront decode state: its top-k list (lane i holds the i-th smallest
// key), the k-th key, and tallies (uniform across the wavefront).
struct WaveState {
    uint64_t wl, kth;
    uint32_t n_ge, n_all, members, gathered;
};

// Broadcast a 64-bit value from one lane (src uniform across the wavefront).
__device__ inline uint64_t bcast64(uint64_t v, int src) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, src);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}

// The value of lane (lane ^ J) (every lane active): quad permutations and a
// row rotation by 8 move data within the VALU (DPP); the other distances go
// through the LDS crossbar (swizzle within 32 lanes, permute across halves).
template <int J>
__device__ inline uint32_t lane_xor(uint32_t v, int lane) {
    if constexpr (J == 1) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);  // quad [1,0,3,2]
    } else if constexpr (J == 2) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);  // quad [2,3,0,1]
    } else if constexpr (J == 8) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, false);  // row rotate 8
    } else if constexpr (J < 32) {
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (J << 10) | 0x1F);  // xor J, 32-lane groups
    } else {
        return (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ J) << 2, (int)v);
    }
}

// One compare-exchange step of a bitonic sort across the wavefront: lanes
// l and l ^ J exchange so that the lower lane keeps the smaller key in
// ascending blocks (bit S of l clear) and the larger one in descending
// blocks.
// Lanes l of a wavefront with bit S of l equal to bit J of l, as a mask
// (a compile-time constant, rematerialised where it is used).
constexpr unsigned long long keep_min_mask(int S, int J) {
    unsigned long long m = 0;
    for (int l = 0; l < 64; ++l)
        if (((l & S) == 0) == ((l & J) == 0)) m |= 1ull << l;
    return m;
}

template <int S, int J>
__device__ inline uint64_t bitonic_step(uint64_t v, int lane) {
    const uint32_t plo = lane_xor<J>((uint32_t)v, lane);
    const uint32_t phi = lane_xor<J>((uint32_t)(v >> 32), lane);
    const uint64_t p = ((uint64_t)phi << 32) | plo;
    // take the partner's key where it is smaller in a keep-min lane, or
    // larger in a keep-max lane
    constexpr unsigned long long km = keep_min_mask(S, J);
    const unsigned long long take = ~(__ballot(p < v) ^ km);
    return __builtin_amdgcn_inverse_ballot_w64(take) ? p : v;
}

// Sort one key per lane ascending across the 64 lanes (every lane active).
__device__ inline uint64_t wave_sort64(uint64_t v, int lane) {
    v = bitonic_step<2, 1>(v, lane);
    v = bitonic_step<4, 2>(v, lane);
    v = bitonic_step<4, 1>(v, lane);
    v = bitonic_step<8, 4>(v, lane);
    v = bitonic_step<8, 2>(v, lane);
    v = bitonic_step<8, 1>(v, lane);
    v = bitonic_step<16, 8>(v, lane);
    v = bitonic_step<16, 4>(v, lane);
    v = bitonic_step<16, 2>(v, lane);
    v = bitonic_step<16, 1>(v, lane);
    v = bitonic_step<32, 16>(v, lane);
    v = bitonic_step<32, 8>(v, lane);
    v = bitonic_step<32, 4>(v, lane);
    v = bitonic_step<32, 2>(v, lane);
    v = bitonic_step<32, 1>(v, lane);
    v = bitonic_step<64, 32>(v, lane);
    v = bitonic_step<64, 16>(v, lane);
    v = bitonic_step<64, 8>(v, lane);
    v = bitonic_step<64, 4>(v, lane);
    v = bitonic_step<64, 2>(v, lane);
    v = bitonic_step<64, 1>(v, lane);
    return v;
}

// Insert the keys of the lanes in `tk` into the wavefront's sorted top-k
// list, all at once (called with every lane of the wavefront active; keys
// are distinct).  Into an empty list many candidates are sorted across the
// wavefront and the first k kept, a few are ranked among themselves and
// permuted to their ranks.  Otherwise each candidate below the k-th key is
// broadcast in turn (readlane) and its place in the merged order found by
// ballot (its rank among the list plus its rank among the candidates); the
// places taken form a lane mask and each place notes its candidate.  Then
// each lane pulls its new entry: the candidate's key, or the list entry
// shifted up by the candidates placed before it.
__device__ inline bool wave_insert(WaveState &ws, uint64_t key, unsigned long long tk, uint32_t k,
                                   int lane) {
    const unsigned long long cm = __ballot(key < ws.kth) & tk;
    if (!cm) return false;
    const bool in = __builtin_amdgcn_inverse_ballot_w64(cm);
    if (bcast64(ws.wl, 0) == ~0ull) {
        // empty list (keys never equal ~0: their cell field is below 2^24 - 1)
        const uint32_t c = (uint32_t)__popcll(cm);
        if (c > 16) {
            const uint64_t v = wave_sort64(in ? key : ~0ull, lane);
            ws.wl = ((uint32_t)lane < k) ? v : ~0ull;
        } else {
            uint32_t rank = 0;
            for (unsigned long long m = cm; m; m &= m - 1) {
                const uint64_t kk = bcast64(key, __ffsll((long long)m) - 1);
                rank += (kk < key) ? 1u : 0u;
            }
            // the other lanes take the places after the candidates, in order
            const uint32_t dest = in ? rank : c + __builtin_amdgcn_mbcnt_hi(
                                                     (uint32_t)(~cm >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)~cm, 0u));
            const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_permute((int)(dest * 4), (int)(uint32_t)key);
            const uint32_t hi =
                (uint32_t)__builtin_amdgcn_ds_permute((int)(dest * 4), (int)(uint32_t)(key >> 32));
            ws.wl = ((uint32_t)lane < (c < k ? c : k)) ? (((uint64_t)hi << 32) | lo) : ~0ull;
        }
        ws.kth = bcast64(ws.wl, (int)k - 1);
        return true;
    }
    unsigned long long placed = 0;  // list places taken by candidates
    int from = 0;                   // the candidate lane placed at this place
    for (unsigned long long m = cm; m; m &= m - 1) {
        const int src = __ffsll((long long)m) - 1;
        const uint64_t kk = bcast64(key, src);
        const uint32_t pos = (uint32_t)__popcll(__ballot(ws.wl < kk)) +
                             (uint32_t)__popcll(__ballot(key < kk) & cm);
        if (pos < k) {
            placed |= 1ull << pos;
            from = (lane == (int)pos) ? src : from;
        }
    }
    // candidates placed before this lane; the list entry that moves here
    const uint32_t before =
        __builtin_amdgcn_mbcnt_hi((uint32_t)(placed >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)placed, 0u));
    const int li = lane - (int)before;
    const bool fromc = __builtin_amdgcn_inverse_ballot_w64(placed);
    const uint32_t clo = (uint32_t)__shfl((int)(uint32_t)key, from, 64);
    const uint32_t chi = (uint32_t)__shfl((int)(uint32_t)(key >> 32), from, 64);
    const uint32_t llo = (uint32_t)__shfl((int)(uint32_t)ws.wl, li, 64);
    const uint32_t lhi = (uint32_t)__shfl((int)(uint32_t)(ws.wl >> 32), li, 64);
    const uint64_t v = fromc ? (((uint64_t)chi << 32) | clo) : (((uint64_t)lhi << 32) | llo);
    ws.wl = ((uint32_t)lane < k) ? v : ~0ull;
    ws.kth = bcast64(ws.wl, (int)k - 1);
    return true;
}

// Compare-exchange of two keys held by the same lane (ascending).
__device__ inline void ce64(uint64_t &a, uint64_t &b) {
    const bool sw = b < a;
    const uint64_t lo = sw ? b : a, hi = sw ? a : b;
    a = lo;
    b = hi;
}

// The group row of one member slot (RP uint16) as (RP + 1) / 2 dwords.
template <int RP>
__device__ inline void load_row1(const uint16_t *p, uint32_t (&w)[(RP + 1) / 2]) {
    if constexpr (RP == 1) {
        w[0] = *p;
    } else if constexpr (RP == 2) {
        w[0] = *reinterpret_cast<const uint32_t *>(p);
    } else if constexpr (RP == 4) {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        w[0] = v.x;
        w[1] = v.y;
    } else {
#pragma unroll
        for (int i = 0; i < RP / 8; ++i) {
            const uint4 v = reinterpret_cast<const uint4 *>(p)[i];
            w[4 * i + 0] = v.x;
            w[4 * i + 1] = v.y;
            w[4 * i + 2] = v.z;
            w[4 * i + 3] = v.w;
        }
    }
}

// Survivor queue of a wavefront: 63 waiting and one more from every lane.
constexpr uint32_t WALK_QUEUE = 128;

// Stream the filter words of the members of the listed cells lbs[0, nl) of one
// repetition and put the members that matter into the wavefront's top-k.
// Work items are runs of 4 << ils member slots of one cell, 1 << ils lanes
// each (fitted to the cell size, set_walk_items), so a wavefront's load covers
// 64 >> ils of them; U loads per lane are in flight while the U before them
// are tested.  A cell's padding slots are walked too (no size is read): they
// hold no id and drop out at the lookup, if not before.
// A member is looked up (its id and group row gathered, its key made) when
// pass(filter word) holds; cflr = nullptr looks up every member.  Survivors go
// to the wavefront's LDS queue and are looked up 64 at a time: whatever lanes
// and rounds they came from, a lookup's fixed cost and its memory latency are
// paid once per 64.
// byte(r, b): 255 - count of cell (r, b).
template <int RP, int QW, int U, class LB, class Pass, class Byte>
__device__ inline void walk_items(const LB *lbs, uint32_t nl, const uint32_t *__restrict__ memr,
                                  const uint16_t *__restrict__ cmgr, const uint32_t *__restrict__ cflr,
                                  uint32_t R, uint32_t Bp, const QArgs &A, uint32_t level, bool keep,
                                  uint32_t *wq, int lane, int wave, WaveState &ws, Pass pass, Byte byte) {
    constexpr int RW = (RP + 1) / 2;
    const uint32_t tmax = (256u - level) << 24;  // m >= level iff the key's high word is below it
    const uint32_t ils = A.ils, cpc = A.cpc, mstride = A.mstride;
    const uint32_t nitems = nl * cpc, ipw = 64u >> ils;
    const uint32_t sub = (uint32_t)lane >> ils, off = 4 * ((uint32_t)lane & ((1u << ils) - 1u));
    uint32_t queued = 0;
    auto take = [&](uint32_t n) {  // look up the first n queued slots, one per lane
        uint32_t xid = ~0u, rw[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) rw[i] = 0;
        if ((uint32_t)lane < n) {
            const uint32_t sl = wq[lane];
            xid = memr[sl];
            load_row1<RP>(cmgr + (uint64_t)sl * RP, rw);
        }
        // the key's high word: max over the member's cells of
        // ((255 - count) << 24 | cell); the padding repetitions r >= R repeat
        // repetition R-1
        uint32_t t = 0;
#pragma unroll
        for (int r = 0; r < RP; ++r) {
            const uint32_t rr = (uint32_t)r < R ? (uint32_t)r : R - 1;
            const uint32_t b = (rw[r >> 1] >> (16 * (r & 1))) & 0xFFFFu;
            const uint32_t tv = (byte(rr, b) << 24) | (rr * Bp + b);
            t = tv > t ? tv : t;
        }
        const bool act = xid != ~0u;
        const unsigned long long am = __ballot(act), gm = __ballot(act && t < tmax);
        const unsigned long long tm = keep ? am : gm;
        ws.gathered += (uint32_t)__popcll(am);
        ws.n_ge += (uint32_t)__popcll(gm);
        ws.n_all += (uint32_t)__popcll(tm);
        wave_insert(ws, ((uint64_t)t << 32) | xid, tm, A.k, lane);
    };
    uint4 fv[U];
    uint32_t slot[U];
    auto load = [&](uint32_t i0) {
#pragma unroll
        for (int g = 0; g < U; ++g) {
            const uint32_t it = (i0 + g * QW) * ipw + sub;
            const uint32_t itc = it < nitems ? it : 0u;
            const uint32_t ci = cpc == 1 ? itc : __umulhi(itc, A.cpc_mul);
            const uint32_t pos = ((itc - ci * cpc) << (ils + 2)) + off;
            const bool in = it < nitems && pos < mstride;
            slot[g] = in ? lbs[ci] * mstride + pos : ~0u;
            fv[g] = make_uint4(0, 0, 0, 0);
            if (in && cflr) fv[g] = *reinterpret_cast<const uint4 *>(cflr + slot[g]);
        }
    };
    if (wave * ipw < nitems) load(wave);
    for (uint32_t i0 = wave; i0 * ipw < nitems; i0 += QW * U) {
        uint4 cf[U];
        uint32_t cs[U];
#pragma unroll
        for (int g = 0; g < U; ++g) {
            cf[g] = fv[g];
            cs[g] = slot[g];
        }
        if ((i0 + QW * U) * ipw < nitems) load(i0 + QW * U);
#pragma unroll
        for (int g = 0; g < U; ++g) {
            const uint32_t fw[4] = {cf[g].x, cf[g].y, cf[g].z, cf[g].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool in = cs[g] != ~0u && (pass(fw[e]) || !cflr);
                const unsigned long long pm = __ballot(in);
                if (pm) {
                    const uint32_t at = queued + __builtin_amdgcn_mbcnt_hi(
                                                     (uint32_t)(pm >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)pm, 0u));
                    if (in) wq[at] = cs[g] + (uint32_t)e;
                    queued += (uint32_t)__popcll(pm);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    if (queued >= 64) {
                        take(64);
                        queued -= 64;
                        uint32_t v = 0;
                        if ((uint32_t)lane < queued) v = wq[64 + lane];
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        if ((uint32_t)lane < queued) wq[lane] = v;
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                    }
                }
            }
        }
    }
    if (queued) take(queued);
}

// Lanes per walk item: the widest of 8 .. 64 lanes (4 members each) whose
// items pad the largest cell by at most a tenth more than the best.
inline void set_walk_items(QArgs &a) {
    uint32_t best = ~0u;
    for (uint32_t ls = 3; ls <= 6; ++ls) {
        const uint32_t w = 4u << ls, pad = (a.gmax + w - 1) / w * w;
        best = pad < best ? pad : best;
    }
    for (uint32_t ls = 3; ls <= 6; ++ls) {
        const uint32_t w = 4u << ls, n = (a.gmax + w - 1) / w;
        if ((uint64_t)n * w * 10 <= (uint64_t)best * 11) {
            a.ils = ls;
            a.cpc = n;
        }
    }
    // item / cpc = umulhi(item, cpc_mul) for items below 2^32 / cpc
    a.cpc_mul = (uint32_t)(0xFFFFFFFFull / a.cpc + 1);
}

// The sparse kernel (query_sparse.hip): its variant for this index and batch,
// 0 where the general kernel serves it; and the launch over a.nq queries, which
// leaves queries that it cannot take marked DEFERRED.
int sparse_variant(const Index &ix, const QArgs &a);
void sparse_query_launch(const Index &ix, int variant, QArgs a, hipStream_t s);

}  // namespace flinng
