// MinHash hashing of item sets on gfx950.
//
// The set-similarity LSH instance (the paper hashes genome n-gram sets with
// MinHash, Section 7, Experiments, "Datasets"; the concatenation trick of Section 3 joins K
// minima per table):
//   a[t][j]  = sm64(key_MH, t*K + j)
//   pi_tj(e) = top 32 bits of splitmix_finalize(e XOR a[t][j])
//   mh_tj(S) = min over e in S of pi_tj(e)        (empty set: 0xFFFFFFFF)
//   h = sm64(key_MH, L*K + t); for j < K: h = splitmix_finalize(h XOR mh_tj)
//   bucket_t = h >> (64 - bucket_bits)
//
// Mapping: one wavefront per set.  The set's items are staged in LDS 128 at a
// time; every lane owns one hash function at a time and takes its minimum over
// the staged items (a broadcast read per item).  The last L*K mod 64 functions
// share the lanes as floor(64 / that) slices of the items each, or in several
// passes where that leaves fewer lanes idle, combined by LDS minima.  Small sets
// and few functions read the items themselves.  Sets may also be given as text: the items of an n-gram set are then
// made from the staged symbols in the wavefront itself and never stored.
//
// What bounds it: vector instructions.  On gfx950 a 32-bit multiply issues like
// any three-operand instruction (4.4-5.1 cycles per wavefront, measured), so
// the count of instructions is what matters: the finaliser's 64-bit products
// are spelled in the 32-bit pieces whose result is used (the second product
// needs its high half only; for 32-bit items half of the first is the same for
// every item), and its last step, h ^ (h >> 31), is left out while the minimum
// runs: it changes only values with the top bit set, so it matters only if
// every value has it (then the minimum is taken again with it).  Measured:
// 10,000 URL sets (70 items, 144 functions) 105 -> 68 us, 1.5 T evaluations a
// second (5M of them 33.7 -> 22.5 ms, 2.2 T/s); 10,000 reads (81 64-bit items,
// 12 functions) 15.6 -> 12.9 us; 7,777 reads given as text, 64 functions, 36 us
// against 64 for offsets, items and hash kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "flinng_internal.h"

namespace flinng {

namespace {

__device__ inline uint64_t murmur_fmix64(uint64_t k) {
    k ^= k >> 33;
    k *= 0xFF51AFD7ED558CCDull;
    k ^= k >> 33;
    k *= 0xC4CEB9FE1A85EC53ull;
    k ^= k >> 33;
    return k;
}

__device__ inline uint32_t murmur_fmix32(uint32_t h) {
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

// High word of splitmix_finalize(e XOR a) before its last xor-shift, for one
// function a.
template <typename ItemT>
struct HashFn {
    static constexpr uint32_t C1L = 0x1CE4E5B9u, C1H = 0xBF58476Du, C2L = 0x133111EBu, C2H = 0x94D049BBu;
    uint32_t al, ah, kk;
    __device__ explicit HashFn(uint64_t a) {
        al = (uint32_t)a;
        ah = (uint32_t)(a >> 32);
        kk = (ah ^ (ah >> 30)) * C1L;  // 32-bit items: the high half never changes
    }
    __device__ uint32_t operator()(ItemT e) const {
        uint32_t lo, hi;
        if constexpr (sizeof(ItemT) == 4) {
            const uint32_t x = (uint32_t)e ^ al;
            const uint32_t l = x ^ __builtin_amdgcn_alignbit(ah, x, 30);
            const uint64_t m = (uint64_t)l * C1L;
            lo = (uint32_t)m;
            hi = (uint32_t)(m >> 32) + l * C1H + kk;
        } else {
            const uint32_t xl = (uint32_t)e ^ al, xh = (uint32_t)((uint64_t)e >> 32) ^ ah;
            const uint32_t l = xl ^ __builtin_amdgcn_alignbit(xh, xl, 30), h = xh ^ (xh >> 30);
            const uint64_t m = (uint64_t)l * C1L;
            lo = (uint32_t)m;
            hi = (uint32_t)(m >> 32) + l * C1H + h * C1L;
        }
        lo ^= __builtin_amdgcn_alignbit(hi, lo, 27);
        hi ^= hi >> 27;
        return __umulhi(lo, C2L) + lo * C2H + hi * C2L;
    }
};

constexpr uint32_t MH_CHUNK = 128;           // items staged at a time
constexpr uint32_t MH_BUF = MH_CHUNK + 64;   // padded with copies of the last for the slices
constexpr uint32_t MH_SYMS = MH_CHUNK + 64;  // symbols of a chunk's windows (n-grams of up to 64)

// Sets are not staged where it is not worth it: up to this many functions, or up to
// 16 items a slice (8 for one slice).  20,000 sets of 64-bit items, staged and not:
// 4 functions, 81 items 22.7 and 18.1 us; 12 functions, 4 items 16.4 and 13.6, 40
// items 22.9 and 20.3, 300 items 63.5 and 74; 31 functions, 81 items 44 and 47.
constexpr uint32_t MH_FEW_FUNCTIONS = 8;
// Items up to which the last functions are taken in one pass.
constexpr uint32_t MH_FEW_ITEMS = 32;

// MANY: the last LK mod 64 functions in several passes (`slices` of the items each)
// for sets of more than MH_FEW_ITEMS.
// (the wavefronts per SIMD are those that the registers of one pass allow)
template <typename ItemT, bool TEXT, bool MANY>
__global__ __launch_bounds__(256, TEXT ? (sizeof(ItemT) == 4 ? 7 : 6) : 8) void minhash_kernel(const ItemT *__restrict__ items,
                                                      const uint64_t *__restrict__ offsets,
                                                      TextSource tx, uint64_t nsets, uint32_t K,
                                                      uint32_t L, uint32_t bbits, uint64_t key,
                                                      uint32_t slices, uint32_t *__restrict__ codes) {
    extern __shared__ uint32_t lds32[];
    const int lane = threadIdx.x % 64;
    const int wave = threadIdx.x / 64;
    const uint64_t set = (uint64_t)blockIdx.x * (blockDim.x / 64) + wave;
    if (set >= nsets) return;
    const uint32_t LK = L * K;
    // per wavefront: staged items, staged symbols, minima
    constexpr uint32_t BW = MH_BUF * sizeof(ItemT) / 4, SW = TEXT ? MH_SYMS / 4 : 0;
    uint32_t *mine = lds32 + wave * ((BW + SW + LK + 1) & ~1u);
    ItemT *buf = reinterpret_cast<ItemT *>(mine);
    uint8_t *sym = reinterpret_cast<uint8_t *>(mine + BW);
    uint32_t *mins = mine + BW + SW;
    auto lds_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (uint32_t f = lane; f < LK; f += 64) mins[f] = 0xFFFFFFFFu;
    const uint64_t *off = TEXT ? tx.offsets : offsets;
    const uint64_t beg = off[set], end = off[set + 1];
    uint64_t n = end > beg ? end - beg : 0;
    if (TEXT) {
        // decreasing offsets: the caller is told, and nothing is read by them
        if (off[nsets] < off[0]) n = 0;
        n = n >= tx.gram ? n - tx.gram + 1 : 0;
    }
    // the last LK mod 64 functions: S slices of the items each
    const uint32_t full = LK & ~63u, rem = LK - full;
    const bool many = MANY && n > MH_FEW_ITEMS;
    const uint32_t S = many ? slices : rem ? 64 / rem : 1;
    const uint32_t rf = (uint32_t)lane / S, rs = (uint32_t)lane - rf * S;
    if (!TEXT && LK <= 64 && (LK <= MH_FEW_FUNCTIONS || n <= (S > 1 ? 16 * S : 8)) && !many) {
        // each lane reads its items itself
        lds_fence();
        if (rf < LK) {
            const HashFn<ItemT> h(sm64(key, rf));
            uint32_t mn = 0xFFFFFFFFu;
            for (const ItemT *p = items + beg + rs, *e = items + beg + n; p < e; p += S) {
                uint32_t v = h(*p);
                v ^= v >> 31;
                mn = v < mn ? v : mn;
            }
            atomicMin(&mins[rf], mn);
        }
        n = 0;
    }
    for (uint64_t c0 = 0; c0 < n; c0 += MH_CHUNK) {
        const uint32_t m = (uint32_t)(n - c0 < MH_CHUNK ? n - c0 : MH_CHUNK);
        lds_fence();  // the last chunk's reads are done
        if constexpr (TEXT) {
            const uint32_t ns = m + tx.gram - 1;
            for (uint32_t j = lane; j < ns; j += 64) sym[j] = tx.symbols[beg + c0 + j];
            lds_fence();
        }
        for (uint32_t j0 = 0; j0 < m + S - 1; j0 += 64) {
            const uint32_t j = j0 + lane, jj = j < m ? j : m - 1;
            if constexpr (TEXT) {
                ItemT v = 0;  // 32-bit items need the window value's low word only
                for (uint32_t i = 0; i < tx.gram; ++i) v = v * (ItemT)tx.radix + sym[jj + i];
                if constexpr (sizeof(ItemT) == 8) buf[j] = murmur_fmix64(v ^ tx.key);
                else buf[j] = murmur_fmix32(v ^ (uint32_t)tx.key);
            } else {
                buf[j] = items[beg + c0 + jj];
            }
        }
        lds_fence();
        // the minimum of function f over items first, first + step, ...
        auto minimum = [&](uint32_t f, uint32_t first, uint32_t step) {
            const HashFn<ItemT> h(sm64(key, f));
            const uint32_t cnt = (m + step - 1) / step;
            uint32_t mn = 0xFFFFFFFFu;
#pragma unroll 4
            for (uint32_t i = 0; i < cnt; ++i) {
                const uint32_t v = h(buf[first + i * step]);
                mn = v < mn ? v : mn;
            }
            if (__ballot(mn >> 31)) {  // the last xor-shift decides (small sets)
                mn = 0xFFFFFFFFu;
                for (uint32_t i = 0; i < cnt; ++i) {
                    uint32_t v = h(buf[first + i * step]);
                    v ^= v >> 31;
                    mn = v < mn ? v : mn;
                }
            }
            return mn;
        };
        for (uint32_t f0 = 0; f0 < full; f0 += 64) {
            uint32_t mn = 0xFFFFFFFFu;
            if (m <= 12) {  // some lane's minimum nearly always has the top bit
                const HashFn<ItemT> h(sm64(key, f0 + lane));
                for (uint32_t i = 0; i < m; ++i) {
                    uint32_t v = h(buf[i]);
                    v ^= v >> 31;
                    mn = v < mn ? v : mn;
                }
            } else {
                mn = minimum(f0 + lane, 0, 1);
            }
            const uint32_t old = mins[f0 + lane];
            mins[f0 + lane] = mn < old ? mn : old;
        }
        if (!many) {
            if (rf < rem) atomicMin(&mins[full + rf], minimum(full + rf, rs, S));
        } else {
            const uint32_t F = 64 / S;
            for (uint32_t f0 = full; f0 < LK; f0 += F)
                if (rf < F && f0 + rf < LK) atomicMin(&mins[f0 + rf], minimum(f0 + rf, rs, S));
        }
    }
    lds_fence();
    for (uint32_t t = lane; t < L; t += 64) {
        uint64_t h = sm64(key, (uint64_t)LK + t);
        for (uint32_t j = 0; j < K; ++j) h = splitmix_finalize(h ^ (uint64_t)mins[t * K + j]);
        codes[set * L + t] = (uint32_t)(h >> (64 - bbits));
    }
}

// Slices of the items for r < 64 functions where several passes over a part of
// them take fewer rounds of evaluations than one pass (0 where not), for a set of
// 64 items, each pass costing about four rounds more: 40 functions in one pass
// leave 24 lanes idle, two passes of 21 in three slices one (20,000 sets of 81
// 64-bit items 69 -> 54 us).
uint32_t choose_slices(uint32_t r) {
    auto cost = [&](uint32_t S) { return (r + 64 / S - 1) / (64 / S) * ((64 + S - 1) / S + 4); };
    uint32_t best = 0, least = r ? cost(64 / r) : 0;
    for (uint32_t S = 1; r && S <= 64; ++S)
        if (cost(S) < least) {
            least = cost(S);
            best = S;
        }
    return best;
}

template <typename ItemT, bool TEXT>
void launch_minhash(const ItemT *items, const uint64_t *offs, const TextSource &tx, uint64_t n, uint32_t K,
                    uint32_t L, uint32_t b, uint64_t key, uint32_t *codes, hipStream_t s) {
    // one wavefront per set, up to four per workgroup: as many as keep the
    // wavefronts' minima (L*K words each) and staged items within 64 KiB of
    // LDS, so every valid (K, L) launches (L*K <= 255*32 needs 34 KiB for one)
    const size_t words = MH_BUF * sizeof(ItemT) / 4 + (TEXT ? MH_SYMS / 4 : 0) + (size_t)L * K + 1;
    const size_t per_wave = (words & ~(size_t)1) * 4;
    unsigned waves = 4;
    while (waves > 1 && waves * per_wave > 65536) waves >>= 1;
    dim3 grid((unsigned)((n + waves - 1) / waves)), block(64 * waves);
    const uint32_t slices = choose_slices(L * K & 63);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, waves * per_wave, s, items, offs, tx, n, K, L, b, key, slices,
                           codes);
        FL_CHECK_LAUNCH();
    };
    if (slices) go(minhash_kernel<ItemT, TEXT, true>);
    else go(minhash_kernel<ItemT, TEXT, false>);
}

}  // namespace

void minhash_hash_text(const Index &ix, const TextSource &tx, uint64_t n, uint32_t *codes_dev,
                       hipStream_t s) {
    if (n == 0) return;
    const uint64_t key = sm64(ix.p.seed, TAG_MINHASH);
    if (ix.p.family == FLINNG_MINHASH_U64)
        launch_minhash<uint64_t, true>(nullptr, nullptr, tx, n, ix.p.K, ix.p.L, ix.nbits, key, codes_dev, s);
    else
        launch_minhash<uint32_t, true>(nullptr, nullptr, tx, n, ix.p.K, ix.p.L, ix.nbits, key, codes_dev, s);
}

void minhash_hash(const Index &ix, const flinng_input &in, uint32_t *codes_dev, hipStream_t s) {
    const uint64_t n = in.count;
    if (n == 0) return;
    const bool u64 = ix.p.family == FLINNG_MINHASH_U64;
    const size_t isz = u64 ? 8 : 4;
    const void *items = in.values;
    const uint64_t *offs = in.offsets;
    DevBuf ibuf, obuf;
    uint64_t first = 0, last = 0;
    if (!in.on_device) {
        first = in.offsets[0];
        last = in.offsets[n];
        if (last < first) fail(FLINNG_EINVAL, "offsets must be nondecreasing");
        // copy offsets rebased to 0 and the item range they cover
        std::vector<uint64_t> ro(n + 1);
        for (uint64_t i = 0; i <= n; ++i) {
            if (i && in.offsets[i] < in.offsets[i - 1])
                fail(FLINNG_EINVAL, "offsets must be nondecreasing");
            ro[i] = in.offsets[i] - first;
        }
        obuf = DevBuf((n + 1) * 8, s);
        FL_HIP(hipMemcpyAsync(obuf.ptr, ro.data(), (n + 1) * 8, hipMemcpyHostToDevice, s));
        const uint64_t nit = last - first;
        ibuf = DevBuf(std::max<uint64_t>(nit, 1) * isz, s);
        if (nit)
            FL_HIP(hipMemcpyAsync(ibuf.ptr, static_cast<const char *>(in.values) + first * isz,
                                  nit * isz, hipMemcpyHostToDevice, s));
        // the host copy must finish before the vector goes out of scope
        FL_HIP(hipStreamSynchronize(s));
        items = ibuf.ptr;
        offs = obuf.as<uint64_t>();
    }
    const uint64_t key = sm64(ix.p.seed, TAG_MINHASH);
    if (u64)
        launch_minhash<uint64_t, false>(static_cast<const uint64_t *>(items), offs, TextSource{}, n, ix.p.K,
                                        ix.p.L, ix.nbits, key, codes_dev, s);
    else
        launch_minhash<uint32_t, false>(static_cast<const uint32_t *>(items), offs, TextSource{}, n, ix.p.K,
                                        ix.p.L, ix.nbits, key, codes_dev, s);
}

void hash_batch(const Index &ix, const flinng_input &in, uint32_t *codes_dev, hipStream_t s,
                unsigned long long *ctr, Arena *ws) {
    if (is_dense(ix.p.family))
        srp_hash(ix, in, codes_dev, s, ctr, ws);
    else
        minhash_hash(ix, in, codes_dev, s);
}

}  // namespace flinng
