// Internal declarations of the gfx950 FLINNG library (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <memory>
#include <mutex>
#include <shared_mutex>
#include <string>
#include <utility>
#include <vector>

#include "../../include/flinng.h"

namespace flinng {

// ---------------------------------------------------------------------------
// Errors: every ABI function catches flinng::Error and maps it to a code and
// the thread-local message.
struct Error {
    int code;
    std::string msg;
};
[[noreturn]] void fail(int code, const std::string &msg);
void set_last_error(const std::string &msg);

#define FL_HIP(call)                                                          \
    do {                                                                      \
        hipError_t e_ = (call);                                               \
        if (e_ != hipSuccess)                                                 \
            ::flinng::fail(e_ == hipErrorOutOfMemory ? FLINNG_ENOMEM          \
                                                     : FLINNG_EDEVICE,        \
                           std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

#define FL_CHECK_LAUNCH() FL_HIP(hipGetLastError())

// ---------------------------------------------------------------------------
// Counter-based generator shared by every random object of the method:
// SplitMix64's output function (Steele, Lea and Flood, OOPSLA 2014) applied to
// state s + (i+1) * 0x9E3779B97F4A7C15, i.e. the i-th output of a SplitMix64
// stream started at s.  Stream keys: sm64(seed, tag).
enum : uint64_t { TAG_HYP = 1, TAG_MINHASH = 2, TAG_GROUP = 3, TAG_STREAM = 4 };

__host__ __device__ inline uint64_t splitmix_finalize(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__host__ __device__ inline uint64_t sm64(uint64_t s, uint64_t i) {
    return splitmix_finalize(s + (i + 1ull) * 0x9E3779B97F4A7C15ull);
}

// ---------------------------------------------------------------------------
// A built index.  Device layout (all arrays owned by the index):
//   offsets   [L][nbuckets+1] uint32  absolute positions into `cells`
//   cells     [list_entries]  uint16 (R*B <= 65536) or uint32 cell ids,
//             each bucket's list ascending (a Bloom filter bit set once)
//   grp       [N][Rp]         uint16 group of point x in repetition r
//             (Rp = R rounded up to a power of two; point-major so one
//             vector load gathers all R groups of a candidate)
//   mem       [R][B][mstride] uint32 members of cell (r,b), ascending id,
//             padded with 0xFFFFFFFF to mstride = ceil(N/B) rounded up to 4,
//             so every cell starts 16-byte aligned (4 ids per lane per load)
//   cmg       [R][B][mstride][Rp] uint16 cell-major copy of the groups: the
//             row of the member in each slot of mem, so a decode pass reads
//             every candidate's R groups sequentially beside its id
//   cfl       [R][B][mstride] uint32 the member's groups in repetitions
//             r+1 and r+2 (mod R), low and high 16 bits: a decode pass of
//             repetition r reads these 4 bytes per member and gathers the
//             id and the full row only for the few members whose counts in
//             those repetitions reach the level
//   gsize     [R][B]          uint32 members of each cell
//   hyp       [L*K][dpad]     bf16 hyperplanes (dense families)
//   hypnorm   [L*K]           fp32 Euclidean norms of the hyperplanes
//   hypt      [ceil(L*K/16)][dpad/32][16][32]  bf16 family: the hyperplanes
//             again, in 16 x 32 tiles (one MFMA operand fragment each, 1 KB
//             contiguous; rows past L*K zero)
// Points inserted after the build (ids N0, N0+1, ...) are added by building
// new offsets/cells/mem/cmg/cfl/gsize arrays beside the old ones and swapping
// them in under `rw` (exclusive), so a query enqueued under `rw` (shared)
// sees one version; the old arrays are freed once the device is idle.
struct Index {
    flinng_params p{};
    uint64_t N = 0;
    uint64_t N0 = 0;             // points of the one-pass build
    uint64_t grp_cap = 0;        // point rows allocated in grp
    uint32_t nbits = 0;          // bucket width (K for SRP)
    uint32_t dpad = 0;           // dense: dim rounded up to 32
    uint32_t Rp = 1;
    uint32_t mstride = 4;        // member slots per cell
    uint32_t cell_bytes = 2;
    uint64_t list_entries = 0;
    double mean_entries = 0;     // list entries one of the points meets as a query
    uint64_t device_bytes = 0;
    uint64_t srp_rechecked = 0, srp_exact = 0;
    int device = 0;
    uint32_t *offsets = nullptr;
    void *cells = nullptr;
    uint16_t *grp = nullptr;
    uint32_t *mem = nullptr;
    uint16_t *cmg = nullptr;
    uint32_t *cfl = nullptr;
    uint16_t *hyp = nullptr;
    float *hypnorm = nullptr;
    uint16_t *hypt = nullptr;
    uint32_t *gsize = nullptr;
    uint32_t gmax = 0;                    // the largest cell
    std::vector<uint32_t> gsize_host;     // host copy of gsize
    mutable std::shared_mutex rw;         // query enqueue (shared) / insert swap
    std::mutex insert_mu;                 // one insert at a time
    // Device scratch of one query batch, one region for each stream the index is
    // queried on: work on one stream runs in order, so a region is reused without
    // waiting.  Its lock is held while a call queues the work that uses it (two
    // threads queueing on one stream must not interleave) and, where its results
    // lie in it, until they are copied out.  The codes grow with the batch (with
    // a synchronous free, as when a region is evicted); a small batch's other
    // scratch lies apart, in a piece of one size, so that only a batch with more
    // codes moves the codes of a captured call.  Released with the index.
    struct StreamScratch {
        hipStream_t stream = nullptr;
        void *ptr = nullptr;    // codes
        size_t cap = 0;
        void *small = nullptr;  // SMALL_SCRATCH bytes, once a call needs them
        void release() {
            if (ptr) (void)hipFree(ptr);
            if (small) (void)hipFree(small);
            ptr = small = nullptr;
            cap = 0;
        }
        bool evicted = false;
        std::mutex mu;
    };
    mutable std::mutex scratch_mu;
    mutable std::vector<std::shared_ptr<StreamScratch>> scratch;
    // Pinned words that a text query reads its first and last offset into,
    // with the event that says they are there: one per call in flight.
    struct Readback {
        uint64_t *host;
        hipEvent_t ready;
    };
    mutable std::mutex readback_mu;
    mutable std::vector<Readback> readbacks;  // the free ones
    bool counted = false;                 // among its device's live indexes
};

// Scratch of a batch that is kept in its stream's region rather than allocated.
constexpr size_t SMALL_SCRATCH = (size_t)1 << 20;

inline uint64_t nbuckets(const Index &ix) { return 1ull << ix.nbits; }
// Bytes allocated for n list entries of csz bytes: rounded up to 16 bytes
// plus 16 more (zeroed), so aligned 16-byte reads covering any entry are in
// bounds.
inline size_t cells_alloc_bytes(uint64_t n, size_t csz) {
    return ((n * csz + 15) & ~(size_t)15) + 16;
}
inline bool is_dense(uint32_t fam) { return fam == FLINNG_SRP_F32 || fam == FLINNG_SRP_BF16; }
// Device bytes an index holds (all its arrays).
inline uint64_t index_device_bytes(const Index &ix) {
    const uint64_t ncells = (uint64_t)ix.p.R * ix.p.B;
    uint64_t b = (uint64_t)ix.p.L * (nbuckets(ix) + 1) * 4 +
                 cells_alloc_bytes(ix.list_entries, ix.cell_bytes) + ix.grp_cap * ix.Rp * 2 +
                 ncells * ix.mstride * (8 + 2ull * ix.Rp) + ncells * 4;
    if (is_dense(ix.p.family)) b += (uint64_t)ix.p.L * ix.p.K * (ix.dpad * 2 + 4);
    if (ix.p.family == FLINNG_SRP_BF16) b += ((uint64_t)ix.p.L * ix.p.K + 15) / 16 * 16 * ix.dpad * 2;
    return b;
}

// The member arrays of an index (mem, cmg, cfl, gsize) lie in one allocation,
// mem first, at 256-byte aligned offsets: an insert replaces them together.
struct MemberLayout {
    size_t cmg, cfl, gsize, total;
    MemberLayout(uint64_t ncells, uint64_t mstride, uint32_t Rp) {
        auto round = [](size_t b) { return (b + 255) & ~(size_t)255; };
        cmg = round(ncells * mstride * 4);
        cfl = cmg + round(ncells * mstride * Rp * 2);
        gsize = cfl + round(ncells * mstride * 4);
        total = gsize + round(ncells * 4);
    }
};

// Device memory of builds and inserts: the arrays of indexes and the scratch
// that makes them, from a stream-ordered pool of the library's own (one per
// GPU).  Mapping and unmapping device memory costs milliseconds per call at
// times (a hipFree 1.6 ms on average, up to 15 ms, in runs where a stream of
// inserts took 155 ms instead of 40), so up to POOL_KEEP bytes that are not in
// use stay mapped for the next build or insert; with the last index of a GPU
// everything is given back.  pool_free: the caller knows that the device no
// longer uses the memory.
constexpr uint64_t POOL_KEEP = 4ull << 30;
void *pool_malloc(size_t bytes, hipStream_t s);
void pool_free(void *p);

// Device scratch allocated on a stream (stream-ordered allocator).
struct DevBuf {
    void *ptr = nullptr;
    hipStream_t stream = nullptr;
    DevBuf() = default;
    DevBuf(size_t bytes, hipStream_t s);
    static DevBuf pooled(size_t bytes, hipStream_t s) {
        DevBuf b;
        b.stream = s;
        if (bytes) b.ptr = pool_malloc(bytes, s);
        return b;
    }
    ~DevBuf();
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    DevBuf(DevBuf &&o) noexcept : ptr(o.ptr), stream(o.stream) { o.ptr = nullptr; }
    DevBuf &operator=(DevBuf &&o) noexcept {
        if (this != &o) {
            release();
            ptr = o.ptr;
            stream = o.stream;
            o.ptr = nullptr;
        }
        return *this;
    }
    void release();
    template <class T> T *as() const { return static_cast<T *>(ptr); }
};

// A device region owned by the caller, handed out by a bump pointer in
// 256-byte aligned pieces.  Running past its end is an internal sizing error.
struct Arena {
    char *base = nullptr;
    size_t cap = 0, used = 0;
    static size_t round(size_t b) { return (b + 255) & ~(size_t)255; }
    void *take(size_t bytes) {
        if (bytes == 0) return nullptr;
        const size_t b = round(bytes);
        if (used + b > cap) fail(FLINNG_EDEVICE, "internal: batch workspace undersized");
        void *p = base + used;
        used += b;
        return p;
    }
};

// Pieces of one allocation: sizes added first, pointers once it exists.
struct Pieces {
    size_t total = 0;
    size_t add(size_t bytes) {
        const size_t at = total;
        total += Arena::round(bytes);
        return at;
    }
};

// Scratch of one call: carved from an arena when one is given, otherwise
// allocated on the stream and freed on it when the Scratch goes away.
struct Scratch {
    Arena *arena;
    hipStream_t stream;
    std::vector<DevBuf> owned;
    Scratch(Arena *a, hipStream_t s) : arena(a), stream(s) {}
    template <class T = void> T *get(size_t bytes) {
        if (bytes == 0) return nullptr;
        if (arena) return static_cast<T *>(arena->take(bytes));
        owned.emplace_back(bytes, stream);
        return static_cast<T *>(owned.back().ptr);
    }
};

// ---------------------------------------------------------------------------
// Hashing (hash_srp.hip, hash_minhash.hip).  All write codes[n][L] uint32.
void srp_make_hyperplanes(Index &ix, hipStream_t s);
// ctr (device, optional): the rechecked and exactly decided projections are
// added to its two counts.  Scratch comes from ws when given (srp_scratch_bytes bounds what it takes).
// proj_dev (optional, device, n*L*K fp32): receives the MFMA projections
// before any recheck.
void srp_hash(const Index &ix, const flinng_input &in, uint32_t *codes_dev,
              hipStream_t s, unsigned long long *ctr, Arena *ws = nullptr,
              float *proj_dev = nullptr);
// The error bound the MFMA stage uses for a trusted sign: |v32 - v| <=
// gamma * |x|_2 * |w|_2 + tau_abs (rounding of the norms included).
void srp_bound(const Index &ix, double *gamma, double *tau_abs);
// Upper bound of the scratch srp_hash takes for n rows already on the device
// (exact when the rows' device address xdev is given).
size_t srp_scratch_bytes(const Index &ix, uint64_t n, const void *xdev = nullptr);
void minhash_hash(const Index &ix, const flinng_input &in, uint32_t *codes_dev, hipStream_t s);
// Device-resident inputs take no scratch beyond ws (MinHash takes none).
void hash_batch(const Index &ix, const flinng_input &in, uint32_t *codes_dev,
                hipStream_t s, unsigned long long *ctr, Arena *ws = nullptr);
void zero_counters(unsigned long long *ctr, hipStream_t s);  // the two of srp_hash
// Symbol sequences on the device, read as n-gram sets (see flinng_text).
struct TextSource {
    const uint8_t *symbols;
    const uint64_t *offsets;
    uint64_t key;
    uint32_t gram, radix;
};
void minhash_hash_text(const Index &ix, const TextSource &tx, uint64_t n, uint32_t *codes_dev,
                       hipStream_t s);
// Device bytes one served batch of nq queries (nitems set items) occupies:
// staged input, codes, results and hash scratch, as the server carves them.
uint64_t batch_device_bytes(const Index &ix, uint64_t nq, uint64_t nitems, uint32_t k,
                            bool text);

// N-gram text (text.hip).  validate_text: argument checks (FLINNG_EINVAL);
// text_symbols: symbols the sequences span (reads two offsets back for a
// device input); text_source: the sequences on the device (host text copied to
// buffers from sc).
void validate_text(const flinng_text *t, uint32_t family);
uint64_t text_symbols(const flinng_text &t);
TextSource text_source(const flinng_text &t, uint64_t nsym, hipStream_t s, Scratch &sc);
// What the server's admission counts for the items of n sequences of nsym
// symbols (its batches make them in registers; the bound is kept, so that a
// memory budget admits what it did).
inline size_t text_scratch_bytes(uint32_t family, uint64_t n, uint64_t nsym) {
    const size_t isz = family == FLINNG_MINHASH_U64 ? 8 : 4;
    return Arena::round((n + 1) * 8) + Arena::round((nsym ? nsym : 1) * isz);
}

// Segment copies by kernel (stage.hip): each segment copies `bytes` from
// src to dst, both device-visible addresses (device memory, or mapped pinned
// host memory).  Segments must not overlap their destinations.
struct CopySeg {
    uint64_t src, dst, bytes;
};
constexpr int MAX_COPY_SEGS = 128;  // per launch (kernel-argument space)
void copy_segments(const CopySeg *segs, size_t nseg, hipStream_t s);

// Sorting and scans (radix.hip).  Exclusive scan of data[0, n) in place, each
// prefix plus base (32-bit, wrapping); *total (device) = base + the sum, 64-bit.
size_t scan_scratch_bytes(uint64_t n);
void device_exclusive_scan_u32(uint32_t *data, uint64_t n, uint64_t base, uint64_t *total,
                               void *scratch, hipStream_t s);
// `count` stable sorts of n keys below 2^bits (sort t: keys[t*n ..]) into
// out[t*n ..] = key << 32 | index; tmp: as large as out.
size_t pair_sort_scratch_bytes(uint64_t n, uint32_t count);
void pair_sort(const uint32_t *keys, uint64_t n, uint32_t count, int bits, uint64_t *out,
               uint64_t *tmp, void *scratch, hipStream_t s);

// The reverse index (lists.hip): offsets [L][2^bits + 1] and cells (with the
// zeroed 16-byte tail that the query kernel's chunk reads need), owned by the
// caller.
struct Lists {
    uint32_t *offsets = nullptr;
    void *cells = nullptr;
    uint64_t entries = 0;
    double mean_entries = 0;  // entries that one of the points meets as a query
};
// Lists of n points with codes [n][L] and group rows [n][Rp].
Lists make_lists(const Index &ix, const uint32_t *codes, const uint16_t *grp, uint64_t n,
                 hipStream_t s);
// The index's lists with the cells of n more points merged in, as new arrays.
Lists merge_lists(const Index &ix, const uint32_t *codes, const uint16_t *grp_rows, uint64_t n,
                  hipStream_t s);
void free_lists(Lists &l);

// Build pieces (build.hip).
void build_groups(Index &ix, hipStream_t s);
void build_lists(Index &ix, const uint32_t *codes_dev, hipStream_t s);
// The filter plane cfl of member arrays `mem` (stride mstride) from the
// point rows `grp`.
void build_filter(const Index &ix, const uint32_t *mem, const uint16_t *grp, uint32_t mstride,
                  uint32_t *cfl, hipStream_t s);
// Add n points (ids ix.N ..) whose codes [n][L] are on the device: groups by
// the arrival rule, members, reverse index; swaps the new arrays in.  The
// caller holds ix.insert_mu.  Synchronizes the device.
void insert_points(Index &ix, const uint32_t *codes_dev, uint64_t n, hipStream_t s);

// Query (query.hip).
void query_launch(const Index &ix, const uint32_t *codes_dev, uint64_t nq,
                  uint32_t k, uint32_t *ids_dev, uint32_t *scores_dev,
                  bool persistent, hipStream_t s, uint32_t *work_counter,
                  unsigned long long *stats = nullptr);
void counts_launch(const Index &ix, const uint32_t *codes_dev, uint64_t nq,
                   uint8_t *counts_dev, hipStream_t s);
uint32_t query_max_k();

// Scratch bytes flinng_query_noalloc carves for nq queries (noalloc.hip).
size_t noalloc_scratch_bytes(const Index &ix, uint64_t nq, const void *xdev);

// Fixed-threshold query (threshold.hip): ids [nq][max_out] of the points with
// m(x) >= t, counts [nq] the size of each answer.
void threshold_launch(const Index &ix, const uint32_t *codes_dev, uint64_t nq, uint32_t t,
                      uint32_t max_out, uint32_t *ids_dev, uint32_t *counts_dev, hipStream_t s);

}  // namespace flinng
