// Exported C ABI: argument validation, orchestration of the build and query
// pipelines, and error mapping (no C++ exception crosses the boundary).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "flinng_internal.h"

namespace flinng {

static thread_local std::string g_err;

void set_last_error(const std::string &msg) { g_err = msg; }

[[noreturn]] void fail(int code, const std::string &msg) { throw Error{code, msg}; }

DevBuf::DevBuf(size_t bytes, hipStream_t s) : stream(s) {
    if (bytes == 0) return;
    hipError_t e = hipMallocAsync(&ptr, bytes, s);
    if (e != hipSuccess) {
        ptr = nullptr;
        (void)hipGetLastError();
        fail(e == hipErrorOutOfMemory ? FLINNG_ENOMEM : FLINNG_EDEVICE,
             "device allocation of " + std::to_string(bytes) + " bytes failed: " +
                 hipGetErrorString(e));
    }
}

void DevBuf::release() {
    if (ptr) (void)hipFreeAsync(ptr, stream);
    ptr = nullptr;
}

DevBuf::~DevBuf() { release(); }

namespace {

constexpr int POOL_DEVICES = 64;

struct BuildPool {
    std::mutex mu;
    hipMemPool_t pool = nullptr;  // stays null where none can be made
    bool tried = false;
    int live = 0;                 // indexes of the device
};

BuildPool &build_pool(int dev) {
    static BuildPool p[POOL_DEVICES];
    return p[dev >= 0 && dev < POOL_DEVICES ? dev : 0];
}

hipMemPool_t pool_of(int dev) {
    BuildPool &b = build_pool(dev);
    std::lock_guard<std::mutex> lk(b.mu);
    if (!b.tried) {
        b.tried = true;
        hipMemPoolProps props{};
        props.allocType = hipMemAllocationTypePinned;
        props.handleTypes = hipMemHandleTypeNone;
        props.location.type = hipMemLocationTypeDevice;
        props.location.id = dev;
        uint64_t keep = POOL_KEEP;
        if (hipMemPoolCreate(&b.pool, &props) != hipSuccess ||
            hipMemPoolSetAttribute(b.pool, hipMemPoolAttrReleaseThreshold, &keep) != hipSuccess) {
            b.pool = nullptr;
            (void)hipGetLastError();
        }
    }
    return b.pool;
}

}  // namespace

void *pool_malloc(size_t bytes, hipStream_t s) {
    int dev = 0;
    FL_HIP(hipGetDevice(&dev));
    hipMemPool_t pool = pool_of(dev);
    void *p = nullptr;
    hipError_t e = pool ? hipMallocFromPoolAsync(&p, bytes, pool, s) : hipMallocAsync(&p, bytes, s);
    if (e == hipErrorOutOfMemory && pool) {  // what the pool keeps may be what is missing
        (void)hipGetLastError();
        (void)hipDeviceSynchronize();
        (void)hipMemPoolTrimTo(pool, 0);
        e = hipMallocFromPoolAsync(&p, bytes, pool, s);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        fail(e == hipErrorOutOfMemory ? FLINNG_ENOMEM : FLINNG_EDEVICE,
             "device allocation of " + std::to_string(bytes) + " bytes failed: " + hipGetErrorString(e));
    }
    return p;
}

void pool_free(void *p) {
    if (p) (void)hipFreeAsync(p, nullptr);
}

// An index joins or leaves its device's live ones; with the last the pool
// gives everything back (the device is idle then).
static void pool_live(int dev, int by) {
    BuildPool &b = build_pool(dev);
    std::lock_guard<std::mutex> lk(b.mu);
    b.live += by;
    if (b.live == 0 && b.pool) {
        (void)hipStreamSynchronize(nullptr);  // the frees have happened
        (void)hipMemPoolTrimTo(b.pool, 0);
    }
}

template <class F>
static int guard(F &&f) {
    try {
        f();
        set_last_error("");
        return FLINNG_OK;
    } catch (const Error &e) {
        set_last_error(e.msg);
        return e.code;
    } catch (const std::bad_alloc &) {
        set_last_error("host allocation failed");
        return FLINNG_ENOMEM;
    } catch (const std::exception &e) {
        set_last_error(std::string("internal error: ") + e.what());
        return FLINNG_EDEVICE;
    } catch (...) {
        set_last_error("internal error");
        return FLINNG_EDEVICE;
    }
}

static void require(bool ok, const std::string &msg) {
    if (!ok) fail(FLINNG_EINVAL, msg);
}

static void validate_params(const flinng_params &p, uint64_t N) {
    require(p.family <= FLINNG_MINHASH_U64, "unknown family");
    require(p.reserved == 0, "reserved must be 0");
    require(p.L >= 1 && p.L <= 255, "L (tables) must be in 1..255");
    require(p.R >= 1 && p.R <= 16, "R (repetitions) must be in 1..16");
    require(p.B >= 1 && p.B <= 65536, "B (groups) must be in 1..65536");
    require(N >= 1, "empty dataset");
    require(N <= 0xFFFFFFFEull, "at most 2^32-2 points");
    require(p.B <= N, "B must not exceed N");
    if (is_dense(p.family)) {
        require(p.dim >= 1 && p.dim <= (1u << 20), "dim must be in 1..2^20");
        require(p.K >= 1 && p.K <= 24, "SRP K (bits per table) must be in 1..24");
        require(p.bucket_bits == 0 || p.bucket_bits == p.K, "SRP bucket_bits must be 0 or K");
    } else {
        require(p.K >= 1 && p.K <= 32, "MinHash K must be in 1..32");
        require(p.bucket_bits >= 1 && p.bucket_bits <= 24, "MinHash bucket_bits must be in 1..24");
    }
}

static void validate_input(const flinng_input *in, uint32_t family, const char *what) {
    require(in != nullptr, std::string(what) + " is NULL");
    require(in->reserved == 0, std::string(what) + ".reserved must be 0");
    require(in->on_device <= 1, std::string(what) + ".on_device must be 0 or 1");
    if (in->count == 0) return;
    require(in->values != nullptr || !is_dense(family), std::string(what) + ".values is NULL");
    if (!is_dense(family)) require(in->offsets != nullptr, std::string(what) + ".offsets is NULL");
}

static flinng_input slice(const flinng_input &in, const Index &ix, uint64_t begin, uint64_t n) {
    flinng_input s = in;
    s.count = n;
    if (is_dense(ix.p.family)) {
        const size_t esz = ix.p.family == FLINNG_SRP_F32 ? 4 : 2;
        s.values = static_cast<const char *>(in.values) + begin * ix.p.dim * esz;
    } else {
        s.offsets = in.offsets + begin;
    }
    return s;
}

static void free_index(Index *ix) {
    if (!ix) return;
    (void)hipSetDevice(ix->device);
    (void)hipDeviceSynchronize();  // queries may still be running on any stream
    for (auto &e : ix->scratch) e->release();
    for (auto &r : ix->readbacks) {
        (void)hipEventDestroy(r.ready);
        (void)hipHostFree(r.host);
    }
    // (mem holds the member arrays, hyp the hyperplanes' arrays)
    for (void *p : {static_cast<void *>(ix->offsets), ix->cells, static_cast<void *>(ix->grp),
                    static_cast<void *>(ix->mem), static_cast<void *>(ix->hyp)})
        pool_free(p);
    if (ix->counted) pool_live(ix->device, -1);
    delete ix;
}

template <class T>
static T *dmalloc(uint64_t n, hipStream_t s) {
    return static_cast<T *>(pool_malloc(std::max<uint64_t>(n, 1) * sizeof(T), s));
}

}  // namespace flinng

using namespace flinng;

extern "C" {

const char *flinng_last_error(void) { return g_err.c_str(); }

}  // extern "C"

static void build_impl(const flinng_params *p, const flinng_input *data, hipStream_t s,
                       flinng_index **out, const TextSource *text = nullptr) {
    require(p && data && out, "NULL argument");
    *out = nullptr;
    validate_input(data, p->family, "data");
    validate_params(*p, data->count);
    Index *ix = new Index();
    try {
        ix->p = *p;
        ix->N = data->count;
        FL_HIP(hipGetDevice(&ix->device));
        pool_live(ix->device, 1);
        ix->counted = true;
        const bool dense = is_dense(p->family);
        ix->nbits = dense ? p->K : p->bucket_bits;
        if (dense) ix->p.bucket_bits = p->K;
        ix->dpad = dense ? ((p->dim + 31) / 32) * 32 : 0;
        ix->Rp = 1;
        while (ix->Rp < p->R) ix->Rp <<= 1;
        const uint32_t Bp = (p->B + 3) & ~3u;
        ix->cell_bytes = ((uint64_t)p->R * Bp <= 65536) ? 2 : 4;
        const uint64_t N = ix->N;
        ix->N0 = N;
        ix->grp_cap = N;
        ix->grp = dmalloc<uint16_t>(N * ix->Rp, s);
        const uint64_t gmax = (N + p->B - 1) / p->B;
        ix->mstride = (uint32_t)((gmax + 3) & ~3ull);
        const MemberLayout ml((uint64_t)p->R * p->B, ix->mstride, ix->Rp);
        char *mem = dmalloc<char>(ml.total, s);
        ix->mem = reinterpret_cast<uint32_t *>(mem);
        ix->cmg = reinterpret_cast<uint16_t *>(mem + ml.cmg);
        ix->cfl = reinterpret_cast<uint32_t *>(mem + ml.cfl);
        ix->gsize = reinterpret_cast<uint32_t *>(mem + ml.gsize);
        if (dense) {
            const uint64_t H = (uint64_t)p->L * p->K;
            Pieces hp;
            const size_t o_hyp = hp.add(H * ix->dpad * 2), o_norm = hp.add(H * 4);
            const size_t o_tiled = hp.add(p->family == FLINNG_SRP_BF16 ? (H + 15) / 16 * 16 * ix->dpad * 2 : 0);
            char *h = dmalloc<char>(hp.total, s);
            ix->hyp = reinterpret_cast<uint16_t *>(h + o_hyp);
            ix->hypnorm = reinterpret_cast<float *>(h + o_norm);
            if (p->family == FLINNG_SRP_BF16) ix->hypt = reinterpret_cast<uint16_t *>(h + o_tiled);
            srp_make_hyperplanes(*ix, s);
        }
        // hash all points (in chunks to bound scratch memory)
        DevBuf codes = DevBuf::pooled(N * p->L * 4, s), ctrs = DevBuf::pooled(dense ? 16 : 0, s);
        unsigned long long *ctr = dense ? ctrs.as<unsigned long long>() : nullptr;
        if (ctr) zero_counters(ctr, s);
        // dense chunks bound the SRP scratch (a device copy of host rows,
        // operand planes): 512 MB of bf16 rows (the fused kernel takes them
        // in place, and larger batches fill more rounds of workgroups), or
        // 512 MB of fp32 rows with their three bf16 planes
        const uint64_t per_row =
            (uint64_t)ix->dpad * (p->family == FLINNG_SRP_BF16 ? 2 : 16);
        const uint64_t chunk = dense ? std::max<uint64_t>(1, (1ull << 29) / per_row) : (1ull << 20);
        for (uint64_t b0 = 0; b0 < N; b0 += chunk) {
            const uint64_t n = std::min(chunk, N - b0);
            if (text) {
                TextSource part = *text;
                part.offsets += b0;
                minhash_hash_text(*ix, part, n, codes.as<uint32_t>() + b0 * p->L, s);
                continue;
            }
            flinng_input part = slice(*data, *ix, b0, n);
            hash_batch(*ix, part, codes.as<uint32_t>() + b0 * p->L, s, ctr);
        }
        build_groups(*ix, s);
        build_lists(*ix, codes.as<uint32_t>(), s);
        uint64_t counted[2] = {0, 0};
        if (ctr) FL_HIP(hipMemcpyAsync(counted, ctr, 16, hipMemcpyDeviceToHost, s));
        FL_HIP(hipStreamSynchronize(s));
        ix->srp_rechecked = counted[0];
        ix->srp_exact = counted[1];
        ix->device_bytes = index_device_bytes(*ix);
    } catch (...) {
        free_index(ix);
        throw;
    }
    *out = reinterpret_cast<flinng_index *>(ix);
}

extern "C" {

int flinng_build(const flinng_params *p, const flinng_input *data, void *stream,
                 flinng_index **out) {
    return guard([&] { build_impl(p, data, static_cast<hipStream_t>(stream), out); });
}

int flinng_build_text(const flinng_params *p, const flinng_text *data, void *stream,
                      flinng_index **out) {
    return guard([&] {
        require(p && data && out, "NULL argument");
        *out = nullptr;
        validate_text(data, p->family);
        hipStream_t s = static_cast<hipStream_t>(stream);
        const uint64_t nsym = text_symbols(*data);
        Scratch sc(nullptr, s);
        const TextSource tx = text_source(*data, nsym, s, sc);
        flinng_input sets{tx.symbols, tx.offsets, data->count, 1, 0};
        build_impl(p, &sets, s, out, &tx);
    });
}

void flinng_index_free(flinng_index *idx) { free_index(reinterpret_cast<Index *>(idx)); }

int flinng_index_insert(flinng_index *idx, const flinng_input *data, void *stream) {
    return guard([&] {
        require(idx != nullptr, "index is NULL");
        Index &ix = *reinterpret_cast<Index *>(idx);
        validate_input(data, ix.p.family, "data");
        const uint64_t n = data->count;
        if (n == 0) return;
        FL_HIP(hipSetDevice(ix.device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        std::lock_guard<std::mutex> one(ix.insert_mu);
        require(ix.N + n <= 0xFFFFFFFEull, "at most 2^32-2 points");
        const bool dense = is_dense(ix.p.family);
        DevBuf codes = DevBuf::pooled(n * ix.p.L * 4, s), ctrs = DevBuf::pooled(dense ? 16 : 0, s);
        unsigned long long *ctr = dense ? ctrs.as<unsigned long long>() : nullptr;
        if (ctr) zero_counters(ctr, s);
        const uint64_t per_row =
            (uint64_t)ix.dpad * (ix.p.family == FLINNG_SRP_BF16 ? 2 : 16);  // as in the build
        const uint64_t chunk = dense ? std::max<uint64_t>(1, (1ull << 29) / per_row)
                                     : (1ull << 20);
        for (uint64_t b0 = 0; b0 < n; b0 += chunk) {
            const uint64_t m = std::min(chunk, n - b0);
            flinng_input part = slice(*data, ix, b0, m);
            hash_batch(ix, part, codes.as<uint32_t>() + b0 * ix.p.L, s, ctr);
        }
        insert_points(ix, codes.as<uint32_t>(), n, s);
        uint64_t counted[2] = {0, 0};
        if (ctr) {
            FL_HIP(hipMemcpyAsync(counted, ctr, 16, hipMemcpyDeviceToHost, s));
            FL_HIP(hipStreamSynchronize(s));
        }
        std::unique_lock<std::shared_mutex> lk(ix.rw);
        ix.srp_rechecked += counted[0];
        ix.srp_exact += counted[1];
    });
}

int flinng_index_get_info(const flinng_index *idx, flinng_index_info *info) {
    return guard([&] {
        require(idx && info, "NULL argument");
        const Index &ix = *reinterpret_cast<const Index *>(idx);
        std::shared_lock<std::shared_mutex> rl(ix.rw);
        std::memset(info, 0, sizeof(*info));
        info->N = ix.N;
        info->list_entries = ix.list_entries;
        info->device_bytes = ix.device_bytes;
        info->family = ix.p.family;
        info->dim = ix.p.dim;
        info->K = ix.p.K;
        info->L = ix.p.L;
        info->R = ix.p.R;
        info->B = ix.p.B;
        info->bucket_bits = ix.nbits;
        info->cell_id_bytes = ix.cell_bytes;
        info->srp_rechecked = ix.srp_rechecked;
        info->srp_exact = ix.srp_exact;
    });
}

}  // extern "C"

static void *region_malloc(size_t bytes) {
    void *p = nullptr;
    const hipError_t err = hipMalloc(&p, bytes);
    if (err != hipSuccess) {
        (void)hipGetLastError();
        fail(err == hipErrorOutOfMemory ? FLINNG_ENOMEM : FLINNG_EDEVICE,
             "device allocation of " + std::to_string(bytes) + " bytes failed");
    }
    return p;
}

// The index's region for stream s, its codes at least `bytes` long, with its
// small piece if asked for, and its lock (see Index::StreamScratch).  At most 8
// streams are remembered; the oldest that no call holds is evicted.
using ScratchLock = std::unique_lock<std::mutex>;
static std::shared_ptr<Index::StreamScratch> lock_scratch(const Index &ix, hipStream_t s, size_t bytes,
                                                          bool small, ScratchLock &lock) {
    std::shared_ptr<Index::StreamScratch> e;
    for (;;) {
        {
            std::lock_guard<std::mutex> lk(ix.scratch_mu);
            e.reset();
            for (auto &x : ix.scratch)
                if (x->stream == s) e = x;
            if (!e) {
                for (auto it = ix.scratch.begin(); ix.scratch.size() >= 8 && it != ix.scratch.end();) {
                    ScratchLock l((*it)->mu, std::try_to_lock);
                    if (!l) {
                        ++it;
                        continue;
                    }
                    (*it)->release();
                    (*it)->evicted = true;
                    l.unlock();
                    it = ix.scratch.erase(it);
                }
                e = std::make_shared<Index::StreamScratch>();
                e->stream = s;
                ix.scratch.push_back(e);
            }
        }
        lock = ScratchLock(e->mu);
        if (!e->evicted) break;
        lock.unlock();
    }
    if (small && !e->small) e->small = region_malloc(SMALL_SCRATCH);
    if (e->cap >= bytes) return e;
    if (e->ptr) (void)hipFree(e->ptr);  // waits for the work using it
    e->ptr = nullptr;
    e->cap = 0;
    const size_t cap = std::max<size_t>(bytes, 64 * 1024);
    e->ptr = region_malloc(cap);
    e->cap = cap;
    return e;
}

namespace {

// A Readback of the index for one call; waited for before it is given back.
struct ReadbackLease {
    const Index &ix;
    Index::Readback r{};
    bool pending = false;
    explicit ReadbackLease(const Index &i) : ix(i) {
        {
            std::lock_guard<std::mutex> lk(ix.readback_mu);
            if (!ix.readbacks.empty()) {
                r = ix.readbacks.back();
                ix.readbacks.pop_back();
                return;
            }
        }
        void *p = nullptr;
        FL_HIP(hipHostMalloc(&p, 16, hipHostMallocDefault));
        r.host = static_cast<uint64_t *>(p);
        if (hipEventCreateWithFlags(&r.ready, hipEventDisableTiming) != hipSuccess) {
            (void)hipHostFree(p);
            fail(FLINNG_EDEVICE, "event creation failed");
        }
    }
    void wait() {
        if (!pending) return;
        pending = false;
        FL_HIP(hipEventSynchronize(r.ready));
    }
    ~ReadbackLease() {
        if (pending) (void)hipEventSynchronize(r.ready);
        try {
            std::lock_guard<std::mutex> lk(ix.readback_mu);
            ix.readbacks.push_back(r);
        } catch (...) {  // no room to remember it: not kept
            (void)hipEventDestroy(r.ready);
            (void)hipHostFree(r.host);
        }
    }
};

}  // namespace

// check: the offsets of a text batch on the device, on their way to the host;
// waited for once the hashing is queued, and nothing is written to the outputs
// of a batch that is refused.
static void query_impl(const flinng_index *idx, const flinng_input *q, uint32_t k, uint32_t *ids,
                       uint32_t *scores, uint32_t out_on_device, uint32_t persistent,
                       void *stream, const TextSource *text = nullptr, ReadbackLease *check = nullptr) {
    require(idx != nullptr, "index is NULL");
    const Index &ix = *reinterpret_cast<const Index *>(idx);
    validate_input(q, ix.p.family, "queries");
    require(ids != nullptr, "ids is NULL");
    require(k >= 1 && k <= query_max_k(), "k must be in 1..4096");
    const uint64_t nq = q->count;
    if (nq == 0) return;
    FL_HIP(hipSetDevice(ix.device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    std::shared_lock<std::shared_mutex> rl(ix.rw);  // one index version per call
    // the region of this stream holds the codes and, for a batch whose other
    // scratch is small, that too (a copy of host rows, the SRP stage's planes,
    // results on their way to the host): a lookup of one row then allocates
    // nothing
    const bool dense = is_dense(ix.p.family), host_rows = dense && !q->on_device;
    const size_t row_bytes = (size_t)ix.p.dim * (ix.p.family == FLINNG_SRP_F32 ? 4 : 2);
    const size_t code_bytes = Arena::round((size_t)nq * ix.p.L * 4) + Arena::round(4);
    const size_t in_bytes = host_rows ? Arena::round(nq * row_bytes) : 0;
    const size_t res_bytes = out_on_device ? 0 : Arena::round((size_t)nq * k * 4) * (scores ? 2 : 1);
    const size_t srp_bytes = dense ? srp_scratch_bytes(ix, nq, host_rows ? nullptr : q->values) : 0;
    const bool all = in_bytes + res_bytes + srp_bytes <= SMALL_SCRATCH;
    ScratchLock lock;
    // (a dense index's regions have the small piece from the first call on, so
    // that a later call under capture finds it)
    const auto region = lock_scratch(ix, s, code_bytes, dense || (all && res_bytes > 0), lock);
    Arena c{static_cast<char *>(region->ptr), code_bytes, 0};
    Arena a{static_cast<char *>(region->small), SMALL_SCRATCH, 0};
    uint32_t *codes = static_cast<uint32_t *>(c.take((size_t)nq * ix.p.L * 4));
    uint32_t *work = static_cast<uint32_t *>(c.take(4));
    if (text) {
        minhash_hash_text(ix, *text, nq, codes, s);
        if (check) {
            check->wait();
            require(check->r.host[1] >= check->r.host[0], "text offsets must be nondecreasing");
        }
    } else if (all && dense) {
        flinng_input in = *q;
        if (host_rows) {
            in.values = a.take(nq * row_bytes);
            in.on_device = 1;
            FL_HIP(hipMemcpyAsync(const_cast<void *>(in.values), q->values, nq * row_bytes,
                                  hipMemcpyHostToDevice, s));
        }
        hash_batch(ix, in, codes, s, nullptr, &a);
    } else {
        hash_batch(ix, *q, codes, s, nullptr);
    }
    if (out_on_device) {
        query_launch(ix, codes, nq, k, ids, scores, persistent != 0, s, work);
        lock.unlock();
        rl.unlock();
    } else {
        DevBuf own;
        uint32_t *dids, *dsc = nullptr;
        if (all) {
            dids = static_cast<uint32_t *>(a.take(nq * k * 4));
            if (scores) dsc = static_cast<uint32_t *>(a.take(nq * k * 4));
        } else {
            own = DevBuf(nq * k * 8, s);
            dids = own.as<uint32_t>();
            if (scores) dsc = dids + nq * k;
        }
        query_launch(ix, codes, nq, k, dids, dsc, persistent != 0, s, work);
        rl.unlock();
        // results in the region: it stays this call's until they are copied
        if (!all) lock.unlock();
        FL_HIP(hipMemcpyAsync(ids, dids, nq * k * 4, hipMemcpyDeviceToHost, s));
        if (scores) FL_HIP(hipMemcpyAsync(scores, dsc, nq * k * 4, hipMemcpyDeviceToHost, s));
        FL_HIP(hipStreamSynchronize(s));
    }
}

extern "C" {

int flinng_query(const flinng_index *idx, const flinng_input *q, uint32_t k, uint32_t *ids,
                 uint32_t *scores, uint32_t out_on_device, uint32_t persistent, void *stream) {
    return guard([&] { query_impl(idx, q, k, ids, scores, out_on_device, persistent, stream); });
}

int flinng_query_text(const flinng_index *idx, const flinng_text *q, uint32_t k, uint32_t *ids,
                      uint32_t *scores, uint32_t out_on_device, uint32_t persistent, void *stream) {
    return guard([&] {
        require(idx != nullptr, "index is NULL");
        const Index &ix = *reinterpret_cast<const Index *>(idx);
        validate_text(q, ix.p.family);
        if (q->count == 0) return;
        FL_HIP(hipSetDevice(ix.device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        Scratch sc(nullptr, s);
        if (!q->on_device) {
            const TextSource tx = text_source(*q, text_symbols(*q), s, sc);
            const flinng_input sets{tx.symbols, tx.offsets, q->count, 1, 0};
            query_impl(idx, &sets, k, ids, scores, out_on_device, persistent, stream, &tx);
            return;
        }
        // nothing may be recorded into a graph: it would write the words read back
        // when another call has them
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cap) != hipSuccess) {  // the legacy stream beside a capture
            (void)hipGetLastError();
            cap = hipStreamCaptureStatusNone;
        }
        require(cap == hipStreamCaptureStatusNone, "device text cannot be queried under stream capture");
        // the first and last offset are read back while the batch is hashed (which
        // reads no symbol where they decrease)
        ReadbackLease rb(ix);
        FL_HIP(hipMemcpyAsync(rb.r.host, q->offsets, 8, hipMemcpyDeviceToHost, s));
        FL_HIP(hipMemcpyAsync(rb.r.host + 1, q->offsets + q->count, 8, hipMemcpyDeviceToHost, s));
        FL_HIP(hipEventRecord(rb.r.ready, s));
        rb.pending = true;
        const TextSource tx = text_source(*q, 0, s, sc);
        const flinng_input sets{tx.symbols, tx.offsets, q->count, 1, 0};
        query_impl(idx, &sets, k, ids, scores, out_on_device, persistent, stream, &tx, &rb);
    });
}

int flinng_query_threshold(const flinng_index *idx, const flinng_input *q, uint32_t t,
                           uint32_t max_per_query, uint32_t *ids, uint32_t *counts,
                           uint32_t out_on_device, void *stream) {
    return guard([&] {
        require(idx != nullptr, "index is NULL");
        const Index &ix = *reinterpret_cast<const Index *>(idx);
        validate_input(q, ix.p.family, "queries");
        require(counts != nullptr, "counts is NULL");
        require(ids != nullptr || max_per_query == 0, "ids is NULL");
        const uint64_t nq = q->count;
        if (nq == 0) return;
        require(nq * (uint64_t)max_per_query <= (1ull << 40), "nq * max_per_query too large");
        FL_HIP(hipSetDevice(ix.device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        DevBuf codes(nq * ix.p.L * 4, s);
        hash_batch(ix, *q, codes.as<uint32_t>(), s, nullptr);
        std::shared_lock<std::shared_mutex> rl(ix.rw);
        if (out_on_device) {
            threshold_launch(ix, codes.as<uint32_t>(), nq, t, max_per_query, ids, counts, s);
        } else {
            DevBuf dids(nq * max_per_query * 4, s), dcnt(nq * 4, s);
            threshold_launch(ix, codes.as<uint32_t>(), nq, t, max_per_query, dids.as<uint32_t>(),
                             dcnt.as<uint32_t>(), s);
            if (max_per_query)
                FL_HIP(hipMemcpyAsync(ids, dids.ptr, nq * max_per_query * 4, hipMemcpyDeviceToHost, s));
            FL_HIP(hipMemcpyAsync(counts, dcnt.ptr, nq * 4, hipMemcpyDeviceToHost, s));
            FL_HIP(hipStreamSynchronize(s));
        }
    });
}

int flinng_query_codes(const flinng_index *idx, const uint32_t *codes, uint64_t nq, uint32_t k,
                       uint32_t *ids, uint32_t *scores, uint32_t persistent, uint64_t *stats,
                       void *stream) {
    return guard([&] {
        require(idx && codes && ids, "NULL argument");
        require(k >= 1 && k <= query_max_k(), "k must be in 1..4096");
        if (nq == 0) return;
        const Index &ix = *reinterpret_cast<const Index *>(idx);
        FL_HIP(hipSetDevice(ix.device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        DevBuf work(persistent ? 4 : 0, s);
        std::shared_lock<std::shared_mutex> rl(ix.rw);
        query_launch(ix, codes, nq, k, ids, scores, persistent != 0, s, work.as<uint32_t>(),
                     reinterpret_cast<unsigned long long *>(stats));
    });
}

int flinng_debug_hash(const flinng_index *idx, const flinng_input *q, uint32_t *codes,
                      uint32_t out_on_device, void *stream) {
    return guard([&] {
        require(idx && codes, "NULL argument");
        const Index &ix = *reinterpret_cast<const Index *>(idx);
        validate_input(q, ix.p.family, "queries");
        const uint64_t nq = q->count;
        if (nq == 0) return;
        FL_HIP(hipSetDevice(ix.device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        if (out_on_device) {
            hash_batch(ix, *q, codes, s, nullptr);
        } else {
            DevBuf d(nq * ix.p.L * 4, s);
            hash_batch(ix, *q, d.as<uint32_t>(), s, nullptr);
            FL_HIP(hipMemcpyAsync(codes, d.ptr, nq * ix.p.L * 4, hipMemcpyDeviceToHost, s));
            FL_HIP(hipStreamSynchronize(s));
        }
    });
}

int flinng_debug_projections(const flinng_index *idx, const flinng_input *q, float *proj,
                             double *bound, uint32_t out_on_device, void *stream) {
    return guard([&] {
        require(idx != nullptr, "index is NULL");
        const Index &ix = *reinterpret_cast<const Index *>(idx);
        require(is_dense(ix.p.family), "projections exist for dense (SRP) indexes only");
        if (bound) srp_bound(ix, &bound[0], &bound[1]);
        if (!proj) return;
        validate_input(q, ix.p.family, "queries");
        const uint64_t nq = q->count;
        if (nq == 0) return;
        FL_HIP(hipSetDevice(ix.device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        const uint64_t H = (uint64_t)ix.p.L * ix.p.K;
        DevBuf codes(nq * ix.p.L * 4, s);
        if (out_on_device) {
            srp_hash(ix, *q, codes.as<uint32_t>(), s, nullptr, nullptr, proj);
        } else {
            DevBuf d(nq * H * 4, s);
            srp_hash(ix, *q, codes.as<uint32_t>(), s, nullptr, nullptr, d.as<float>());
            FL_HIP(hipMemcpyAsync(proj, d.ptr, nq * H * 4, hipMemcpyDeviceToHost, s));
            FL_HIP(hipStreamSynchronize(s));
        }
    });
}

int flinng_debug_counts(const flinng_index *idx, const flinng_input *q, uint8_t *counts,
                        uint32_t out_on_device, void *stream) {
    return guard([&] {
        require(idx && counts, "NULL argument");
        const Index &ix = *reinterpret_cast<const Index *>(idx);
        validate_input(q, ix.p.family, "queries");
        const uint64_t nq = q->count;
        if (nq == 0) return;
        FL_HIP(hipSetDevice(ix.device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        const uint64_t nc = (uint64_t)ix.p.R * ix.p.B;
        DevBuf codes(nq * ix.p.L * 4, s);
        hash_batch(ix, *q, codes.as<uint32_t>(), s, nullptr);
        std::shared_lock<std::shared_mutex> rl(ix.rw);
        if (out_on_device) {
            counts_launch(ix, codes.as<uint32_t>(), nq, counts, s);
        } else {
            DevBuf d(nq * nc, s);
            counts_launch(ix, codes.as<uint32_t>(), nq, d.as<uint8_t>(), s);
            FL_HIP(hipMemcpyAsync(counts, d.ptr, nq * nc, hipMemcpyDeviceToHost, s));
            FL_HIP(hipStreamSynchronize(s));
        }
    });
}

int flinng_index_export(const flinng_index *idx, uint64_t *offsets, uint32_t *cells,
                        uint32_t *groups, void *stream) {
    return guard([&] {
        require(idx != nullptr, "index is NULL");
        const Index &ix = *reinterpret_cast<const Index *>(idx);
        FL_HIP(hipSetDevice(ix.device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        std::shared_lock<std::shared_mutex> rl(ix.rw);
        const uint64_t nbk = nbuckets(ix);
        const uint32_t B = ix.p.B, Bp = (B + 3) & ~3u;
        if (offsets) {
            std::vector<uint32_t> o((size_t)ix.p.L * (nbk + 1));
            FL_HIP(hipMemcpyAsync(o.data(), ix.offsets, o.size() * 4, hipMemcpyDeviceToHost, s));
            FL_HIP(hipStreamSynchronize(s));
            for (size_t i = 0; i < o.size(); ++i) offsets[i] = o[i];
        }
        if (cells) {
            const uint64_t n = ix.list_entries;
            if (ix.cell_bytes == 2) {
                std::vector<uint16_t> c(n);
                if (n) FL_HIP(hipMemcpyAsync(c.data(), ix.cells, n * 2, hipMemcpyDeviceToHost, s));
                FL_HIP(hipStreamSynchronize(s));
                for (uint64_t i = 0; i < n; ++i) cells[i] = (c[i] / Bp) * B + c[i] % Bp;
            } else {
                std::vector<uint32_t> c(n);
                if (n) FL_HIP(hipMemcpyAsync(c.data(), ix.cells, n * 4, hipMemcpyDeviceToHost, s));
                FL_HIP(hipStreamSynchronize(s));
                for (uint64_t i = 0; i < n; ++i) cells[i] = (c[i] / Bp) * B + c[i] % Bp;
            }
        }
        if (groups) {
            std::vector<uint16_t> g(ix.N * ix.Rp);
            FL_HIP(hipMemcpyAsync(g.data(), ix.grp, g.size() * 2, hipMemcpyDeviceToHost, s));
            FL_HIP(hipStreamSynchronize(s));
            for (uint32_t r = 0; r < ix.p.R; ++r)
                for (uint64_t x = 0; x < ix.N; ++x) groups[(uint64_t)r * ix.N + x] = g[x * ix.Rp + r];
        }
    });
}

}  // extern "C"
