// N-gram item sets of symbol sequences: argument checks and the staging of
// host text; the items themselves are made inside the MinHash kernel
// (hash_minhash.hip), the step after (the paper hashes genome reads and URLs as
// sets of n-grams, Section 7, Experiments, "Datasets").
//
// Sequence s (symbols s_0 .. s_{len-1}, each below the radix) is the set of
// its windows p = 0 .. len - n: the window's value is the base-radix number
// v = sum_i s_{p+i} radix^(n-1-i), and its item is MurmurHash3's 64-bit
// finaliser of v XOR key (64-bit items) or its 32-bit finaliser of the low
// 32 bits of v XOR key (32-bit items) (Appleby, MurmurHash3, public domain).
// A sequence shorter than n has no items (its MinHash is that of the empty
// set).  Duplicate windows give duplicate items, which MinHash ignores.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "flinng_internal.h"

namespace flinng {

void validate_text(const flinng_text *t, uint32_t family) {
    if (!t) fail(FLINNG_EINVAL, "text input is NULL");
    if (t->reserved != 0) fail(FLINNG_EINVAL, "text.reserved must be 0");
    if (t->on_device > 1) fail(FLINNG_EINVAL, "text.on_device must be 0 or 1");
    if (family != FLINNG_MINHASH_U32 && family != FLINNG_MINHASH_U64)
        fail(FLINNG_EINVAL, "n-gram text feeds a MinHash index");
    if (t->radix < 2 || t->radix > 256) fail(FLINNG_EINVAL, "text.radix must be in 2..256");
    if (t->gram < 1) fail(FLINNG_EINVAL, "text.gram must be >= 1");
    // radix^gram <= 2^64: the window value fits 64 bits
    long double cap = 1.0L;
    for (uint32_t i = 0; i < t->gram; ++i) {
        cap *= t->radix;
        if (cap > 18446744073709551616.0L) fail(FLINNG_EINVAL, "text.radix^gram exceeds 2^64");
    }
    if (t->count && !t->offsets) fail(FLINNG_EINVAL, "text.offsets is NULL");
}

uint64_t text_symbols(const flinng_text &t) {
    if (t.count == 0) return 0;
    uint64_t first = 0, last = 0;
    if (t.on_device) {
        FL_HIP(hipMemcpy(&first, t.offsets, 8, hipMemcpyDeviceToHost));
        FL_HIP(hipMemcpy(&last, t.offsets + t.count, 8, hipMemcpyDeviceToHost));
    } else {
        first = t.offsets[0];
        last = t.offsets[t.count];
    }
    if (last < first) fail(FLINNG_EINVAL, "text offsets must be nondecreasing");
    return last - first;
}

TextSource text_source(const flinng_text &t, uint64_t nsym, hipStream_t s, Scratch &sc) {
    const uint64_t n = t.count;
    TextSource tx{t.symbols, t.offsets, t.key, t.gram, t.radix};
    if (t.on_device) return tx;
    // symbols of the sequences and their offsets rebased to them
    std::vector<uint64_t> ro(n + 1);
    for (uint64_t i = 0; i <= n; ++i) {
        if (i && t.offsets[i] < t.offsets[i - 1])
            fail(FLINNG_EINVAL, "text offsets must be nondecreasing");
        ro[i] = t.offsets[i] - t.offsets[0];
    }
    uint8_t *dsym = sc.get<uint8_t>(std::max<uint64_t>(nsym, 1));
    uint64_t *doff = sc.get<uint64_t>((n + 1) * 8);
    if (nsym) FL_HIP(hipMemcpyAsync(dsym, t.symbols + t.offsets[0], nsym, hipMemcpyHostToDevice, s));
    FL_HIP(hipMemcpyAsync(doff, ro.data(), (n + 1) * 8, hipMemcpyHostToDevice, s));
    FL_HIP(hipStreamSynchronize(s));  // ro is the copy's source
    tx.symbols = dsym;
    tx.offsets = doff;
    return tx;
}

}  // namespace flinng
