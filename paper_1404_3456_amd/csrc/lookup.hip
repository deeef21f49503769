// lookup.hip -- the suffix-array interval of the suffixes that start with a pattern.
//
// Sec. IV: the paper builds the suffix array in order to search it, deciding whether one
// string (a fragment, the paper's "ID matching") is a prefix of a suffix.  For a pattern P over
// A, C, G, T the suffixes that start with P form one interval [lo, hi) of the array: lo is the
// first index whose suffix does not sort below P, hi the first whose suffix sorts above it.
// One thread per pattern searches for both ends of the interval together until it meets a
// suffix that starts with P, then for each end in its half.  Every suffix between two suffixes that
// share x bases with P shares them too, so each comparison resumes at the smaller of the
// prefix lengths P shares with the current interval's two ends (Manber and Myers) and then
// compares 32 bases per step from 2-bit windows; a separator ends a suffix below any base.
//
// The search starts between two samples: every stride-th suffix's first kSampleD bases as one
// word that orders like them, so that a step is one load from an array that stays in L2 (the
// first steps read a part of it held in LDS) instead of a position and a window of the text,
// one after the other.
#include "device.hpp"
#include "internal.hpp"
#include "text.hpp"

namespace saasm {

constexpr int kSampleD = 29;          // bases of a sample: 58 bits, and their number in 5
constexpr uint32_t kTopSamples = 512; // samples a workgroup of k_lookup holds
constexpr uint64_t kNoSample = ~uint64_t(0);  // of a position that is not in the text

// The first kSampleD bases of a string (the codes' top bits) of which l are there, and l: orders
// like the strings, an end below any base.
__device__ __forceinline__ uint64_t sample_key(uint64_t codes, uint32_t l) {
    l = l < uint32_t(kSampleD) ? l : uint32_t(kSampleD);
    return (l ? (codes & (~uint64_t(0) << (64 - 2 * l))) >> 1 : 0) | l;
}

// Common prefix of two strings as far as their sample keys tell.
__device__ __forceinline__ uint32_t sample_lcp(uint64_t a, uint64_t b) {
    const uint32_t la = uint32_t(a) & 31u, lb = uint32_t(b) & 31u, l = la < lb ? la : lb;
    const uint64_t d = (a ^ b) >> 5;
    const uint32_t same = d ? (uint32_t(__clzll((long long)d)) - 6) >> 1 : uint32_t(kSampleD);
    return same < l ? same : l;
}

// The first pblocks blocks: pattern bytes to 2-bit codes, 16 per word (word w: bytes 16w ..
// 16w+15 of the concatenated patterns, byte 16w in the top bits); bytes other than A, C, G, T
// raise kErrAlphabet.  The others: the samples, one a thread.
// Bound by memory: the bytes of 1 M patterns of 40, 16 a load at any alignment, and half a million
// samples take 31 us (the bytes alone, one a load, 44).
__global__ __launch_bounds__(256) void k_lookup_prep(const uint8_t *__restrict__ pat, int64_t total,
                                                     uint32_t *__restrict__ packed, int64_t nwords,
                                                     uint32_t pblocks, const uint4 *__restrict__ blk,
                                                     const int32_t *__restrict__ sa, uint32_t n,
                                                     uint64_t *__restrict__ samples, uint32_t ns,
                                                     uint32_t stride, uint32_t *err) {
    if (blockIdx.x >= pblocks) {
        const uint32_t j = (blockIdx.x - pblocks) * 256u + threadIdx.x;
        if (j >= ns) return;
        const uint32_t p = uint32_t(sa[size_t(j) * stride]);  // (ns - 1) * stride < n
        uint64_t k = kNoSample;
        if (p < n) {
            const Window t = window_at(blk, p);
            k = sample_key(t.code, t.sep ? uint32_t(__clz(t.sep)) : 32u);
        }
        samples[j] = k;
        return;
    }
    const int64_t w = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (w >= nwords) return;
    uint32_t x = 0;
    bool bad = false;
    if (w * 16 + 16 <= total) {
        const Bytes16 b = *reinterpret_cast<const Bytes16 *>(pat + w * 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bad |= bases_of(b.w[j]) != 0x80808080u;
            x |= codes_packed(codes_of(b.w[j])) << (24 - 8 * j);
        }
    } else {
        for (int j = 0; w * 16 + j < total; ++j) {
            const uint32_t c = pat[w * 16 + j];
            bad |= !(bases_of(c) & 128u);
            x |= (codes_of(c) & 3u) << (30 - 2 * j);
        }
    }
    packed[w] = x;
    if (bad) raise_err(err, kErrAlphabet);
}

// A pattern: m bases from base `at` of the packed patterns; c0 and c1 are its first 64 (bases
// past its end are whatever follows).
struct Pattern {
    uint64_t at, c0, c1;
    uint32_t m;
    // 32 bases from base k <= m on, those past the end anything
    __device__ __forceinline__ uint64_t codes(const uint32_t *__restrict__ ppk, uint32_t k) const {
        if (k < 32) return k ? (c0 << (2 * k)) | (c1 >> (64 - 2 * k)) : c0;
        if (m <= 64 && k < 64) return c1 << (2 * (k - 32));
        return codes_at(ppk, at + k);
    }
};

// Compares P with the suffix at p, whose first k bases are known to equal P's.  Returns < 0 when
// the suffix sorts below P without starting with it, 0 when it starts with P, > 0 when it sorts
// above P; *l = their common prefix (<= P.m).  One record of the text a step: most suffixes
// differ from P within the first.  The text ends with a separator (k_lookup does not search one
// that does not), so no record past it is read.
__device__ __forceinline__ int cmp_suffix(const uint4 *__restrict__ blk,
                                          const uint32_t *__restrict__ ppk, const Pattern &P,
                                          uint32_t p, uint32_t k, uint32_t *l) {
    while (true) {
        const uint32_t rem = P.m - k;
        if (rem == 0) { *l = P.m; return 0; }
        const uint32_t o = (p + k) & 31u, held = 32 - o;  // bases of the record from p + k on
        const uint4 x = blk[(p + k) >> 5];
        const uint64_t text = ((uint64_t(x.x) << 32) | x.y) << (2 * o);
        const uint32_t sep = x.z << o;
        const uint64_t pw = P.codes(ppk, k);
        const uint64_t d = pw ^ text;
        const uint32_t md = d ? uint32_t(__clzll((long long)d)) >> 1 : 32u;
        const uint32_t ms = sep ? uint32_t(__clz(sep)) : 32u;
        const uint32_t c = md < ms ? md : ms;
        if (rem <= (c < held ? c : held)) { *l = P.m; return 0; }  // P ends before any difference
        if (c >= held) { k += held; continue; }
        *l = k + c;
        if (ms <= md) return -1;  // the suffix reaches its separator first
        const uint32_t tb = uint32_t(text >> (62 - 2 * c)) & 3u;
        const uint32_t pb = uint32_t(pw >> (62 - 2 * c)) & 3u;
        return tb < pb ? -1 : 1;
    }
}

// What bounds it: the lines that the last steps' positions and records of the text take from
// beyond L2, at random.  A million patterns of 40 bases over 50.1 M suffixes: 400 us for 20 such
// lines a pattern, 51 G lines a second of the 56 to 73 a plain gather reaches; without the
// samples, with two records a step and the pattern read again at each, 720 us.  A thousand over
// 80,000 suffixes, a serial chain of loads: 30 us, before 60.
__global__ __launch_bounds__(256) void k_lookup(const uint4 *__restrict__ blk,
                                                const int32_t *__restrict__ sa, uint32_t n,
                                                const uint32_t *__restrict__ ppk,
                                                const int64_t *__restrict__ off, int64_t total,
                                                uint32_t npat, const uint64_t *__restrict__ samples,
                                                uint32_t ns, uint32_t stride,
                                                int32_t *__restrict__ lohi, uint32_t *err) {
    __shared__ uint64_t s_top[kTopSamples];
    const uint32_t found = *err;  // by the packing
    const uint32_t step = (ns + kTopSamples - 1) / kTopSamples;  // samples per held one
    const uint32_t nt = ns ? (ns + step - 1) / step : 0;
    for (uint32_t t = threadIdx.x; t < nt; t += 256) s_top[t] = samples[t * step];
    __syncthreads();
    // Without a separator at its end nothing stops a comparison there: a long pattern would be
    // compared with whatever follows the text's records.  (The call fails.)
    if (found & kErrNoSepEnd) return;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= npat) return;
    const int64_t a = off[i], b = off[i + 1];
    if (a < 0 || b < a || b > total || b - a > int64_t(0x7fffffff)) {
        raise_err(err, kErrRange);
        lohi[2 * i] = lohi[2 * i + 1] = 0;
        return;
    }
    const Pattern P = {uint64_t(a), codes_at(ppk, uint64_t(a)),
                       b - a > 32 ? codes_at(ppk, uint64_t(a) + 32) : 0, uint32_t(b - a)};
    const uint32_t m = P.m;
    // All bounds below are found together: L and R, outside which every suffix sorts below P
    // or above it, with P's common prefixes lL and lR with the suffixes just outside; and once
    // a suffix that starts with P is met, mL and mR, between which (mL <= i < mR) all do.
    uint32_t L = 0, R = n, lL = 0, lR = 0, mL = 0, mR = 0;
    bool met = false;
    if (ns) {
        // first: the least key of a string P may be a prefix of; last: the greatest.  A
        // sample below first belongs to a suffix below P, one above last to a suffix above
        // it; a sample between them starts with P, if P is no longer than a sample.
        const uint64_t first = sample_key(P.c0, m);
        const uint64_t last = first | 31u |
                              (m < uint32_t(kSampleD) ? (uint64_t(1) << (63 - 2 * m)) - 1 : 0);
        uint32_t lo = 0, hi = nt;
        while (lo < hi) {
            const uint32_t t = lo + (hi - lo) / 2;
            if (s_top[t] < first) lo = t + 1;
            else hi = t;
        }
        // the samples before lo and at hi, where there are such
        uint64_t below = lo ? s_top[lo - 1] : 0, above = lo < nt ? s_top[lo] : 0;
        hi = lo < nt ? lo * step : ns;
        lo = lo ? (lo - 1) * step + 1 : 0;
        while (lo < hi) {
            const uint32_t t = lo + (hi - lo) / 2;
            const uint64_t k = samples[t];
            if (k < first) { lo = t + 1; below = k; }
            else { hi = t; above = k; }
        }
        const uint32_t c0 = lo;  // samples below first
        uint32_t c1 = c0;        // samples not above last
        if (c0 < ns && above <= last) {
            lo = c0 + 1;
            hi = ns;
            for (uint32_t d = 1; lo + d < hi; d *= 2) {
                if (samples[lo + d] > last) hi = lo + d;
                else lo += d + 1;
            }
            while (lo < hi) {
                const uint32_t t = lo + (hi - lo) / 2;
                if (samples[t] > last) hi = t;
                else lo = t + 1;
            }
            c1 = lo;
            if (c1 < ns) above = samples[c1];
        }
        if (c0 > 0) {
            L = (c0 - 1) * stride + 1;
            lL = sample_lcp(below, first);
        }
        if (c1 < ns) {
            R = c1 * stride;
            if (above == kNoSample) raise_err(err, kErrRange);
            else lR = sample_lcp(above, first);
        }
        if (c1 > c0 && m <= uint32_t(kSampleD)) {
            met = true;
            mL = c0 * stride;
            mR = (c1 - 1) * stride + 1;
        }
    }
    // No suffix that starts with P is known: one below P moves L, one above it R.  An absent
    // pattern thus costs one search, a present one shares most of its path.
    while (!met && L < R) {
        const uint32_t mid = L + (R - L) / 2, k = lL < lR ? lL : lR;
        const uint32_t p = uint32_t(sa[mid]);
        if (p >= n || k >= n - p) { raise_err(err, kErrRange); break; }
        uint32_t l;
        const int c = cmp_suffix(blk, ppk, P, p, k, &l);
        if (c < 0) { L = mid + 1; lL = l; }
        else if (c > 0) { R = mid; lR = l; }
        else { met = true; mL = mid; mR = mid + 1; }
    }
    if (met) {
        // the first in [L, mL] that does not sort below P; P's prefix with the right end is m
        while (L < mL) {
            const uint32_t mid = L + (mL - L) / 2;
            const uint32_t p = uint32_t(sa[mid]);
            if (p >= n || lL >= n - p) { raise_err(err, kErrRange); break; }
            uint32_t l;
            if (cmp_suffix(blk, ppk, P, p, lL, &l) < 0) { L = mid + 1; lL = l; }
            else mL = mid;
        }
        // the first in [mR, R] that sorts above P
        while (mR < R) {
            const uint32_t mid = mR + (R - mR) / 2;
            const uint32_t p = uint32_t(sa[mid]);
            if (p >= n || lR >= n - p) { raise_err(err, kErrRange); break; }
            uint32_t l;
            if (cmp_suffix(blk, ppk, P, p, lR, &l) <= 0) mR = mid + 1;
            else { R = mid; lR = l; }
        }
    } else {
        mL = mR = L;
    }
    lohi[2 * i] = int32_t(mL);
    lohi[2 * i + 1] = int32_t(mR);
}

static int64_t pat_words(int64_t total) { return (total + 15) / 16 + 4; }

constexpr int64_t kMaxSamples = int64_t(1) << 19;
static int64_t max_samples(int64_t n) { return n / 16 + 1 < kMaxSamples ? n / 16 + 1 : kMaxSamples; }

// Bytes of everything but the samples.
static int64_t lookup_base_bytes(int64_t n, int64_t pat_total) {
    Carver c(nullptr, INT64_MAX);
    c.take<uint4>(sepmask_words(n));
    c.take<uint32_t>(pat_words(pat_total));
    c.take<uint32_t>(64);
    return c.off + 256;
}

}  // namespace saasm

using namespace saasm;

extern "C" int64_t sa_lookup_ws_bytes(int64_t n, int64_t pat_total) {
    if (n < 1 || pat_total < 0) return -1;
    Carver c(nullptr, INT64_MAX);
    c.take<uint64_t>(max_samples(n));
    return lookup_base_bytes(n, pat_total) + c.off + 256;
}

extern "C" int sa_lookup(const uint8_t *text, int64_t n, const int32_t *sa, const uint8_t *pat,
                         const int64_t *pat_off, int64_t pat_total, int32_t n_pat, int32_t *lohi,
                         void *ws, int64_t ws_bytes, hipStream_t stream) {
    if (!text || !sa || !pat_off || !ws || (n_pat > 0 && !lohi) || (pat_total > 0 && !pat))
        return fail(SA_ERR_INVALID, "sa_lookup: NULL pointer");
    if (n < 1) return fail(SA_ERR_INVALID, "sa_lookup: n must be >= 1");
    if (n >= kMaxN) return fail(SA_ERR_TOO_LARGE, "sa_lookup: n >= 2^31-2");
    if (n_pat < 0 || pat_total < 0) return fail(SA_ERR_INVALID, "sa_lookup: negative count");
    if (ws_bytes < lookup_base_bytes(n, pat_total))
        return fail(SA_ERR_NOMEM, "sa_lookup: workspace too small");
    if (n_pat == 0) return SA_OK;
    Carver c(ws, ws_bytes);
    uint4 *blk = c.take<uint4>(sepmask_words(n));
    uint32_t *ppk = c.take<uint32_t>(pat_words(pat_total));
    uint32_t *err = c.take<uint32_t>(64);
    // Samples: one for every two patterns and at least 4,096, at most a sixteenth of the
    // suffixes and 2^19 (4 MB, as large as an L2).  Both kernels for a million patterns over
    // 50.1 M suffixes took 496 us with one for every four, 484 for every two, 486 for each:
    // more save steps of the search but cost as much to make.  A workspace without room for
    // them still does: the search then starts from the whole array.
    int64_t ns = 0, stride = 1;
    if (ws_bytes >= sa_lookup_ws_bytes(n, pat_total)) {
        ns = int64_t(n_pat) / 2 > 4096 ? int64_t(n_pat) / 2 : 4096;
        if (ns > max_samples(n)) ns = max_samples(n);
        stride = (n + ns - 1) / ns;
        ns = (n + stride - 1) / stride;
    }
    uint64_t *samples = ns ? c.take<uint64_t>(ns) : nullptr;
    SA_TRY(launch_fill_u32(err, 1, 0, stream));
    SA_TRY(launch_pack(text, n, nullptr, nullptr, nullptr, blk, err, stream));
    const int64_t pw = pat_words(pat_total);
    const uint32_t pblocks = uint32_t((pw + 255) / 256);
    hipLaunchKernelGGL(k_lookup_prep, dim3(pblocks + unsigned((ns + 255) / 256)), dim3(256), 0, stream,
                       pat, pat_total, ppk, pw, pblocks, blk, sa, uint32_t(n), samples, uint32_t(ns),
                       uint32_t(stride), err);
    SA_HIP(hipGetLastError());
    {
        // algorithmic bytes: the pattern and its two result words
        TimedScope ts("lookup", double(pat_total) + 8.0 * double(n_pat), stream, double(n_pat));
        hipLaunchKernelGGL(k_lookup, dim3(unsigned((int64_t(n_pat) + 255) / 256)), dim3(256), 0,
                           stream, blk, sa, uint32_t(n), ppk, pat_off, pat_total,
                           uint32_t(n_pat), samples, uint32_t(ns), uint32_t(stride), lohi, err);
        ts.finish();
    }
    SA_HIP(hipGetLastError());
    uint32_t host[kStWords];
    SA_TRY(read_words(err, host, stream));
    const uint32_t e = host[0];
    if (e & kErrAlphabet)
        return fail(SA_ERR_ALPHABET, "sa_lookup: text or pattern holds a byte other than A, C, G, T (or $ in the text)");
    if (e & kErrNoSepEnd) return fail(SA_ERR_INVALID, "sa_lookup: the text must end with '$'");
    if (e & kErrRange) return fail(SA_ERR_INVALID, "sa_lookup: pattern offsets or suffix array out of range");
    if (e) return fail(SA_ERR_HIP, "sa_lookup: device check failed (code " + std::to_string(e) + ")");
    return SA_OK;
}
