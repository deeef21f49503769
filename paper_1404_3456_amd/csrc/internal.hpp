// internal.hpp -- host-side plumbing shared by the library's translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <new>
#include <string>

#include "../../include/saasm.h"

namespace saasm {

// ---- errors --------------------------------------------------------------------------------
void set_error(const std::string &msg);
int fail(int code, const std::string &msg);

#define SA_HIP(call)                                                                     \
    do {                                                                                 \
        hipError_t e_ = (call);                                                          \
        if (e_ != hipSuccess)                                                            \
            return ::saasm::fail(SA_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

// Runs an entry point's body; a host exception (an allocation that fails, a thread that cannot
// start) becomes an error status instead of crossing the C interface.  The messages are short
// enough to need no allocation themselves.
template <class R, class F>
R guard(F &&body) noexcept {
    try {
        return body();
    } catch (const std::bad_alloc &) {
        set_error("host alloc fail");
        return R(SA_ERR_NOMEM);
    } catch (...) {
        set_error("host failure");
        return R(SA_ERR_HIP);
    }
}

#define SA_TRY(expr)                 \
    do {                             \
        int r_ = (expr);             \
        if (r_ != SA_OK) return r_;  \
    } while (0)

constexpr int64_t kMaxN = (int64_t(1) << 31) - 2;  // n <= kMaxN - 1: labels fit in 31 bits
constexpr uint32_t kDone = 1u << 31;      // bit 31 flag: first member of a group (positions), singleton (rank update)
constexpr uint32_t kRankMask = kDone - 1;
constexpr int kH0 = 29;                   // bases in the first-round key (58 code bits + 5)

// ---- workspace carving -----------------------------------------------------------------------
struct Carver {
    char *base;
    int64_t off = 0;
    int64_t cap;
    Carver(void *p, int64_t c) : base(static_cast<char *>(p)), cap(c) {}
    template <class T>
    T *take(int64_t count) {
        off = (off + 255) & ~int64_t(255);
        T *p = reinterpret_cast<T *>(base ? base + off : nullptr);
        off += count * int64_t(sizeof(T));
        return p;
    }
    bool ok() const { return off <= cap; }
};

// ---- tuning --------------------------------------------------------------------------------
// The shape of a radix pass's workgroup.  Unless the caller fixed it, it depends on the items a
// sort has: small tiles spread few items over the chip, large ones write longer digit runs and
// look back less.  One 9-bit pass, 512 x 8 / 512 x 16 / 1024 x 16: 80 k items 12.5 / 15.8 /
// 21.4 us, 565 k 18.1 / 19.4 / 23.3, 1.6 M 26.3 / 23.4 / 25.7, 3.2 M 38.7 / 32.5 / 28.9, 26 M
// 243 / 202 / 185.
constexpr int64_t kTuneSmallN = int64_t(1) << 20, kTuneMidN = int64_t(1) << 21;
struct Tune {
    int dbits = 9;
    int block = 1024;  // 512 when digits are wider than 9 bits (resolve_tuning)
    int items = 16;
    bool fixed = false;  // the caller's shape, for any number of items
    int tile() const { return block * items; }
    int radix() const { return 1 << dbits; }
    // 11-bit digits have four times the look-back words a tile, so 8 items a thread pay up to half
    // as many items: a 64-bit sort of 500 k 248 us with 8, 251 with 16, of 600 k 262 and 257, of 1 M
    // 298 and 280.
    int64_t small_n() const { return dbits > 9 ? kTuneSmallN / 2 : kTuneSmallN; }
    Tune at(int64_t n) const {
        Tune t = *this;
        if (!fixed && n <= kTuneMidN) {
            t.block = 512;
            t.items = n <= small_n() ? 8 : 16;
        }
        t.fixed = true;
        return t;
    }
};
int resolve_tuning(const sa_tuning *t, Tune *out);

// ---- timing --------------------------------------------------------------------------------
bool timing_on();
struct TimedScope {
    // Records a start event on `stream` when timing is on; finish() records the end event and
    // files the launch under `key` with `bytes` algorithmic bytes.  The second form is for
    // launches whose item count is only known on the device: the record waits until
    // timing_round_items() gives the count for the calling thread's current round tag.
    // `items` counts the launch's units of work (suffixes, reads, pass items); the per-item
    // form takes it from its round's count.
    const char *key;
    double bytes;
    double per_item = 0.0;
    double items = 0.0;
    int64_t tag = -1;
    int mode = 0;
    hipStream_t stream;
    hipEvent_t start = nullptr;
    TimedScope(const char *k, double b, hipStream_t s, double n_items = 0.0);
    TimedScope(const char *k, double fixed_bytes, double per_item_bytes, hipStream_t s);
    void finish();
};
int64_t timing_round_begin();                       // new tag for the calling thread's round
// Units of work of that round: scopes opened in kModeRadix count the items of its large
// groups (sorted by radix passes), the others every active item (0: no bytes).
void timing_round_items(int64_t tag, int64_t items, int64_t big_items);
constexpr int kModeAny = 0, kModeRadix = 1, kModeRuns = 2;
// The unit count that scopes opened by the calling thread from now on take from their round
// (kModeRadix: the large groups' items; otherwise all active items).
void timing_scope_mode(int mode);
void timing_flush();  // resolve pending events (waits for them)
void timing_poll();   // resolve only the pending events that have already completed
void timing_pause(bool on);  // calling thread: no events while a stream is being captured

// ---- kernels exposed across translation units ----------------------------------------------
int64_t packed_words(int64_t n);
int64_t sepmask_words(int64_t n);

// pack: validates the text (err bits OR-ed into *err) and writes those of its forms that are
// asked for (NULL: not): the 2-bit codes, the separator bits, the separators per word, and the
// records for random-access windows (text.hpp; sepmask_words(n) of them).
int launch_pack(const uint8_t *text, int64_t n, uint32_t *packed, uint32_t *sepmask,
                uint32_t *wordcnt, uint4 *blk, uint32_t *err, hipStream_t s);
// exclusive scan of uint32 values into int32 (out[i] = sum of in[0..i)); total -> *total_out
int64_t scan_flags_words(int64_t n);
int launch_scan_u32_i32(const uint32_t *in, int32_t *out, int64_t n, int32_t *total_out,
                        uint64_t *lbflags, uint32_t *ticket, uint32_t *err, hipStream_t s);
int launch_scan_u32_i64(const uint32_t *in, int64_t *out, int64_t n, int64_t *total_out,
                        uint64_t *lbflags, uint32_t *ticket, uint32_t *err, hipStream_t s);
int launch_read_ends(const uint32_t *sepmask, const int32_t *sepcnt, int64_t n, int32_t *read_end,
                     hipStream_t s);
int launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s);
int launch_fill_u64(uint64_t *p, int64_t n, uint64_t v, hipStream_t s);

// LCP array (Kasai's scan; lcp.hip): workspace bytes and the body of sa_lcp.  A failure found
// on the device is written to flag[0] (default: lcp[0]) as the negative status.  `span` bounds
// the range of suffix-array indices and text positions one text's accesses fall in (a batch of
// texts: its largest text; 0: n); it chooses between the two forms of the scan.
int64_t lcp_ws_bytes(int64_t n);
int lcp_run(const uint8_t *text, int64_t n, const int32_t *sa, const int32_t *isa, int32_t *lcp,
            void *ws, int64_t ws_bytes, hipStream_t stream, int32_t *flag = nullptr,
            int64_t span = 0);

// Finishes an LCP array whose negative entries are -1 - (symbols the suffix is known to share with
// its predecessor), by comparing on in the text.  Sets *too_long, and may leave entries
// negative, when some pair shares more than kLcpRestMax symbols past those (then Kasai's scan
// is the way).  list: the indices of `count` entries among which the negative ones are (NULL:
// the first `count` entries).
constexpr uint32_t kLcpRestMax = 2048;
int launch_lcp_rest(const uint8_t *text, const uint32_t *packed, const uint32_t *sepmask, int64_t n,
                    const int32_t *sa, const uint32_t *list, int64_t count, int32_t *lcp, void *ws,
                    int64_t ws_bytes, uint32_t *too_long, uint32_t *err, hipStream_t s);

// radix sort plumbing
struct SortBufs {
    uint64_t *keys[2];
    uint32_t *vals[2];
    uint32_t *hist;     // [kHistParts][passes][radix] per-workgroup partial counts
    uint32_t *gbase;    // [passes][radix] exclusive bases
    uint32_t *tickets;  // [passes]; cleared, with the flags, by the kernel that builds hist
    uint32_t *flags;    // [passes][tiles][radix] look-back words
    uint32_t *err;
};
int sort_passes(int bits, const Tune &t);
int64_t sort_flag_words(int64_t n, int bits, const Tune &t);
void carve_sort(Carver &c, int64_t n, int bits, const Tune &t, SortBufs *b, bool with_items);
// Upper bound on the workgroups of a histogram-producing launch; each writes one partial
// histogram (no global atomics) that the per-pass scan kernel reduces.
constexpr int kHistParts = 1024;
// Histogram (and cleared tickets and flags) of keys[cur] for all passes (when the producer did not build it); the number of
// partial histograms written goes to *nparts.
int launch_hist(const SortBufs &b, int cur, int64_t n, int bit_lo, int bits, const Tune &t,
                hipStream_t s, int *nparts);
// Runs the passes over n items (or, when count_dev is given, over the count read from device
// memory, at most n); returns the buffer index holding the sorted data in *cur_out.
// index_vals: vals[cur] is not read, each item's value is its index.
int sort_run(const SortBufs &b, int cur, const uint32_t *count_dev, int64_t n, int bit_lo,
             int bits, const Tune &t, int nparts, hipStream_t s, int *cur_out,
             bool index_vals = false);

// Device-side round state of a suffix-array build (words of a uint32 array).
constexpr int kStErr = 0;      // error bits
constexpr int kStActive = 1;   // suffixes in non-singleton groups entering the next round
constexpr int kStH = 3;        // prefix length the groups are sorted by
constexpr int kStRounds = 4;   // rounds completed
constexpr int kStNext = 5;     // active count produced by the round's rank update
constexpr int kStBig = 6;      // 1: some group entering the round has more than kRunMax members
constexpr int kStRadixN = 7;   // items of large groups the round sorts by radix passes
constexpr int kStBigNext = 8;  // set by the rank update for the next round
constexpr int kStBigLast = 9;  // kStRadixN of the round that ended (read back for timing)
constexpr int kStLongRun = 10; // first round: a run of equal top key bits is too long for LDS
constexpr int kStNoExt = 11;   // first round: some group is equal on the h0 symbols of its key only
constexpr int kStLcpLong = 12; // the LCP array needs Kasai's scan (launch_lcp_rest)
constexpr int kStTopN = 13;    // first round: items its passes over the top bits sort (n, or 0)
constexpr int kStSample = 14;  // launch_sample_runs: its counts (64 bits)
constexpr int kStWords = 16;   // state words the host reads back
constexpr int kStValid = 16;   // launch_sample_runs: positions that could be sampled
constexpr int kStAll = 17;     // state words
constexpr int kRunMax = 32;    // largest group the run sort handles

// Pinned host words and events for reading device words without a full stream sync (two slots so
// one round's state can be in flight while the other is read, and a third for read_words).
struct PinnedState {
    uint32_t *h = nullptr;
    hipEvent_t ev[2] = {nullptr, nullptr};
    int device = 0;
    PinnedState *next = nullptr;
};
// The calling thread's for the current device, until the thread ends; NULL when none can be made.
PinnedState *pinned_state();
// Copies kStWords device words to the host and waits for the stream: one copy to pinned memory
// (a copy to pageable memory takes two more steps on the host).
int read_words(const uint32_t *dev, uint32_t host[kStWords], hipStream_t s);

// key builders (fused with the histogram of the sort that follows, over key bits
// [lo_bit, key_bits)); a value is its item's index and is left to the first pass.  count_dev: the
// count that the passes read, if they do; no keys are made where it is 0
int launch_key0(const uint32_t *packed, const uint32_t *sepmask, int64_t n, int h0, int top_d, const int64_t *set_off_dev,
                int n_sets, int lo_bit, int key_bits, const uint32_t *count_dev, const SortBufs &b, int cur,
                const Tune &t, hipStream_t s, int *nparts);
// First round (first_round.hip): from items ordered by key bits [lo_bit, key_bits), which tell
// their first top_d bases apart, to labelled groups equal on h0 + kExtBases symbols; and the
// items of runs too long for it, taken out.  Both need their ticket and look-back words (one
// per kFirstMinTile items) cleared.
constexpr int kKeyLenShift = 55;          // a key's top 9 bits: distance to the separator, capped
constexpr uint32_t kKeyLenMax = 511;
constexpr int kExtStage = 57;             // bases one comparison of the extension takes
constexpr int kExtWindows = 4;            // windows of two stages each
constexpr int kExtBases = 2 * kExtStage * kExtWindows;
static_assert(kH0 + kExtBases <= int(kKeyLenMax), "the extension needs exact distances");
constexpr int kFirstMinTile = 896;
int launch_first_runs(const uint64_t *K, const uint32_t *V, const uint32_t *packed, int64_t n,
                      int lo_bit, int key_bits, int top_d, int h0, bool mixed, int32_t *sa,
                      uint32_t *rank, uint32_t *S_new, uint32_t *P_new, int32_t *lcp_or_null,
                      uint64_t *lbflags, int64_t lb_words, uint32_t *tick, uint32_t *state,
                      hipStream_t s);
// Samples the text's suffixes at random, some 2^12 to 2^13 (all positions looked at, `looked`, a
// multiple of kSampleStep and at most kMaxLooked, that fall into a part of the hashes), and sets
// state[kStTopN] to 0 and state[kStLongRun] to 1 when the share of them that are equal to another
// position looked at on top_d bases is at least `enough`, or most positions hold so few different
// bases that the sample misses them.  table: kSampleSlots cleared words.
constexpr int kSampleBlock = 256;
constexpr int kSampleRow = 8;  // positions in a row a thread looks at
constexpr int64_t kSampleStep = int64_t(kSampleBlock) * kSampleRow;
constexpr int64_t kMaxLooked = int64_t(1) << 20;
constexpr int64_t kSampleSlots = int64_t(1) << 14;
int launch_sample_runs(const uint32_t *packed, const uint32_t *sepmask, int64_t n, int top_d,
                       const int64_t *set_off_dev, int n_sets, int64_t looked, double enough,
                       uint32_t *table, uint32_t *state, hipStream_t s);
int launch_first_extract(const uint64_t *K, const uint32_t *V, int64_t n, int lo_bit, int top_d,
                         int key_bits,
                         const SortBufs &b, uint32_t *idx, uint64_t *lbflags, int64_t lb_words,
                         uint32_t *tick, uint32_t *state, const Tune &t, hipStream_t s,
                         int *nparts);
// Keys of the items in groups of more than kRunMax members (sa_build.hip's doubling rounds),
// into b.keys[0]/b.vals[0] with their list indices in bigidx, fused with the histograms.
int launch_big_extract(const uint32_t *P, const uint32_t *S, const uint32_t *rank, int64_t n,
                       int rbits, int64_t a_bound, const SortBufs &b, uint32_t *bigidx,
                       uint64_t *lbflags, int64_t lb_words, uint32_t *tick, uint32_t *state,
                       const Tune &t, hipStream_t s, int *nparts);
// The sorted large items to their indices in the round's full key/value list.
int launch_big_place(const uint64_t *ks, const uint32_t *vs, const uint32_t *bigidx,
                     int64_t a_bound, const uint32_t *state, uint64_t *K, uint32_t *V,
                     uint32_t *err, hipStream_t s);

}  // namespace saasm
