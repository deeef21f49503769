// first_round.hip -- the first round of a suffix-array build, from suffixes ordered by the top
// bits of their first-round keys to groups equal on top_d + kExtBases symbols.
//
// Sec. IV sorts integer keys by radix passes, one digit at a time.  A key of 29 bases (63 bits)
// takes seven 9-bit passes, but two or three passes over its top bits already leave runs of
// equal top bits that are about as short as the final groups: the reads of a 10x coverage put
// about ten copies of a genome stretch side by side, and that is what a run holds.  So only the
// top bits go through passes over HBM; each run is then sorted in LDS by the next kExtBases
// symbols, read from the packed text.  The same kernel finishes the round: it labels groups,
// writes the ranks, the final suffixes and the common prefixes it saw, and compacts the rest
// for the doubling rounds, which start at top_d + kExtBases symbols instead of 29.
//
// A run is a stretch of equal top bits, that is, of suffixes equal on their first top_d bases
// (suffixes that end before top_d bases share theirs only with their equals and are runs of
// their own).  Runs of more than kFrRun suffixes (repeats) do not fit the context a tile loads.
// The plain form of the kernel only reports them; the host then has their items taken out,
// sorted by radix passes over the whole key and put back in place (k_first_extract,
// k_big_place), and runs the other form, which takes such runs as sorted by h0 symbols and
// first sorts the others by them too.  Where nearly all runs are that long, all of this is in vain: a
// sample of the suffixes tells before the first pass (k_sample_runs), and the round sorts by
// whole keys alone.
#include "device.hpp"
#include "internal.hpp"
#include "text.hpp"

namespace saasm {

constexpr int kFrRun = 128;                      // longest run sorted in LDS
constexpr uint32_t kFrNone = 0xffffffffu;        // no item
constexpr int kFrReach = kFrRun / kWave;         // words of a mask a run can reach into
constexpr int kFrNowhere = -2 * kFrRun;          // no start, no end
static_assert(kFrRun % kWave == 0 && kFrRun <= 128, "7 bits tell the members of a group apart");

// The shape of a workgroup and its tile.
template <int BLOCK, int ITEMS, int WAVES_PER_SIMD>
struct FrShape {
    static constexpr int kBlock = BLOCK, kItems = ITEMS, kOcc = WAVES_PER_SIMD;
    static constexpr int kSpan = BLOCK * ITEMS;      // items loaded per tile
    static constexpr int kTile = kSpan - kFrRun;     // items whose runs a tile finishes
    static constexpr int kRows = kSpan / kWave;
    static constexpr int kWaves = BLOCK / kWave;
    static_assert(kTile % kWave == 0 && kRows <= kWave, "rows of the scan");
    static_assert(kTile >= kFirstMinTile, "look-back words are sized for tiles of kFirstMinTile items");
};

// First item of the run that holds item x, from a mask of run starts (bit x % 64 of word
// x / 64 of `rows`; kFrReach words before word 0 are there too): the nearest start at or before x, sought
// kFrReach words back; kFrNowhere if there is none.
__device__ __forceinline__ int run_start(const uint64_t *m, int x) {
    const int w = x >> 6, b = x & 63;
    const uint64_t le = b == 63 ? ~uint64_t(0) : ((uint64_t(2) << b) - 1);
    uint64_t v = m[w] & le;
    int at = w;
    for (int k = 1; k <= kFrReach && !v; ++k) {
        v = m[w - k];
        at = w - k;
    }
    return v ? at * 64 + 63 - int(__clzll((long long)v)) : kFrNowhere;
}

// First item after the run that holds item x: the next start, sought kFrReach words on;
// kFrNowhere if there is none.
__device__ __forceinline__ int run_end(const uint64_t *m, int rows, int x) {
    const int w = x >> 6, b = x & 63;
    const uint64_t le = b == 63 ? ~uint64_t(0) : ((uint64_t(2) << b) - 1);
    uint64_t v = m[w] & ~le;
    int at = w;
    for (int k = 1; k <= kFrReach && !v && w + k < rows; ++k) {
        v = m[w + k];
        at = w + k;
    }
    return v ? at * 64 + int(__ffsll((long long)v)) - 1 : kFrNowhere;
}

// Bounds of the run of item x; whether it is known to have at most kFrRun items.
__device__ __forceinline__ bool run_bounds(const uint64_t *m, int rows, int x, int *st, int *en) {
    *st = run_start(m, x);
    *en = run_end(m, rows, x);
    return *st != kFrNowhere && *en != kFrNowhere && *en - *st <= kFrRun;
}

// The first start at or after item x (word-aligned) of the span; the span's size if none.
__device__ __forceinline__ int first_start(const uint64_t *m, int rows, int x) {
    for (int w = x >> 6; w < rows; ++w) {
        const uint64_t v = m[w];
        if (v) return w * 64 + int(__ffsll((long long)v)) - 1;
    }
    return rows * 64;
}

// 128 bases of the packed text from position a on (base 0 in the top bits of b[0]).
struct Bases {
    uint64_t b[4];
};
struct __attribute__((packed, aligned(4))) Words9 {
    uint32_t w[9];
};
__device__ __forceinline__ Bases bases_at(const uint32_t *__restrict__ packed, uint32_t a) {
    const Words9 q = *reinterpret_cast<const Words9 *>(packed + (a >> 4));
    const uint32_t o = 2 * (a & 15);
    uint32_t r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = __builtin_amdgcn_alignbit(q.w[i], q.w[i + 1], (32 - o) & 31);
    Bases x;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        x.b[i] = o ? (uint64_t(r[2 * i]) << 32) | r[2 * i + 1]
                   : (uint64_t(q.w[2 * i]) << 32) | q.w[2 * i + 1];
    return x;
}

// The kExtStage bases at the top of (w0, w1), of which l are before the separator, as two words
// that order like the symbols: 32 bases; then 25 bases, l in 6 bits, and 7 bits left zero.
// Bases past the separator are zero, so a suffix that ends sorts below those that go on.
__device__ __forceinline__ void stage_key(uint64_t w0, uint64_t w1, uint32_t l, uint64_t *c0,
                                          uint64_t *c1) {
    if (l > uint32_t(kExtStage)) l = kExtStage;
    if (l < 32) {
        w0 &= l ? ~uint64_t(0) << (64 - 2 * l) : 0;
        w1 = 0;
    } else {
        w1 &= l > 32 ? ~uint64_t(0) << (128 - 2 * l) : 0;  // 7 bases and more cleared
    }
    *c0 = w0;
    *c1 = w1 | (uint64_t(l) << 7);
}

// How many of four words q[i], in the lanes of in[i], are below k, added to c: the borrows of
// 32-bit subtraction chains.  As comparisons a two-word key takes four 64-bit ones and their logic,
// twice the instructions, and the compiler turns a chain in C back into them.  The four chains
// take turns, each with its borrow in a register pair of its own: gfx950 wants two wait states
// between a vector instruction that writes a carry and the one that takes it in (the compiler
// puts s_nop 1 there, but looks into no inline assembly), and three instructions lie between.
__device__ __forceinline__ uint32_t add_below(uint32_t c, const uint64_t (&q)[4], uint64_t k,
                                              const uint64_t (&in)[4]) {
    uint32_t t;
    uint64_t b1, b2, b3;
    asm("v_sub_co_u32_e64 %[t], vcc, %[q0l], %[kl]\n\t"
        "v_sub_co_u32_e64 %[t], %[b1], %[q1l], %[kl]\n\t"
        "v_sub_co_u32_e64 %[t], %[b2], %[q2l], %[kl]\n\t"
        "v_sub_co_u32_e64 %[t], %[b3], %[q3l], %[kl]\n\t"
        "v_subb_co_u32_e64 %[t], vcc, %[q0h], %[kh], vcc\n\t"
        "v_subb_co_u32_e64 %[t], %[b1], %[q1h], %[kh], %[b1]\n\t"
        "v_subb_co_u32_e64 %[t], %[b2], %[q2h], %[kh], %[b2]\n\t"
        "v_subb_co_u32_e64 %[t], %[b3], %[q3h], %[kh], %[b3]\n\t"
        "s_and_b64 vcc, vcc, %[i0]\n\t"
        "s_and_b64 %[b1], %[b1], %[i1]\n\t"
        "s_and_b64 %[b2], %[b2], %[i2]\n\t"
        "s_and_b64 %[b3], %[b3], %[i3]\n\t"
        "v_addc_co_u32_e64 %[c], vcc, 0, %[c], vcc\n\t"
        "v_addc_co_u32_e64 %[c], %[b1], 0, %[c], %[b1]\n\t"
        "v_addc_co_u32_e64 %[c], %[b2], 0, %[c], %[b2]\n\t"
        "v_addc_co_u32_e64 %[c], %[b3], 0, %[c], %[b3]"
        : [t] "=&v"(t), [c] "+&v"(c), [b1] "=&s"(b1), [b2] "=&s"(b2), [b3] "=&s"(b3)
        : [q0l] "v"(uint32_t(q[0])), [q0h] "v"(uint32_t(q[0] >> 32)), [q1l] "v"(uint32_t(q[1])),
          [q1h] "v"(uint32_t(q[1] >> 32)), [q2l] "v"(uint32_t(q[2])), [q2h] "v"(uint32_t(q[2] >> 32)),
          [q3l] "v"(uint32_t(q[3])), [q3h] "v"(uint32_t(q[3] >> 32)), [kl] "v"(uint32_t(k)),
          [kh] "v"(uint32_t(k >> 32)), [i0] "s"(in[0]), [i1] "s"(in[1]), [i2] "s"(in[2]), [i3] "s"(in[3])
        : "vcc", "scc");
    return c;
}
// The same for two-word keys (q0, q1) and (k0, k1).
__device__ __forceinline__ uint32_t add_below2(uint32_t c, const uint64_t (&q0)[4],
                                               const uint64_t (&q1)[4], uint64_t k0, uint64_t k1,
                                               const uint64_t (&in)[4]) {
    uint32_t t;
    uint64_t b1, b2, b3;
    asm("v_sub_co_u32_e64 %[t], vcc, %[q0l], %[kl]\n\t"
        "v_sub_co_u32_e64 %[t], %[b1], %[q1l], %[kl]\n\t"
        "v_sub_co_u32_e64 %[t], %[b2], %[q2l], %[kl]\n\t"
        "v_sub_co_u32_e64 %[t], %[b3], %[q3l], %[kl]\n\t"
        "v_subb_co_u32_e64 %[t], vcc, %[q0m], %[km], vcc\n\t"
        "v_subb_co_u32_e64 %[t], %[b1], %[q1m], %[km], %[b1]\n\t"
        "v_subb_co_u32_e64 %[t], %[b2], %[q2m], %[km], %[b2]\n\t"
        "v_subb_co_u32_e64 %[t], %[b3], %[q3m], %[km], %[b3]\n\t"
        "v_subb_co_u32_e64 %[t], vcc, %[q0n], %[kn], vcc\n\t"
        "v_subb_co_u32_e64 %[t], %[b1], %[q1n], %[kn], %[b1]\n\t"
        "v_subb_co_u32_e64 %[t], %[b2], %[q2n], %[kn], %[b2]\n\t"
        "v_subb_co_u32_e64 %[t], %[b3], %[q3n], %[kn], %[b3]\n\t"
        "v_subb_co_u32_e64 %[t], vcc, %[q0h], %[kh], vcc\n\t"
        "v_subb_co_u32_e64 %[t], %[b1], %[q1h], %[kh], %[b1]\n\t"
        "v_subb_co_u32_e64 %[t], %[b2], %[q2h], %[kh], %[b2]\n\t"
        "v_subb_co_u32_e64 %[t], %[b3], %[q3h], %[kh], %[b3]\n\t"
        "s_and_b64 vcc, vcc, %[i0]\n\t"
        "s_and_b64 %[b1], %[b1], %[i1]\n\t"
        "s_and_b64 %[b2], %[b2], %[i2]\n\t"
        "s_and_b64 %[b3], %[b3], %[i3]\n\t"
        "v_addc_co_u32_e64 %[c], vcc, 0, %[c], vcc\n\t"
        "v_addc_co_u32_e64 %[c], %[b1], 0, %[c], %[b1]\n\t"
        "v_addc_co_u32_e64 %[c], %[b2], 0, %[c], %[b2]\n\t"
        "v_addc_co_u32_e64 %[c], %[b3], 0, %[c], %[b3]"
        : [t] "=&v"(t), [c] "+&v"(c), [b1] "=&s"(b1), [b2] "=&s"(b2), [b3] "=&s"(b3)
        : [q0l] "v"(uint32_t(q1[0])), [q0m] "v"(uint32_t(q1[0] >> 32)), [q0n] "v"(uint32_t(q0[0])),
          [q0h] "v"(uint32_t(q0[0] >> 32)), [q1l] "v"(uint32_t(q1[1])), [q1m] "v"(uint32_t(q1[1] >> 32)),
          [q1n] "v"(uint32_t(q0[1])), [q1h] "v"(uint32_t(q0[1] >> 32)), [q2l] "v"(uint32_t(q1[2])),
          [q2m] "v"(uint32_t(q1[2] >> 32)), [q2n] "v"(uint32_t(q0[2])), [q2h] "v"(uint32_t(q0[2] >> 32)),
          [q3l] "v"(uint32_t(q1[3])), [q3m] "v"(uint32_t(q1[3] >> 32)), [q3n] "v"(uint32_t(q0[3])),
          [q3h] "v"(uint32_t(q0[3] >> 32)), [kl] "v"(uint32_t(k1)), [km] "v"(uint32_t(k1 >> 32)),
          [kn] "v"(uint32_t(k0)), [kh] "v"(uint32_t(k0 >> 32)), [i0] "s"(in[0]), [i1] "s"(in[1]),
          [i2] "s"(in[2]), [i3] "s"(in[3])
        : "vcc", "scc");
    return c;
}

// Items y of [st, en) whose word s[y] is below k, four reads at a time (s has four words more
// than it has items).
__device__ __forceinline__ int count_below(const uint64_t *s, int st, int en, uint64_t k) {
    uint32_t c = 0;
    for (int y = st; y < en; y += 4) {
        uint64_t q[4], in[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            q[i] = s[y + i];
            in[i] = ballot(y + i < en);
        }
        c = add_below(c, q, k, in);
    }
    return int(c);
}

// The same for two-word keys.
__device__ __forceinline__ int count_below2(const uint64_t *s0, const uint64_t *s1, int st, int en,
                                             uint64_t k0, uint64_t k1) {
    uint32_t c = 0;
    for (int y = st; y < en; y += 4) {
        uint64_t q0[4], q1[4], in[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            q0[i] = s0[y + i];
            q1[i] = s1[y + i];
            in[i] = ballot(y + i < en);
        }
        c = add_below2(c, q0, q1, k0, k1, in);
    }
    return int(c);
}

// The codes of a key's h0 bases (zeros past its separator).  The string of its first D bases is
// number at = |w| + (4 c - sum w_i) / 3 among all strings (key0_of), so 4 c - sum w_i is known
// and rises by at least 3 with every c: steps by a quarter of what is left, rounded away from
// zero, close in on c (three at most over every case tried up to 20 bases).
__device__ __forceinline__ uint64_t key_codes(uint64_t key, uint32_t lo_bit, uint32_t top_d,
                                              uint32_t h0, uint32_t *err) {
    const uint32_t len = uint32_t(key) & 31u;
    const uint64_t at = (key >> lo_bit) & ((uint64_t(1) << (2 * top_d + 1)) - 1);
    const int64_t m = 3 * int64_t(at - (len < top_d ? len : top_d));
    int64_t c = m >> 2;
    for (int k = 0;; ++k) {
        const int64_t d = m - 4 * c + popc64(uint64_t(c) & 0x5555555555555555ull) +
                          2 * popc64(uint64_t(c) & 0xaaaaaaaaaaaaaaaaull);
        if (d == 0) break;
        if (k == 32) {  // not reached by a key that key0_of made
            raise_err(err, kErrRange);
            break;
        }
        c += d > 0 ? (d + 3) >> 2 : -((3 - d) >> 2);
    }
    const uint32_t rest = 2 * (h0 - top_d);
    return (uint64_t(c) << rest) | ((key >> 5) & ((uint64_t(1) << rest) - 1));
}

// Common prefix of two suffixes that differ within their first h0 symbols, from their keys'
// codes and lengths (the last 5 bits of a and b).
__device__ __forceinline__ uint32_t key_lcp(uint64_t ca, uint64_t cb, uint32_t a, uint32_t b,
                                            uint32_t h0) {
    const uint32_t la = a & 31u, lb = b & 31u, l = la < lb ? la : lb;
    const uint64_t d = ca ^ cb;
    const uint32_t same = d ? (uint32_t(__clzll((long long)d)) - (64 - 2 * h0)) >> 1 : h0;
    return same < l ? same : l;
}

using FrLarge = FrShape<256, 6, 3>;
using FrSmall = FrShape<512, 2, 4>;
constexpr int64_t kFrFewItems = int64_t(1) << 21;

// One tile of the order by the keys' top bits (bits lo_bit and up): sorts its runs, labels its
// groups and writes rank[], the final sa[] entries and the compacted slots and positions of
// the suffixes still in groups, as k_rank_update does for a doubling round.  MIXED: runs of
// more than kFrRun items are in order of the whole key already; otherwise such a run sets
// state[kStLongRun], after which the tiles give up (the host sees the flag and starts over).
// A tile finishes the runs that start among its kFrTile items; kFrRun items more are loaded, so
// they lie in the loaded span as a whole, and of the kFrRun items before it the starts.  In a
// long run the groups equal on the whole key take the runs' part, and single items where those
// are long too.
// LCP: also writes lcp[i] of every suffix told apart from its predecessor here (the keys and
// windows compared hold their common prefix); for the others, which leave in groups, the
// negative of one more than the symbols they are known to share.
// What bounds it: the lines of its gathers, 36 bytes of packed text an item and window, and of the
// ranks it scatters (11.6 GB counted beyond L2 for the 50.1 M suffixes of 10x reads, 3.9 TB/s in
// 3.0 ms, where a copy reaches 5.1), and beside them the comparisons in LDS (about ten items a
// run are compared with each other twice a window).  The four passes, rank updates, sorts of
// runs and Kasai's scan it took the place of were 8.1 ms.
// The plain form's windows follow the run's top bits at once: sorting by the rest of the key
// first costs 18.0 ms against 16.8 over a batch of 210 M suffixes in small sets, and 3.0 either
// way at 50.1 M.  The mixed form does sort by it: repeats make its runs long (40 items and more),
// and comparing one word of the key instead of two of the text tells most of them apart: 23.5
// against 28.7 ms at 400 M suffixes with planted repeats.
template <class Shape, bool MIXED, bool LCP>
__global__ __launch_bounds__(Shape::kBlock, Shape::kOcc) void k_first_runs(
    const uint64_t *__restrict__ K, const uint32_t *__restrict__ V,
    const uint32_t *__restrict__ packed, uint32_t n, uint32_t lo_bit, uint32_t key_bits,
    uint32_t top_d, uint32_t h0, int32_t *__restrict__ sa, uint32_t *__restrict__ rank,
    uint32_t *__restrict__ S_new, uint32_t *__restrict__ P_new, int32_t *__restrict__ lcp,
    uint64_t *lbflags, uint32_t *tick, uint32_t *state, uint32_t *err) {
    constexpr int kFrBlock = Shape::kBlock, kFrItems = Shape::kItems, kFrSpan = Shape::kSpan;
    constexpr int kFrTile = Shape::kTile, kFrRows = Shape::kRows, kFrWaves = Shape::kWaves;
    __shared__ uint64_t s_k[kFrSpan + 4];        // keys; first words of the extension keys
    __shared__ uint64_t s_c[kFrSpan + 4];        // (rest of key, item); second words
    __shared__ uint32_t s_v[kFrSpan];            // text positions, in order
    __shared__ uint16_t s_reach[kFrSpan];        // symbols before the separator (511: or more)
    __shared__ uint16_t s_list[kFrSpan];         // places of the items in groups; s_at
    __shared__ int16_t s_l[LCP ? kFrSpan : 1];   // lcp entries
    uint16_t *const s_at = s_list;               // where a sorted item's words lie
    __shared__ uint32_t s_cnt[kFrRows];
    __shared__ uint64_t s_mw[kFrReach + kFrRows];
    uint64_t *const s_m = s_mw + kFrReach;       // starts of groups
    __shared__ uint64_t s_m0w[MIXED ? kFrReach + kFrRows : 1];
    uint64_t *const s_m0 = MIXED ? s_m0w + kFrReach : s_m;  // starts of runs
    __shared__ uint64_t s_u[MIXED ? kFrRows : 1];  // starts of what a tile takes as a whole
    __shared__ uint64_t s_row[kFrRows];   // (count, last start) before each row
    __shared__ uint32_t s_tile, s_quit;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    // Once a long run is known no workgroup takes another ticket (all take them from one word,
    // one every 11 ns, 3.3 ms for the tiles of 400 M suffixes, 0.2 without): tiles look back at
    // lower tickets only, and every one taken is published.
    if (tid == 0) {
        s_quit = MIXED ? 0u : ld_agent(state + kStLongRun);
        if (!s_quit) s_tile = ticket(tick);
    }
    __syncthreads();
    if (s_quit) return;
    const uint32_t tile = s_tile;
    const uint32_t ntiles = (n + kFrTile - 1) / kFrTile;
    if (tile >= ntiles) return;
    const int64_t lo = int64_t(tile) * kFrTile;
    const uint64_t kmask = (uint64_t(1) << key_bits) - 1;  // key_bits <= kKeyLenShift
    {
        uint64_t k[kFrItems];
        uint32_t v[kFrItems];
#pragma unroll
        for (int j = 0; j < kFrItems; ++j) {
            const int64_t gi = lo + j * kFrBlock + tid;
            const bool in = gi < int64_t(n);
            k[j] = in ? K[gi] : 0;
            v[j] = in ? V[gi] : 0;
        }
        const uint64_t rest = (uint64_t(1) << lo_bit) - 1;  // 31 bits at most
#pragma unroll
        for (int j = 0; j < kFrItems; ++j) {
            const int x = j * kFrBlock + tid;
            s_k[x] = k[j];
            if (MIXED) {
                s_c[x] = ((k[j] & rest) << 32) | uint32_t(x);
            } else {
                s_v[x] = v[j];
                s_reach[x] = uint16_t(k[j] >> kKeyLenShift);
                if (LCP) s_c[x] = key_codes(k[j], lo_bit, top_d, h0, err);  // for neighbours
            }
        }
        // the rows before the span: their starts (in a long run, in order, also of its groups)
        if (wave < uint32_t(kFrReach)) {
            const int64_t gi = lo - kFrRun + int64_t(tid);
            bool h = gi <= 0, g = gi <= 0;
            if (!h) {
                const uint64_t a = K[gi], d = (a ^ K[gi - 1]) & kmask;
                h = d >> lo_bit || (a & 31u) < uint64_t(top_d);
                g = d != 0 || (a & 31u) < uint64_t(h0);
            }
            const uint64_t mh = ballot(h), mg = ballot(g);
            if (lane == 0) {
                s_m0[int(wave) - kFrReach] = mh;
                if (MIXED) s_mw[wave] = mg;
            }
        }
        __syncthreads();
        if (MIXED) {
#pragma unroll
            for (int j = 0; j < kFrItems; ++j) {
                const int x = j * kFrBlock + tid;
                const int64_t gi = lo + x;
                bool h = gi <= 0 || gi >= int64_t(n);
                if (!h) {
                    const uint64_t prev = x > 0 ? s_k[x - 1] : K[gi - 1];
                    h = ((k[j] ^ prev) & kmask) >> lo_bit || (k[j] & 31u) < uint64_t(top_d);
                }
                const uint64_t m = ballot(h);
                if (lane == 0) s_m0[x >> 6] = m;
            }
            __syncthreads();
            int pos[kFrItems];
#pragma unroll
            for (int j = 0; j < kFrItems; ++j) {
                const int x = j * kFrBlock + tid;
                int st, en;
                pos[j] = x;
                if (run_bounds(s_m0, kFrRows, x, &st, &en)) {  // equal keys keep their order
                    if (st >= 0 && en - st > 1)
                        pos[j] = st + count_below(s_c, st, en, ((k[j] & rest) << 32) | uint32_t(x));
                }
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kFrItems; ++j) {
                s_k[pos[j]] = k[j];
                s_v[pos[j]] = v[j];
                s_reach[pos[j]] = uint16_t(k[j] >> kKeyLenShift);
                if (LCP) s_c[pos[j]] = key_codes(k[j], lo_bit, top_d, h0, err);
            }
            __syncthreads();
        }
    }
    // Starts of the groups that the windows begin with.  Positions outside the array count as
    // groups of their own, and so does a suffix of fewer than depth0 bases: it shares its key
    // only with its equals, which are in position order.
    const uint32_t depth0 = MIXED ? h0 : top_d;  // symbols a group shares
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        const int x = j * kFrBlock + tid;
        const int64_t gi = lo + x;
        const uint64_t key = s_k[x];
        const bool edge = gi <= 0 || gi >= int64_t(n);
        // before the span: the last item of another run, which differs in its top bits whatever
        // its order, or one of the same long run, in order
        const uint64_t prev = edge ? 0 : x > 0 ? s_k[x - 1] : K[gi - 1];
        const uint64_t d = (key ^ prev) & kmask;
        const bool h = edge || (MIXED ? d : d >> lo_bit) != 0 || (key & 31u) < uint64_t(depth0);
        if (LCP) {
            int l = -1 - int(depth0);
            if (edge) {
                l = 0;
            } else if (h) {
                const uint64_t before = x > 0 ? s_c[x - 1] : key_codes(prev, lo_bit, top_d, h0, err);
                l = int(key_lcp(before, s_c[x], uint32_t(prev), uint32_t(key), h0));
            }
            s_l[x] = int16_t(l);
        }
        const uint64_t m = ballot(h);
        if (lane == 0) s_m[x >> 6] = m;
    }
    __syncthreads();
    // the tile's own items: from the first start of a unit on, up to the first after its kFrTile
    const uint64_t *unit = s_m0;
    if (MIXED) {
#pragma unroll
        for (int j = 0; j < kFrItems; ++j) {
            const int x = j * kFrBlock + tid;
            int st, en, gs, ge;
            bool u = (s_m0[x >> 6] >> (x & 63)) & 1u;
            if (!u && !run_bounds(s_m0, kFrRows, x, &st, &en) && st < kFrTile)
                u = ((s_m[x >> 6] >> (x & 63)) & 1u) || !run_bounds(s_m, kFrRows, x, &gs, &ge);
            const uint64_t m = ballot(u);
            if (lane == 0) s_u[x >> 6] = m;
        }
        __syncthreads();
        unit = s_u;
    }
    const int own0 = first_start(unit, kFrRows, 0), own1 = first_start(unit, kFrRows, kFrTile);
    // Groups of the tile are told apart by the text: windows of two stages, kExtStage bases
    // each, while there are such groups.  Each window takes a list of their items, so that one
    // which few items need takes few waves.
    uint32_t *const s_m32 = reinterpret_cast<uint32_t *>(s_m);
    const auto list_items = [&](const uint64_t (&in)[kFrItems], const uint32_t (&place)[kFrItems]) {
        // the places of the lanes of in[j], in the order of j and the threads; how many
#pragma unroll
        for (int j = 0; j < kFrItems; ++j)
            if (lane == 0) s_cnt[j * kFrWaves + wave] = uint32_t(popc64(in[j]));
        __syncthreads();
        const uint32_t cnt = lane < uint32_t(kFrRows) ? s_cnt[lane] : 0u;
        const uint32_t inc = wave_incl_scan<Sum32>(cnt);
#pragma unroll
        for (int j = 0; j < kFrItems; ++j) {
            const uint32_t before = __shfl(inc - cnt, j * kFrWaves + int(wave));
            if ((in[j] >> lane) & 1u)
                s_list[before + uint32_t(popc64(in[j] & lanemask_lt()))] = uint16_t(place[j]);
        }
        const uint32_t total = __shfl(inc, kFrRows - 1);
        __syncthreads();
        return total;
    };
    uint32_t total;
    {
        uint64_t in[kFrItems];
        uint32_t place[kFrItems];
#pragma unroll
        for (int j = 0; j < kFrItems; ++j) {
            const int x = j * kFrBlock + tid;
            int st, en;
            const bool small = run_bounds(s_m, kFrRows, x, &st, &en);
            if (!small && x < kFrTile) {
                if (!MIXED) s_quit = 1;
                else if (x >= own0 && x < own1) state[kStNoExt] = 1u;
            }
            in[j] = ballot(small && en - st > 1 && st >= own0 && st < own1);
            place[j] = uint32_t(x);
        }
        total = list_items(in, place);
        if (!MIXED && s_quit) {
            if (tid == 0) {
                st_agent(state + kStLongRun, 1u);
                st_agent(lbflags + tile, kLb64Inc);
            }
            return;
        }
    }
#pragma unroll 1
    for (int w = 0; w < kExtWindows && total > 0; ++w) {
        // opaque in the loop: what hangs on it is cheaper made again than kept in registers
        uint32_t id = tid;
        asm volatile("" : "+v"(id));
        const uint32_t depth = depth0 + uint32_t(w) * 2 * kExtStage;
        // an item of the thread: its place, where its position and reach lie (its place at the
        // window's start) and its group's bounds in one word each, 11 bits a place; and the
        // second stage's words.  What a barrier separates is read again from LDS: registers
        // bound the waves in flight.
        uint32_t at[kFrItems], grp[kFrItems];
        uint64_t d0[kFrItems], d1[kFrItems];
#pragma unroll
        for (int j = 0; j < kFrItems; ++j) {
            const uint32_t t = j * kFrBlock + id;
            at[j] = kFrNone;
            if (t >= total) continue;
            const uint32_t x = s_list[t];
            at[j] = x | (x << 16);
            grp[j] = uint32_t(run_start(s_m, int(x))) | (uint32_t(run_end(s_m, kFrRows, int(x))) << 16);
            uint32_t a = s_v[x] + depth;
            if (a >= n) {  // inconsistent input: report only
                raise_err(err, kErrRange);
                a = 0;
            }
            const Bases q = bases_at(packed, a);
            const uint32_t l = s_reach[x] - depth;
            uint64_t c0, c1;
            stage_key(q.b[0], q.b[1], l, &c0, &c1);
            s_k[x] = c0;
            s_c[x] = c1 | (x - (grp[j] & 0xffffu));  // equal symbols: in order of their positions
            // 57 bases are 114 bits: 50 bits into the second word
            stage_key((q.b[1] << 50) | (q.b[2] >> 14), (q.b[2] << 50) | (q.b[3] >> 14),
                      l > uint32_t(kExtStage) ? l - kExtStage : 0u, &d0[j], &d1[j]);
        }
#pragma unroll
        for (int stage = 0; stage < 2; ++stage) {
            if (stage == 1) {
#pragma unroll
                for (int j = 0; j < kFrItems; ++j) {
                    if (at[j] == kFrNone || !grp[j]) continue;
                    const uint32_t x = at[j] & 0xffffu;
                    s_k[x] = d0[j];
                    s_c[x] = d1[j] | (x - (grp[j] & 0xffffu));
                }
            }
            __syncthreads();
            uint32_t to[kFrItems];  // its place after the stage
#pragma unroll
            for (int j = 0; j < kFrItems; ++j) {
                if (at[j] == kFrNone || !grp[j]) continue;
                const uint32_t x = at[j] & 0xffffu;
                const int st = int(grp[j] & 0xffffu), en = int(grp[j] >> 16);
                to[j] = uint32_t(st + count_below2(s_k, s_c, st, en, s_k[x], s_c[x]));
                s_at[to[j]] = uint16_t(x);
            }
            __syncthreads();
            // an item starts a group when its symbols are not its predecessor's, or when they
            // end with a separator (every such suffix is alone)
#pragma unroll
            for (int j = 0; j < kFrItems; ++j) {
                if (at[j] == kFrNone || !grp[j]) continue;
                const uint32_t x = at[j] & 0xffffu, y = to[j];
                at[j] = (at[j] & 0xffff0000u) | y;
                if (y == (grp[j] & 0xffffu)) continue;  // a group's first: known
                const uint32_t z = s_at[y - 1];
                const uint64_t c1 = s_c[x], e1 = s_c[z];
                const uint64_t x0 = s_k[x] ^ s_k[z], x1 = (c1 ^ e1) >> 7;
                const uint32_t lb = uint32_t(c1 >> 7) & 63u;
                const bool head = x0 != 0 || x1 != 0 || lb < uint32_t(kExtStage);
                if (head) atomicOr(&s_m32[y >> 5], 1u << (y & 31));
                if (LCP) {
                    // equal words: all the stage's symbols, or those before the separator
                    const uint32_t same = x0        ? uint32_t(__clzll((long long)x0)) >> 1
                                          : x1 >> 7 ? 32u + ((uint32_t(__clzll((long long)x1)) - 7u) >> 1)
                                                    : uint32_t(kExtStage);
                    const uint32_t la = uint32_t(e1 >> 7) & 63u, most = la < lb ? la : lb;
                    s_l[y] = int16_t(head ? int(depth) + stage * kExtStage + int(same < most ? same : most)
                                          : -1 - int(depth) - (stage + 1) * kExtStage);
                }
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kFrItems; ++j) {
                if (at[j] == kFrNone || !grp[j]) continue;
                const int x = int(at[j] & 0xffffu);
                const uint32_t st = uint32_t(run_start(s_m, x)), en = uint32_t(run_end(s_m, kFrRows, x));
                grp[j] = en - st > 1 ? st | (en << 16) : 0u;  // 0: alone
            }
        }
        uint32_t v2[kFrItems], r2[kFrItems];
#pragma unroll
        for (int j = 0; j < kFrItems; ++j) {
            if (at[j] == kFrNone) continue;
            v2[j] = s_v[at[j] >> 16];
            r2[j] = s_reach[at[j] >> 16];
        }
        __syncthreads();
        uint64_t in[kFrItems];
#pragma unroll
        for (int j = 0; j < kFrItems; ++j) {
            in[j] = ballot(at[j] != kFrNone && grp[j] != 0);
            if (at[j] == kFrNone) continue;
            at[j] &= 0xffffu;
            s_v[at[j]] = v2[j];
            s_reach[at[j]] = uint16_t(r2[j]);
        }
        total = list_items(in, at);
    }
    __syncthreads();
    // Wave 0: per row of 64, the tile's suffixes still in groups (not both they and the next
    // item start one) and the last start, scanned over the rows and then over tiles.  The
    // other waves meanwhile write the ranks and the final suffixes, which need only the
    // starts at hand (unless a long group began before them).
    const auto own_row = [&](int r) {  // the tile's own items of row r that are in the array
        int64_t a = own0 - r * 64, b = own1 - r * 64;
        if (int64_t(n) - lo - r * 64 < b) b = int64_t(n) - lo - r * 64;
        if (a < 0) a = 0;
        if (b > 64) b = 64;
        if (a >= b) return uint64_t(0);
        const uint64_t to = b == 64 ? ~uint64_t(0) : ((uint64_t(1) << b) - 1);
        return to & ~((uint64_t(1) << a) - 1);
    };
    const auto singles = [&](int r) {  // items alone in their group
        const uint64_t m = s_m[r];
        return m & ((m >> 1) | (r + 1 < kFrRows ? s_m[r + 1] << 63 : 0));
    };
    if (wave == 0) {
        uint64_t mine = 0;
        const int r = int(lane);
        if (r < kFrRows) {
            const uint64_t in = own_row(r), hm = s_m[r] & in;
            const uint32_t last = hm ? uint32_t(lo + r * 64) + 64u - uint32_t(__clzll((long long)hm)) : 0u;
            mine = (uint64_t(popc64(~singles(r) & in)) << 31) | last;
        }
        const uint64_t inc = wave_incl_scan<CountLastOp>(mine);
        uint64_t ex = __shfl_up(inc, 1);
        if (lane == 0) ex = 0;
        const uint64_t agg = __shfl(inc, kWave - 1);
        const uint64_t before = lookback_tile<CountLastOp>(lbflags, int(tile), agg, err);
        if (r < kFrRows) s_row[r] = CountLastOp::combine(before, ex);
        if (lane == 0 && tile == ntiles - 1)
            state[kStNext] = uint32_t(CountLastOp::combine(before, agg) >> 31);
    } else {
        for (int r = int(wave) - 1; r < kFrRows; r += kFrWaves - 1) {
            if (!((own_row(r) >> lane) & 1u)) continue;
            const int x = r * 64 + int(lane);
            const uint32_t p = s_v[x];
            const int st = run_start(s_m, x);
            if (p >= n || st < own0) continue;  // see below
            rank[p] = uint32_t(lo + st);
            if ((singles(r) >> lane) & 1u) sa[lo + x] = int32_t(p);
        }
    }
    __syncthreads();
    for (int r = int(wave); r < kFrRows; r += kFrWaves) {
        const uint64_t in = own_row(r), bit = uint64_t(1) << lane;
        if (!(in & bit)) continue;
        const int x = r * 64 + int(lane);
        const uint32_t i = uint32_t(lo + x);
        if (LCP) lcp[i] = s_l[x];
        const uint32_t p = s_v[x];
        if (p >= n) {  // inconsistent input: report only
            raise_err(err, kErrRange);
            continue;
        }
        const uint64_t many = ~singles(r) & in;
        if (!(many & bit)) continue;
        // the last start at or before i: one of the tile's, else from the rows and tiles before
        const int st = run_start(s_m, x);
        uint32_t g = uint32_t(lo + st);
        if (st < own0) {
            g = uint32_t(s_row[r] & CountLastOp::kLastMask) - 1u;
            if (!MIXED || g > i) {
                if (MIXED) raise_err(err, kErrRange);
                continue;
            }
            rank[p] = g;
        }
        const uint32_t o = uint32_t(s_row[r] >> 31) + uint32_t(popc64(many & (bit - 1)));
        if (o >= n) {
            raise_err(err, kErrRange);
            continue;
        }
        S_new[o] = i;
        P_new[o] = p | (s_m[r] & bit ? kDone : 0u);
        if (i - g == uint32_t(kRunMax)) state[kStBigNext] = 1u;
    }
}

// What share of sampled suffixes have an equal among the positions looked at, on their first
// top_d bases (and in the same text of a batch); see launch_sample_runs.  A thread looks at
// kSampleRow positions in a row, somewhere in its part of the text, and takes those of which
// skip bits of a hash are zero: the members of a run are taken or left together, so that few of
// them tell as much of the runs' sizes as all would.  Each taken takes a slot of an open-addressed
// table of (31 bits of the hash, "met twice") words; one that finds its word there, and marked
// already, needs no atomic, so a text of one repeated base does not serialise on one word.  The
// last workgroup decides, by the share or because far fewer were taken than should be (the few
// different strings of a tandem repeat may all fall into another part).
// Bound by latency, so the taken are listed in LDS first and then probe all at once: 12 to 14 us at
// 20 M and 50 M suffixes, 19 at 400 M (54 to 61 with the probes in the loop over the row; 20 to 53
// with every position taken of 2^16 to 2^18).
__global__ __launch_bounds__(kSampleBlock) void k_sample_runs(
    const uint32_t *__restrict__ packed, const uint32_t *__restrict__ sepmask, uint32_t n,
    uint32_t top_d, const int64_t *__restrict__ set_off, uint32_t n_sets, uint32_t part,
    uint32_t skip, float enough, uint32_t *table, uint32_t *state) {
    constexpr int kFirst = 21, kSecond = 42;  // fields of the counts: paired, taken, workgroups
    static_assert(kMaxLooked < int64_t(1) << kFirst, "counts fit their fields");
    static_assert(kSampleSlots <= 1 << 14, "slots come from 14 bits of the hash");
    static_assert(kSampleRow - 1 + 24 < 32, "a row's bases lie in one word");
    __shared__ uint32_t s_h[kSampleStep];
    __shared__ uint32_t s_taken, s_paired, s_valid;
    if (threadIdx.x == 0) s_taken = s_paired = s_valid = 0;
    __syncthreads();
    const uint32_t t = blockIdx.x * kSampleBlock + threadIdx.x;
    // part positions a thread, at least 2 kSampleRow; (t + 1) * part <= n
    const uint32_t a = t * part + uint32_t((uint64_t(t * 2654435769u) * (part - kSampleRow)) >> 32);
    const uint64_t codes = codes_at(packed, a);
    const uint32_t sep = bits_at(sepmask, a);
    uint32_t valid = 0;
#pragma unroll
    for (int j = 0; j < kSampleRow; ++j) {
        if ((sep << j) >> (32 - top_d)) continue;  // ends before top_d <= 24 bases
        ++valid;
        uint64_t h = (codes << (2 * j)) >> (64 - 2 * top_d);
        h = (h ^ (h >> 29)) * 0x9e3779b97f4a7c15ull;
        if (skip && h >> (64 - skip)) continue;
        if (set_off) h += uint64_t(set_of(set_off, n_sets, a + j)) * 0xd1342543de82ef95ull;
        h = (h ^ (h >> 32)) * 0x9e3779b97f4a7c15ull;
        s_h[atomicAdd(&s_taken, 1u)] = uint32_t(h >> 32);
    }
    __syncthreads();
    const uint32_t taken = s_taken;
    uint32_t paired = 0;
    for (uint32_t i = threadIdx.x; i < taken; i += kSampleBlock) {
        const uint32_t tag = (s_h[i] | 2u) & ~1u;
        uint32_t at = (tag >> 18) & uint32_t(kSampleSlots - 1);
        for (int k = 0; k < 64; ++k, at = (at + 1) & uint32_t(kSampleSlots - 1)) {
            uint32_t w = ld_agent(table + at);
            if (w == 0) {
                w = atomicCAS(table + at, 0u, tag);
                if (w == 0) break;  // the first
            }
            if ((w & ~1u) != tag) continue;
            // the second counts for the first too
            paired += (w & 1u) || (atomicOr(table + at, 1u) & 1u) ? 1u : 2u;
            break;
        }
    }
    for (int o = 1; o < kWave; o <<= 1) {
        paired += __shfl_xor(paired, o);
        valid += __shfl_xor(valid, o);
    }
    if (lane_id() == 0) {
        atomicAdd(&s_paired, paired);
        atomicAdd(&s_valid, valid);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    __hip_atomic_fetch_add(state + kStValid, s_valid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence();  // before this workgroup counts as ended
    const uint64_t mine = (uint64_t(1) << kSecond) | (uint64_t(taken) << kFirst) | s_paired;
    const uint64_t all = mine + __hip_atomic_fetch_add(reinterpret_cast<uint64_t *>(state + kStSample), mine,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (all >> kSecond != gridDim.x) return;
    const uint32_t field = (1u << kFirst) - 1;
    const uint32_t pairs = uint32_t(all) & field, of = uint32_t(all >> kFirst) & field;
    __threadfence();
    const uint32_t could = ld_agent(state + kStValid);
    // far fewer taken than a part of the hashes should hold: a text of a few bases over and over
    const bool few = could >= 1024 && (of << skip) < could / 4;
    if (!few && (of < 256 || float(pairs) < enough * float(of))) return;
    st_agent(state + kStTopN, 0u);
    st_agent(state + kStLongRun, 1u);
}

// The items of runs (as in k_first_runs) of more than kFrRun items, in order, with their whole
// keys and their places in the list, and the digit counts of the passes that sort them.  The
// runs' starts come from masks of 64 items: an item's run is long when the distance back to its
// start plus the distance on to the next, each sought two rows away, exceeds kFrRun.
// Bound by the waves in flight (keys read, and a look-back a tile): 1.9 ms over 400 M suffixes,
// 0.6 for the read alone.  One row at a time 2.1, four 2.3 (fewer waves fit); with one LDS add
// an item for the counts, 1.3 ms more: a long run's items share their upper digits.
constexpr int kFxBlock = 512;
constexpr int kFxWaves = kFxBlock / kWave;
constexpr int kFxRows = 128;                  // rows of 64 items per tile
constexpr int kFxTile = kFxRows * kWave;
constexpr int kFxLoad = 2;                    // rows a wave has on their way
static_assert(kFxRows % (kFxLoad * kFxWaves) == 0, "whole steps over a tile's rows");
static_assert(kFxTile >= kFirstMinTile, "look-back words are sized for tiles of kFirstMinTile items");

template <int D>
__global__ __launch_bounds__(kFxBlock) void k_first_extract(
    const uint64_t *__restrict__ K, const uint32_t *__restrict__ V, uint32_t n, uint32_t lo_bit,
    uint32_t key_bits, uint32_t top_d, uint64_t *__restrict__ keys, uint32_t *__restrict__ vals, uint32_t *__restrict__ idx,
    int passes, uint32_t *__restrict__ hist, uint64_t *lbflags, uint32_t *tick, uint32_t *state,
    uint32_t *err, uint32_t *clear, uint64_t nclear) {
    constexpr int R = 1 << D;
    extern __shared__ uint32_t s_h[];
    // what the passes need cleared (a multiple of 4 words)
    for (uint64_t i = blockIdx.x * kFxBlock + threadIdx.x; i < nclear / 4; i += gridDim.x * kFxBlock)
        reinterpret_cast<uint4 *>(clear)[i] = make_uint4(0, 0, 0, 0);
    __shared__ uint64_t s_m[kFxRows + 4];  // starts per row, two rows of context on either side
    __shared__ uint64_t s_big[kFxRows];
    __shared__ uint32_t s_cnt[kFxRows];
    __shared__ uint32_t s_tile;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const uint32_t ntiles = (n + kFxTile - 1) / kFxTile;
    const uint64_t le = lane == 63 ? ~uint64_t(0) : ((uint64_t(2) << lane) - 1);
    const uint64_t kmask = (uint64_t(1) << key_bits) - 1;
    for (int i = tid; i < passes * R; i += kFxBlock) s_h[i] = 0;
    while (true) {
        __syncthreads();
        if (tid == 0) s_tile = ticket(tick);
        __syncthreads();
        const uint32_t tile = s_tile;
        if (tile >= ntiles) break;
        const int64_t tbase = int64_t(tile) * kFxTile;
        for (int r0 = int(wave); r0 < kFxRows + 4; r0 += kFxLoad * kFxWaves) {
            uint64_t k[kFxLoad], q[kFxLoad];  // the row's keys; the one before it, in lane 0
#pragma unroll
            for (int j = 0; j < kFxLoad; ++j) {
                const int r = r0 + j * kFxWaves;
                const int64_t i = tbase + int64_t(r - 2) * kWave + lane;
                const bool in = r < kFxRows + 4 && i >= 0 && i < int64_t(n);
                k[j] = in ? K[i] : 0;
                q[j] = in && lane == 0 && i > 0 ? K[i - 1] : 0;
            }
#pragma unroll
            for (int j = 0; j < kFxLoad; ++j) {
                const int r = r0 + j * kFxWaves;
                const int64_t i = tbase + int64_t(r - 2) * kWave + lane;
                const uint64_t up = __shfl_up((unsigned long long)k[j], 1);
                const uint64_t d = (k[j] ^ (lane ? up : q[j])) & kmask;
                const uint64_t m = ballot(i <= 0 || i >= int64_t(n) || d >> lo_bit ||
                                          (k[j] & 31u) < uint64_t(top_d));
                if (lane == 0 && r < kFxRows + 4) s_m[r] = m;
            }
        }
        __syncthreads();
        for (int r = int(wave); r < kFxRows; r += kFxWaves) {
            const int64_t i = tbase + int64_t(r) * kWave + lane;
            const uint64_t *m = s_m + r + 2;
            int back = 4 * kWave, fwd = 4 * kWave;
            const uint64_t mb = m[0] & le, mf = m[0] & ~le;
            if (mb) back = int(lane) - (63 - int(__clzll((long long)mb)));
            else if (m[-1]) back = int(lane) + 1 + int(__clzll((long long)m[-1]));
            else if (m[-2]) back = int(lane) + 65 + int(__clzll((long long)m[-2]));
            if (mf) fwd = int(__ffsll((long long)mf)) - 1 - int(lane);
            else if (m[1]) fwd = kWave - int(lane) + int(__ffsll((long long)m[1])) - 1;
            else if (m[2]) fwd = 2 * kWave - int(lane) + int(__ffsll((long long)m[2])) - 1;
            const uint64_t b = ballot(i < int64_t(n) && back + fwd > kFrRun);
            if (lane == 0) {
                s_big[r] = b;
                s_cnt[r] = uint32_t(popc64(b));
            }
        }
        __syncthreads();
        if (wave == 0) {  // two rows per lane: exclusive counts over the rows, then over the tiles
            const uint64_t a = s_cnt[2 * lane], b = s_cnt[2 * lane + 1];
            const uint64_t inc = wave_incl_scan<SumOp>(a + b);
            const uint64_t agg = __shfl(inc, kWave - 1);
            const uint64_t before = lookback_tile<SumOp>(lbflags, int(tile), agg, err);
            const uint64_t ex = before + inc - a - b;
            s_cnt[2 * lane] = uint32_t(ex);
            s_cnt[2 * lane + 1] = uint32_t(ex + a);
            if (lane == 0 && tile == ntiles - 1) state[kStRadixN] = uint32_t(before + agg);
        }
        __syncthreads();
        for (int r0 = int(wave); r0 < kFxRows; r0 += kFxLoad * kFxWaves) {
            uint64_t k[kFxLoad];
            uint32_t v[kFxLoad];
#pragma unroll
            for (int j = 0; j < kFxLoad; ++j) {
                const int r = r0 + j * kFxWaves;
                if (!((s_big[r] >> lane) & 1u)) continue;
                const int64_t i = tbase + int64_t(r) * kWave + lane;
                k[j] = K[i];
                v[j] = V[i];
            }
#pragma unroll
            for (int j = 0; j < kFxLoad; ++j) {
                const int r = r0 + j * kFxWaves;
                const uint64_t b = s_big[r];
                if (!((b >> lane) & 1u)) continue;
                const uint32_t at = s_cnt[r] + uint32_t(popc64(b & lanemask_lt()));
                if (at >= n) {
                    raise_err(err, kErrRange);
                    continue;
                }
                keys[at] = k[j];
                vals[at] = v[j];
                idx[at] = uint32_t(tbase) + uint32_t(r) * kWave + lane;
                hist_add_streaks<D>(s_h, k[j] & kmask, passes);
            }
        }
    }
    __syncthreads();
    uint32_t *dst = hist + size_t(blockIdx.x) * passes * R;
    for (int i = tid; i < passes * R; i += kFxBlock) dst[i] = s_h[i];
}

template <class Shape>
static int launch_first_runs_t(const uint64_t *K, const uint32_t *V, const uint32_t *packed,
                               int64_t n, int lo_bit, int key_bits, int top_d, int h0, bool mixed,
                               int32_t *sa, uint32_t *rank, uint32_t *S_new, uint32_t *P_new,
                               int32_t *lcp, uint64_t *lbflags, int64_t lb_words, uint32_t *tick,
                               uint32_t *state, hipStream_t s) {
    const int64_t tiles = (n + Shape::kTile - 1) / Shape::kTile;
    if (tiles > lb_words) return fail(SA_ERR_HIP, "first round: look-back array too small");
    // per suffix: key 8 and position 4 read; rank 4, and sa 4 or slot and position 8, written;
    // 36 bytes of packed text per window of a suffix still in a group; lcp 4
    // (counted by the caller, who learns whether the launch gave up)
    TimedScope ts("keyruns", 0.0, lcp ? 28.0 : 24.0, s);
    TimedScope own("first_runs", 0.0, lcp ? 28.0 : 24.0, s);
    auto k = mixed ? (lcp ? k_first_runs<Shape, true, true> : k_first_runs<Shape, true, false>)
                   : (lcp ? k_first_runs<Shape, false, true> : k_first_runs<Shape, false, false>);
    hipLaunchKernelGGL(k, dim3(unsigned(tiles)), dim3(Shape::kBlock), 0, s, K, V, packed, uint32_t(n),
                       uint32_t(lo_bit), uint32_t(key_bits), uint32_t(top_d), uint32_t(h0), sa, rank,
                       S_new, P_new, lcp, lbflags, tick, state, state + kStErr);
    own.finish();
    ts.finish();
    SA_HIP(hipGetLastError());
    return SA_OK;
}

int launch_first_runs(const uint64_t *K, const uint32_t *V, const uint32_t *packed, int64_t n,
                      int lo_bit, int key_bits, int top_d, int h0, bool mixed, int32_t *sa,
                      uint32_t *rank, uint32_t *S_new, uint32_t *P_new, int32_t *lcp,
                      uint64_t *lbflags, int64_t lb_words, uint32_t *tick, uint32_t *state,
                      hipStream_t s) {
    if (n <= kFrFewItems)
        return launch_first_runs_t<FrSmall>(K, V, packed, n, lo_bit, key_bits, top_d, h0, mixed, sa, rank,
                                            S_new, P_new, lcp, lbflags, lb_words, tick, state, s);
    return launch_first_runs_t<FrLarge>(K, V, packed, n, lo_bit, key_bits, top_d, h0, mixed, sa, rank,
                                        S_new, P_new, lcp, lbflags, lb_words, tick, state, s);
}

int launch_sample_runs(const uint32_t *packed, const uint32_t *sepmask, int64_t n, int top_d,
                       const int64_t *set_off_dev, int n_sets, int64_t looked, double enough,
                       uint32_t *table, uint32_t *state, hipStream_t s) {
    const int64_t part = looked > 0 ? n / (looked / kSampleRow) : 0;
    if (looked % kSampleStep || looked > kMaxLooked || part < 2 * kSampleRow || top_d < 1 || top_d > 24)
        return fail(SA_ERR_HIP, "first round: bad sample");
    uint32_t skip = 0;  // half as many hashes while half of the slots would be taken
    while ((looked >> skip) >= kSampleSlots / 2) ++skip;
    hipLaunchKernelGGL(k_sample_runs, dim3(unsigned(looked / kSampleStep)), dim3(kSampleBlock), 0, s, packed,
                       sepmask, uint32_t(n), uint32_t(top_d), set_off_dev, uint32_t(n_sets),
                       uint32_t(part), skip, float(enough), table, state);
    SA_HIP(hipGetLastError());
    return SA_OK;
}

int launch_first_extract(const uint64_t *K, const uint32_t *V, int64_t n, int lo_bit, int top_d,
                         int key_bits,
                         const SortBufs &b, uint32_t *idx, uint64_t *lbflags, int64_t lb_words,
                         uint32_t *tick, uint32_t *state, const Tune &t, hipStream_t s,
                         int *nparts) {
    const int P = sort_passes(key_bits, t);
    const int64_t tiles = (n + kFxTile - 1) / kFxTile;
    if (tiles > lb_words) return fail(SA_ERR_HIP, "first round: look-back array too small");
    int64_t grid = kHistParts < tiles ? kHistParts : tiles;
    *nparts = int(grid);
    const size_t lds = size_t(P) * t.radix() * 4;
    const uint64_t nclear = uint64_t(64 + sort_flag_words(n, key_bits, t));
    const uint32_t lb = uint32_t(lo_bit);
    // every key read; per item of a long run, its key, value and place written
    TimedScope ts("first_extract", double(n) * 8.0, s, double(n));
    switch (t.dbits) {
        case 4: hipLaunchKernelGGL(k_first_extract<4>, dim3(unsigned(grid)), dim3(kFxBlock), lds, s, K, V, uint32_t(n), lb, uint32_t(key_bits), uint32_t(top_d), b.keys[0], b.vals[0], idx, P, b.hist, lbflags, tick, state, b.err, b.tickets, nclear); break;
        case 8: hipLaunchKernelGGL(k_first_extract<8>, dim3(unsigned(grid)), dim3(kFxBlock), lds, s, K, V, uint32_t(n), lb, uint32_t(key_bits), uint32_t(top_d), b.keys[0], b.vals[0], idx, P, b.hist, lbflags, tick, state, b.err, b.tickets, nclear); break;
        case 9: hipLaunchKernelGGL(k_first_extract<9>, dim3(unsigned(grid)), dim3(kFxBlock), lds, s, K, V, uint32_t(n), lb, uint32_t(key_bits), uint32_t(top_d), b.keys[0], b.vals[0], idx, P, b.hist, lbflags, tick, state, b.err, b.tickets, nclear); break;
        case 11: hipLaunchKernelGGL(k_first_extract<11>, dim3(unsigned(grid)), dim3(kFxBlock), lds, s, K, V, uint32_t(n), lb, uint32_t(key_bits), uint32_t(top_d), b.keys[0], b.vals[0], idx, P, b.hist, lbflags, tick, state, b.err, b.tickets, nclear); break;
        default: return fail(SA_ERR_INVALID, "unsupported digit width");
    }
    ts.finish();
    SA_HIP(hipGetLastError());
    return SA_OK;
}

}  // namespace saasm
