// first_round.hip -- the first round of a suffix-array build, from suffixes ordered by the top
// bits of their first-round keys to groups equal on h0 + kExtBases symbols.
//
// Sec. IV sorts integer keys by radix passes, one digit at a time.  A first-round key holds 29
// bases (63 bits, seven 9-bit passes), but two or three passes over its top bits already leave
// runs of equal top bits that are about as short as the final groups: the reads of a 10x
// coverage put about ten copies of a genome stretch side by side, and that is what a run
// holds.  So only the top bits go through passes over HBM; the rest of the key is sorted run by
// run in LDS here, and each group still equal on all of it is sorted by the next kExtBases
// symbols read from the packed text.  The same kernel then finishes the round: it labels
// groups, writes the ranks and the final suffixes, and compacts the rest for the doubling
// rounds, which start at h0 + kExtBases symbols instead of h0.
//
// A run is a stretch of equal top bits, that is, of suffixes equal on their first top_d bases
// (suffixes that end before top_d bases share theirs only with their equals and are runs of
// their own).  Runs of more than kFrRun suffixes (repeats) do not fit the context a tile loads.  The plain
// form of the kernel only reports them; the host then has their items taken out, sorted by
// radix passes over the whole key and put back in place (k_first_extract, k_big_place), and
// runs the other form, which takes such runs as sorted.
#include "device.hpp"
#include "internal.hpp"
#include "text.hpp"

namespace saasm {

constexpr int kFrRun = 128;                      // longest run sorted in LDS
constexpr int kFrBlock = 512;
constexpr int kFrItems = 4;
constexpr int kFrSpan = kFrBlock * kFrItems;     // items loaded per tile
constexpr int kFrTile = kFrSpan - 2 * kFrRun;    // items a tile finishes
constexpr int kFrRows = kFrSpan / kWave;
constexpr int kFrWaves = kFrBlock / kWave;
constexpr int kFrRow0 = kFrRun / kWave;              // first and last + 1 row of the tile's own items
constexpr int kFrRow1 = kFrRows - kFrRun / kWave;
static_assert(kFrRun % kWave == 0 && kFrRun == 2 * kWave, "the bounds of a run are sought two words away");
static_assert(kFrTile >= kFirstMinTile, "look-back words are sized for tiles of kFirstMinTile items");

// First item of the run that holds item x, from a mask of run starts (bit x % 64 of word
// x / 64): the nearest start at or before x, sought two words back; -1 if there is none.
__device__ __forceinline__ int run_start(const uint64_t *m, int x) {
    const int w = x >> 6, b = x & 63;
    const uint64_t le = b == 63 ? ~uint64_t(0) : ((uint64_t(2) << b) - 1);
    uint64_t v = m[w] & le;
    int at = w;
    for (int k = 1; k <= 2 && !v && w - k >= 0; ++k) {
        v = m[w - k];
        at = w - k;
    }
    return v ? at * 64 + 63 - int(__clzll((long long)v)) : -1;
}

// First item after the run that holds item x: the next start, sought two words on; -1 if none.
__device__ __forceinline__ int run_end(const uint64_t *m, int x) {
    const int w = x >> 6, b = x & 63;
    const uint64_t le = b == 63 ? ~uint64_t(0) : ((uint64_t(2) << b) - 1);
    uint64_t v = m[w] & ~le;
    int at = w;
    for (int k = 1; k <= 2 && !v && w + k < kFrRows; ++k) {
        v = m[w + k];
        at = w + k;
    }
    return v ? at * 64 + int(__ffsll((long long)v)) - 1 : -1;
}

// Bounds of the run of item x when it has at most kFrRun items inside the loaded span.
__device__ __forceinline__ bool run_bounds(const uint64_t *m, int x, int *st, int *en) {
    *st = run_start(m, x);
    *en = run_end(m, x);
    return *st >= 0 && *en >= 0 && *en - *st <= kFrRun;
}

// The kExtBases symbols from text position a on, as two words that order like them: 32 bases,
// then 29 bases and, in the last 6 bits, how many there are before the separator (61: all).
// Bases past the separator are zero, so a suffix that ends sorts below those that go on.
__device__ __forceinline__ void ext_key(const uint4 *__restrict__ blk, uint32_t a, uint64_t *c0,
                                        uint64_t *c1) {
    const uint32_t b = a >> 5, o = a & 31;
    const uint4 x = blk[b], y = blk[b + 1], z = blk[b + 2];
    const uint64_t w0 = (uint64_t(x.x) << 32) | x.y, w1 = (uint64_t(y.x) << 32) | y.y,
                   w2 = (uint64_t(z.x) << 32) | z.y;
    uint64_t p0 = o ? (w0 << (2 * o)) | (w1 >> (64 - 2 * o)) : w0;
    uint64_t p1 = o ? (w1 << (2 * o)) | (w2 >> (64 - 2 * o)) : w1;
    const uint64_t s01 = (uint64_t(x.z) << 32) | y.z;
    const uint64_t sm = o ? (s01 << o) | (uint64_t(z.z) >> (32 - o)) : s01;  // bits of a .. a+63
    uint32_t L = sm ? uint32_t(__clzll((long long)sm)) : 64u;
    if (L < 32) {
        p0 &= L ? ~uint64_t(0) << (64 - 2 * L) : 0;
        p1 = 0;
    } else if (L < 64) {
        p1 &= L > 32 ? ~uint64_t(0) << (128 - 2 * L) : 0;
    }
    if (L > uint32_t(kExtBases)) L = kExtBases;
    *c0 = p0;
    *c1 = (p1 & ~uint64_t(63)) | L;
}

// One tile of the order by the keys' top bits (bits lo_bit and up): sorts its runs, labels its
// groups and writes rank[], the final sa[] entries and the compacted slots and positions of
// the suffixes still in groups, as k_rank_update does for a doubling round.  MIXED: runs of
// more than kFrRun items are in order of the whole key already; otherwise such a run sets
// state[kStLongRun], after which the tiles give up (the host sees the flag and starts over).
// A tile loads kFrRun items of context on either side, so every run of at most kFrRun items
// that meets it, or meets the item after it, lies in the loaded span, and both tiles that share
// a run sort it alike.
template <bool MIXED>
__global__ __launch_bounds__(kFrBlock) void k_first_runs(
    const uint64_t *__restrict__ K, const uint32_t *__restrict__ V, const uint4 *__restrict__ blk,
    uint32_t n, uint32_t lo_bit, uint32_t top_d, uint32_t h0, int32_t *__restrict__ sa,
    uint32_t *__restrict__ rank, uint32_t *__restrict__ S_new, uint32_t *__restrict__ P_new,
    uint64_t *lbflags, uint32_t *tick, uint32_t *state, uint32_t *err) {
    __shared__ uint64_t s_k[kFrSpan];     // keys; then the first words of the extension keys
    __shared__ uint64_t s_c[kFrSpan];     // second words of the extension keys
    __shared__ uint32_t s_v[kFrSpan];     // text positions; then with bit 31 on group starts
    __shared__ uint64_t s_m0[kFrRows];    // starts of runs
    __shared__ uint64_t s_m1[kFrRows];    // starts of groups equal on the whole key
    __shared__ uint64_t s_m2[kFrRows];    // starts of the final groups
    __shared__ uint64_t s_row[kFrRows];   // (count, last start) before each row
    __shared__ uint32_t s_tile, s_quit;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    if (tid == 0) {
        s_tile = ticket(tick);
        s_quit = MIXED ? 0u : ld_agent(state + kStLongRun);
    }
    __syncthreads();
    const uint32_t tile = s_tile;
    const uint32_t ntiles = (n + kFrTile - 1) / kFrTile;
    if (tile >= ntiles) return;
    if (s_quit) {  // later tiles look back at this one: publish something and stop
        if (tid == 0) st_agent(lbflags + tile, kLb64Inc);
        return;
    }
    const int64_t lo = int64_t(tile) * kFrTile - kFrRun;
    uint64_t k[kFrItems];
    uint32_t v[kFrItems];
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        const int64_t gi = lo + j * kFrBlock + tid;
        const bool in = gi >= 0 && gi < int64_t(n);
        k[j] = in ? K[gi] : 0;
        v[j] = in ? V[gi] : 0;
    }
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) s_k[j * kFrBlock + tid] = k[j];
    __syncthreads();
    // starts of runs (positions outside the array count as runs of their own, and so does a
    // suffix of fewer than top_d bases: it shares its top bits only with its equals, which are
    // in position order)
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        const int x = j * kFrBlock + tid;
        const int64_t gi = lo + x;
        bool h = gi <= 0 || gi >= int64_t(n);
        if (!h && x > 0)
            h = (k[j] >> lo_bit) != (s_k[x - 1] >> lo_bit) || (k[j] & 31u) < uint64_t(top_d);
        const uint64_t m = ballot(h);
        if (lane == 0) s_m0[x >> 6] = m;
    }
    __syncthreads();
    // each run in order of the whole key (equal keys keep their order)
    int pos[kFrItems];
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        const int x = j * kFrBlock + tid;
        int st, en;
        pos[j] = x;
        if (run_bounds(s_m0, x, &st, &en)) {
            int before = 0;
            for (int y = st; y < en; ++y) {
                const uint64_t q = s_k[y];
                before += (q < k[j] || (q == k[j] && y < x)) ? 1 : 0;
            }
            pos[j] = st + before;
        } else if (!MIXED && x >= kFrRun && x < kFrRun + kFrTile) {
            s_quit = 1;
        }
    }
    __syncthreads();
    if (!MIXED && s_quit) {
        if (tid == 0) {
            st_agent(state + kStLongRun, 1u);
            st_agent(lbflags + tile, kLb64Inc);
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        s_k[pos[j]] = k[j];
        s_v[pos[j]] = v[j];
    }
    __syncthreads();
    // starts of groups equal on the whole key; a key of fewer than h0 symbols is a suffix that
    // ended at its separator, alone in its group
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        const int x = j * kFrBlock + tid;
        const int64_t gi = lo + x;
        k[j] = s_k[x];
        v[j] = s_v[x];
        bool h = gi <= 0 || gi >= int64_t(n);
        if (!h && x > 0) h = k[j] != s_k[x - 1] || (k[j] & 31u) < uint64_t(h0);
        const uint64_t m = ballot(h);
        if (lane == 0) s_m1[x >> 6] = m;
    }
    __syncthreads();
    // groups that meet the tile or the item after it: their members' next kExtBases symbols
    int st[kFrItems], en[kFrItems];
    uint64_t c0[kFrItems], c1[kFrItems];
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        const int x = j * kFrBlock + tid;
        const bool small = run_bounds(s_m1, x, &st[j], &en[j]);
        if (!small && x >= kFrRun && x < kFrRun + kFrTile) state[kStNoExt] = 1u;
        const bool ext = small && en[j] - st[j] > 1 && st[j] <= kFrRun + kFrTile && en[j] > kFrRun;
        if (!ext) {
            en[j] = 0;
            continue;
        }
        const uint32_t a = v[j] + h0;
        if (a < n) {
            ext_key(blk, a, &c0[j], &c1[j]);
        } else {
            raise_err(err, kErrRange);
            c0[j] = c1[j] = 0;
        }
    }
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        const int x = j * kFrBlock + tid;
        if (en[j]) {
            s_k[x] = c0[j];
            s_c[x] = c1[j];
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        const int x = j * kFrBlock + tid;
        pos[j] = x;
        bool head = (s_m1[x >> 6] >> (x & 63)) & 1u;
        if (en[j]) {
            int before = 0;
            bool first = true;
            for (int y = st[j]; y < en[j]; ++y) {
                const uint64_t q0 = s_k[y], q1 = s_c[y];
                const bool eq = q0 == c0[j] && q1 == c1[j];
                before += (q0 < c0[j] || (q0 == c0[j] && q1 < c1[j]) || (eq && y < x)) ? 1 : 0;
                if (eq && y < x) first = false;
            }
            pos[j] = st[j] + before;
            head = first || (c1[j] & 63u) < uint64_t(kExtBases);
        }
        s_v[pos[j]] = v[j] | (head ? kDone : 0u);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kFrItems; ++j) {
        const int x = j * kFrBlock + tid;
        const uint64_t m = ballot((s_v[x] & kDone) != 0);
        if (lane == 0) s_m2[x >> 6] = m;
    }
    __syncthreads();
    // per row of 64: suffixes still in groups (neither they nor the next item start a group on
    // both sides) and the last start; scanned over the tile's rows, then over tiles
    if (wave == 0) {
        uint64_t mine = 0;
        const int r = kFrRow0 + int(lane);
        if (r < kFrRow1) {
            const int64_t g = lo + r * 64;
            const uint64_t m = s_m2[r];
            const uint64_t nxt = (m >> 1) | (s_m2[r + 1] << 63);
            const int64_t left = int64_t(n) - g;
            const uint64_t in = left >= 64 ? ~uint64_t(0) : left <= 0 ? 0 : ((uint64_t(1) << left) - 1);
            const uint64_t hm = m & in;
            const uint32_t last = hm ? uint32_t(g) + 64u - uint32_t(__clzll((long long)hm)) : 0u;
            mine = (uint64_t(popc64(~(m & nxt) & in)) << 31) | last;
        }
        const uint64_t inc = wave_incl_scan<CountLastOp>(mine);
        uint64_t ex = __shfl_up(inc, 1);
        if (lane == 0) ex = 0;
        const uint64_t agg = __shfl(inc, kWave - 1);
        const uint64_t before = lookback_tile<CountLastOp>(lbflags, int(tile), agg, err);
        if (r < kFrRow1) s_row[r] = CountLastOp::combine(before, ex);
        if (lane == 0 && tile == ntiles - 1)
            state[kStNext] = uint32_t(CountLastOp::combine(before, agg) >> 31);
    }
    __syncthreads();
    for (int r = kFrRow0 + int(wave); r < kFrRow1; r += kFrWaves) {
        const int64_t gi = lo + r * 64 + lane;
        if (gi >= int64_t(n)) break;
        const uint32_t i = uint32_t(gi);
        const uint64_t m = s_m2[r];
        const uint64_t nxt = (m >> 1) | (s_m2[r + 1] << 63);
        const uint64_t single = m & nxt, bit = uint64_t(1) << lane;
        const uint64_t le = bit | (bit - 1);
        const uint64_t mb = m & le;
        const uint32_t head = uint32_t((m >> lane) & 1u);
        // the last start at or before i: in this row, else in the rows and tiles before
        const uint32_t g = mb ? uint32_t(lo + r * 64) + 63u - uint32_t(__clzll((long long)mb))
                              : uint32_t(s_row[r] & CountLastOp::kLastMask) - 1u;
        const uint32_t p = s_v[r * 64 + lane] & kRankMask;
        if (p >= n || g > i) {  // inconsistent input: report only (a tile that gave up also
                                // leaves the tiles after it without a start: not an error)
            if (MIXED || p >= n) raise_err(err, kErrRange);
            continue;
        }
        rank[p] = g;
        if (single & bit) {
            sa[i] = int32_t(p);
        } else {
            const uint32_t o = uint32_t(s_row[r] >> 31) + uint32_t(popc64(~single & (bit - 1)));
            if (o >= n) {
                raise_err(err, kErrRange);
                continue;
            }
            S_new[o] = i;
            P_new[o] = p | (head ? kDone : 0u);
            if (i - g == uint32_t(kRunMax)) state[kStBigNext] = 1u;
        }
    }
}

// The items of runs (as in k_first_runs) of more than kFrRun items, in order, with their whole keys and
// their places in the list, and the digit counts of the passes that sort them.  The runs'
// starts come from masks of 64 items: an item's run is long when the distance back to its
// start plus the distance on to the next, each sought two rows away, exceeds kFrRun.
constexpr int kFxBlock = 512;
constexpr int kFxWaves = kFxBlock / kWave;
constexpr int kFxRows = 128;                  // rows of 64 items per tile
constexpr int kFxTile = kFxRows * kWave;
static_assert(kFxTile >= kFirstMinTile, "look-back words are sized for tiles of kFirstMinTile items");

template <int D>
__global__ __launch_bounds__(kFxBlock) void k_first_extract(
    const uint64_t *__restrict__ K, const uint32_t *__restrict__ V, uint32_t n, uint32_t lo_bit,
    uint32_t top_d, uint64_t *__restrict__ keys, uint32_t *__restrict__ vals, uint32_t *__restrict__ idx,
    int passes, uint32_t *__restrict__ hist, uint64_t *lbflags, uint32_t *tick, uint32_t *state,
    uint32_t *err) {
    constexpr int R = 1 << D;
    extern __shared__ uint32_t s_h[];
    __shared__ uint64_t s_m[kFxRows + 4];  // starts per row, two rows of context on either side
    __shared__ uint64_t s_big[kFxRows];
    __shared__ uint32_t s_cnt[kFxRows];
    __shared__ uint32_t s_tile;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const uint32_t ntiles = (n + kFxTile - 1) / kFxTile;
    const uint64_t le = lane == 63 ? ~uint64_t(0) : ((uint64_t(2) << lane) - 1);
    for (int i = tid; i < passes * R; i += kFxBlock) s_h[i] = 0;
    while (true) {
        __syncthreads();
        if (tid == 0) s_tile = ticket(tick);
        __syncthreads();
        const uint32_t tile = s_tile;
        if (tile >= ntiles) break;
        const int64_t tbase = int64_t(tile) * kFxTile;
        for (int r = int(wave); r < kFxRows + 4; r += kFxWaves) {
            const int64_t i = tbase + int64_t(r - 2) * kWave + lane;
            bool h = i <= 0 || i >= int64_t(n);
            if (!h) {
                const uint64_t k = K[i];
                h = (k >> lo_bit) != (K[i - 1] >> lo_bit) || (k & 31u) < uint64_t(top_d);
            }
            const uint64_t m = ballot(h);
            if (lane == 0) s_m[r] = m;
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
        for (int r = int(wave); r < kFxRows; r += kFxWaves) {
            const uint64_t b = s_big[r];
            if (!((b >> lane) & 1u)) continue;
            const uint32_t i = uint32_t(tbase) + uint32_t(r) * kWave + lane;
            const uint32_t j = s_cnt[r] + uint32_t(popc64(b & lanemask_lt()));
            if (j >= n) {
                raise_err(err, kErrRange);
                continue;
            }
            const uint64_t key = K[i];
            keys[j] = key;
            vals[j] = V[i];
            idx[j] = i;
            for (int p = 0; p < passes; ++p)
                atomicAdd(&s_h[p * R + uint32_t((key >> (p * D)) & (R - 1))], 1u);
        }
    }
    __syncthreads();
    uint32_t *dst = hist + size_t(blockIdx.x) * passes * R;
    for (int i = tid; i < passes * R; i += kFxBlock) dst[i] = s_h[i];
}

int launch_first_runs(const uint64_t *K, const uint32_t *V, const uint4 *blk, int64_t n,
                      int lo_bit, int top_d, int h0, bool mixed, int32_t *sa, uint32_t *rank,
                      uint32_t *S_new, uint32_t *P_new, uint64_t *lbflags, int64_t lb_words,
                      uint32_t *tick, uint32_t *state, hipStream_t s) {
    const int64_t tiles = (n + kFrTile - 1) / kFrTile;
    if (tiles > lb_words) return fail(SA_ERR_HIP, "first round: look-back array too small");
    SA_TRY(launch_fill_u64(lbflags, tiles, 0, s));
    SA_TRY(launch_fill_u32(tick, 1, 0, s));
    // per suffix: key 8 and position 4 read; rank 4, and sa 4 or slot and position 8, written;
    // 24 bytes of packed text for a suffix still in a group
    TimedScope ts("first_runs", double(n) * 24.0, s, double(n));
    if (mixed)
        hipLaunchKernelGGL(k_first_runs<true>, dim3(unsigned(tiles)), dim3(kFrBlock), 0, s, K, V, blk,
                           uint32_t(n), uint32_t(lo_bit), uint32_t(top_d), uint32_t(h0), sa, rank, S_new, P_new,
                           lbflags, tick, state, state + kStErr);
    else
        hipLaunchKernelGGL(k_first_runs<false>, dim3(unsigned(tiles)), dim3(kFrBlock), 0, s, K, V, blk,
                           uint32_t(n), uint32_t(lo_bit), uint32_t(top_d), uint32_t(h0), sa, rank, S_new, P_new,
                           lbflags, tick, state, state + kStErr);
    ts.finish();
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
    SA_TRY(launch_fill_u64(lbflags, tiles, 0, s));
    SA_TRY(launch_fill_u32(tick, 1, 0, s));
    const size_t lds = size_t(P) * t.radix() * 4;
    const uint32_t lb = uint32_t(lo_bit);
    // every key read; per item of a long run, its key, value and place written
    TimedScope ts("first_extract", double(n) * 8.0, s, double(n));
    switch (t.dbits) {
        case 4: hipLaunchKernelGGL(k_first_extract<4>, dim3(unsigned(grid)), dim3(kFxBlock), lds, s, K, V, uint32_t(n), lb, uint32_t(top_d), b.keys[0], b.vals[0], idx, P, b.hist, lbflags, tick, state, b.err); break;
        case 8: hipLaunchKernelGGL(k_first_extract<8>, dim3(unsigned(grid)), dim3(kFxBlock), lds, s, K, V, uint32_t(n), lb, uint32_t(top_d), b.keys[0], b.vals[0], idx, P, b.hist, lbflags, tick, state, b.err); break;
        case 9: hipLaunchKernelGGL(k_first_extract<9>, dim3(unsigned(grid)), dim3(kFxBlock), lds, s, K, V, uint32_t(n), lb, uint32_t(top_d), b.keys[0], b.vals[0], idx, P, b.hist, lbflags, tick, state, b.err); break;
        case 11: hipLaunchKernelGGL(k_first_extract<11>, dim3(unsigned(grid)), dim3(kFxBlock), lds, s, K, V, uint32_t(n), lb, uint32_t(top_d), b.keys[0], b.vals[0], idx, P, b.hist, lbflags, tick, state, b.err); break;
        default: return fail(SA_ERR_INVALID, "unsupported digit width");
    }
    ts.finish();
    SA_HIP(hipGetLastError());
    return SA_OK;
}

}  // namespace saasm
