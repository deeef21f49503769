// overlaps.hip -- longest suffix-prefix overlap of every ordered pair of reads, by walks over
// LCP intervals of the suffix array.
//
// Sec. III: a fragment is 'fir' when it is a prefix of another (or another is a prefix of it),
// and the weighted overlap graph's edges carry overlap lengths; Sec. IV: the suffix array is
// built to answer such prefix tests.  In suffix-array order, the suffixes that share at least l
// symbols with read b's first suffix form one interval around it.  A suffix s of read a whose
// whole remainder (up to a's separator) equals the first l symbols of b ends with a separator
// that sorts below every base, so it lies just before b's suffix in that interval with
// LCP(s, b) == l == length of s; when l == |b| (b is all of s) it lies before b when a < b and
// after b when a > b (separator order).  Hence, per read b with |b| >= min_len:
//   left walk:  k = j-1, j-2, ...  (j = isa[start of b]) with run = min lcp over (k, j];
//               stop when run < min_len; report (a, b, run) when suffix sa[k] has exactly
//               run symbols before its separator and a != b;
//   right walk: k = j+1, ...  while lcp[k] >= |b|; report (a, b, |b|) when suffix sa[k] has
//               exactly |b| symbols before its separator and a != b.
// A pair can be reported more than once (a read with periodic structure); the longest wins.
// Candidates are written in order of b as (a << 32 | b, l), sorted by a with the stable radix
// sort (keeping b order within a), and reduced to one row per (a, b) with the largest l.
//
// Prefix sums come from look-backs over tiles (separators to read ids and ends; candidates to
// their places; rows to theirs), so the host waits twice: for the candidate count, which sizes
// the sort, and for the row count.  The walks are a kernel without one: a look-back's wait is
// bounded, and a walk is as long as its input makes it.
#include "device.hpp"
#include "internal.hpp"

namespace saasm {

__device__ __forceinline__ uint32_t read_of(const uint32_t *__restrict__ sepmask,
                                            const int32_t *__restrict__ sepcnt, uint32_t s) {
    const uint32_t w = s >> 5, o = s & 31;
    const uint32_t before = o ? (sepmask[w] >> (32 - o)) : 0u;  // separators at 32w .. s-1
    return uint32_t(sepcnt[w]) + __popc(before);
}

// Device words of a call: error bits, lcp[0], reads, candidates and rows (64 bits each).
constexpr int kOvErr = 0, kOvLcp0 = 1, kOvReads = 2, kOvHits = 4, kOvRows = 6;
constexpr int kOvTick = 16;  // tickets of the reads, the placing and the rows

// Validates the text and finds its reads: separator bits and the separators before each word
// of 32 positions, the read ends while they fit, and the read count.
// (1024 threads: 55 us on 50.1 M characters, where tiles of 256 words look back four times as
// often and take 94.)
constexpr int kRdBlock = 1024;
constexpr int kRdWords = 1;                     // words of 32 positions a thread
constexpr int kRdTile = kRdBlock * kRdWords;
__global__ __launch_bounds__(kRdBlock) void k_ovl_reads(const uint8_t *__restrict__ text, int64_t n,
                                                        const int32_t *__restrict__ lcp,
                                                        uint32_t *__restrict__ sepmask,
                                                        int32_t *__restrict__ sepcnt,
                                                        int32_t *__restrict__ read_end,
                                                        int64_t cap_reads, uint32_t nwords,
                                                        uint64_t *lbflags, uint32_t *ctr) {
    __shared__ uint32_t s_tile, s_excl;
    __shared__ uint32_t s_w[kRdBlock / kWave];
    if (threadIdx.x == 0) s_tile = ticket(ctr + kOvTick);
    __syncthreads();
    const uint32_t tile = s_tile;
    const uint32_t w0 = (tile * uint32_t(kRdBlock) + threadIdx.x) * kRdWords;
    uint32_t sep[kRdWords];
    bool bad = false;
#pragma unroll
    for (int q = 0; q < kRdWords; ++q) {
        const int64_t p0 = int64_t(w0 + q) * 32;
        sep[q] = 0;
        if (p0 >= n) continue;
        uint32_t c[8];  // four bytes each, position p0 in the low byte of the first
        if (p0 + 32 <= n && (reinterpret_cast<uintptr_t>(text) & 15) == 0) {
            const uint4 a = *reinterpret_cast<const uint4 *>(text + p0);
            const uint4 b = *reinterpret_cast<const uint4 *>(text + p0 + 16);
            c[0] = a.x, c[1] = a.y, c[2] = a.z, c[3] = a.w;
            c[4] = b.x, c[5] = b.y, c[6] = b.z, c[7] = b.w;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                c[j] = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t p = p0 + 4 * j + k;
                    c[j] |= uint32_t(p < n ? text[p] : uint8_t('A')) << (8 * k);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            const uint32_t x = (c[j >> 2] >> (8 * (j & 3))) & 255u;
            const bool is = x == '$';
            bad |= !(is || x == 'A' || x == 'C' || x == 'G' || x == 'T');
            sep[q] |= uint32_t(is) << (31 - j);
        }
        if (p0 <= n - 1 && n - 1 < p0 + 32 && !((sep[q] >> (31 - uint32_t(n - 1 - p0))) & 1u))
            raise_err(ctr + kOvErr, kErrNoSepEnd);
    }
    uint32_t cnt = 0;
#pragma unroll
    for (int q = 0; q < kRdWords; ++q) {
        if (w0 + q < nwords) sepmask[w0 + q] = sep[q];
        cnt += uint32_t(__popc(sep[q]));
    }
    if (bad) raise_err(ctr + kOvErr, kErrAlphabet);
    uint32_t total;
    const uint32_t mine = block_excl_sum<kRdBlock>(cnt, s_w, &total);
    if (threadIdx.x < kWave) {
        const uint64_t ex = lookback_tile<SumOp>(lbflags, int(tile), total, ctr + kOvErr);
        if (threadIdx.x == 0) s_excl = uint32_t(ex);
    }
    __syncthreads();
    uint32_t k = s_excl + mine;
#pragma unroll
    for (int q = 0; q < kRdWords; ++q) {
        if (w0 + q < nwords) sepcnt[w0 + q] = int32_t(k);
        for (uint32_t v = sep[q]; v;) {
            const int j = __clz(v);  // bit 31-j <-> position 32w+j
            if (int64_t(k) < cap_reads) read_end[k] = int32_t(int64_t(w0 + q) * 32 + j);
            ++k;
            v &= ~(0x80000000u >> j);
        }
    }
    if (threadIdx.x == 0 && (uint64_t(tile) + 1) * kRdTile >= nwords) {
        ctr[kOvReads] = s_excl + total;
        ctr[kOvLcp0] = uint32_t(lcp[0]);
    }
}

// The walks of a read's two sides; hit(a, l) for every suffix of another read a that equals
// the first l symbols of read b.
template <class F>
__device__ __forceinline__ void walk_read(const int32_t *__restrict__ sa, const int32_t *__restrict__ isa,
                                          const int32_t *__restrict__ lcp,
                                          const int32_t *__restrict__ read_end,
                                          const uint32_t *__restrict__ sepmask,
                                          const int32_t *__restrict__ sepcnt, uint32_t n, uint32_t m,
                                          int32_t min_len, uint32_t b, uint32_t *err, F hit) {
    const int32_t start = b == 0 ? 0 : read_end[b - 1] + 1;
    const int32_t len = read_end[b] - start;
    if (len < min_len) return;
    const int32_t j = isa[start];
    if (j < 0 || uint32_t(j) >= n) {
        raise_err(err, kErrRange);
        return;
    }
    int32_t run = len;
    for (int32_t k = j; k > 0; --k) {
        const int32_t l = lcp[k];
        run = l < run ? l : run;
        if (run < min_len) break;
        const uint32_t s = uint32_t(sa[k - 1]);
        const uint32_t a = read_of(sepmask, sepcnt, s < n ? s : n - 1);
        if (a >= m || s >= n) {
            raise_err(err, kErrRange);
            break;
        }
        if (read_end[a] - int32_t(s) == run && a != b) hit(a, uint32_t(run));
    }
    for (uint32_t k = uint32_t(j) + 1; k < n && lcp[k] >= len; ++k) {
        const uint32_t s = uint32_t(sa[k]);
        const uint32_t a = read_of(sepmask, sepcnt, s < n ? s : n - 1);
        if (a >= m || s >= n) {
            raise_err(err, kErrRange);
            break;
        }
        if (read_end[a] - int32_t(s) == len && a != b) hit(a, uint32_t(len));
    }
}

// The matches of a tile of reads: how many, and where among the unplaced ones they lie.
struct OvlTile {
    uint64_t count, at;
};

// One read per thread, tiles dealt out in turn (the read count is only on the device).  A thread
// keeps its first kWkKeep matches in LDS while its tile takes room for all of its own, one addition
// to the count; a read with more is walked again.  A tile's matches are written together, in order,
// if they fit in cap_hits; k_ovl_place puts the tiles in order.  Nothing is walked when the text
// or the LCP array is not valid.
// No workgroup waits for another: the matches of one read can take seconds to find (a short
// read of one letter beside a read of millions of it), longer than a look-back polls.
// Bound by each walk's chain of reads: 43 us for 100,000 reads in 50.1 M suffixes, and 12 to place
// their matches (72 in one kernel that looked back between the two; a walk to count, a scan and
// a walk to write took 90).
constexpr int kWkBlock = 256;
constexpr int kWkKeep = 12;
__global__ __launch_bounds__(kWkBlock) void k_ovl_walk(
    const int32_t *__restrict__ sa, const int32_t *__restrict__ isa,
    const int32_t *__restrict__ lcp, const int32_t *__restrict__ read_end,
    const uint32_t *__restrict__ sepmask, const int32_t *__restrict__ sepcnt, uint32_t n,
    int64_t cap_reads, int32_t min_len, uint64_t *__restrict__ hkeys, uint32_t *__restrict__ hvals,
    int64_t cap_hits, OvlTile *__restrict__ tiles, uint32_t *ctr) {
    __shared__ uint64_t s_at;
    __shared__ uint64_t s_w[kWkBlock / kWave];
    __shared__ uint32_t s_a[kWkKeep][kWkBlock], s_l[kWkKeep][kWkBlock];
    const uint32_t tid = threadIdx.x;
    uint32_t *err = ctr + kOvErr;
    const uint32_t reads = ctr[kOvReads];
    // reads beyond the room for their ends are not walked: the host asks for more first
    const bool valid = (ctr[kOvErr] & (kErrAlphabet | kErrNoSepEnd)) == 0 && ctr[kOvLcp0] == 0 &&
                       int64_t(reads) <= cap_reads;
    const uint32_t m = valid ? reads : 0u;
    const uint32_t ntiles = (m + kWkBlock - 1) / kWkBlock;
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        __syncthreads();  // what the tile before left in LDS has been read
        const uint32_t b = tile * kWkBlock + tid;
        uint32_t c = 0;
        if (b < m)
            walk_read(sa, isa, lcp, read_end, sepmask, sepcnt, n, m, min_len, b, err,
                      [&](uint32_t a, uint32_t l) {
                          if (c < uint32_t(kWkKeep)) {
                              s_a[c][tid] = a;
                              s_l[c][tid] = l;
                          }
                          ++c;
                      });
        const uint64_t inc = wave_incl_scan<SumOp>(uint64_t(c));
        if (lane_id() == kWave - 1) s_w[tid / kWave] = inc;
        __syncthreads();
        uint64_t before = inc - c, total = 0;
#pragma unroll
        for (int w = 0; w < kWkBlock / kWave; ++w) {
            if (uint32_t(w) < tid / kWave) before += s_w[w];
            total += s_w[w];
        }
        if (tid == 0) {
            s_at = total ? __hip_atomic_fetch_add(reinterpret_cast<uint64_t *>(ctr + kOvHits), total,
                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                         : 0;
            tiles[tile] = OvlTile{total, s_at};
        }
        __syncthreads();
        if (c == 0 || s_at + total > uint64_t(cap_hits)) continue;
        uint64_t o = s_at + before;
        if (c <= uint32_t(kWkKeep)) {
            for (uint32_t k = 0; k < c; ++k, ++o) {
                hkeys[o] = (uint64_t(s_a[k][tid]) << 32) | b;
                hvals[o] = s_l[k][tid];
            }
        } else {
            walk_read(sa, isa, lcp, read_end, sepmask, sepcnt, n, m, min_len, b, err,
                      [&](uint32_t a, uint32_t l) {
                          hkeys[o] = (uint64_t(a) << 32) | b;
                          hvals[o] = l;
                          ++o;
                      });
        }
    }
}

// The tiles' matches, put in the order of the tiles, and the rows' look-back words cleared;
// nothing when they did not all fit in cap_hits.  Units of work by ticket, one for about
// kPlUnit matches: all tiles are cut into as many slices, and the first slice of a tile looks
// back for the others, which wait for what it publishes (26 M matches of two tiles of reads: 0.2
// ms, a tile a workgroup 36).  Bound by memory (24 bytes a match).
constexpr int kPlBlock = 256;
constexpr uint32_t kPlUnit = 2048;
constexpr int kRwBlock = 256;  // of the rows' kernel
constexpr int kRwItems = 4;
constexpr int kRwTile = kRwBlock * kRwItems;
__global__ __launch_bounds__(kPlBlock) void k_ovl_place(
    const OvlTile *__restrict__ tiles, const uint64_t *__restrict__ hkeys,
    const uint32_t *__restrict__ hvals, uint64_t *__restrict__ keys, uint32_t *__restrict__ vals,
    int64_t cap_hits, uint64_t *__restrict__ lb_rows, uint64_t *lbflags, uint32_t *ctr) {
    __shared__ uint32_t s_unit;
    __shared__ uint64_t s_to;
    const uint64_t hits = *reinterpret_cast<const uint64_t *>(ctr + kOvHits);
    if (hits == 0 || hits > uint64_t(cap_hits)) return;  // 0 too where nothing was walked
    const uint32_t ntiles = (ctr[kOvReads] + kWkBlock - 1) / kWkBlock;
    const uint32_t slices = uint32_t(hits / (uint64_t(ntiles) * kPlUnit)) + 1u;
    const uint32_t units = ntiles * slices;  // at most ntiles + hits / kPlUnit
    if (blockIdx.x >= units) return;  // the others are enough (a ticket takes 11 ns of all)
    const uint32_t groups = gridDim.x < units ? gridDim.x : units;  // those that go on
    for (uint64_t i = blockIdx.x * kPlBlock + threadIdx.x; i * kRwTile < hits; i += groups * kPlBlock)
        lb_rows[i] = 0;
    while (true) {
        __syncthreads();
        if (threadIdx.x == 0) s_unit = ticket(ctr + kOvTick + 1);
        __syncthreads();
        const uint32_t tile = s_unit / slices, slice = s_unit % slices;
        if (s_unit >= units) break;
        const OvlTile t = tiles[tile];
        if (slice == 0) {
            if (threadIdx.x < kWave) {
                const uint64_t to = lookback_tile<SumOp>(lbflags, int(tile), t.count, ctr + kOvErr);
                if (threadIdx.x == 0) s_to = to;
            }
        } else if (threadIdx.x == 0) {
            uint64_t v = ld_agent(lbflags + tile);  // of a lower ticket
            for (uint32_t spins = 0; v >> 62 != 2; v = ld_agent(lbflags + tile)) {
                if (++spins > kSpinLimit) {
                    raise_err(ctr + kOvErr, kErrSpin);
                    v = kLb64Inc | (hits + t.count + 1);  // out of range below
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            s_to = (v & kLb64Val) - t.count;
        }
        __syncthreads();
        const uint64_t to = s_to;
        if (to + t.count > hits) continue;  // a wait that gave up: reported
        for (uint64_t i = uint64_t(slice) * kPlBlock + threadIdx.x; i < t.count; i += slices * kPlBlock) {
            keys[to + i] = hkeys[t.at + i];
            vals[to + i] = hvals[t.at + i];
        }
    }
}

// Rows of the sorted candidates: one per run of equal (a, b) keys, with the longest length.
__global__ __launch_bounds__(kRwBlock) void k_ovl_rows(const uint64_t *__restrict__ keys,
                                                       const uint32_t *__restrict__ vals, uint32_t r,
                                                       int32_t *__restrict__ out, int64_t cap,
                                                       uint64_t *lbflags, uint32_t *ctr) {
    constexpr int W = kRwBlock / kWave;
    __shared__ uint32_t s_tile;
    __shared__ uint64_t s_excl;
    __shared__ uint32_t s_cnt[kRwItems * W];
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    if (tid == 0) s_tile = ticket(ctr + kOvTick + 2);
    __syncthreads();
    const uint32_t tile = s_tile, base = tile * uint32_t(kRwTile);
    uint64_t key[kRwItems], heads[kRwItems];
#pragma unroll
    for (int j = 0; j < kRwItems; ++j) {
        const uint32_t i = base + j * kRwBlock + tid;
        key[j] = i < r ? keys[i] : 0;
        heads[j] = ballot(i < r && (i == 0 || keys[i - 1] != key[j]));
        if (lane == 0) s_cnt[j * W + wave] = uint32_t(popc64(heads[j]));
    }
    __syncthreads();
    if (wave == 0) {
        const uint32_t c = lane < uint32_t(kRwItems * W) ? s_cnt[lane] : 0u;
        const uint32_t inc = wave_incl_scan<Sum32>(c);
        const uint64_t ex = lookback_tile<SumOp>(lbflags, int(tile), __shfl(inc, kWave - 1), ctr + kOvErr);
        if (lane < uint32_t(kRwItems * W)) s_cnt[lane] = inc - c;
        if (lane == 0) s_excl = ex;
        if (lane == kWave - 1 && (uint64_t(tile) + 1) * kRwTile >= r)
            *reinterpret_cast<uint64_t *>(ctr + kOvRows) = ex + inc;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kRwItems; ++j) {
        if (!((heads[j] >> lane) & 1u)) continue;
        const uint32_t i = base + j * kRwBlock + tid;
        const uint64_t o = s_excl + s_cnt[j * W + wave] + uint32_t(popc64(heads[j] & lanemask_lt()));
        if (o >= uint64_t(cap)) continue;
        uint32_t best = vals[i];
        for (uint32_t y = i + 1; y < r && keys[y] == key[j]; ++y) best = vals[y] > best ? vals[y] : best;
        out[3 * o] = int32_t(key[j] >> 32);
        out[3 * o + 1] = int32_t(key[j] & 0xffffffffu);
        out[3 * o + 2] = int32_t(best);
    }
}

// Clears a call's words, with the active launch's look-back words.
__global__ __launch_bounds__(256) void k_ovl_init(uint32_t *ctr, uint64_t *lb0, uint32_t n0,
                                                  uint64_t *lb1, uint32_t n1) {
    const uint32_t stride = gridDim.x * 256u;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n0; i += stride) lb0[i] = 0;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n1; i += stride) lb1[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x < 64) ctr[threadIdx.x] = 0;
}

// Text-sized part, read-sized part, candidates.
struct OvlFixed {
    uint32_t *ctr, *sepmask;
    int32_t *sepcnt;
    uint64_t *lb_reads;
};
static int64_t reads_tiles(int64_t n) { return (sepmask_words(n) + kRdTile - 1) / kRdTile; }
static void carve_fixed(Carver &c, int64_t n, OvlFixed *F) {
    F->ctr = c.take<uint32_t>(64);
    F->sepmask = c.take<uint32_t>(sepmask_words(n));
    F->sepcnt = c.take<int32_t>(sepmask_words(n));
    F->lb_reads = c.take<uint64_t>(reads_tiles(n));
}
struct OvlReads {
    int32_t *read_end;
    uint64_t *lb_place;
    OvlTile *tiles;
};
static void carve_reads(Carver &c, int64_t m, OvlReads *R) {
    R->read_end = c.take<int32_t>(m);
    R->lb_place = c.take<uint64_t>((m + kWkBlock - 1) / kWkBlock + 1);
    R->tiles = c.take<OvlTile>((m + kWkBlock - 1) / kWkBlock + 1);
}
// The rows' look-back words, and keys[0] and vals[0], where the matches are placed, come first:
// their places do not depend on r.  The sort's other half, which follows, holds the matches
// before that.
struct OvlHits {
    SortBufs sb;
    uint64_t *lb_rows;
};
static void take_hits(Carver &c, int64_t hits, int64_t r, OvlHits *H) {
    H->lb_rows = c.take<uint64_t>((hits + kRwTile - 1) / kRwTile + 1);
    H->sb.keys[0] = c.take<uint64_t>(hits);
    H->sb.vals[0] = c.take<uint32_t>(hits);
    H->sb.keys[1] = c.take<uint64_t>(r);
    H->sb.vals[1] = c.take<uint32_t>(r);
}
static void carve_hits(Carver &c, int64_t hits, int64_t r, const Tune &t, OvlHits *H) {
    take_hits(c, hits, r, H);
    carve_sort(c, r, 32, t, &H->sb, false);
}

// Bytes to find, place and sort r candidates; the most of them that fit in so many bytes.
static int64_t hits_bytes(int64_t r, const Tune &t) {
    Carver c(nullptr, INT64_MAX);
    OvlHits H;
    carve_hits(c, r, r, t, &H);
    return c.off;
}
static int64_t hits_in(int64_t bytes, const Tune &t) {
    int64_t lo = 0, hi = bytes / 24 < int64_t(1) << 31 ? bytes / 24 : int64_t(1) << 31;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo + 1) / 2;
        if (hits_bytes(mid, t) <= bytes) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

static int bits_for_u(int64_t v) {
    int b = 0;
    while ((int64_t(1) << b) <= v) ++b;
    return b;
}

}  // namespace saasm

using namespace saasm;

extern "C" int64_t sa_overlaps_ws_bytes(int64_t n, int64_t m, int64_t candidates) {
    if (n < 1 || candidates < 0) return -1;
    if (m <= 0 || m > n) m = n;
    Tune t;
    resolve_tuning(nullptr, &t);
    Carver c(nullptr, INT64_MAX);
    OvlFixed F;
    carve_fixed(c, n, &F);
    OvlReads R;
    carve_reads(c, m, &R);
    if (candidates > 0) {
        OvlHits H;
        carve_hits(c, candidates, candidates, t, &H);
    }
    return c.off + 256;
}

// The reads and, while they fit, the candidates of the text: kOv* words to host[].
static int find_hits(const uint8_t *text, int64_t n, const int32_t *sa, const int32_t *isa,
                     const int32_t *lcp, int32_t min_len, const OvlFixed &F, const OvlReads &R,
                     int64_t cap_reads, const OvlHits &H, int64_t cap_hits,
                     uint32_t host[kStWords], hipStream_t s) {
    const int64_t tag = timing_round_begin();
    timing_scope_mode(kModeAny);
    const int64_t rt = reads_tiles(n), wt = (cap_reads + kWkBlock - 1) / kWkBlock;
    const int64_t most = rt > wt ? rt : wt;
    hipLaunchKernelGGL(k_ovl_init, dim3(unsigned(most / 256 + 1 < 256 ? most / 256 + 1 : 256)), dim3(256), 0, s,
                       F.ctr, F.lb_reads, uint32_t(rt), R.lb_place, uint32_t(wt));
    {
        TimedScope ts("pack", double(n) + double(sepmask_words(n)) * 8.0, s, double(n));
        hipLaunchKernelGGL(k_ovl_reads, dim3(unsigned(rt)), dim3(kRdBlock), 0, s, text, n, lcp, F.sepmask,
                           F.sepcnt, R.read_end, cap_reads, uint32_t(sepmask_words(n)), F.lb_reads, F.ctr);
        ts.finish();
    }
    {
        TimedScope ts("overlap_walk", 0.0, 12.0, s);  // per read, counted below
        // at most eight workgroups a CU
        const unsigned g = unsigned(wt < 1 ? 1 : wt < 2048 ? wt : 2048);
        hipLaunchKernelGGL(k_ovl_walk, dim3(g), dim3(kWkBlock), 0, s, sa, isa,
                           lcp, R.read_end, F.sepmask, F.sepcnt, uint32_t(n), cap_reads, min_len,
                           H.sb.keys[1], H.sb.vals[1], cap_hits, R.tiles, F.ctr);
        hipLaunchKernelGGL(k_ovl_place, dim3(1024), dim3(kPlBlock), 0, s, R.tiles, H.sb.keys[1],
                           H.sb.vals[1], H.sb.keys[0], H.sb.vals[0], cap_hits, H.lb_rows, R.lb_place, F.ctr);
        ts.finish();
    }
    SA_HIP(hipGetLastError());
    SA_TRY(read_words(F.ctr, host, s));
    timing_round_items(tag, host[kOvReads], 0);
    timing_flush();
    // sa_lcp leaves a failure it found on the device in lcp[0] (0 in every valid array)
    const int32_t lcp0 = int32_t(host[kOvLcp0]);
    if (lcp0 < 0) return fail(lcp0 == SA_ERR_ALPHABET || lcp0 == SA_ERR_INVALID ? lcp0 : SA_ERR_HIP,
                              "sa_overlaps: the LCP array carries a failure from sa_lcp");
    if (lcp0 != 0) return fail(SA_ERR_INVALID, "sa_overlaps: lcp[0] must be 0");
    const uint32_t e = host[kOvErr];
    if (e & kErrAlphabet) return fail(SA_ERR_ALPHABET, "text holds a byte other than A, C, G, T, $");
    if (e & kErrNoSepEnd) return fail(SA_ERR_INVALID, "text must end with '$'");
    if (e) return fail(SA_ERR_HIP, "sa_overlaps: device consistency check failed (code " + std::to_string(e) + ")");
    if (host[kOvReads] < 1 || int64_t(host[kOvReads]) > n) return fail(SA_ERR_HIP, "sa_overlaps: bad read count");
    return SA_OK;
}

static int64_t words64(const uint32_t host[kStWords], int at) {
    return int64_t((uint64_t(host[at + 1]) << 32) | host[at]);
}

static int sa_overlaps_impl(const uint8_t *text, int64_t n, const int32_t *sa, const int32_t *isa,
                            const int32_t *lcp, int32_t min_len, int32_t *out, int64_t cap,
                            int64_t *n_out_h, void *ws, int64_t ws_bytes, int64_t *ws_needed_h,
                            hipStream_t s) {
    if (!text || !sa || !isa || !lcp || !ws || !n_out_h || (cap > 0 && !out))
        return fail(SA_ERR_INVALID, "sa_overlaps: NULL pointer");
    if (n < 1) return fail(SA_ERR_INVALID, "sa_overlaps: n must be >= 1");
    if (n >= kMaxN) return fail(SA_ERR_TOO_LARGE, "sa_overlaps: n >= 2^31-2");
    if (min_len < 1) return fail(SA_ERR_INVALID, "sa_overlaps: min_len must be >= 1");
    if (cap < 0) return fail(SA_ERR_INVALID, "sa_overlaps: cap < 0");
    // the text-sized part must fit before the read count is known
    const int64_t fixed = sa_overlaps_ws_bytes(n, 1, 0);
    if (ws_needed_h) *ws_needed_h = fixed;
    if (ws_bytes < fixed) return fail(SA_ERR_NOMEM, "sa_overlaps: workspace too small");
    Tune t;
    resolve_tuning(nullptr, &t);
    // What the text-sized part leaves is split before the counts are known: of what a sort needs
    // for however few candidates (8 MB of digit counts) and more, an eighth of the rest is room
    // for read ends and tile words (under 5 bytes a read), all else for candidates.  Where the
    // counts do not fit that split, the search runs again with the sizes it found; where every
    // read has some candidates, a workspace a quarter larger than it asks for spares that.
    Carver c(ws, ws_bytes - 256);
    OvlFixed F;
    carve_fixed(c, n, &F);
    const int64_t left = ws_bytes - 256 - c.off, least = hits_bytes(1, t);
    const int64_t reads_room = (left > least ? left - least : left) / 8;
    int64_t cap_reads = reads_room / 5 < n ? reads_room / 5 : n, cap_hits = 0;
    const Carver at_reads = c;
    OvlReads R{};
    OvlHits H{};
    uint32_t host[kStWords];
    carve_reads(c, cap_reads, &R);
    Carver at_hits = c;
    if (cap_reads > 0) cap_hits = hits_in(ws_bytes - 256 - ((c.off + 255) & ~int64_t(255)), t);
    take_hits(c, cap_hits, cap_hits, &H);
    SA_TRY(find_hits(text, n, sa, isa, lcp, min_len, F, R, cap_reads, H, cap_hits, host, s));
    const int64_t m = host[kOvReads];
    int64_t r = words64(host, kOvHits);
    bool known = m <= cap_reads;  // the walks ran
    if (!known || r > cap_hits) {
        for (int again = 0;; ++again) {
            const int64_t need = sa_overlaps_ws_bytes(n, m, known ? r : 0);
            if (ws_needed_h) *ws_needed_h = need;
            if (known && r >= kMaxN) return fail(SA_ERR_TOO_LARGE, "sa_overlaps: more than 2^31-2 candidate matches");
            if (ws_bytes < need)
                return fail(SA_ERR_NOMEM, known ? "sa_overlaps: workspace too small for " + std::to_string(r) + " candidates"
                                                : "sa_overlaps: workspace too small for the reads");
            if (again == 2) return fail(SA_ERR_HIP, "sa_overlaps: the candidate count changed between walks");
            c = at_reads;
            carve_reads(c, m, &R);
            at_hits = c;
            cap_hits = known ? r : 0;
            take_hits(c, cap_hits, cap_hits, &H);
            SA_TRY(find_hits(text, n, sa, isa, lcp, min_len, F, R, m, H, cap_hits, host, s));
            r = words64(host, kOvHits);
            if (known && r <= cap_hits) break;
            known = true;
            if (r == 0) break;
        }
    }
    if (ws_needed_h) *ws_needed_h = sa_overlaps_ws_bytes(n, m, r);
    if (r >= kMaxN) return fail(SA_ERR_TOO_LARGE, "sa_overlaps: more than 2^31-2 candidate matches");
    if (r == 0) {
        *n_out_h = 0;
        return SA_OK;
    }
    c = at_hits;
    carve_hits(c, cap_hits, r, t, &H);
    if (!c.ok()) {  // the first split left too little for the sort: walk once more, exactly sized
        const int64_t need = sa_overlaps_ws_bytes(n, m, r);
        if (ws_bytes < need)
            return fail(SA_ERR_NOMEM, "sa_overlaps: workspace too small for " + std::to_string(r) + " candidates");
        c = at_reads;
        carve_reads(c, m, &R);
        carve_hits(c, r, r, t, &H);
        const int64_t r0 = r;
        SA_TRY(find_hits(text, n, sa, isa, lcp, min_len, F, R, m, H, r, host, s));
        r = words64(host, kOvHits);
        if (r != r0) return fail(SA_ERR_HIP, "sa_overlaps: the candidate count changed between walks");
    }
    H.sb.err = F.ctr + kOvErr;
    int cur = 0;
    const int abits = bits_for_u(m - 1);
    const int64_t row_tiles = (r + kRwTile - 1) / kRwTile;
    if (abits > 0) {
        int nparts = 0;
        SA_TRY(launch_hist(H.sb, 0, r, 32, abits, t, s, &nparts));
        SA_TRY(sort_run(H.sb, 0, nullptr, r, 32, abits, t, nparts, s, &cur));
    }
    hipLaunchKernelGGL(k_ovl_rows, dim3(unsigned(row_tiles)), dim3(kRwBlock), 0, s, H.sb.keys[cur],
                       H.sb.vals[cur], uint32_t(r), out, cap, H.lb_rows, F.ctr);
    SA_HIP(hipGetLastError());
    SA_TRY(read_words(F.ctr, host, s));
    timing_flush();
    if (host[kOvErr])
        return fail(SA_ERR_HIP, "sa_overlaps: device consistency check failed (code " + std::to_string(host[kOvErr]) + ")");
    const int64_t u = words64(host, kOvRows);
    *n_out_h = u;
    if (u > cap) return fail(SA_ERR_CAPACITY, "sa_overlaps: output holds " + std::to_string(cap) + " rows, need " + std::to_string(u));
    return SA_OK;
}

extern "C" int sa_overlaps(const uint8_t *text, int64_t n, const int32_t *sa, const int32_t *isa,
                           const int32_t *lcp, int32_t min_len, int32_t *out, int64_t cap,
                           int64_t *n_out_h, void *ws, int64_t ws_bytes, int64_t *ws_needed_h,
                           hipStream_t stream) {
    return guard<int>([&] {
        return sa_overlaps_impl(text, n, sa, isa, lcp, min_len, out, cap, n_out_h, ws, ws_bytes,
                                ws_needed_h, stream);
    });
}
