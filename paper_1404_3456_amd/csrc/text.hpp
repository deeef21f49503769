// text.hpp -- random-access 32-position windows of the packed text (device side).
//
// Record b of the block layout holds the 2-bit codes of positions 32b .. 32b+31 (two words,
// position 32b in the top bits of the first) and their separator bits (position 32b in bit
// 31), padded to 16 bytes; launch_pack writes it.
// A window starting anywhere is then two aligned 16-byte loads.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace saasm {

struct __attribute__((packed, aligned(1))) Bytes16 {
    uint32_t w[4];
};

// Four bytes at once: 128 in every byte of v that equals c.
__device__ __forceinline__ uint32_t bytes_equal(uint32_t v, uint32_t c) {
    const uint32_t x = v ^ (c * 0x01010101u);
    return ~(((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x | 0x7f7f7f7fu);
}
// 128 in every byte that is a base.
__device__ __forceinline__ uint32_t bases_of(uint32_t v) {
    return bytes_equal(v, 'A') | bytes_equal(v, 'C') | bytes_equal(v, 'G') | bytes_equal(v, 'T');
}
// Their codes, a byte each (A0 C1 G2 T3); and four such in 8 bits, byte 0's on top.
__device__ __forceinline__ uint32_t codes_of(uint32_t v) { return ((v >> 1) ^ (v >> 2)) & 0x03030303u; }
__device__ __forceinline__ uint32_t codes_packed(uint32_t c) { return (c * 0x40100401u) >> 24; }

struct Window {
    uint64_t code;  // 32 bases from position a, base a in bits 63..62
    uint32_t sep;   // separator bits of positions a .. a+31, position a in bit 31
};

// Needs records a/32 and a/32 + 1.
__device__ __forceinline__ Window window_at(const uint4 *__restrict__ blk, uint32_t a) {
    const uint32_t b = a >> 5, o = a & 31;
    const uint4 x = blk[b], y = blk[b + 1];
    const uint64_t c0 = (uint64_t(x.x) << 32) | x.y, c1 = (uint64_t(y.x) << 32) | y.y;
    Window w;
    w.code = o ? (c0 << (2 * o)) | (c1 >> (64 - 2 * o)) : c0;
    w.sep = o ? (x.z << o) | (y.z >> (32 - o)) : x.z;
    return w;
}

// Separator bits of positions a .. a+31 (position a in bit 31); reads words a/32 and a/32 + 1.
__device__ __forceinline__ uint32_t bits_at(const uint32_t *__restrict__ sepmask, uint32_t a) {
    const uint32_t o = a & 31;
    const uint32_t x = sepmask[a >> 5], y = sepmask[(a >> 5) + 1];
    return o ? (x << o) | (y >> (32 - o)) : x;
}

// 32 bases of a packed code array (16 per word, base 0 in the top bits) from base a; reads
// words a/16 .. a/16 + 2.
__device__ __forceinline__ uint64_t codes_at(const uint32_t *__restrict__ packed, uint64_t a) {
    const uint64_t w = a >> 4;
    const uint32_t o = uint32_t(a & 15);
    uint64_t x = (uint64_t(packed[w]) << 32) | packed[w + 1];
    x <<= 2 * o;
    if (o) x |= uint64_t(packed[w + 2]) >> (32 - 2 * o);
    return x;
}

// Index of the text of a batch that holds position p: largest s with set_off[s] <= p.
__device__ __forceinline__ uint32_t set_of(const int64_t *__restrict__ set_off, uint32_t n_sets,
                                           uint32_t p) {
    uint32_t lo = 0, hi = n_sets;  // invariant: set_off[lo] <= p < set_off[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (set_off[mid] <= int64_t(p)) lo = mid;
        else hi = mid;
    }
    return lo;
}

}  // namespace saasm
