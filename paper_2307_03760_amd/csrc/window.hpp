// Output of the LZ77 codecs (Deflate, LZ4) by one wavefront: the history
// window in LDS, its kilobyte flushes to HBM ("coalesced on-demand writing",
// CODAG Section IV-F) and the back-references ("memcpy").
#pragma once

#include "../../include/codag.h"
#include "share.hpp"
#include "stream.hpp"

namespace codag {

typedef uint64_t u64_any __attribute__((aligned(1), may_alias));
typedef uint32_t u32_any __attribute__((aligned(1), may_alias));
typedef uint16_t u16_any __attribute__((aligned(1), may_alias));

typedef uint32_t u128_any __attribute__((ext_vector_type(4), aligned(1), may_alias));

// len bytes from src to dst in HBM (not overlapping) by one wave: sixteen
// bytes a lane at any alignment, four kilobytes in flight.  (A byte a lane,
// each load waited for, 256 KiB took about as long as inflating them.)
__device__ __forceinline__ void wave_stream(uint8_t *dst, const uint8_t *src, uint32_t len) {
    const uint32_t l16 = 16 * lane();
    uint32_t i = 0;
    for (; i + 4096 <= len; i += 4096) {
        u128_any v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; k++) v[k] = *reinterpret_cast<const u128_any *>(src + i + 1024 * k + l16);
#pragma unroll
        for (uint32_t k = 0; k < 4; k++) *reinterpret_cast<u128_any *>(dst + i + 1024 * k + l16) = v[k];
    }
    for (; i < len; i += 1024) {
        const uint32_t a = i + l16;
        if (a + 16 <= len) *reinterpret_cast<u128_any *>(dst + a) = *reinterpret_cast<const u128_any *>(src + a);
    }
    const uint32_t a = (len & ~15u) + lane();
    if (a < len) dst[a] = src[a];
}

// Output through an LDS history window.  Positions are 32-bit offsets from
// `base`, the chunk's output address rounded down to a block (uniform values
// stay in scalar registers; there are no scalar 64-bit ordered compares).
// Bytes below `fa` are in HBM, those in [fa, o0 + pos) only in the window.
// The window is linear: it holds offsets [wlo, o0 + pos) at win[x - wlo];
// when an append would pass its end, the complete blocks are flushed and the
// newest bytes slide to the front (5 of 16 bytes per lane, a few hundred
// cycles per kilobyte and a half of output), so runs of bytes never wrap and
// may be read and written eight at a time at any alignment.  wlo and fa are
// multiples of kBlock, and everything below wlo + 512 is in HBM once wlo > 0
// (appends are of at most kAppend bytes), so a copy of at most 512 bytes
// whose source starts below wlo reads HBM alone.
// `room` = wlo + H - (o0 + pos).
template <uint32_t H>
struct LinearOut {
    static_assert(H >= 3072 && H % 1024 == 0, "an append, a slide and a copy must fit");
    static constexpr uint32_t kBlock = 512, kAppend = H - 3 * kBlock;
    uint8_t *base;  // kBlock aligned
    uint8_t *win;
    uint32_t o0, wlo, fa, cap, pos, room;

    __device__ __forceinline__ void init(uint8_t *out, uint32_t capacity, uint8_t *window) {
        o0 = (uint32_t)(reinterpret_cast<uintptr_t>(out) & (kBlock - 1));
        base = out - o0;
        win = window;
        wlo = 0;
        fa = 0;
        cap = capacity;
        pos = 0;
        room = H - o0;
    }
    // (The slot of an offset outside the window is in bounds too.)
    __device__ __forceinline__ uint32_t slot(uint32_t x) const { return min(x - wlo, H); }

    // Writes the block [fa, fa + kBlock) to HBM, restricted to the bytes of
    // the chunk's range below `limit` (relative).
    __device__ __forceinline__ void flush_block(uint32_t limit) {
        const uint32_t a = fa + 16 * lane(), sl = a - wlo;
        if (16 * lane() < kBlock) {
            if (a >= o0 && a + 16 <= limit) {
                *reinterpret_cast<uint4 *>(base + a) = *reinterpret_cast<const uint4 *>(win + sl);
            } else if (a + 16 > o0 && a < limit) {
                for (uint32_t k = 0; k < 16; k++)
                    if (a + k >= o0 && a + k < limit) base[a + k] = win[sl + k];
            }
        }
        fa += kBlock;
    }
    // Room for len <= kAppend more bytes.  A slide makes room for `want` bytes: a
    // window slid by the few bytes that an append needs is copied whole for each
    // of them (with a 32 KiB window, 64 KiB of zeros in Deflate took 252
    // us, a random LZ4 block 106, and take 191 and 85; half a window of history
    // stays).
    __device__ __forceinline__ void make_room(uint32_t len, uint32_t want = H > 4096 ? H / 2 : 0) {
        if (room >= len) return;
        len = max(len, want);
        wave_sync();
        const uint32_t at = o0 + pos;
        // Complete blocks go out, a kilobyte per store where the chunk's
        // first bytes are past.
        while (fa >= o0 && fa + 2 * kBlock <= at) {
            *reinterpret_cast<uint4 *>(base + fa + 16 * lane()) =
                *reinterpret_cast<const uint4 *>(win + (fa - wlo) + 16 * lane());
            fa += 2 * kBlock;
        }
        while (fa + kBlock <= at) flush_block(o0 + cap);
        const uint32_t lo = (at + len - H + kBlock - 1) & ~(kBlock - 1), d = lo - wlo;
        // (A step's reads are at or past its writes; what the last one reads
        // past the output lands past the output.)
        for (uint32_t i = 0; i < at - lo; i += 1024) {
            const uint4 v = *reinterpret_cast<const uint4 *>(win + slide_from(d + i + 16 * lane(), H));
            wave_sync();
            *reinterpret_cast<uint4 *>(win + i + 16 * lane()) = v;
        }
        wlo = lo;
        room = wlo + H - at;
        wave_sync();
    }
    __device__ __forceinline__ void put_literal(uint32_t b) {
        make_room(1);
        win[slot(o0 + pos)] = (uint8_t)b;  // same byte from every lane
        pos++;
        room--;
    }
    // Back-reference: len bytes (at most 258) from dist bytes back (dist <=
    // pos).  With len > dist the bytes repeat with period dist.
    __device__ __forceinline__ void copy(uint32_t dist, uint32_t len) {
        make_room(len);
        const uint32_t dst = o0 + pos, src = dst - dist;
        if (src < wlo) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            for (uint32_t i = lane(); i < len; i += kWave) win[slot(dst + i)] = base[src + i];
        } else {
            copy_near(src, dst, dist, len);
        }
        pos += len;
        room -= len;
    }
    // A copy within the window by the whole wave, overlapping or not.
    __device__ __forceinline__ void copy_near(uint32_t src, uint32_t dst, uint32_t dist, uint32_t len) const {
        const uint8_t *from = win + (src - wlo);
        uint8_t *to = win + (dst - wlo);
        if (dist >= len) {
            for (uint32_t i = lane(); i < len; i += kWave) to[i] = from[i];
        } else {
            // Byte i is byte i mod dist of the period.  m is above 2^21 / dist
            // by at most 1 (the reciprocal's error is below a quarter of the
            // distance to the next multiple of 1 / dist), so with i and dist
            // below 1,024 the quotient i m >> 21 is exact.
            const uint32_t m = (uint32_t)(2097152.0f * __builtin_amdgcn_rcpf((float)dist)) + 1;
            for (uint32_t i = lane(); i < len; i += kWave) to[i] = from[i - dist * ((i * m) >> 21)];
        }
        wave_sync();
    }
    // Appends len >= kStream bytes of src (HBM): straight to the output, then
    // the window is filled from there.
    static constexpr uint32_t kStream = 4096;
    __device__ __forceinline__ void stream(const uint8_t *src, uint32_t len) {
        wave_sync();
        finish();
        wave_stream(base + o0 + pos, src, len);
        pos += len;
        const uint32_t end = o0 + pos;
        fa = end & ~(kBlock - 1);
        wlo = fa - 2 * kBlock;
        room = wlo + H - end;
        // The wave's own stores, read back.
        wait_vm();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        for (uint32_t a = wlo + 16 * lane(); a < end; a += 1024) {
            if (a + 16 <= end) {
                *reinterpret_cast<uint4 *>(win + (a - wlo)) = *reinterpret_cast<const uint4 *>(base + a);
            } else {
                for (uint32_t k = a; k < end; k++) win[k - wlo] = base[k];
            }
        }
        wave_sync();
    }
    // Writes every byte produced so far to HBM.
    __device__ __forceinline__ void finish() {
        const uint32_t end = o0 + pos;
        while (fa < end) flush_block(end);
    }
};

// Copies waiting to be made, in output order: length (3 to kMaxCopy) |
// offset of the output from the step's start << 16 | distance << 32.
constexpr uint32_t kCopyQueue = 152, kMaxCopy = 512;
__device__ __forceinline__ uint64_t copy_entry(uint32_t len, uint32_t at, uint32_t dist) {
    return ((uint64_t)dist << 32) | (at << 16) | len;
}

// Copies longer than this are made by the whole wave, one after another.
constexpr uint32_t kLongCopy = 32;

// Makes the copies of the lanes that are `ready` (sources final, in the window
// or, `far`, in HBM; no copy overlaps its own output), eight bytes per access
// at any alignment.
template <uint32_t H>
__device__ __forceinline__ void make_copies(const LinearOut<H> &o, bool ready, bool far, uint32_t src, uint32_t dst,
                                            uint32_t len) {
    const uint32_t l = lane();
    if (ready && len <= kLongCopy) {
        uint8_t *const to = o.win + (dst - o.wlo);
        const uint32_t tail = len > 8 ? len - 8 : 0u;
        uint64_t a, b;
        if (far) {
            a = *reinterpret_cast<const u64_any *>(o.base + src);
            b = *reinterpret_cast<const u64_any *>(o.base + src + tail);
        } else {
            const uint8_t *from = o.win + (src - o.wlo);
            a = *reinterpret_cast<const u64_any *>(from);
            b = *reinterpret_cast<const u64_any *>(from + tail);
        }
        if (len >= 8) {
            *reinterpret_cast<u64_any *>(to) = a;
            for (uint32_t j = 8; j < tail; j += 8) {
                uint64_t m;
                if (far) m = *reinterpret_cast<const u64_any *>(o.base + src + j);
                else m = *reinterpret_cast<const u64_any *>(o.win + (src - o.wlo) + j);
                *reinterpret_cast<u64_any *>(to + j) = m;
            }
            *reinterpret_cast<u64_any *>(to + tail) = b;
        } else if (len >= 4) {
            *reinterpret_cast<u32_any *>(to) = (uint32_t)a;
            *reinterpret_cast<u32_any *>(to + len - 4) = (uint32_t)(a >> (8 * (len - 4)));
        } else {
            *reinterpret_cast<u16_any *>(to) = (uint16_t)a;
            to[2] = (uint8_t)(a >> 16);
        }
    }
    for (uint64_t lm = ballot(ready && len > kLongCopy); lm; lm &= lm - 1) {
        const uint32_t k = (uint32_t)__builtin_ctzll(lm);
        const uint32_t cs = readlane(src, k), cd = readlane(dst, k), cl = readlane(len, k);
        for (uint32_t i = 8 * l; i < cl; i += 8 * kWave) {
            const uint32_t j = min(i, cl - 8);
            uint64_t a;
            if (cs < o.wlo) a = *reinterpret_cast<const u64_any *>(o.base + cs + j);
            else a = *reinterpret_cast<const u64_any *>(o.win + (cs - o.wlo) + j);
            *reinterpret_cast<u64_any *>(o.win + (cd - o.wlo) + j) = a;
        }
    }
}

// Runs the nq queued copies of an emission step whose output starts at
// `start`.  Their sources are the output before them: 64 copies at a time,
// every copy whose source ends before the lowest pending copy's output goes
// at once, eight bytes per access at any alignment (byte by byte, sixteen
// masked stores a piece, this was the larger half of a step).
template <uint32_t H>
__device__ __forceinline__ void run_copies(const LinearOut<H> &o, const uint64_t *queue, uint32_t nq,
                                           uint32_t start) {
    const uint32_t l = lane();
    for (uint32_t k0 = 0; k0 < nq; k0 += kWave) {
        const bool v = k0 + l < nq;
        const uint32_t at = min(k0 + l, kCopyQueue - 1);
        const uint64_t q = queue[at];
        const uint32_t len = v ? (uint32_t)q & 0xffff : 0u, dist = (uint32_t)(q >> 32);
        const uint32_t dst = start + ((uint32_t)q >> 16), src = dst - dist;
        const bool far = v && src < o.wlo;  // left the window: wholly in HBM
        if (ballot(far)) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        uint64_t pend = ballot(v);
        while (pend) {
            const uint32_t t = (uint32_t)__builtin_ctzll(pend), front = readlane(dst, t);
            const bool ready = ((pend >> l) & 1) && src + len <= front;
            const uint64_t rm = ballot(ready);
            if (!rm) {  // the lowest pending copy repeats its own output
                o.copy_near(readlane(src, t), front, readlane(dist, t), readlane(len, t));
                pend &= pend - 1;
                continue;
            }
            make_copies(o, ready, far, src, dst, len);
            pend &= ~rm;
            wave_sync();
        }
    }
}

}  // namespace codag
