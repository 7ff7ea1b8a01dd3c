// LZ4 block decode, one wavefront per chunk: an LDS input buffer
// (input_stream) and Deflate's LDS history window with kilobyte flushes to
// HBM (output_stream).  CODAG presents new codecs as device functions written
// against these two streams (Section III, Section IV-E); LZ4 is the
// byte-aligned member of the LZ77 family: a lane-parallel parse of the
// sequence chain, literals written as they are found, and the matches queued
// and made 64 at a time.
//
// A block is a list of sequences: a token byte (literal count in the high
// nibble, match length minus 4 in the low one; a nibble of 15 continues in
// bytes that add to it until one below 255), the literals, a 2-byte
// little-endian offset and the match length's continuation bytes.  The
// block ends right after some sequence's literals.
//
// Status order, field by field as they are read: a field cut off by the end
// of the chunk is TRUNCATED; a literal run longer than the output range left
// is OVERFLOW (before its bytes are looked at, as for a stored Deflate
// block); offset 0 or one past the bytes produced is CORRUPT (no dictionary)
// once the sequence's match length is read; a match past the range is
// OVERFLOW; a block that ends before the range is full is UNDERFLOW unless
// the range is a capacity.
#pragma once

#include "../../include/codag.h"
#include "stream.hpp"
#include "window.hpp"

namespace codag {

template <uint32_t H>
struct Lz4Lds {
    uint8_t window[H];
    uint8_t window_pad[16];  // eight-byte reads may pass the window's end
    uint64_t queue[kCopyQueue + 1];
};

// The chunk's input through one linear LDS buffer of 65 x 16 bytes from
// position a0 on, so fields are read at any alignment with one access.
// Bytes past the chunk read as zero within the buffer.
struct LinearIn {
    static constexpr uint32_t kPieces = 65, kBytes = 16 * kPieces;
    static constexpr uint32_t kLdsWords = kBytes / 4, kLand = 0;
    static constexpr uint32_t kMost = kBytes - 16;  // any so many bytes can be had at once

    const uint8_t *gbase;  // 16-byte aligned
    uint32_t skip;         // chunk start relative to gbase (0..15)
    uint32_t gend;         // one past the chunk's last byte, relative to gbase
    uint32_t a0;
    uint32_t *buf;

    __device__ __forceinline__ void init(const uint8_t *chunk, uint32_t len, uint32_t *lds, uint32_t *) {
        skip = (uint32_t)(reinterpret_cast<uintptr_t>(chunk) & 15);
        gbase = chunk - skip;
        gend = skip + len;
        buf = lds;
        load(0);
    }
    __device__ __forceinline__ void load(uint32_t pos) {
        a0 = pos & ~15u;
        wave_sync();
        load_pieces<kPieces, kWave>(gbase, gend, a0, buf, lane());
        wave_sync();
    }
    // Bytes [pos, pos + n) readable (n <= kMost).
    __device__ __forceinline__ void ensure(uint32_t pos, uint32_t n) {
        if (pos < a0 || pos + n > a0 + kBytes) load(pos);
    }
    __device__ __forceinline__ const uint8_t *at(uint32_t pos) const {
        return reinterpret_cast<const uint8_t *>(buf) + (pos - a0);
    }
    // Four bytes at pos, the same on every lane.
    __device__ __forceinline__ uint32_t peek4(uint32_t pos) {
        ensure(pos, 4);
        return uni(*reinterpret_cast<const u32_any *>(at(pos)));
    }
};

// A step's output in the making: literals are in the window, matches queued.
struct Lz4Step {
    uint32_t start, made, nq;
    uint32_t most;  // bytes it may take
};

// Room for a new step.
template <uint32_t H>
__device__ __forceinline__ void lz4_begin(LinearOut<H> &o, Lz4Step &s) {
    o.make_room(s.most);
    s.start = o.o0 + o.pos;
    s.made = s.nq = 0;
}
// Makes the queued matches; the step's bytes are output.
template <uint32_t H>
__device__ __forceinline__ void lz4_end(LinearOut<H> &o, const Lz4Lds<H> *lds, Lz4Step &s) {
    wave_sync();
    run_copies<H>(o, lds->queue, s.nq, s.start);
    o.pos += s.made;
    o.room -= s.made;
    s.made = s.nq = 0;
}

// Adds continuation bytes from position q on to len (a nibble was 15), 64 at a
// time: returns the position after the last one, or 0 if the chunk ends first.
// (One at a time the 257 of a 64 KiB field took 20 us.)
__device__ __forceinline__ uint32_t lz4_more(LinearIn &in, uint32_t q, uint32_t end, uint32_t &len) {
    for (;;) {
        if (q >= end) return 0;
        in.ensure(q, kWave);
        const uint32_t b = in.at(q)[lane()];
        const uint64_t m = ballot(b != 255);
        const uint32_t full = m ? (uint32_t)__builtin_ctzll(m) : (uint32_t)kWave;
        if (full >= end - q) return 0;  // (bytes past the end are not 255)
        // A run over 2^32 cannot fit any output range; saturate instead of
        // wrapping so the range check still fails.
        const uint32_t more = 255 * full + (m ? readlane(b, full) : 0u);
        len = len + more < len ? 0xffffffffu : len + more;
        if (m) return q + full + 1;
        q += kWave;
    }
}

// One sequence the general way (any field length, the last sequence, every
// status): returns kLz4More to go on, else the block's status (OK when this
// was its last sequence).  Fields that fit go into the step.
enum : int { kLz4More = 1 };

template <uint32_t H>
__device__ __forceinline__ int lz4_sequence(LinearIn &in, LinearOut<H> &o, Lz4Lds<H> *lds, Lz4Step &s, uint32_t &p,
                                            uint32_t end, uint32_t cap) {
    const uint32_t l = lane();
    const uint32_t tok = in.peek4(p) & 255;
    uint32_t lit = tok >> 4, q = p + 1;
    if (lit == 15) {
        q = lz4_more(in, q, end, lit);
        if (!q) return CODAG_E_TRUNCATED;
    }
    if (lit > cap - o.pos - s.made) return CODAG_E_OVERFLOW;
    if (lit > end - q) return CODAG_E_TRUNCATED;
    while (lit) {
        const uint32_t n = min(lit, 512u);  // eight bytes a lane
        if (s.made + n > s.most) {
            lz4_end(o, lds, s);
            lz4_begin(o, s);
        }
        in.ensure(q, n);
        uint8_t *const to = o.win + (s.start + s.made - o.wlo);
        if (n >= 8) {
            const uint32_t j = min(8 * l, n - 8);
            if (8 * l < n) *reinterpret_cast<u64_any *>(to + j) = *reinterpret_cast<const u64_any *>(in.at(q) + j);
        } else if (l < n) {
            to[l] = in.at(q)[l];
        }
        s.made += n;
        q += n;
        lit -= n;
    }
    if (q == end) return CODAG_OK;  // the last sequence carries no match
    if (end - q < 2) return CODAG_E_TRUNCATED;
    const uint32_t off = in.peek4(q) & 0xffff;
    q += 2;
    uint32_t mlen = tok & 15;
    if (mlen == 15) {
        q = lz4_more(in, q, end, mlen);
        if (!q) return CODAG_E_TRUNCATED;
    }
    mlen = mlen + 4 < mlen ? 0xffffffffu : mlen + 4;
    if (off == 0 || off > o.pos + s.made) return CODAG_E_CORRUPT;
    if (mlen > cap - o.pos - s.made) return CODAG_E_OVERFLOW;
    // Pieces of at most kMaxCopy bytes, none below the three that a copy has at
    // least; each repeats the bytes `off` back, so splitting a match does not
    // change what it writes.  A piece longer than the offset may as well read
    // any multiple of the offset back that the match has come: pieces after the
    // first do not overlap themselves, and two go at once (a 64 KiB block of
    // zeros 127 to 95 us).
    for (uint32_t done = 0; done < mlen;) {
        const uint32_t n = mlen - done > kMaxCopy ? kMaxCopy - 8 : mlen - done;
        if (s.made + n > s.most || s.nq == kCopyQueue) {
            lz4_end(o, lds, s);
            lz4_begin(o, s);
        }
        const uint32_t dist = off >= n || done == 0 ? off : off * ((off + min(done, 2 * kMaxCopy)) / off);
        lds->queue[s.nq] = copy_entry(n, s.made, dist);  // the same from every lane
        s.nq++;
        s.made += n;
        done += n;
    }
    p = q;
    return kLz4More;
}

__device__ __forceinline__ uint64_t lz4_bit(uint32_t x) { return x < 64 ? 1ull << x : 0ull; }

// Every lane parses the sequence that would start at its own byte of a
// 64-byte input window (at most 14 literals, a match length with at most one
// continuation byte).  The real sequence starts are the chain of next-start
// links from the window's first byte; each lane gathers, by lane permutes,
// where its links lead over eight steps and which lanes they pass, so a
// wave-uniform walk covers eight sequences with two lane reads.  The window's
// share of the step is the chain's prefix up to anything the general step
// must judge: a long field, the block's last sequence, a cut-off stream,
// output past the range, an offset reaching before the chunk's output (the
// last two found with a prefix sum over the chain).  Its lanes write their
// literals into the window, eight bytes at a time, and queue their matches;
// the step ends when the queue or kAppend bytes are full, so 64 matches are
// made at once instead of a window's ten to twenty.  What bounds it is the
// parse: some 60 vector instructions and five dependent lane permutes a
// window.  Measured against a batch per window with byte-wise copies: 4,096
// chunks of 64 KiB 2.43 to 1.38 ms, 97 lone blocks of 64 KiB 1.69 to 1.03 ms.
template <uint32_t H>
__device__ __forceinline__ int decode_lz4(LinearIn &in, uint8_t *out, uint32_t cap, Lz4Lds<H> *lds,
                                          uint32_t *made = nullptr) {
    constexpr uint32_t kAppend = LinearOut<H>::kAppend;
    const uint32_t l = lane();
    LinearOut<H> o;
    o.init(out, cap, lds->window);
    const uint32_t end = in.gend;
    uint32_t p = in.skip;
    int st = CODAG_OK;
    Lz4Step s;
    s.most = kAppend;
    lz4_begin(o, s);
    for (;;) {
        if (p >= end) { st = CODAG_E_TRUNCATED; break; }
        in.ensure(p, kWave + 32);
        // This lane's candidate.
        const uint32_t x = p + l;
        const uint8_t *const at = in.at(x);
        const uint32_t tok = at[0], lit = tok >> 4, ml = tok & 15;
        const uint32_t f = *reinterpret_cast<const u32_any *>(at + 1 + lit);  // offset, a continuation byte
        const uint32_t off = f & 0xffff, more = ml == 15 ? 1u : 0u, ext = (f >> 16) & 255;
        const uint32_t inl = 3 + lit + more, mlen = ml + 4 + (more ? ext : 0u), outl = lit + mlen;
        // What a sequence needs on its own: short fields, a nonzero offset,
        // its bytes inside the chunk and followed by more (the last sequence
        // has no offset).
        const bool ok = lit < 15 && !(more && ext == 255) && off != 0 && x + inl <= end;
        // Links: the next start (64 = none in this window, or stop here).
        const uint32_t n1 = ok ? min(l + inl, 64u) : 64u;
        const uint32_t n2 = lane_follow(n1, n1);
        const uint32_t n3 = lane_follow(n1, n2);
        const uint32_t n4 = lane_follow(n1, n3);
        const uint64_t m4 = lz4_bit(l) | lz4_bit(n1) | lz4_bit(n2) | lz4_bit(n3);
        const uint32_t n8 = lane_follow(n4, n4);
        const uint32_t m8h = lane_pull((uint32_t)(m4 >> 32), n4), m8l = lane_pull((uint32_t)m4, n4);
        const uint64_t m8 = m4 | (n4 < 64 ? (uint64_t)m8h << 32 | m8l : 0ull);
        // Links only lead forward, so eight steps of eight cover the window;
        // the bound is a second guard.
        uint64_t chain = 0;
        for (uint32_t t = 0, step = 0; t < 64 && step < 8; step++) {
            chain |= readlane64(m8, t);
            t = readlane(n8, t);
        }
        // The chain runs through sequences that are fine on their own and
        // ends at (and includes) the first that is not, if any.
        uint64_t exe = chain & ballot(ok);
        const uint32_t my_out = (exe >> l) & 1 ? outl : 0u;
        const uint32_t incl = wave_inclusive_sum32(my_out), before = incl - my_out;
        const uint32_t done = o.pos + s.made;
        const uint64_t fm = ballot(((exe >> l) & 1) && (incl > cap - done || off > done + before + lit));
        if (fm) exe &= (fm & (0 - fm)) - 1;
        if (!exe) {
            st = lz4_sequence(in, o, lds, s, p, end, cap);
            if (st != kLz4More) break;
            st = CODAG_OK;
            continue;
        }
        // What the step has room for: its first sequence always goes into an
        // empty step.
        const uint64_t nofit = ballot(((exe >> l) & 1) && (s.made + incl > kAppend ||
                                                            s.nq + count_below(exe) >= kCopyQueue));
        if (nofit) exe &= (nofit & (0 - nofit)) - 1;
        if (exe) {
            const uint32_t last = 63 - (uint32_t)__builtin_clzll(exe);
            const bool mine = (exe >> l) & 1;
            const uint32_t dl = s.made + before;  // this sequence's literals, from the step's start
            if (ballot(mine && lit)) {
                const uint64_t a = *reinterpret_cast<const u64_any *>(at + 1);
                const uint64_t b = *reinterpret_cast<const u64_any *>(at + 1 + (lit >= 8 ? lit - 8 : 0u));
                uint8_t *const to = o.win + (s.start + dl - o.wlo);
                if (mine && lit >= 8) {
                    *reinterpret_cast<u64_any *>(to) = a;
                    *reinterpret_cast<u64_any *>(to + lit - 8) = b;
                } else if (mine && lit >= 4) {
                    *reinterpret_cast<u32_any *>(to) = (uint32_t)a;
                    *reinterpret_cast<u32_any *>(to + lit - 4) = (uint32_t)(a >> (8 * (lit - 4)));
                } else if (mine && lit) {
                    to[0] = (uint8_t)a;
                    if (lit > 1) to[1] = (uint8_t)(a >> 8);
                    if (lit > 2) to[2] = (uint8_t)(a >> 16);
                }
            }
            if (mine) lds->queue[s.nq + count_below(exe)] = copy_entry(mlen, dl + lit, off);
            s.nq += (uint32_t)__builtin_popcountll(exe);
            s.made += readlane(incl, last);
            p += last + readlane(inl, last);
        }
        if (nofit || s.nq == kCopyQueue) {
            lz4_end(o, lds, s);
            lz4_begin(o, s);
        }
    }
    lz4_end(o, lds, s);
    o.finish();
    if (st) return st;
    if (made) {
        *made = o.pos;
        return CODAG_OK;
    }
    return o.pos == cap ? CODAG_OK : CODAG_E_UNDERFLOW;
}

}  // namespace codag
