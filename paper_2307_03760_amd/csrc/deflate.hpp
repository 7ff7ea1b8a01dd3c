// Deflate (RFC 1951) decoding by one wavefront.
//
// CODAG (Section II-A, III) locates Deflate's cost in Huffman decoding and
// dictionary copies.  Here:
//   * A block's symbols are decoded by all lanes at once, each lane decoding
//     its own stretch of the input with lookups in LDS tables that the whole
//     wave builds in parallel for each block (inflate_lanes below).  Headers
//     and whatever is rare are wave-uniform scalar code: a 64-bit bit buffer
//     in scalar registers, refilled one 32-bit word at a time from the LDS
//     input ring.
//   * Output goes first to a per-wave history window in LDS (the last H bytes
//     of output) and reaches HBM behind the decoder, 1 KiB at a time, as one
//     16-byte store per lane of an aligned kilobyte ("coalesced on-demand
//     writing", Section IV-F).  Literals ("write_byte") are one LDS byte write
//     each; back-references ("memcpy", Section IV-F) are copied by all lanes
//     at once from the window, including the overlapping case where the
//     length exceeds the distance.  Only a reference reaching further back
//     than the window reads HBM.  Reading just-written output from HBM would
//     make each copy wait for all outstanding stores of the wave.
#pragma once

#include "../../include/codag.h"
#include "stream.hpp"
#include "window.hpp"

namespace codag {

// Table entry (32 bits).  Bits 0-4: input bits of the code and its extra bits
// together; 5-8: code length; 9-12: extra-bit count.
//   literal/length table: 12-20 output bytes (1 for a literal, the base
//     length for a copy; ex is at most 5, bits 9-11), 21-28 the literal;
//   distance table: 13-27 the base distance;
//   code-length table: 13-17 the symbol.
// With kEntStop, bits 21-22 say why: end of block, no code starts with these
// bits, or a code for a symbol that may not appear (286, 287; 30, 31).
// Everything a token needs is in its two entries, so decoding a token takes
// no arithmetic on symbols (16-bit entries with the bases in closed form
// cost about 20 more vector instructions per candidate).
constexpr uint32_t kEntSlow = 1u << 29;  // code longer than the table: canonical decode
constexpr uint32_t kEntStop = 1u << 30;
constexpr uint32_t kEntCopy = 1u << 31;  // length symbol
enum : uint32_t { kWhyEob = 1, kWhyInvalid = 2, kWhyBadSym = 3 };
constexpr uint32_t kEntInvalid = kEntStop | (kWhyInvalid << 21);

enum TableUse { kLitLen = 0, kDist = 1, kCodeLen = 2 };

__device__ __forceinline__ uint32_t ent_bits(uint32_t e) { return e & 31; }
__device__ __forceinline__ uint32_t ent_cl(uint32_t e) { return (e >> 5) & 15; }
__device__ __forceinline__ uint32_t ent_ex(uint32_t e) { return (e >> 9) & 15; }     // distance entries
__device__ __forceinline__ uint32_t ent_lex(uint32_t e) { return (e >> 9) & 7; }     // literal/length entries
__device__ __forceinline__ uint32_t ent_len(uint32_t e) { return (e >> 12) & 511; }
__device__ __forceinline__ uint32_t ent_byte(uint32_t e) { return (e >> 21) & 255; }
__device__ __forceinline__ uint32_t ent_why(uint32_t e) { return (e >> 21) & 3; }
__device__ __forceinline__ uint32_t ent_dist(uint32_t e) { return (e >> 13) & 0x7fff; }
__device__ __forceinline__ uint32_t ent_sym(uint32_t e) { return (e >> 13) & 31; }   // code lengths

// Length and distance bases and extra-bit counts (RFC 1951 section 3.2.5)
// in closed form.
__device__ __forceinline__ uint32_t length_extra(uint32_t k) {  // k = symbol - 257
    return (k < 8 || k == 28) ? 0 : (k >> 2) - 1;
}
__device__ __forceinline__ uint32_t length_base(uint32_t k) {
    return k < 8 ? k + 3 : k == 28 ? 258 : ((4 + (k & 3)) << ((k >> 2) - 1)) + 3;
}
__device__ __forceinline__ uint32_t dist_extra(uint32_t d) { return d < 4 ? 0 : (d >> 1) - 1; }
__device__ __forceinline__ uint32_t dist_base(uint32_t d) {
    return d < 4 ? d + 1 : ((2 + (d & 1)) << ((d >> 1) - 1)) + 1;
}

// The entry of symbol s with a code of cl bits.
__device__ __forceinline__ uint32_t table_entry(int use, uint32_t s, uint32_t cl) {
    if (use == kCodeLen) return cl | (cl << 5) | (s << 13);
    if (use == kLitLen) {
        if (s < 256) return cl | (cl << 5) | (1u << 12) | (s << 21);
        if (s == 256) return cl | (cl << 5) | kEntStop | (kWhyEob << 21);
        if (s > 285) return cl | (cl << 5) | kEntStop | (kWhyBadSym << 21);
        const uint32_t ex = length_extra(s - 257);
        return (cl + ex) | (cl << 5) | (ex << 9) | (length_base(s - 257) << 12) | kEntCopy;
    }
    if (s > 29) return cl | (cl << 5) | kEntStop | (kWhyBadSym << 21);
    const uint32_t ex = dist_extra(s);
    return (cl + ex) | (cl << 5) | (ex << 9) | (dist_base(s) << 13);
}

// Canonical decoding of one code: codes of length k, left-aligned to 15
// bits, lie below lim[k] (and at or above lim[k - 1]); their symbols are
// sorted[base[k] + code].
struct CodeMeta {
    uint16_t lim[16];
    uint16_t base[16];  // modulo 2^16
};

struct BuildResult {
    int32_t left;    // unused codes scaled to 2^15 (< 0: over-subscribed)
    uint32_t total;  // number of symbols with a code
    uint32_t ones;   // number of codes of length 1
};

// Builds the lookup table (2^tb entries) of the canonical code whose lengths
// are lens[0..n) (n <= 320), lane-parallel: per-length counts and each
// symbol's rank come from ballots, then every slot of the table decodes its
// own index.  (13,000 cycles for a literal/length table, 14,000 to 35,000 with
// the symbols filling their slots; 5,000 instead of 11,000 for distances.)
__device__ __forceinline__ BuildResult build_table(const uint8_t *lens, uint32_t n, uint32_t tb,
                                                   int use, uint32_t *tab, uint16_t *sorted,
                                                   CodeMeta *meta) {
    const uint32_t l = lane();
    uint32_t cnt[16];
#pragma unroll
    for (int k = 0; k < 16; k++) cnt[k] = 0;
    uint32_t rank[5];
#pragma unroll
    for (int p = 0; p < 5; p++) {
        rank[p] = 0;
        if (64u * p >= n) break;
        uint32_t s = 64 * p + l;
        uint32_t m = s < n ? lens[s] : 0;
#pragma unroll
        for (int len = 1; len < 16; len++) {
            uint64_t b = ballot(m == (uint32_t)len);
            if (m == (uint32_t)len) rank[p] = cnt[len] + count_below(b);
            cnt[len] += (uint32_t)__builtin_popcountll(b);
        }
    }
    BuildResult r;
    int32_t left = 1;
    uint32_t total = 0;
#pragma unroll
    for (int len = 1; len < 16; len++) {
        left = 2 * left - (int32_t)cnt[len];
        total += cnt[len];
        if (left < 0) break;
    }
    r.left = left;
    r.total = total;
    r.ones = cnt[1];
    if (left < 0) return r;
    {
        uint32_t code = 0, off = 0, lim = 0, base = 0;
#pragma unroll
        for (int len = 1; len < 16; len++) {
            if ((uint32_t)len == l) {
                lim = (code + cnt[len]) << (15 - len);
                base = off - code;
            }
            off += cnt[len];
            code = (code + cnt[len]) << 1;
        }
        if (l < 16) {
            meta->lim[l] = (uint16_t)lim;
            meta->base[l] = (uint16_t)base;
        }
    }
    wave_sync();
#pragma unroll
    for (int p = 0; p < 5; p++) {
        if (64u * p >= n) break;
        uint32_t s = 64 * p + l;
        uint32_t m = s < n ? lens[s] : 0;
        if (m != 0) {
            // The first code of length m is the limit below it at m bits.
            const uint32_t code = ((uint32_t)meta->lim[m - 1] >> (15 - m)) + rank[p];
            sorted[(uint16_t)(meta->base[m] + code)] = (uint16_t)s;
        }
    }
    wave_sync();
    // Every slot decodes its own index: the same work for every code, where a
    // symbol filling its own slots takes up to 2^tb / 2 stores on one lane.
    for (uint32_t i = l; i < (1u << tb); i += kWave) {
        const uint32_t rev = __builtin_bitreverse32(i) >> 17;
        uint32_t len = 1;
#pragma unroll
        for (uint32_t k = 1; k < 16; k++) len += rev >= meta->lim[k] ? 1u : 0u;
        uint32_t e = kEntInvalid;  // past the last code of an incomplete set
        if (len <= tb) e = table_entry(use, sorted[(uint16_t)(meta->base[len] + (rev >> (15 - len)))], len);
        else if (len < 16) e = kEntSlow;
        tab[i] = e;
    }
    wave_sync();
    return r;
}

constexpr uint32_t kDistBits = 8;
constexpr uint32_t kCodeLenBits = 7;

// The tables of the fixed code (RFC 1951 3.2.6), every entry from its index: no
// code is longer than a table's bits, so nothing looks at the canonical lists.
// (Through build_table they took 18,000 cycles: 256 chunks of 11 compressed
// bytes 15.2 us that way and 9.9 so, of 97 bytes 21.1 and 15.1.)
template <int TB>
__device__ __forceinline__ void build_fixed(uint32_t *lit, uint32_t *dist) {
    static_assert(TB >= 9 && kDistBits >= 5, "fixed codes fit the tables");
    for (uint32_t i = lane(); i < (1u << TB); i += kWave) {
        const uint32_t c = __builtin_bitreverse32(i) >> 23, c8 = c >> 1;
        uint32_t len = 8, sym = c8 - 48;                     // 00110000 on: 0..143
        if (c8 < 48) len = 7, sym = 256 + (c >> 2);          // 0000000 on: 256..279
        else if (c8 >= 200) len = 9, sym = c - 400 + 144;    // 110010000 on: 144..255
        else if (c8 >= 192) sym = c8 - 192 + 280;            // 11000000 on: 280..287
        lit[i] = table_entry(kLitLen, sym, len);
    }
    for (uint32_t i = lane(); i < (1u << kDistBits); i += kWave)
        dist[i] = table_entry(kDist, __builtin_bitreverse32(i) >> 27, 5);
    wave_sync();
}

// Order in which the code-length code's lengths are sent (RFC 1951 3.2.7).
__constant__ const uint8_t kCodeLenOrder[19] = {16, 17, 18, 0, 8,  7, 9,  6, 10, 5,
                                                11, 4,  12, 3, 13, 2, 14, 1, 15};

// A round of the lane-parallel decoder takes 64 lanes x 256 bits of input,
// each lane's share cut into four segments of 64 bits.
constexpr uint32_t kLaneBits = 256, kSegBits = 64, kLaneSegs = kLaneBits / kSegBits;
constexpr uint32_t kRoundSegs = kWave * kLaneSegs;
// The round's input: 64 x 32 bytes, up to 8 bytes of alignment before them
// and the eight-byte reads past the last bit, in 16-byte pieces.
constexpr uint32_t kRoundPieces = kWave * kLaneBits / 128 + 2, kRoundInWords = 4 * kRoundPieces;

// A block's Huffman tables.
template <int TB>
struct DeflateTables {
    // Literal/length codes, distance codes (their part also serves the
    // code-length code), and one zero: the entry of a lane with nothing to
    // decode, which takes no bits and makes no output.
    static constexpr uint32_t kIdle = (1u << TB) + (1u << kDistBits);
    uint32_t tab[(1u << TB) + (1u << kDistBits) + 1];
    CodeMeta meta[2];
    uint16_t sorted[288 + 32];

    __device__ __forceinline__ uint32_t *dist() { return tab + (1u << TB); }
    __device__ __forceinline__ const uint32_t *dist() const { return tab + (1u << TB); }
    __device__ __forceinline__ uint16_t *dist_sorted() { return sorted + 288; }
};

// What one wave keeps in LDS while inflating, besides its input: the Huffman
// tables, the output history window and the lane-parallel decoder's lists.
template <int TB, uint32_t H>
struct DeflateLds : DeflateTables<TB> {
    union {
        uint8_t lens[320];          // while a block's tables are built
        uint32_t segs[kRoundSegs];  // while its symbols decode
    };
    uint64_t queue[kCopyQueue];  // pending copies
    __attribute__((aligned(16))) uint8_t window[H];
    union {
        uint8_t window_pad[16];  // eight-byte reads may pass the window's end; nothing is written here
        uint32_t block[4];       // BlockLength's
    };
};

// Wave-uniform LSB-first bit reader over the ring.
struct BitIn {
    uint64_t buf;    // valid bits are the low `cnt`
    uint32_t cnt;
    uint32_t next;   // byte position of the next (aligned) word to load
    int32_t remain;  // input bits not yet consumed (negative: past the end);
                     // 32 bits because there is no scalar 64-bit ordered
                     // compare (chunks are below 256 MiB)

    template <class Ring>
    __device__ __forceinline__ void seek(Ring &in, uint32_t pos) {
        if (pos >= in.loaded + Ring::kFetch) in.restart(pos);
        uint32_t a = pos & ~3u;
        in.ensure(a + 4);
        uint32_t w = uni(in.word(a >> 2));
        uint32_t sh = 8 * (pos & 3);
        buf = w >> sh;
        cnt = 32 - sh;
        next = a + 4;
        remain = 8 * ((int32_t)in.gend - (int32_t)pos);
    }
    template <class Ring>
    __device__ __forceinline__ void refill(Ring &in) {
        if (cnt <= 32) {
            if (in.loaded < next + 4) in.ensure(next + 4);
            uint32_t w = uni(in.word(next >> 2));
            buf |= (uint64_t)w << cnt;
            cnt += 32;
            next += 4;
        }
    }
    // Consume n bits (n <= cnt); false if that runs past the end of input.
    __device__ __forceinline__ bool drop(uint32_t n) {
        buf >>= n;
        cnt -= n;
        remain -= (int32_t)n;
        return remain >= 0;
    }
    // Consume n bits without the end-of-input test.  Bits past the end read
    // as zero; `remain` only decreases, so a decoder that tests it wherever
    // it stops (an error, the end of a block) reports running past the end
    // exactly where a bit-by-bit reader would have.
    __device__ __forceinline__ void skip(uint32_t n) {
        buf >>= n;
        cnt -= n;
        remain -= (int32_t)n;
    }
    // Refill with at most one ring advance (the reader moves 4 bytes at a
    // time, the ring 1 KiB), keeping the hot loop free of inner loops.
    template <class Ring>
    __device__ __forceinline__ void refill1(Ring &in) {
        if (cnt <= 32) {
            if (in.loaded < next + 4) in.commit();
            uint32_t w = uni(in.word(next >> 2));
            buf |= (uint64_t)w << cnt;
            cnt += 32;
            next += 4;
        }
    }
    __device__ __forceinline__ uint32_t peek(uint32_t n) const {
        return (uint32_t)(buf & ((1ull << n) - 1));
    }
    // Bit position of the next unconsumed bit.
    __device__ __forceinline__ uint32_t pos() const { return 8 * next - cnt; }
    // Byte position of the next unconsumed bit (on a byte boundary).
    __device__ __forceinline__ uint32_t byte_pos() const { return next - cnt / 8; }
};

// Canonical decode of a code longer than a table of tb bits (CODAG's
// "Huffman tree traversal"): the code's length is where its bits, left-
// aligned, fall below that length's limit.  x holds the next 15 bits at
// least; per lane, and the same code serves the wave-uniform reader.
__device__ __forceinline__ uint32_t slow_entry(uint32_t x, uint32_t tb, const CodeMeta *meta,
                                               const uint16_t *sorted, int use) {
    const uint32_t rev = __builtin_bitreverse32(x) >> 17;
    uint32_t len = tb + 1;
#pragma unroll
    for (uint32_t k = 1; k < 16; k++)
        if (k > tb) len += rev >= meta->lim[k] ? 1u : 0u;
    if (len > 15) return kEntInvalid;
    const uint32_t at = (uint16_t)(meta->base[len] + (rev >> (15 - len)));
    return table_entry(use, sorted[min(at, use == kLitLen ? 287u : 31u)], len);
}

// Single-byte LDS writes in the decode loops are issued by all lanes with
// the same address and value rather than by one lane: a one-lane branch
// inside a loop that also has early exits makes the compiler treat the loop
// exit as divergent, which moves the whole bit reader out of scalar
// registers.

// Reads a dynamic block's header up to its code lengths (RFC 1951 3.2.7):
// HLIT, HDIST, HCLEN, the code-length code (built into cltab, 7-bit
// table), then the HLIT + HDIST lengths into lens.  Returns a status.
template <class Ring>
__device__ __forceinline__ int read_code_lengths(Ring &in, BitIn &bi, uint32_t *cltab,
                                                 CodeMeta *meta, uint16_t *sorted, uint8_t *lens,
                                                 uint32_t &hlit, uint32_t &hdist, uint32_t &hclen) {
    const uint32_t l = lane();
    bi.refill(in);
    hlit = bi.peek(5) + 257;
    hdist = ((uint32_t)(bi.buf >> 5) & 31) + 1;
    hclen = ((uint32_t)(bi.buf >> 10) & 15) + 4;
    if (!bi.drop(14)) return CODAG_E_TRUNCATED;
    if (hlit > 286 || hdist > 30) return CODAG_E_CORRUPT;
    if (l < 19) lens[l] = 0;
    __builtin_amdgcn_wave_barrier();
    for (uint32_t i = 0; i < hclen; i++) {
        bi.refill(in);
        uint32_t v = bi.peek(3);
        if (!bi.drop(3)) return CODAG_E_TRUNCATED;
        lens[kCodeLenOrder[i]] = (uint8_t)v;  // same byte from every lane
    }
    __builtin_amdgcn_wave_barrier();
    BuildResult cl = build_table(lens, 19, kCodeLenBits, kCodeLen, cltab, sorted, meta);
    if (cl.left != 0) return CODAG_E_CORRUPT;
    uint32_t idx = 0, total = hlit + hdist, prev = 0;
    // The lengths a 64-bit window at a time: every lane decodes the symbol
    // that would start at its bit, a walk marks the real ones, a prefix sum
    // gives their places.  (Symbol by symbol a block's 300 lengths took about
    // 350 cycles each, a tenth of a 64 KiB chunk's time.)  Anything unusual --
    // the end of the input near, a repeat past the last length or without one
    // before it -- is left to the loop below.
    for (uint32_t s = l; s < 320; s += kWave) lens[s] = 0;
    wave_sync();
    uint32_t p = bi.pos();
    while (idx < total && p + 128 <= 8 * in.gend) {
        in.ensure((p >> 3) + 24);
        const uint32_t a = p + l;
        const uint32_t x = __builtin_amdgcn_alignbit(in.word((a >> 5) + 1), in.word(a >> 5), a & 31);
        const uint32_t e = cltab[x & ((1u << kCodeLenBits) - 1)];
        const uint32_t sym = ent_sym(e), cl = ent_cl(e);
        const uint32_t ex = sym < 16 ? 0u : sym == 16 ? 2u : sym == 17 ? 3u : 7u;
        const uint32_t rep = (sym < 16 ? 1u : sym == 18 ? 11u : 3u) + ((x >> cl) & ((1u << ex) - 1));
        const uint32_t step = (cl + ex) | (rep << 8);
        uint32_t t = 0, n = idx;
        uint64_t mark = 0;
        while (t < kWave && n < total) {
            const uint32_t w = readlane(step, t);
            mark |= 1ull << t;
            t += w & 255;
            n += w >> 8;
        }
        const uint64_t m16 = ballot(sym == 16);
        if (n > total || (idx == 0 && (m16 & 1))) break;
        const bool mine = (mark >> l) & 1;
        const uint32_t reps = mine ? rep : 0u;
        const uint32_t at = idx + wave_inclusive_sum32(reps) - reps;
        const uint32_t own = sym < 16 ? sym : 0u;
        const uint64_t below = mark & ~m16 & ((1ull << l) - 1);
        const uint32_t pulled = lane_pull(own, 63 - (uint32_t)__builtin_clzll(below | 1));
        const uint32_t val = sym != 16 ? own : below ? pulled : prev;
        if (mine && val) {
            const uint32_t k = sym == 16 ? rep : 1u;  // 1, or 3..6
            for (uint32_t j = 0; j < k; j++) lens[at + j] = (uint8_t)val;
        }
        prev = readlane(val, 63 - (uint32_t)__builtin_clzll(mark));
        idx = n;
        p += t;
    }
    bi.seek(in, p >> 3);
    bi.skip(p & 7);
    while (idx < total) {
        bi.refill(in);
        uint32_t e = uni(cltab[bi.peek(kCodeLenBits)]);
        uint32_t sym = ent_sym(e);
        if (!bi.drop(ent_cl(e))) return CODAG_E_TRUNCATED;
        if (sym < 16) {
            lens[idx] = (uint8_t)sym;  // same byte from every lane
            prev = sym;
            idx++;
            continue;
        }
        uint32_t rep, val;
        if (sym == 16) {
            if (idx == 0) return CODAG_E_CORRUPT;
            rep = 3 + bi.peek(2);
            if (!bi.drop(2)) return CODAG_E_TRUNCATED;
            val = prev;
        } else if (sym == 17) {
            rep = 3 + bi.peek(3);
            if (!bi.drop(3)) return CODAG_E_TRUNCATED;
            val = 0;
        } else {
            rep = 11 + bi.peek(7);
            if (!bi.drop(7)) return CODAG_E_TRUNCATED;
            val = 0;
        }
        if (idx + rep > total) return CODAG_E_CORRUPT;
        for (uint32_t k = l; k < rep; k += kWave) lens[idx + k] = (uint8_t)val;
        prev = val;
        idx += rep;
    }
    __builtin_amdgcn_wave_barrier();
    return CODAG_OK;
}

// Not statuses: a symbol was decoded and the block goes on; the next symbol
// is for inflate_symbol.
enum : int { kMore = 1, kOneSymbol = 2 };

// One symbol of a Huffman block, however unusual: kMore after a literal or a
// copy, CODAG_OK at the end of the block, or an error status; running past
// the end of input at or before that point is CODAG_E_TRUNCATED.
template <int TB, uint32_t H, class Ring>
__device__ __forceinline__ int inflate_symbol(Ring &in, BitIn &bi, LinearOut<H> &o, DeflateLds<TB, H> *lds) {
    bi.refill1(in);
    uint32_t e = uni(lds->tab[bi.peek(TB)]);
    if (e & kEntSlow) e = uni(slow_entry((uint32_t)bi.buf, TB, &lds->meta[0], lds->sorted, kLitLen));
    bi.skip(ent_cl(e));
    int st;
    if (e & kEntStop) {  // end of block, or an invalid code
        st = ent_why(e) == kWhyEob ? CODAG_OK : CODAG_E_CORRUPT;
    } else if (!(e & kEntCopy)) {
        if (o.pos != o.cap) {
            o.put_literal(ent_byte(e));
            return kMore;
        }
        st = CODAG_E_OVERFLOW;
    } else {
        // Length, then distance.
        const uint32_t lex = ent_lex(e);
        const uint32_t len = ent_len(e) + bi.peek(lex);
        bi.skip(lex);
        bi.refill1(in);
        uint32_t d = uni(lds->dist()[bi.peek(kDistBits)]);
        if (d & kEntSlow) d = uni(slow_entry((uint32_t)bi.buf, kDistBits, &lds->meta[1], lds->dist_sorted(), kDist));
        bi.skip(ent_cl(d));
        st = CODAG_E_CORRUPT;  // an invalid code, or a block without distance codes
        if (!(d & kEntStop)) {
            const uint32_t dist = ent_dist(d) + bi.peek(ent_ex(d));
            bi.skip(ent_ex(d));
            if (dist <= o.pos) {
                if (o.pos + len <= o.cap) {
                    o.copy(dist, len);
                    return kMore;
                }
                st = CODAG_E_OVERFLOW;
            }
        }
    }
    return bi.remain < 0 ? CODAG_E_TRUNCATED : st;
}

// ---------------------------------------------------------------------------
// Batched symbol decoding.
//
// The serial dependency of Huffman decoding is the position of the next
// code.  Here every lane decodes, from its own bit offset b + lane, the whole
// token that would start there -- a literal, or a length code with its extra
// bits and the distance code with its extra bits -- with two table lookups
// issued by all lanes at once.  A wave-uniform walk then follows the real
// token starts through those 64 candidates with one lane read per token, and
// collects up to 64 tokens (at most kBatchOut output bytes) in registers.
// The batch is then written out: literals by one store per lane, copies
// whose source lies before the batch lane-parallel (one lane per copy), and
// the few copies that read bytes of the batch itself one after another.
// Anything unusual (codes longer than the tables, invalid codes, an output
// overflow, a distance reaching before the chunk) ends the batch and goes
// through one step of the symbol-at-a-time loop above, so the statuses are
// exactly that loop's.
// ---------------------------------------------------------------------------

constexpr uint32_t kBatchOut = 1024;

// Token words: a literal is 1 << 16 | byte, a copy is length << 16 | 0x8000;
// bits 8-13 hold the bits the token takes in the input; 0x4000 marks a
// token the batch cannot take (0x4000: end of block, 0xc000: anything that
// needs the symbol-at-a-time path).
constexpr uint32_t kTokCopy = 0x8000u, kTokStop = 0x4000u, kTokOther = 0xc000u;

// The token starting at bit b + lane (b + 63 at most), as a token word, and
// a copy's distance (0 otherwise).  The lane's 64 input bits come from the
// wave-uniform words s0..s4 (input words b/32 .. b/32 + 4); a length code
// with its extra bits, the distance code and its extra bits take at most 36
// bits.
template <int TB, uint32_t H, bool ALIGNED = false>
__device__ __forceinline__ void lane_token(uint32_t s0, uint32_t s1, uint32_t s2, uint32_t s3,
                                           uint32_t s4, uint32_t b, const DeflateLds<TB, H> *lds,
                                           uint32_t &info, uint32_t &dist) {
    // ALIGNED: b is a multiple of 32, so lane l starts in word l / 32 and
    // s4 is not needed.
    const uint32_t a = (ALIGNED ? 0u : (b & 31)) + lane();
    const uint32_t k = a >> 5, sh = a & 31;
    const uint32_t wa = ALIGNED ? (k ? s1 : s0) : k == 0 ? s0 : k == 1 ? s1 : s2;
    const uint32_t wb = ALIGNED ? (k ? s2 : s1) : k == 0 ? s1 : k == 1 ? s2 : s3;
    const uint32_t wc = ALIGNED ? (k ? s3 : s2) : k == 0 ? s2 : k == 1 ? s3 : s4;
    const uint64_t x = ((uint64_t)__builtin_amdgcn_alignbit(wc, wb, sh) << 32) |
                       __builtin_amdgcn_alignbit(wb, wa, sh);
    const uint32_t xl = (uint32_t)x;
    const uint32_t e = lds->tab[xl & ((1u << TB) - 1)];
    // Every lane also decodes a length/distance pair from its bits (the
    // distance lookup reads the table whatever the entry was) and the kind
    // picks the result: no branches, so no scalar mask bookkeeping.  The
    // length code and its extra bits end by bit 20, the distance code's
    // index by bit 28, its extra bits by bit 50.  The choices are
    // all-ones/zero masks rather than conditionals, which the compiler would
    // turn back into branches.
    const uint32_t cl = ent_cl(e), p2 = ent_bits(e);
    const uint32_t len = ent_len(e) + ((xl >> cl) & ((1u << ent_lex(e)) - 1));
    const uint32_t d = lds->dist()[(xl >> p2) & ((1u << kDistBits) - 1)];
    const uint32_t q = p2 + ent_cl(d), dex = ent_ex(d);
    const uint32_t dv = ent_dist(d) + ((uint32_t)(x >> q) & ((1u << dex) - 1));
    const uint32_t odd = e & (kEntSlow | kEntStop);
    const uint32_t m_lit = 0u - (uint32_t)(odd == 0 && !(e & kEntCopy));
    const uint32_t m_eob = 0u - (uint32_t)((e & kEntStop) && ent_why(e) == kWhyEob);
    const uint32_t m_copy = 0u - (uint32_t)(odd == 0 && (e & kEntCopy) && !(d & (kEntSlow | kEntStop)));
    info = (((1u << 16) | (cl << 8) | ent_byte(e)) & m_lit) | ((kTokStop | (cl << 8)) & m_eob) |
           (((len << 16) | kTokCopy | ((q + dex) << 8)) & m_copy) | (kTokOther & ~(m_lit | m_eob | m_copy));
    dist = dv & m_copy;
}

// A copy's distance packed into its token word: distance - 1 (15 bits) in
// bits 0-7 and 25-31, which a copy does not otherwise use.
__device__ __forceinline__ uint32_t pack_token(uint32_t info, uint32_t dist) {
    const uint32_t d = dist - 1;
    return (info & kTokCopy) ? info | (d & 0xff) | ((d >> 8) << 25) : info;
}
__device__ __forceinline__ uint32_t token_dist(uint32_t w) { return ((w & 0xff) | ((w >> 25) << 8)) + 1; }
__device__ __forceinline__ uint32_t token_len(uint32_t w) { return (w >> 16) & 511; }

// The walk's view of a candidate: its bits plus, from bit 8, its output
// length plus 12, so one add advances both the bit position within the
// window (bits 0-7) and the batch budget (from bit 8); bit 31 marks a token
// the batch cannot take.  The budget starts at kBudget0 and the batch is
// full once it reaches 1024 (bit 18): at most 60 tokens, and at most 766
// output bytes before the last token, so at most kBatchOut in all.
constexpr uint32_t kWalkStop = 1u << 31, kBudget0 = 257, kBudgetFull = 1u << 18;
constexpr uint32_t kWindowEnd = 1u << 6;  // bit position 64 or beyond
__device__ __forceinline__ uint32_t walk_word(uint32_t info) {
    return (info & kTokStop) ? kWalkStop : ((info >> 8) & 63) + ((((info >> 16) & 511) + 12) << 8);
}

// Returns kMore once a batch ends at bit position `until` or past it.
template <int TB, uint32_t H, class Ring>
__device__ __forceinline__ int inflate_batched(Ring &in, BitIn &bi, LinearOut<H> &o,
                                               DeflateLds<TB, H> *lds, uint32_t until) {
    const uint32_t l = lane();
    // Candidates are decoded for fixed 64-bit windows of the input (lane l:
    // the token at bit 64 w + l).  The walk's tokens are staged, as packed
    // token words, in the code-length scratch (free while symbols decode),
    // one word per token of the batch.
    uint32_t *stage = reinterpret_cast<uint32_t *>(lds->lens);
    constexpr uint32_t kStageSpare = 64;  // 16 words no batch uses (at most 60 tokens)
    static_assert(sizeof(lds->lens) >= 4 * (kStageSpare + 16), "staging space");
    uint32_t p = bi.pos();  // bit position of the next code
    // Input words [cend - 64, cend), one per lane, read from the ring once
    // per 240 bytes or so; a window takes its four words out with readlane.
    uint32_t cache = 0, cend = 0;
    uint32_t wk = p >> 6;      // the window being walked (64-bit units)
    uint32_t cur = 0, walk = 0;  // packed token and walk word of this lane's candidate in window wk
    bool have = false;
    for (;;) {
        o.make_room(kBatchOut, H / 2);
        // ---- collect a batch of tokens
        uint32_t ntok = 0;
        uint32_t stop = 0;  // 1 full, 2 end of block, 3 one symbol the slow way
        const uint32_t total0 = o.pos, p0 = p;
        uint32_t budget = kBudget0;
        // Candidates of window wk: every lane's packed token and walk word.
        auto candidates = [&]() {
            const uint32_t wi = 2 * wk;
            if (wi + 4 > cend || wi + 64 < cend) {
                in.ensure(4 * (wi + 64) + 4);
                cache = in.word(wi + l);
                cend = wi + 64;
            }
            const uint32_t c0 = wi + 64 - cend;
            uint32_t info, dist;
            lane_token<TB, H, true>(readlane(cache, c0), readlane(cache, c0 + 1), readlane(cache, c0 + 2),
                                    readlane(cache, c0 + 3), 0u, 64 * wk, lds, info, dist);
            cur = pack_token(info, dist);
            walk = walk_word(info);
        };
        if (!have) candidates();
        for (;;) {
            // The walk follows token starts only, one lane read and one add
            // per token, until a token the batch cannot take, the end of the
            // window or a full batch (output bounds are checked lane-parallel
            // once the batch is complete).
            uint32_t T = (p - 64 * wk) | (budget << 8);
            uint32_t w = readlane(walk, T & 63);
            uint64_t mark = 0;
            while (!((w | T) & (kWalkStop | kWindowEnd | kBudgetFull))) {
                // One scalar instruction sets the bit (bit T mod 64).
                asm volatile("s_bitset1_b64 %0, %1" : "+s"(mark) : "s"(T));
                T += w;
                w = readlane(walk, T & 63);
            }
            // Stage this window's tokens in walk order.  Lanes without one
            // write a spare staging word past the batch's 60, so the store
            // needs no lane mask.
            const bool staged = (mark >> l) & 1;
            stage[staged ? ntok + count_below(mark) : kStageSpare + (l & 15)] = cur;
            ntok += (uint32_t)__builtin_popcountll(mark);
            budget = T >> 8;
            const uint32_t t = T & 255;
            p = 64 * wk + t;
            if (t < 64) {  // the batch ends in this window; its candidates stay
                if (budget >= 1024) {
                    stop = 1;  // batch full
                } else {
                    const uint32_t inf = readlane(cur, t);
                    if (inf == (kTokStop | (inf & 0x3f00))) {  // end of block
                        p += (inf >> 8) & 63;
                        stop = 2;
                    } else {
                        stop = 3;
                    }
                }
                have = true;
                break;
            }
            wk++;  // into the next window (a token ends at most 48 bits past this one)
            candidates();
        }
        uint32_t bout = budget - kBudget0 - 12 * ntok;
        __builtin_amdgcn_wave_barrier();
        // Every lane reads a staging word (all in bounds); lanes past the
        // batch drop it.
        const uint32_t staged = stage[l];
        const uint32_t tok = l < ntok ? staged : 0u;
        uint8_t *const trash = reinterpret_cast<uint8_t *>(stage) + 4 * l;
        const uint32_t tdist = (tok & kTokCopy) ? token_dist(tok) : 0u;
        // Each token's output length and offset in the chunk (one prefix sum
        // for the bounds and the writes).
        const uint32_t vlen = token_len(tok);
        const uint32_t before = total0 + wave_inclusive_sum32(vlen) - vlen;
        // Output bounds, lane-parallel: the first token whose distance
        // reaches before the chunk or whose output would pass the end ends
        // the batch, and goes through the symbol-at-a-time path.
        if (ntok) {
            const uint64_t badm = ballot(l < ntok && (tdist > before || before + vlen > o.cap));
            if (badm) {
                const uint32_t j = (uint32_t)__builtin_ctzll(badm);
                const uint32_t bits = l < j ? (tok >> 8) & 63 : 0u;
                ntok = j;
                bout = readlane(before, j) - total0;
                p = p0 + readlane(wave_inclusive_sum32(bits), 63);
                stop = 3;
            }
        }

        // ---- write the batch
        if (ntok) {
            const bool valid = l < ntok;
            const uint32_t len = valid ? vlen : 0;
            const bool is_copy = valid && (tok & kTokCopy);
            const uint32_t start = o.o0 + total0;  // first byte of the batch
            const uint32_t dst = o.o0 + before;    // this token's first byte
            uint8_t *const lit_to = valid && !is_copy ? o.win + o.slot(dst) : trash;
            *lit_to = (uint8_t)tok;
            const uint32_t src = dst - tdist;
            const bool before = is_copy && src + len <= start;  // source entirely before the batch
            // Bytes below lds_from have left the window; they were flushed to
            // HBM before this batch started.
            const int32_t lds_from = (int32_t)o.wlo;
            const bool far = ballot(before && (int32_t)src < lds_from) != 0;
            if (!far) {
                // Every source byte is in the window: no global loads, so
                // nothing waits for the flushes still in flight.
                for (uint32_t r = 0; ballot(before && r < len); r += 16) {
                    if (before && r < len) {
                        const uint32_t n = min(len - r, 16u), q0 = src + r;
                        const uint32_t a0 = q0 & ~3u, sh = q0 & 3;
                        uint32_t w[5];
#pragma unroll
                        for (uint32_t j = 0; j < 5; j++)
                            w[j] = *reinterpret_cast<const uint32_t *>(o.win + o.slot(a0 + 4 * j));
#pragma unroll
                        for (uint32_t j = 0; j < 4; j++) {
                            const uint32_t v = __builtin_amdgcn_alignbyte(w[j + 1], w[j], sh);
#pragma unroll
                            for (uint32_t b = 0; b < 4; b++) {
                                // Bytes past the copy go to this lane's slot
                                // of the (already read) token staging words,
                                // so the sixteen stores need no lane masks.
                                uint8_t *to = 4 * j + b < n ? o.win + o.slot(dst + r + 4 * j + b) : trash;
                                *to = (uint8_t)(v >> (8 * b));
                            }
                        }
                    }
                }
            } else {
                // Some source bytes were flushed: read them from HBM.
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                for (uint32_t r = 0; ballot(before && r < len); r += 16) {
                    if (before && r < len) {
                        // Sixteen source bytes as five aligned words (from the
                        // window, and from HBM where they fall below lds_from),
                        // all loads issued before any is used; then byte stores.
                        // HBM words may take up to three bytes either side of the
                        // copy's range: the same aligned word, so the same
                        // allocation; those bytes are discarded.
                        const uint32_t n = min(len - r, 16u), q0 = src + r;
                        const uint32_t a0 = q0 & ~3u, sh = q0 & 3;
                        uint32_t w[5], g[5] = {0, 0, 0, 0, 0};
#pragma unroll
                        for (uint32_t j = 0; j < 5; j++)
                            w[j] = *reinterpret_cast<const uint32_t *>(o.win + o.slot(a0 + 4 * j));
                        const int32_t nglob = lds_from - (int32_t)q0;  // leading bytes taken from HBM
                        if (nglob > 0) {
                            const uint32_t *gp = reinterpret_cast<const uint32_t *>(o.base + a0);
#pragma unroll
                            for (uint32_t j = 0; j < 5; j++) g[j] = gp[j];
                        }
                        // Every loaded word is used here (masked), so no load
                        // is left in flight past this loop: the wait for it
                        // would also wait for every flush store.
#pragma unroll
                        for (uint32_t j = 0; j < 4; j++) {
                            uint32_t v = __builtin_amdgcn_alignbyte(w[j + 1], w[j], sh);
                            const uint32_t gv = __builtin_amdgcn_alignbyte(g[j + 1], g[j], sh);
                            const int32_t kb = nglob - 4 * (int32_t)j;  // bytes of this word from HBM
                            const uint32_t m = kb >= 4 ? 0xffffffffu : kb <= 0 ? 0u : (1u << (8 * kb)) - 1;
                            v = (gv & m) | (v & ~m);
#pragma unroll
                            for (uint32_t b = 0; b < 4; b++) {
                                uint8_t *to = 4 * j + b < n ? o.win + o.slot(dst + r + 4 * j + b) : trash;
                                *to = (uint8_t)(v >> (8 * b));
                            }
                        }
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
            // Copies that read bytes of this batch, in order (their sources
            // are recent, so always in the window).
            uint64_t m = ballot(is_copy && !before);
            while (m) {
                uint32_t k = (uint32_t)__builtin_ctzll(m);
                m &= m - 1;
                uint32_t cd = readlane(dst, k), cs = readlane(tdist, k), cl = readlane(len, k);
                if (cs >= cl) {
                    for (uint32_t i = l; i < cl; i += kWave) o.win[o.slot(cd + i)] = o.win[o.slot(cd - cs + i)];
                } else {
                    uint32_t rr = l % cs, step = kWave % cs;
                    for (uint32_t i = l; i < cl; i += kWave) {
                        o.win[o.slot(cd + i)] = o.win[o.slot(cd - cs + rr)];
                        rr += step;
                        if (rr >= cs) rr -= cs;
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
            o.pos += bout;
            o.room -= bout;
        }
        if (stop == 1 && p < until) continue;
        bi.seek(in, p >> 3);
        bi.skip(p & 7);
        if (stop == 1) return kMore;
        if (stop == 2) return bi.remain < 0 ? CODAG_E_TRUNCATED : CODAG_OK;
        return kOneSymbol;
    }
}

// ---------------------------------------------------------------------------
// Lane-parallel symbol decoding.
//
// A round takes the next 64 x 256 bits of input, and lane l decodes, token
// after token, the tokens that start in its own 256 bits.  Only lane 0 knows
// where its first token starts; the others begin at their first bit, which is
// usually inside a token.  A Huffman decoder started off the track falls back
// onto it after a few tokens, so most lanes end at a true token start all the
// same: each lane then starts over where the lane before it ended, and the
// pass is repeated until no start moves (4 to 5 passes on text, 4 on columns,
// 6 to 9 with the fixed code).  Every lane works on tokens it alone decodes,
// so a pass costs about 25 loop trips for some 1,400 tokens, where one
// candidate per bit of a 64-bit window costs a trip and a serial walk for
// every five.  Each lane notes per 64-bit segment where the segment's first
// token starts and how many output bytes and copies its tokens make.
//
// The segments are then written out, up to 64 at a time, one per lane (as
// many as fit kAppend output bytes and the copy queue): a prefix sum gives
// each segment's place in the output, its lane decodes it once more, puts
// literals into the window and queues copies, and the queue is run 64 copies
// at a time.  A segment too large by itself is written by one lane, in parts.
//
// Sizes: with 256 bits a lane the passes take 6 trips per 64 tokens of text,
// with 128 and 64 bits 10 and 17 (counted on the CPU); 512 bits would take
// 4.6 but 4 KiB of input and two KiB of segment notes per wave.  Segments are
// 64 bits because the output window bounds one step to about 340 tokens.
// Measured against the window-by-window decoder: 16,384 chunks of 64 KiB
// 12.5 to 4.2 ms, 48 chunks of 60 KB (one wave each, nothing else
// running) 1,814 to 624 us, a learned batch of 2,000 chunks 15.8 to 4.4 ms.
// Chunks and blocks too short for it are decoded window by window (kShortBits).
// A wave holds 12 KiB of LDS instead of 8 (13 instead of 20 waves per CU),
// which the shorter work more than pays for.  Smaller footprints measured
// over 20,480 chunks: 14 waves (a 3 KiB window, 128 copies) 6.81 against 6.96
// ms but 10% slower for a lone wave, 16 waves (192 bits a lane besides) 7.41.
// Codes that hardly ever fall back (all of one length) would need a pass per
// lane: past kMaxPasses a round keeps the lanes that are on the track and the
// rest of the block goes to the window-by-window decoder.
// ---------------------------------------------------------------------------

constexpr uint32_t kMaxPasses = 20;

// One token per lane and loop trip.  x holds the next TB bits, so the
// literal/length lookup goes out together with the read of the eight input
// bytes that the distance code and the extra bits come from; the distance
// lookup is the trip's second wait.  Every lane goes through every trip, the
// idle ones on a table entry of zero: with the loops' conditions as branches
// around their effects, a trip spent more on execution masks than on decoding
// (700 cycles of a lone wave).  What is rare (codes longer than the tables,
// stops) is behind one branch that the wave takes when any lane needs it.
template <int TB>
struct LaneToken {
    const uint8_t *at;    // the stretch's first byte (LDS)
    const uint8_t *idle;  // where lanes with nothing to decode read: one place (each reading its own
                          // kept LDS busy 54% of the time instead of 47; 5.75 to 5.52 ms, 16,384 chunks)
    uint32_t r, x;      // next token's first bit in the stretch; its TB bits
    uint32_t e, d;      // its entries; d is 0 for a literal
    uint64_t raw;

    __device__ __forceinline__ void read() { raw = *reinterpret_cast<const u64_any *>(at + (r >> 3)); }
    __device__ __forceinline__ void start(const uint8_t *stretch, uint32_t bit, const uint8_t *nothing) {
        at = stretch;
        idle = nothing;
        r = bit;
        read();
        x = (uint32_t)(raw >> (r & 7));
    }
    // The low 32 bits from the token on: length code and extra bits end by
    // bit 20, the distance lookup's index by bit 28.
    __device__ __forceinline__ uint32_t bits() const { return (uint32_t)(raw >> (r & 7)); }
    // Looks the token up; true if some lane's needs resolve().
    __device__ __forceinline__ bool look(const DeflateTables<TB> *lds, bool on) {
        e = lds->tab[on ? x & ((1u << TB) - 1) : DeflateTables<TB>::kIdle];
        raw = *reinterpret_cast<const u64_any *>(on ? at + (r >> 3) : idle);
        // (A bit field's position is e's low five bits.  Lanes without a copy
        // all look one entry up.)
        const uint32_t m = (uint32_t)((int32_t)e >> 31);
        d = lds->dist()[bit_field(bits(), e, kDistBits) & m] & m;
        return ballot(((e | d) & (kEntSlow | kEntStop)) != 0) != 0;
    }
    // Codes longer than the tables; true if the lane's token is a stop.
    __device__ __forceinline__ bool resolve(const DeflateTables<TB> *lds) {
        if (!((e | d) & (kEntSlow | kEntStop))) return false;
        const uint64_t b = raw >> (r & 7);
        if (e & kEntSlow) {
            e = slow_entry((uint32_t)b, TB, &lds->meta[0], lds->sorted, kLitLen);
            d = (e & kEntCopy) ? lds->dist()[(uint32_t)(b >> ent_bits(e)) & ((1u << kDistBits) - 1)] : 0u;
        }
        if (d & kEntSlow)
            d = slow_entry((uint32_t)(b >> ent_bits(e)), kDistBits, &lds->meta[1], lds->sorted + 288, kDist);
        return ((e | d) & kEntStop) != 0;
    }
    __device__ __forceinline__ uint32_t length() const {
        return ent_len(e) + bit_field(bits(), ent_cl(e), ent_lex(e));
    }
    __device__ __forceinline__ uint32_t distance() const {
        return ent_dist(d) + bit_field((uint32_t)(raw >> ((r & 7) + ent_bits(e) + ent_cl(d))), 0, ent_ex(d));
    }
    // Past the token.  Of raw's 57 bits from r on, the longest token leaves
    // nine.
    __device__ __forceinline__ void next() {
        const uint32_t n = ent_bits(e) + ent_bits(d), old = r;
        r += n;
        x = (uint32_t)(raw >> ((old & 7) + n));
        if constexpr (TB > 9) {
            if (ballot(n > 57 - TB)) {
                read();
                x = bits();
            }
        }
    }
};

// One pass of the lanes with `need`: the tokens from bit rs of the lane's
// stretch on.  re is where the lane ended, rz the token it stopped at (why:
// kWhyEob, ...; 0: it did not); segs gets its segments' first tokens, output
// bytes << 12 and copies << 6.
template <int TB>
__device__ __forceinline__ void lane_pass(const DeflateTables<TB> *lds, uint32_t *segs, const uint8_t *inb,
                                          const uint8_t *mine, bool need, uint32_t rs, uint32_t &tried, uint32_t &re, uint32_t &rz, uint32_t &why) {
    LaneToken<TB> t;
    t.start(mine, rs, inb);
    bool on = need;
    uint32_t sp = rs, acc = 0;
    if (need) {
        tried = rs;
        why = 0;
    }
    do {
        if (t.look(lds, on) && t.resolve(lds)) {
            why = (t.e & kEntStop) ? ent_why(t.e) : (uint32_t)kWhyInvalid;
            rz = t.r;
            re = why == kWhyEob ? t.r + ent_cl(t.e) : t.r;
            segs[t.r / kSegBits] = (sp & (kSegBits - 1)) | acc;
            t.e = t.d = 0;
            on = false;
        }
        acc += (t.length() << 12) + ((t.e >> 31) << 6);
        const uint32_t from = t.r;
        t.next();
        if ((from ^ t.r) & ~(kSegBits - 1)) {
            segs[from / kSegBits] = (sp & (kSegBits - 1)) | acc;
            sp = t.r;
            acc = 0;
        }
        on = on && t.r < kLaneBits;
    } while (ballot(on));
    if (need && !why) rz = re = t.r;
}

// Writes the looked-up token of an emitting lane: a literal into the window, a
// copy into the queue at qi.  (The other lanes' stores sent to a spare place
// instead would spare two branches, but stores of many lanes to one address
// are serialised.)  A token whose distance reaches before the chunk or whose
// output passes its end sets bad and stops the lane.
template <int TB, uint32_t H>
__device__ __forceinline__ void emit_token(LaneToken<TB> &t, const LinearOut<H> &o, uint64_t *queue, uint32_t start, uint32_t lim, bool tight, bool &on,
                                           uint32_t er, uint32_t &dst, uint32_t &qi, int &bad) {
    const uint32_t len = t.length();
    const bool copy = (int32_t)t.e < 0;
    const uint32_t dist = t.distance();
    if (ballot(copy && dist > dst - o.o0) || tight) {
        if (on && dst + len > lim) bad = CODAG_E_OVERFLOW;
        if (copy && dist > dst - o.o0) bad = CODAG_E_CORRUPT;
    }
    const bool lit = on && !copy && !bad;
    if (lit) o.win[dst - o.wlo] = (uint8_t)ent_byte(t.e);
    const bool queued = copy && !bad;
    if (queued) queue[qi] = copy_entry(len, dst - start, dist);
    qi += queued ? 1u : 0u;
    dst += bad ? 0u : len;
    t.next();
    on = on && t.r < er && !bad;
}

// Returns kMore once a round ends at bit position `until` or past it, and where
// the block is for the window-by-window decoder (windows).
template <int TB, uint32_t H, class Ring>
__device__ __forceinline__ int inflate_lanes(Ring &in, BitIn &bi, LinearOut<H> &o, DeflateLds<TB, H> *lds,
                                             uint32_t until, bool &windows) {
    static_assert(Ring::kLdsWords <= kRoundInWords, "the round's input takes the ring's place");
    const uint32_t l = lane();
    uint8_t *const inb = reinterpret_cast<uint8_t *>(in.ring);
    const uint32_t endbit = 8 * in.gend;
    uint32_t p = bi.pos();  // bit position of the next code
    for (;;) {
        // Bits past the end read as zero; a block that goes on there is cut
        // off, whatever they decode to.
        if (p >= endbit) return CODAG_E_TRUNCATED;
        // ---- the round's input
        const uint32_t b0 = p & ~(kSegBits - 1), a0 = (b0 >> 3) & ~15u, ofs = (b0 >> 3) & 15;
        wave_sync();
        load_pieces<kRoundPieces, kWave>(in.gbase, in.gend, a0, in.ring, l);
        wave_sync();

        // ---- passes: every lane's tokens, until every start is true
        const uint8_t *const mine = inb + ofs + (kLaneBits / 8) * l;
        uint32_t live = min((uint32_t)kWave, (endbit - b0 + kLaneBits - 1) / kLaneBits);
        uint32_t rs = l == 0 ? p - b0 : 0u;  // this lane's first token, relative to its first bit
        uint32_t tried = ~0u, re = 0, rz = 0, why = 0;  // where it started, ended, stopped and why
        uint32_t m = 0;                                 // lanes whose tokens are true
        bool poor = false;
        for (uint32_t pass = 0;; pass++) {
            const bool need = l < live && rs != tried;
            const uint64_t nm = ballot(need);
            if (!nm) {
                m = live;
                break;
            }
            if (pass == kMaxPasses) {
                m = (uint32_t)__builtin_ctzll(nm);
                poor = true;
                break;
            }
            lane_pass<TB>(lds, lds->segs + kLaneSegs * l, inb, mine, need, rs, tried, re, rz, why);
            // Start over where the lane before ended (if it did not stop).
            const uint32_t ue = wave_shift_up1(why ? ~0u : re);
            if (l != 0 && l < live && ue != ~0u) rs = ue - kLaneBits;
            const uint64_t moved = ballot(l < live && rs != tried);
            const uint64_t stops = ballot(l < live && why != 0) & (moved ? (moved & (0 - moved)) - 1 : ~0ull);
            if (stops) live = (uint32_t)__builtin_ctzll(stops) + 1;  // a true stop: nothing follows it
        }
        wave_sync();
        const uint32_t whyl = readlane(why, m - 1), zl = readlane(rz, m - 1);
        const uint32_t nseg = kLaneSegs * (m - 1) + (whyl ? zl / kSegBits + 1 : kLaneSegs);
        p = b0 + kLaneBits * (m - 1) + readlane(re, m - 1);

        // ---- write the segments
        for (uint32_t g0 = 0; g0 < nseg;) {
            const uint32_t g = g0 + l;
            const uint32_t c = g < nseg ? lds->segs[g] : 0u;
            const uint32_t so = c >> 12, sc = (c >> 6) & 63;
            const uint32_t incl = wave_inclusive_sum32((so << 12) | sc);
            const uint64_t over = ballot(g >= nseg || (incl >> 12) > LinearOut<H>::kAppend || (incl & 4095) > kCopyQueue);
            uint32_t cnt = over ? (uint32_t)__builtin_ctzll(over) : (uint32_t)kWave;
            const bool part = cnt == 0;  // one segment does not fit: its lane writes what does
            if (part) cnt = 1;
            uint32_t made = part ? LinearOut<H>::kAppend : readlane(incl, cnt - 1) >> 12;
            uint32_t nq = readlane(incl, cnt - 1) & 4095;
            o.make_room(made);
            const uint32_t start = o.o0 + o.pos, lim = o.o0 + o.cap;
            uint32_t dst = start + (incl >> 12) - so, qi = (incl & 4095) - sc;
            const uint32_t er = whyl && g == nseg - 1 ? zl & (kSegBits - 1) : kSegBits;
            const bool tight = start + made > lim;  // the output range ends in this step
            int bad = CODAG_OK;
            LaneToken<TB> t;
            t.start(inb + ofs + (kSegBits / 8) * min(g, nseg - 1), c & (kSegBits - 1), inb);
            bool on = l < cnt && t.r < er;
            while (ballot(on)) {
                if (t.look(lds, on)) t.resolve(lds);
                if (part && on && (dst - start + t.length() > LinearOut<H>::kAppend || qi == kCopyQueue)) {
                    t.e = t.d = 0;  // the step is full
                    on = false;
                }
                emit_token<TB, H>(t, o, lds->queue, start, lim, tight, on, er, dst, qi, bad);
            }
            const uint32_t r = t.r;
            wave_sync();
            const uint64_t badm = ballot(bad != CODAG_OK);
            const uint32_t bl = badm ? (uint32_t)__builtin_ctzll(badm) : 0u;  // the first bad token's lane
            if (badm || part) {
                nq = readlane(qi, bl);
                made = readlane(dst, bl) - start;
            }
            run_copies<H>(o, lds->queue, nq, start);
            o.pos += made;
            o.room -= made;
            if (badm)
                return b0 + kSegBits * (g0 + bl) + readlane(r, bl) > endbit ? CODAG_E_TRUNCATED
                                                                           : (int)readlane((uint32_t)bad, bl);
            if (part) {
                const uint32_t r0 = readlane(r, 0);
                if (r0 >= readlane(er, 0)) {
                    g0++;
                } else {
                    if (l == 0) lds->segs[g0] = ((c - (made << 12) - (nq << 6)) & ~(kSegBits - 1)) | r0;
                    wave_sync();
                }
            } else {
                g0 += cnt;
            }
        }
        if (!whyl && !poor && p < until) continue;
        in.restart(p >> 3);
        bi.seek(in, p >> 3);
        bi.skip(p & 7);
        if (whyl == kWhyEob) return p > endbit ? CODAG_E_TRUNCATED : CODAG_OK;
        windows = !whyl && poor;
        return whyl ? kOneSymbol : kMore;
    }
}

// Leader-lane symbol loop: lane 0 decodes the token at the current bit
// position (the same per-lane token decoder the batched path runs on every
// lane), writes it to an LDS slot, and the wave reads it back and writes the
// literal or copy.  Every token takes one decode by one lane and one LDS
// round trip.  Anything but a plain literal or an in-range copy goes through
// one step of the symbol-at-a-time loop, so statuses are that loop's.
template <int TB, uint32_t H, class Ring>
__device__ __forceinline__ int inflate_leader(Ring &in, BitIn &bi, LinearOut<H> &o,
                                              DeflateLds<TB, H> *lds) {
    uint32_t p = bi.pos();  // bit position of the next code
    uint32_t *slot = reinterpret_cast<uint32_t *>(lds->lens);  // free while symbols decode
    for (;;) {
        const uint32_t wi = p >> 5;
        in.ensure(4 * (wi + 5) + 4);
        if (lane() == 0) {
            uint32_t info, dist;
            lane_token<TB, H>(in.word(wi), in.word(wi + 1), in.word(wi + 2), in.word(wi + 3),
                              in.word(wi + 4), p, lds, info, dist);
            slot[0] = info;
            slot[1] = dist;
        }
        __builtin_amdgcn_wave_barrier();
        const uint32_t info = uni(slot[0]), dist = uni(slot[1]);
        __builtin_amdgcn_wave_barrier();
        const uint32_t bits = (info >> 8) & 63;
        if (!(info & kTokStop)) {
            if (!(info & kTokCopy)) {
                if (o.pos < o.cap) {
                    o.put_literal(info & 0xff);
                    p += bits;
                    continue;
                }
            } else {
                const uint32_t len = info >> 16;
                if (dist <= o.pos && o.pos + len <= o.cap) {
                    o.copy(dist, len);
                    p += bits;
                    continue;
                }
            }
        }
        bi.seek(in, p >> 3);
        bi.skip(p & 7);
        const int st = inflate_symbol<TB, H>(in, bi, o, lds);
        if (st != kMore) return st;
        p = bi.pos();
    }
}

// MODE kAllLanes: the decoders above, rounds or windows; kLeaderLane: lane 0
// alone decodes each token and hands it to the wave through LDS (the
// single-thread decoding CODAG compares against, Section V-E).
enum : int { kAllLanes = 0, kLeaderLane = 1 };

// With `made` non-null the output range is a capacity: a final block that
// ends inside it is OK and *made receives the bytes produced.  `symbols`
// decodes a Huffman block's symbols once its tables are built, up to and
// including end-of-block, and returns a status.
template <int TB, uint32_t H, class Ring, class Symbols>
__device__ __forceinline__ int inflate_chunk(Ring &in, LinearOut<H> &o, DeflateLds<TB, H> *lds, uint32_t *made,
                                             Symbols symbols) {
    const uint32_t l = lane(), cap = o.cap;
    BitIn bi;
    bi.seek(in, in.skip);
    lds->tab[DeflateTables<TB>::kIdle] = 0;
    bool fixed_ready = false;
    int st = CODAG_OK;

    for (;;) {
        bi.refill(in);
        uint32_t hdr = bi.peek(3);
        if (!bi.drop(3)) { st = CODAG_E_TRUNCATED; break; }
        uint32_t btype = hdr >> 1;
        bool last = hdr & 1;
        if (btype == 0) {
            // Stored block: byte-align, LEN, NLEN = ~LEN, then LEN raw bytes.
            bi.drop(bi.cnt & 7);
            bi.refill(in);
            uint32_t len = bi.peek(16), nlen = (uint32_t)(bi.buf >> 16) & 0xffff;
            if (!bi.drop(32)) { st = CODAG_E_TRUNCATED; break; }
            if (nlen != (~len & 0xffff)) { st = CODAG_E_CORRUPT; break; }
            if (o.pos + len > cap) { st = CODAG_E_OVERFLOW; break; }
            uint32_t p = bi.byte_pos();
            if (p + len > in.gend) { st = CODAG_E_TRUNCATED; break; }
            uint32_t done = 0;
            if constexpr (Ring::kLaneRounds) {
                if (len >= LinearOut<H>::kStream) {
                    o.stream(in.gbase + p, len);
                    done = len;
                }
            }
            while (done < len) {
                uint32_t piece = min(len - done, Ring::kFetch / 2);
                o.make_room(piece);
                in.ensure(p + done + piece + 4);
                uint32_t dst = o.o0 + o.pos;
                for (uint32_t i = l; i < piece; i += kWave) {
                    uint32_t q = p + done + i;
                    o.win[o.slot(dst + i)] = (uint8_t)(in.word(q >> 2) >> (8 * (q & 3)));
                }
                o.pos += piece;
                o.room -= piece;
                done += piece;
            }
            bi.seek(in, p + len);
        } else if (btype == 3) {
            st = CODAG_E_CORRUPT;
            break;
        } else {
            if (btype == 1) {
                if (!fixed_ready) {
                    build_fixed<TB>(lds->tab, lds->dist());
                    fixed_ready = true;
                }
            } else {
                // Dynamic block header (RFC 1951 section 3.2.7).
                fixed_ready = false;
                uint32_t hlit, hdist, hclen;
                st = read_code_lengths(in, bi, lds->dist(), &lds->meta[1], lds->dist_sorted(),
                                       lds->lens, hlit, hdist, hclen);
                if (st) break;
                __builtin_amdgcn_wave_barrier();
                if (uni((uint32_t)lds->lens[256]) == 0) { st = CODAG_E_CORRUPT; break; }
                BuildResult lr = build_table(lds->lens, hlit, TB, kLitLen, lds->tab, lds->sorted,
                                             &lds->meta[0]);
                if (lr.left < 0 || (lr.left > 0 && !(lr.total == 1 && lr.ones == 1))) {
                    st = CODAG_E_CORRUPT;
                    break;
                }
                BuildResult dr = build_table(lds->lens + hlit, hdist, kDistBits, kDist, lds->dist(),
                                             lds->dist_sorted(), &lds->meta[1]);
                if (dr.left < 0 || (dr.left > 0 && dr.total != 0 && !(dr.total == 1 && dr.ones == 1))) {
                    st = CODAG_E_CORRUPT;
                    break;
                }
                // Without distance codes (total 0) every table entry is invalid.
            }
            st = symbols(bi);
            if (st) break;
        }
        if (last) break;
    }
    o.finish();
    if (st) return st;
    if (made) {
        *made = o.pos;
        return CODAG_OK;
    }
    return o.pos == cap ? CODAG_OK : CODAG_E_UNDERFLOW;
}

// Blocks that are likely to be shorter than this many bits are decoded window by
// window: a round's passes take as long for a few lanes' input as for all.  One
// block of text with its tables, window by window and in a round: 181 bytes 36
// and 49 us, 313 bytes 49 and 61, 399 bytes 56 and 49; of 4-byte integers, 316
// bytes 37 and 67, 498 bytes 68 and 58.  Streams flushed every 100 bytes take
// 3.4 ms per 64 KiB, 18.9 in rounds.  A block that goes on past this goes on
// in rounds.
//
// Blocks with much output for their bits are copies mostly, which rounds make
// many at a time: runs of integers, 8 KiB from 2,372 bits 70 and 72 us, 16 KiB
// from 4,263 bits 132 and 89; but not where every copy repeats the one before:
// 64 KiB of zeros from 624 bits 190 and 299.
constexpr uint32_t kShortBits = 3072, kShortOut = 8192, kRepeatsPerBit = 32;

// How long a Huffman block of a chunk is likely to be, in bits and in output
// bytes: as long as the one before it or half as long as was likely for that
// (long and short ones may alternate), or what is left of the chunk.  Kept in
// LDS: in scalar registers its four words cost the loops of the batched kernel
// 2%.
struct BlockLength {
    uint32_t *w;  // likely bits and output (~0: none yet), the block's first bit and output position

    __device__ __forceinline__ void init(uint32_t *words) {
        w = words;
        w[0] = w[1] = ~0u;
    }
    __device__ __forceinline__ uint32_t likely() const { return uni(w[0]); }
    // A block starts at bit p and output position out, with so much left.
    __device__ __forceinline__ bool is_short(uint32_t p, uint32_t rest, uint32_t out, uint32_t rest_out) {
        w[2] = p;
        w[3] = out;
        const uint32_t b = min(rest, likely()), n = min(rest_out, uni(w[1]));
        return b < kShortBits && (n <= kShortOut || n > kRepeatsPerBit * b);
    }
    __device__ __forceinline__ void ended(uint32_t p, uint32_t out) {
        const uint32_t b = p - uni(w[2]), n = out - uni(w[3]);
        if (b < 16) return;  // a flush's empty block
        const bool first = likely() == ~0u;
        w[0] = first ? b : max(b, likely() / 2);
        w[1] = first ? n : max(n, uni(w[1]) / 2);
    }
};

template <int TB, uint32_t H, int MODE = kAllLanes, class Ring>
__device__ __forceinline__ int decode_deflate(Ring &in, uint8_t *out, uint32_t cap,
                                              DeflateLds<TB, H> *lds, uint32_t *made = nullptr) {
    LinearOut<H> o;
    o.init(out, cap, lds->window);
    BlockLength blocks;
    blocks.init(lds->block);
    return inflate_chunk<TB, H>(in, o, lds, made, [&](BitIn &bi) {
        if constexpr (MODE == kLeaderLane) {
            return inflate_leader<TB, H>(in, bi, o, lds);
        } else {
            int st;
            uint32_t until = ~0u;  // window by window up to here
            if constexpr (Ring::kLaneRounds)
                until = blocks.is_short(bi.pos(), 8 * in.gend - bi.pos(), o.pos, o.cap - o.pos) ? bi.pos() + kShortBits : 0u;
            do {
                if (bi.pos() < until) {
                    st = inflate_batched<TB, H>(in, bi, o, lds, until);
                } else if constexpr (Ring::kLaneRounds) {
                    bool windows = false;
                    st = inflate_lanes<TB, H>(in, bi, o, lds, ~0u, windows);
                    if (windows) until = ~0u;
                }
                if (st == kOneSymbol) st = inflate_symbol<TB, H>(in, bi, o, lds);
            } while (st == kMore);
            if constexpr (Ring::kLaneRounds) {
                if (8 * in.gend - bi.pos() >= 16) blocks.ended(bi.pos(), o.pos);  // not after the chunk's last block
            }
            return st;
        }
    });
}

}  // namespace codag
