// Deflate and LZ4 by one workgroup per chunk, for launches with few chunks.
//
// One wave per chunk leaves most of the GPU idle when there are a few dozen
// chunks, and each wave's time is a chain of dependent steps.  Here kTeam
// waves decode a chunk together: a round of the lane-parallel decoder takes
// kTeam x 64 x 256 bits, and the emission steps, the copies, the window's
// flushes and slides are shared the same way.  Wave 0 alone reads block
// headers, builds tables and takes whatever is rare; the others wait for
// rounds.  The passes' trip count hardly grows with the number of lanes, so
// a round costs about what a wave's round costs and takes kTeam times the
// input.
//
// Measured against one wave per chunk: 48 chunks of 60 KB 624 to 162 us, 49
// ORC blocks of 256 KiB 2.58 to 0.65 ms, 256 chunks of 64 KiB 689 to 195 us
// with teams of 16; 512 chunks of 64 KiB 727 to 302 us with teams of 8.  1,024
// chunks fill the GPU a wave each (780 us against 899 in teams of 8), hence
// the limits.  Of a 64 KiB text chunk's 372,000 cycles the passes take some
// 120,000, the copies 70,000, the block header and its tables 40,000.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "../../include/codag.h"
#include "decode.hpp"
#include "internal.hpp"
#include "share.hpp"

namespace codag {

constexpr uint32_t kTeamH = 32768;  // output window
// Blocks in the middle of a chunk that are likely to be shorter than this are
// wave 0's alone: they fit a round of one wave, and a team's round would take its
// 32 KiB of input, and its passes over the blocks after, for each (64 KiB
// flushed every 2,000 bytes, 48 chunks 1.76 against 2.04 ms).  The last block of
// a chunk is the team's however short: 24 KiB of runs from 5,846 bits 98 us
// against 124.
constexpr uint32_t kAloneBits = 8192;

// Room for len <= kAppend more bytes, by the whole team (the same decision on
// every wave).
template <uint32_t kTeamThreads>
__device__ __forceinline__ void team_room(LinearOut<kTeamH> &o, uint32_t len, uint32_t tid) {
    if (o.room >= len) return;
    constexpr uint32_t kBlock = LinearOut<kTeamH>::kBlock;
    const uint32_t at = o.o0 + o.pos;
    if (o.fa < o.o0 && o.fa + kBlock <= at) {  // the chunk starts inside its first block
        if (tid < kWave) o.flush_block(o.o0 + o.cap);
        else o.fa += kBlock;
    }
    const uint32_t fe = at & ~(kBlock - 1);
    for (uint32_t a = o.fa + 16 * tid; a < fe; a += 16 * kTeamThreads)
        *reinterpret_cast<uint4 *>(o.base + a) = *reinterpret_cast<const uint4 *>(o.win + (a - o.wlo));
    o.fa = max(o.fa, fe);
    const uint32_t lo = (at + len - kTeamH + kBlock - 1) & ~(kBlock - 1), d = lo - o.wlo;
    static_assert(kTeamH % (16 * kTeamThreads) == 0, "a slide's steps end at the window's end");
    for (uint32_t i = 0; i < at - lo; i += 16 * kTeamThreads) {
        const uint4 v = *reinterpret_cast<const uint4 *>(o.win + slide_from(d + i + 16 * tid, kTeamH));
        __syncthreads();
        *reinterpret_cast<uint4 *>(o.win + i + 16 * tid) = v;
        __syncthreads();
    }
    o.wlo = lo;
    o.room = lo + kTeamH - at;
    wait_vm();  // the flushed bytes are there for any wave's copies
    __syncthreads();
}

// Copies whose output starts below offset x of the step (they are in output
// order).
template <uint32_t kTeamQueue>
__device__ __forceinline__ uint32_t team_copies_below(const uint64_t *queue, uint32_t nq, uint32_t x) {
    uint32_t lo = 0;
#pragma unroll
    for (uint32_t step = kTeamQueue >= 2048 ? 2048 : 1024; step; step >>= 1) {
        const uint32_t k = lo + step;
        const uint32_t at = ((uint32_t)queue[min(k, kTeamQueue) - 1] >> 16) & 0xffff;
        if (k <= nq && at < x) lo = k;
    }
    return lo;
}

// The nq queued copies of a step that starts at `start`.  The waves take them
// 64 at a time, in order; a copy is made once the copies that overlap its
// source are -- found by bisection, and looked up in a bitmap of the copies
// made -- so a step takes as many rounds as copies of copies are deep.  (With
// every copy waiting for all the copies below its source's end, 1,100 copies
// of text took 64,000 cycles, this way 28,000.)
//
// With `hops` (one word per copy), depth is cut first: a copy whose source is
// part of one earlier copy's output takes its bytes from that copy's source
// instead, and from that one's in turn, each hop going as far as the copy
// hopped to has come, so a chain of n copies takes about log2 n hops.  Words
// of running text repeat their last occurrence, which repeats its last: 690
// LZ4 matches took 93,000 cycles without hops and 18,000 with them.
struct CopyHop {
    // lo: source relative to the step's start + 2^19 | the copy its bytes come
    // from << 20 (kNone: none); hi: first and one past the last copy that
    // overlaps the source.  Other waves read a copy's word while its lane
    // hops, and need its halves from one write: the words are only accessed
    // by load and store.
    static constexpr uint32_t kNone = 0xfff, kBias = 1u << 19;

    static __device__ __forceinline__ uint64_t load(const uint64_t *w) {
        return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    static __device__ __forceinline__ void store(uint64_t *w, uint32_t lo, uint32_t hi) {
        __hip_atomic_store(w, ((uint64_t)hi << 32) | lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};
template <uint32_t kTeamThreads, uint32_t kTeamQueue>
__device__ __forceinline__ void team_copies(const LinearOut<kTeamH> &o, const uint64_t *queue, uint64_t *hops,
                                            unsigned long long *made_bits, uint32_t nq, uint32_t start, uint32_t wave) {
    static_assert(kTeamQueue < CopyHop::kNone, "copies count in 12 bits");
    const uint32_t l = lane();
    if (threadIdx.x < kTeamQueue / kWave) made_bits[threadIdx.x] = 0;
    // Copies d0 .. d1 - 1 overlap the source [src, min(src + len, dst)) of copy
    // k; `from` is that copy's hop.
    auto overlaps = [&](uint64_t q, bool v, uint32_t &d0, uint32_t &d1, uint32_t &hop) {
        const uint32_t len = (uint32_t)q & 0xffff, dist = (uint32_t)(q >> 32), at = ((uint32_t)q >> 16) & 0xffff;
        const bool inside = v && at + len > dist;  // the source's end, from the step's start, is past it
        d0 = d1 = 0;
        hop = CopyHop::kNone;
        if (!ballot(inside)) return;
        const uint32_t from = at > dist ? at - dist : 0u, to = min(at, at - dist + len);
        d1 = inside ? team_copies_below<kTeamQueue>(queue, nq, to) : 0u;
        // Few copies fit between the source's ends: walk down to the first
        // that reaches past `from`.
        d0 = d1;
        bool more = d0 != 0;
        while (ballot(more)) {
            const uint32_t p = (uint32_t)queue[d0 - (more ? 1 : 0)];
            more = more && (p >> 16) + (p & 0xffff) > from;
            d0 -= more ? 1u : 0u;
            more = more && d0 != 0;
        }
        if (d1 - d0 == 1 && dist >= len && at >= dist) {
            const uint64_t p = queue[d0];
            const uint32_t pl = (uint32_t)p & 0xffff, pa = ((uint32_t)p >> 16) & 0xffff;
            if (pa <= from && from + len <= pa + pl && (uint32_t)(p >> 32) >= pl) hop = d0;
        }
    };
    if (hops) {
        for (uint32_t k0 = wave * kWave; k0 < nq; k0 += kTeamThreads) {
            const uint32_t k = k0 + l;
            const uint64_t q = queue[min(k, kTeamQueue - 1)];
            uint32_t d0, d1, hop;
            overlaps(q, k < nq, d0, d1, hop);
            const uint32_t rel = (((uint32_t)q >> 16) & 0xffff) - (uint32_t)(q >> 32);
            if (k < nq) CopyHop::store(&hops[k], (rel + CopyHop::kBias) | (hop << 20), d0 | (d1 << 16));
        }
    }
    __syncthreads();
    for (uint32_t k0 = wave * kWave; k0 < nq; k0 += kTeamThreads) {
        const uint32_t k = k0 + l;
        const bool v = k < nq;
        const uint64_t q = queue[min(k, kTeamQueue - 1)];
        const uint32_t len = v ? (uint32_t)q & 0xffff : 0u, dist = (uint32_t)(q >> 32);
        const uint32_t at = ((uint32_t)q >> 16) & 0xffff, dst = start + at;
        const bool repeats = v && dist < len;  // its own output
        uint32_t src = dst - dist, d0, d1, hop;
        if (hops) {
            const uint64_t h = v ? CopyHop::load(&hops[k]) : (uint64_t)(CopyHop::kNone << 20);
            hop = ((uint32_t)h >> 20) & 0xfff;
            uint32_t over = (uint32_t)(h >> 32);
            while (ballot(hop != CopyHop::kNone)) {
                if (hop != CopyHop::kNone) {
                    const uint64_t hp = CopyHop::load(&hops[hop]), qp = queue[hop];
                    src += ((uint32_t)hp & 0xfffff) - CopyHop::kBias - (((uint32_t)qp >> 16) & 0xffff);
                    hop = ((uint32_t)hp >> 20) & 0xfff;
                    over = (uint32_t)(hp >> 32);
                    CopyHop::store(&hops[k], (src - start + CopyHop::kBias) | (hop << 20), over);
                }
            }
            d0 = v ? over & 0xffff : 0u;
            d1 = v ? over >> 16 : 0u;
        } else {
            overlaps(q, v, d0, d1, hop);
        }
        const bool far = v && src < o.wlo;
        if (ballot(far)) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        uint64_t pend = ballot(v);
        const uint64_t all = pend;
        while (pend) {
            bool ready = (pend >> l) & 1;
            for (uint32_t w = d0 / 64; ballot(ready && 64 * w < d1); w++) {
                if (ready && 64 * w < d1) {
                    uint64_t need = ~0ull;
                    if (64 * w < d0) need &= ~0ull << (d0 & 63);
                    if (64 * w + 64 > d1) need &= ~(~0ull << (d1 & 63));
                    const uint64_t done = __hip_atomic_load(&made_bits[w], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
                    ready = (need & ~done) == 0;
                }
            }
            const uint64_t rm = ballot(ready);
            if (!rm) {
                __builtin_amdgcn_s_sleep(1);  // the lowest pending copy of all goes on
                continue;
            }
            make_copies(o, ready && !repeats, far, src, dst, len);
            for (uint64_t m = ballot(ready && repeats); m; m &= m - 1) {
                const uint32_t t = (uint32_t)__builtin_ctzll(m);
                o.copy_near(readlane(src, t), readlane(dst, t), readlane(dist, t), readlane(len, t));
            }
            pend &= ~rm;
            wave_sync();
            if (l == 0)
                __hip_atomic_store(&made_bits[k0 / kWave], all & ~pend, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    __syncthreads();
}

// Decoding by kTeam waves (8 or 16).
template <uint32_t kTeam>
struct Team {
static constexpr uint32_t kTeamThreads = kTeam * kWave;
static constexpr uint32_t kTeamQueue = kTeam * 160;
static constexpr bool kHops = kTeam == 16;  // a team of 8 shares its CU's LDS with another
static constexpr uint32_t kTeamPieces = kTeamThreads * kLaneBits / 128 + 2;
// Lanes off the track at the end of a pass pass it on; a longer line of them
// is a little likelier with more lanes.
static constexpr uint32_t kTeamPasses = kMaxPasses + 4;
// A step always takes a segment: at most 32 copies, 258 bytes each.
static_assert(LinearOut<kTeamH>::kAppend >= 32 * 258 && kTeamQueue >= 32, "a step fits a segment");

struct Lds {
    DeflateLds<9, kTeamH> d;  // tables, window, and wave 0's own lists
    uint32_t in[4 * kTeamPieces];
    uint32_t segs[kTeam * kRoundSegs];
    uint64_t queue[kTeamQueue], hops[kHops ? kTeamQueue : 1];
    // Wave 0's orders: rounds from bit p on, or no more; and its output state.
    uint32_t go, p, pos, wlo, fa, room;
    // What the waves tell each other: where the last lane of each ended
    // (~0: it stopped), its first lane of interest, its sums.
    uint32_t edge[kTeam], first[kTeam], stop[kTeam], sum_out[kTeam], sum_cop[kTeam];
    uint32_t last_why, last_z, last_e, made, nq;
    uint32_t bad_lane[kTeam], bad_st[kTeam], bad_r[kTeam], bad_dst[kTeam], bad_qi[kTeam];
    unsigned long long made_bits[kTeamQueue / kWave];  // copies made, a bit each
};

// The smallest wave * 64 + v[wave] over the waves (v < 64, or 64 for none):
// kTeamThreads when there is none.
static __device__ __forceinline__ uint32_t first_lane(const uint32_t *v) {
    uint32_t r = kTeamThreads;
#pragma unroll
    for (uint32_t w = 0; w < kTeam; w++) {
        const uint32_t x = uni(v[w]);
        if (x < kWave && w * kWave + x < r) r = w * kWave + x;
    }
    return r;
}

// Rounds from bit p on until the block ends, an error, or something for wave
// 0 alone: as inflate_lanes, with the same result on every wave.  p is left
// at the next bit.
static __device__ __forceinline__ int rounds(const uint8_t *gbase, uint32_t gend, uint32_t &p, LinearOut<kTeamH> &o,
                                           Lds *s, uint32_t wave, bool &windows) {
    constexpr uint32_t kAppend = LinearOut<kTeamH>::kAppend;
    const uint32_t l = lane(), tid = wave * kWave + l;
    uint8_t *const inb = reinterpret_cast<uint8_t *>(s->in);
    const uint32_t endbit = 8 * gend;
    for (;;) {
        if (p >= endbit) return CODAG_E_TRUNCATED;
        const uint32_t b0 = p & ~(kSegBits - 1), a0 = (b0 >> 3) & ~15u, ofs = (b0 >> 3) & 15;
        load_pieces<kTeamPieces, kTeamThreads>(gbase, gend, a0, s->in, tid);
        __syncthreads();

        // ---- passes
        const uint8_t *const mine = inb + ofs + (kLaneBits / 8) * tid;
        uint32_t live = min(kTeamThreads, (endbit - b0 + kLaneBits - 1) / kLaneBits);
        uint32_t rs = tid == 0 ? p - b0 : 0u;
        uint32_t tried = ~0u, re = 0, rz = 0, why = 0;
        uint32_t m = 0;
        bool poor = false;
        for (uint32_t pass = 0;; pass++) {
            const bool need = tid < live && rs != tried;
            if (ballot(need))
                lane_pass<9>(&s->d, s->segs + kLaneSegs * tid, inb, mine, need, rs, tried, re, rz, why);
            if (l == kWave - 1) s->edge[wave] = why ? ~0u : re;
            __syncthreads();
            uint32_t ue = wave_shift_up1(why ? ~0u : re);
            const uint32_t ee = wave ? s->edge[wave - 1] : ~0u;
            if (l == 0) ue = ee;
            if (tid != 0 && tid < live && ue != ~0u) rs = ue - kLaneBits;
            const uint64_t mv = ballot(tid < live && rs != tried), sm = ballot(tid < live && why != 0);
            if (l == 0) {
                s->first[wave] = mv ? (uint32_t)__builtin_ctzll(mv) : kWave;
                s->stop[wave] = sm ? (uint32_t)__builtin_ctzll(sm) : kWave;
            }
            __syncthreads();
            const uint32_t fm = first_lane(s->first), fs = first_lane(s->stop);
            if (fs < fm) live = min(live, fs + 1);  // a true stop: nothing follows it
            if (fm >= live) {
                m = live;
                break;
            }
            if (pass + 1 == kTeamPasses) {
                m = fm;
                poor = true;
                break;
            }
        }
        if (wave == (m - 1) / kWave) {
            const uint32_t ll = (m - 1) % kWave;
            const uint32_t a = readlane(why, ll), b = readlane(rz, ll), c = readlane(re, ll);
            if (l == 0) {
                s->last_why = a;
                s->last_z = b;
                s->last_e = c;
            }
        }
        __syncthreads();
        const uint32_t whyl = uni(s->last_why), zl = uni(s->last_z);
        const uint32_t nseg = kLaneSegs * (m - 1) + (whyl ? zl / kSegBits + 1 : kLaneSegs);
        p = b0 + kLaneBits * (m - 1) + uni(s->last_e);

        // ---- write the segments
        for (uint32_t g0 = 0; g0 < nseg;) {
            const uint32_t g = g0 + tid;
            const uint32_t c = g < nseg ? s->segs[g] : 0u;
            const uint32_t so = c >> 12, sc = (c >> 6) & 63;
            uint32_t io = wave_inclusive_sum32(so), ic = wave_inclusive_sum32(sc);
            if (l == kWave - 1) {
                s->sum_out[wave] = io;
                s->sum_cop[wave] = ic;
            }
            __syncthreads();
            for (uint32_t w = 0; w < wave; w++) {
                io += uni(s->sum_out[w]);
                ic += uni(s->sum_cop[w]);
            }
            const uint64_t over = ballot(g >= nseg || io > kAppend || ic > kTeamQueue);
            if (l == 0) s->first[wave] = over ? (uint32_t)__builtin_ctzll(over) : kWave;
            __syncthreads();
            const uint32_t cnt = first_lane(s->first);  // 1 or more
            if (tid == cnt - 1) {
                s->made = io;
                s->nq = ic;
            }
            __syncthreads();
            uint32_t made = uni(s->made), nq = uni(s->nq);
            team_room<kTeamThreads>(o, made, tid);
            const uint32_t start = o.o0 + o.pos, lim = o.o0 + o.cap;
            const bool tight = start + made > lim;  // the output range ends in this step
            uint32_t dst = start + io - so, qi = ic - sc;
            const uint32_t er = whyl && g == nseg - 1 ? zl & (kSegBits - 1) : kSegBits;
            int bad = CODAG_OK;
            LaneToken<9> t;
            t.start(inb + ofs + (kSegBits / 8) * min(g, nseg - 1), c & (kSegBits - 1), inb);
            bool on = tid < cnt && t.r < er;
            while (ballot(on)) {
                if (t.look(&s->d, on)) t.resolve(&s->d);
                emit_token<9, kTeamH>(t, o, s->queue, start, lim, tight, on, er, dst, qi, bad);
            }
            const uint64_t badm = ballot(bad != CODAG_OK);
            if (badm) {
                const uint32_t bl = (uint32_t)__builtin_ctzll(badm);
                const uint32_t bs = readlane((uint32_t)bad, bl), br = readlane(t.r, bl), bd = readlane(dst, bl),
                               bq = readlane(qi, bl);
                if (l == 0) {
                    s->bad_st[wave] = bs;
                    s->bad_r[wave] = br;
                    s->bad_dst[wave] = bd;
                    s->bad_qi[wave] = bq;
                }
            }
            if (l == 0) s->bad_lane[wave] = badm ? (uint32_t)__builtin_ctzll(badm) : kWave;
            __syncthreads();
            const uint32_t fb = first_lane(s->bad_lane);  // the first bad token's lane
            if (fb < kTeamThreads) {
                nq = uni(s->bad_qi[fb / kWave]);
                made = uni(s->bad_dst[fb / kWave]) - start;
            }
            team_copies<kTeamThreads, kTeamQueue>(o, s->queue, kHops ? s->hops : nullptr, s->made_bits, nq, start, wave);
            o.pos += made;
            o.room -= made;
            if (fb < kTeamThreads) {
                const int st = (int)uni(s->bad_st[fb / kWave]);
                return b0 + kSegBits * (g0 + fb) + uni(s->bad_r[fb / kWave]) > endbit ? CODAG_E_TRUNCATED : st;
            }
            g0 += cnt;
            __syncthreads();
        }
        if (whyl == kWhyEob) return p > endbit ? CODAG_E_TRUNCATED : CODAG_OK;
        if (whyl) return kOneSymbol;
        if (poor) {
            windows = true;
            return kMore;
        }
        __syncthreads();  // the round's input is done with
    }
}

// One chunk by the workgroup; the status is wave 0's.
static __device__ __forceinline__ int chunk(const uint8_t *chunk, uint32_t len, uint8_t *out, uint32_t cap,
                                          uint32_t *made, Lds *s, uint32_t *ring, uint32_t wave) {
    DirectRing<512> in;
    in.init(chunk, len, ring, nullptr);
    LinearOut<kTeamH> o;
    o.init(out, cap, s->d.window);
    if (wave != 0) {
        for (;;) {
            __syncthreads();  // wave 0's orders
            const uint32_t go = uni(s->go);
            uint32_t p = uni(s->p);
            o.pos = uni(s->pos);
            o.wlo = uni(s->wlo);
            o.fa = uni(s->fa);
            o.room = uni(s->room);
            __syncthreads();  // everyone has read them
            if (!go) break;
            bool windows = false;
            rounds(in.gbase, in.gend, p, o, s, wave, windows);
        }
        return CODAG_OK;
    }
    BlockLength blocks;
    blocks.init(s->d.block);
    const int st = inflate_chunk<9, kTeamH>(in, o, &s->d, made, [&](BitIn &bi) {
        int r;
        const uint32_t p0 = bi.pos(), rest = 8 * in.gend - p0;
        // Window by window up to here, then in rounds of one wave, then the team's.
        uint32_t until = blocks.is_short(p0, rest, o.pos, o.cap - o.pos) ? p0 + kShortBits : 0u;
        const uint32_t alone = blocks.likely() < kAloneBits && rest >= kAloneBits ? p0 + kAloneBits : 0u;
        do {
            bool windows = false;
            if (bi.pos() < until) {
                r = inflate_batched<9, kTeamH>(in, bi, o, &s->d, until);
            } else if (bi.pos() < alone) {
                r = inflate_lanes<9, kTeamH>(in, bi, o, &s->d, alone, windows);
            } else {
                uint32_t p = bi.pos();
                if (lane() == 0) {
                    s->go = 1;
                    s->p = p;
                    s->pos = o.pos;
                    s->wlo = o.wlo;
                    s->fa = o.fa;
                    s->room = o.room;
                }
                wait_vm();  // what wave 0 wrote out is there for the others
                __syncthreads();
                __syncthreads();
                r = rounds(in.gbase, in.gend, p, o, s, 0, windows);
                in.restart(p >> 3);
                bi.seek(in, p >> 3);
                bi.skip(p & 7);
            }
            if (windows) until = ~0u;
            if (r == kOneSymbol) r = inflate_symbol<9, kTeamH>(in, bi, o, &s->d);
        } while (r == kMore);
        blocks.ended(bi.pos(), o.pos);
        return r;
    });
    if (lane() == 0) s->go = 0;
    __syncthreads();
    __syncthreads();
    return st;
}

};  // Team

// A team of 16 takes a CU's LDS, of 8 half of it.
constexpr uint32_t kBigTeamMaxChunks = 256;

template <uint32_t kTeam>
__global__ void __launch_bounds__(kTeam * kWave) __attribute__((amdgpu_waves_per_eu(4)))
    deflate_team(const uint8_t *comp, const uint64_t *coff, uint8_t *out, const uint64_t *ooff, uint32_t n,
                 int32_t *status, unsigned long long *err) {
    __shared__ __align__(16) typename Team<kTeam>::Lds s;
    __shared__ __align__(16) uint32_t s_ring[kRoundInWords];
    const uint32_t wave = uni(threadIdx.x / kWave), c = blockIdx.x;
    if (c >= n) return;
    const uint64_t i0 = coff[c], i1 = coff[c + 1], o0 = ooff[c], o1 = ooff[c + 1];
    int st = CODAG_E_INVALID_ARGUMENT;
    if ((((i1 - i0) | (o1 - o0)) >> 31) == 0 && i1 - i0 < (1u << 28))
        st = Team<kTeam>::chunk(comp + i0, (uint32_t)(i1 - i0), out + o0, (uint32_t)(o1 - o0), nullptr, &s, s_ring, wave);
    if (wave == 0) report(c, st, status, err);
}

int launch_deflate_team(const uint8_t *comp, const uint64_t *coff, uint8_t *out, const uint64_t *ooff, uint32_t n,
                        int32_t *status, unsigned long long *err, hipStream_t s) {
    if (n <= kBigTeamMaxChunks)
        hipLaunchKernelGGL(deflate_team<16>, dim3(n), dim3(16 * kWave), 0, s, comp, coff, out, ooff, n, status, err);
    else
        hipLaunchKernelGGL(deflate_team<8>, dim3(n), dim3(8 * kWave), 0, s, comp, coff, out, ooff, n, status, err);
    return hipGetLastError() == hipSuccess ? CODAG_OK : CODAG_E_HIP;
}

// ---- LZ4 -------------------------------------------------------------------
//
// A block is a chain of sequences of three bytes and more, and one wave spends
// its time on the chain and on matches of matches.  A team takes the input in
// windows of 3,072 byte positions: every thread parses the sequences that
// would start at three of them (continuation bytes included, for literal runs
// below 270 bytes and matches of up to 1,024), six rounds of link doubling in
// LDS give where 64 sequences end, one read per 64 follows the real chain, and
// each thread finds and parses one of its sequences.  A prefix sum places
// them; literals go to the window and matches to the copy queue.  What the
// parse leaves out (longer fields, the last sequence, every error) is a
// general step of wave 0; blocks with little else are set aside for one wave.
//
// Measured against one wave per block: 97 ORC blocks of 64 KiB 1,028 to 246 us,
// one block of 64 KiB 840 to 174, 256 chunks 968 to 220, 1,024 chunks 1,025 to
// 690; two teams fit neither a CU's LDS nor its waves, so from some 1,300
// chunks on a wave each is faster.  Of a text window's 40,000 cycles the
// copies take 18,000, the links 6,600, finding the sequences 7,700.
constexpr uint32_t kLzTeam = 16, kLzThreads = kLzTeam * kWave;
constexpr uint32_t kLzStep = 3 * kLzThreads;  // byte positions of a window: one sequence a thread at most
constexpr uint32_t kLzPieces = kLzStep / 16 + 20;  // a sequence's fields and literals past the last position
constexpr uint32_t kLzLevels = 7;             // links over 1, 2, ... 64 sequences
constexpr uint32_t kLzMatch = 1024;           // longest match of a parsed sequence
// Copies of up to kLzMatch bytes: as much more of what lies below the window
// has to be in HBM (see LinearOut).
constexpr uint32_t kLzMost = LinearOut<kTeamH>::kAppend - (kLzMatch - 512);

// Workgroups of a launch, one a CU: they take more blocks than that in turn.
constexpr uint32_t kLzGrid = 256, kLzGroup = kLzTeamMaxChunks / kLzGrid;

// Which blocks a workgroup of a launch of n takes: with more than one each, the
// blocks in order of what they are likely to cost (cost(i) of block i, from its
// lengths, to a quarter of an octave) are dealt out forth and back.  Every
// workgroup finds the same order, by counting, in about 1 us.  1,024 blocks of
// log-normal sizes take 1,143 us, 1,335 with a workgroup each as CUs come free
// and 1,844 with every 256th block; 300 ORC blocks of 64 KiB 324, 479 and 542.
struct LzDeal {
    uint32_t count[kLzTeam][kWave];  // blocks of each class, by the wave that looked at them
    uint32_t mine[kLzGroup];
};
template <class Cost>
__device__ __forceinline__ uint32_t lz_deal(LzDeal *s, uint32_t n, uint32_t b, Cost cost) {
    static_assert(kLzTeamMaxChunks <= kLzThreads, "a thread a block");
    const uint32_t t = threadIdx.x, wave = uni(t / kWave), l = lane();
    if (n <= kLzGrid) {  // (a stream's chunks may be fewer than its capacity's)
        if (t == 0) s->mine[0] = b;
        __syncthreads();
        return 1;
    }
    // Class 0 is the costliest (2^23 and more), 63 the cheapest (below 320).
    const uint32_t v = max(t < n ? cost(t) : 0u, 256u), e = 31 - (uint32_t)__builtin_clz(v);
    const uint32_t cls = 95 - min(4 * e + ((v >> (e - 2)) & 3), 95u);
    uint64_t same = ballot(t < n);  // lanes of this one's class
#pragma unroll
    for (uint32_t i = 0; i < 6; i++) {
        const uint64_t m = ballot((cls >> i) & 1);
        same &= (cls >> i) & 1 ? m : ~m;
    }
    s->count[wave][l] = 0;
    __syncthreads();
    const uint32_t earlier = count_below(same);
    if (t < n && earlier == 0) s->count[wave][cls] = (uint32_t)__builtin_popcountll(same);
    __syncthreads();
    // Lane l: blocks of class l in all waves and in those before this one.
    uint32_t all = 0, before = 0;
#pragma unroll
    for (uint32_t w = 0; w < kLzTeam; w++) {
        const uint32_t c = s->count[w][l];
        all += c;
        before += w < wave ? c : 0u;
    }
    const uint32_t rank = lane_pull(wave_inclusive_sum32(all) - all + before, cls) + earlier;
    // Rank r goes to workgroup r mod 256 in even turns, 255 minus that in odd ones.
    const uint32_t turn = rank / kLzGrid, at = rank % kLzGrid;
    if (t < n && (turn & 1 ? kLzGrid - 1 - at : at) == b) s->mine[turn] = t;
    __syncthreads();
    const uint32_t turns = n / kLzGrid, rest = n % kLzGrid;
    return turns + ((turns & 1 ? kLzGrid - 1 - b : b) < rest ? 1 : 0);
}
// A block that hardly compressed is literals mostly.
__device__ __forceinline__ uint32_t lz_cost(uint32_t in, uint32_t out) {
    return in + in / 16 < out ? in : in / 16;
}

// Blocks that a team is no better at than one wave are set aside, and when the
// workgroup is done with the others its waves decode one each, side by side:
// blocks of at most kLzTiny compressed bytes, and those whose general steps
// would take the team longer than its share of the waves takes for everything,
// by the costs below (hundreds of cycles).  Literal runs of 300 to 2,000 bytes,
// 64 blocks 147 us (484 with every run a turn of the team, 133 by a wave each in
// a launch of their own), 1,024 blocks 231 (1,872; 159); 1,024 blocks of 200
// bytes 18.5 (50; 14.4).
constexpr uint32_t kLzTiny = 256;
constexpr uint32_t kLzTurnCost = 130, kLzLinkCost = 100;  // a turn of a team's loop; a window's links
constexpr uint32_t kLzFastCost = 2, kLzSlowCost = 30;     // a sequence by one wave: parsed by a lane, or general (18 bytes and more on average)
constexpr uint32_t kLzHuge = 8192;  // fields this long are wave 0's work for longer than all of these
enum : int { kLzAside = 2 };        // not a status

struct LzAloneLds {
    Lz4Lds<4096> d;
    uint32_t in[LinearIn::kLdsWords];
};

struct LzTeamLds {
    Lz4Lds<kTeamH> d;  // the window; wave 0's queue
    uint32_t buf[2][4 * kLzPieces];
    uint16_t link[kLzLevels][kLzStep];
    uint64_t queue[kLzThreads], hops[kLzThreads];
    unsigned long long made_bits[kLzThreads / kWave];
    uint32_t unit[kLzTeam + 2], units, chain_end;
    uint32_t sum[kLzTeam], first[kLzTeam], made, next;
    uint32_t st, p, pos, wlo, fa, room;  // wave 0's general step
};

// A workgroup's LDS: a team's, then that of the waves with a block each.
union LzLds {
    LzTeamLds t;
    LzAloneLds a[kLzGroup];
};

struct LzSeq {
    uint32_t lit, at, off, mlen, next;  // at: its literals' first position
    bool ok;
};
// The sequence at position x of a window, `room` positions before the chunk's
// end: ok if a thread can take it.
__device__ __forceinline__ LzSeq lz_parse(const uint8_t *bytes, uint32_t x, uint32_t room) {
    LzSeq q;
    const uint32_t tok = bytes[x];
    q.lit = tok >> 4;
    q.at = x + 1;
    q.ok = true;
    if (q.lit == 15) {
        const uint32_t e = bytes[x + 1];
        q.lit += e;
        q.at++;
        q.ok = e != 255;
    }
    const uint64_t f = *reinterpret_cast<const u64_any *>(bytes + q.at + q.lit);
    q.off = (uint32_t)f & 0xffff;
    q.mlen = (tok & 15) + 4;
    q.next = q.at + q.lit + 2;
    if ((tok & 15) == 15) {
        const uint32_t full = (uint32_t)(__builtin_ctzll(~(f >> 16)) >> 3);  // continuation bytes of 255; 6 or more: too long
        q.ok = q.ok && full < 6;
        q.mlen += 255 * full + ((uint32_t)(f >> (16 + 8 * min(full, 5u))) & 255);
        q.next += full + 1;
    }
    q.ok = q.ok && q.off != 0 && q.mlen <= kLzMatch && q.next <= room;
    return q;
}

// Whether the general sequence at p has a field of kLzHuge bytes or more.
__device__ __forceinline__ bool lz_huge(LinearIn &in, uint32_t p, uint32_t end) {
    const uint32_t tok = in.peek4(p) & 255;
    uint32_t lit = tok >> 4, mlen = tok & 15, q = p + 1;
    if (lit == 15) q = lz4_more(in, q, end, lit);
    if (!q || lit >= kLzHuge || lit > end - q) return q != 0 && lit >= kLzHuge;
    q += lit + 2;
    return mlen == 15 && q < end && lz4_more(in, q, end, mlen) && mlen >= kLzHuge;
}

// One block by the workgroup; the same status on every wave.  kLzAside: it is
// for one wave, from its start (`group` blocks, at most, are the workgroup's).
__device__ __forceinline__ int lz_team_chunk(const uint8_t *chunk, uint32_t len, uint8_t *out, uint32_t cap,
                                             uint32_t *made_out, LzTeamLds *s, uint32_t *lin, uint32_t wave,
                                             uint32_t group) {
    if (len <= kLzTiny) return kLzAside;
    const uint32_t l = lane(), tid = wave * kWave + l;
    LinearOut<kTeamH> o;
    o.init(out, cap, s->d.window);
    LinearIn in;  // wave 0's
    in.skip = (uint32_t)(reinterpret_cast<uintptr_t>(chunk) & 15);
    in.gbase = chunk - in.skip;
    in.gend = in.skip + len;
    in.buf = lin;
    in.a0 = 0;
    if (wave == 0) in.load(0);
    const uint32_t end = in.gend;
    uint32_t p = in.skip;
    uint32_t cur = ~0u, nxt = ~0u;  // the window in use, and one in (or on its way to) the other buffer
    uint32_t turns = 0, linked = 0;    // turns of the loop, windows linked
    uint32_t general = 0, alone = 0;   // general steps (wave 0's count); what one wave would have taken for the rest
    int st = CODAG_OK;
    auto issue = [&](uint32_t w) {
        const uint32_t at = w * kLzStep + 16 * tid;
        if (tid < kLzPieces && at < end)
            __builtin_amdgcn_global_load_lds(in.gbase + at, (lds_void *)(s->buf[w & 1] + 256 * wave), 16, 0, 0);
    };
    for (;;) {
        if (p >= end) {
            st = CODAG_E_TRUNCATED;
            break;
        }
        const uint32_t w = p / kLzStep, W = w * kLzStep, room = end - W;
        const uint8_t *const bytes = reinterpret_cast<const uint8_t *>(s->buf[w & 1]);
        turns++;
        if (w != cur) {  // (after a general step the window and its links may still be there)
            if (w != nxt) {
                wait_vm();  // a window not wanted any more may be landing
                issue(w);
            }
            cur = w;
            linked++;
            if (wave < (kLzPieces + kWave - 1) / kWave) wait_vm();
            __syncthreads();
            if (W + kLzStep < end && nxt != w + 1) {
                issue(w + 1);
                nxt = w + 1;
            }
            // Links; a position whose sequence no thread can take links to itself.
            uint32_t to[3];
#pragma unroll
            for (uint32_t i = 0; i < 3; i++) {
                const uint32_t x = tid + kLzThreads * i;
                const LzSeq q = lz_parse(bytes, x, room);
                to[i] = q.ok && x < room ? q.next : x;
                s->link[0][x] = (uint16_t)to[i];
            }
            __syncthreads();
#pragma unroll
            for (uint32_t k = 1; k < kLzLevels; k++) {
#pragma unroll
                for (uint32_t i = 0; i < 3; i++) {
                    const uint32_t f = s->link[k - 1][min(to[i], kLzStep - 1)];
                    if (to[i] < kLzStep) to[i] = f;
                    s->link[k][tid + kLzThreads * i] = (uint16_t)to[i];
                }
                __syncthreads();
            }
        }
        // The chain, 64 sequences a step.
        if (wave == 0) {
            uint32_t x = p - W, u = 0;
            while (x < kLzStep && u < kLzTeam + 2) {
                if (l == 0) s->unit[u] = x;
                const uint32_t f = uni((uint32_t)s->link[kLzLevels - 1][x]);
                if (f == x) break;
                u++;
                x = f;
            }
            if (l == 0) {
                s->units = u;
                s->chain_end = x;
            }
        }
        __syncthreads();
        // One sequence a thread: wave u's are those of unit u.
        const uint32_t units = uni(s->units), chain_end = uni(s->chain_end);
        uint32_t x = wave < units ? s->unit[wave] : kLzStep;
#pragma unroll
        for (uint32_t k = kLzLevels - 1; k-- > 0;) {
            const uint32_t f = s->link[k][min(x, kLzStep - 1)];
            if (((l >> k) & 1) && x < kLzStep) x = f;
        }
        const LzSeq q = lz_parse(bytes, min(x, kLzStep - 1), room);
        const bool valid = x < kLzStep && x < room && q.ok;
        const uint32_t outl = valid ? q.lit + q.mlen : 0u;
        uint32_t incl = wave_inclusive_sum32(outl);
        if (l == kWave - 1) s->sum[wave] = incl;
        __syncthreads();
        for (uint32_t v = 0; v < wave; v++) incl += uni(s->sum[v]);
        const uint32_t before = incl - outl, done = o.pos;
        // Sequences up to the first that is not one, or breaks a bound.
        const uint64_t no = ballot(!valid || incl > cap - done || q.off > done + before + q.lit);
        if (l == 0) s->first[wave] = no ? (uint32_t)__builtin_ctzll(no) : kWave;
        if (tid == 0) s->next = W + chain_end;
        __syncthreads();
        uint32_t cnt = kLzThreads;
        for (uint32_t v = kLzTeam; v-- > 0;) {
            const uint32_t fv = uni(s->first[v]);
            if (fv < kWave) cnt = v * kWave + fv;
        }
        // A sequence left to the general step (a bound): the chain stops there.
        if (tid == cnt && valid) s->next = W + x;
        // Steps of at most kLzMost output bytes.
        for (uint32_t g = 0, base = 0; g < cnt;) {
            const uint64_t over = ballot(tid >= cnt || (tid >= g && incl - base > kLzMost));
            __syncthreads();
            if (l == 0) s->first[wave] = over ? (uint32_t)__builtin_ctzll(over) : kWave;
            __syncthreads();
            uint32_t g1 = cnt;
            for (uint32_t v = kLzTeam; v-- > 0;) {
                const uint32_t fv = uni(s->first[v]);
                if (fv < kWave) g1 = min(g1, v * kWave + fv);
            }
            if (tid == g1 - 1) s->made = incl;
            __syncthreads();
            const uint32_t upto = uni(s->made), made = upto - base;
            team_room<kLzThreads>(o, made, tid);
            const uint32_t start = o.o0 + o.pos;
            if (tid >= g && tid < g1) {
                const uint32_t dl = before - base;
                uint8_t *const dst = o.win + (start + dl - o.wlo);
                const uint8_t *const src = bytes + q.at;
                if (q.lit >= 8) {
                    for (uint32_t j = 0; j < q.lit; j += 8) {
                        const uint32_t k = min(j, q.lit - 8);
                        *reinterpret_cast<u64_any *>(dst + k) = *reinterpret_cast<const u64_any *>(src + k);
                    }
                } else {
                    for (uint32_t j = 0; j < q.lit; j++) dst[j] = src[j];
                }
                s->queue[tid - g] = copy_entry(q.mlen, dl + q.lit, q.off);
            }
            __syncthreads();
            team_copies<kLzThreads, kLzThreads>(o, s->queue, s->hops, s->made_bits, g1 - g, start, wave);
            o.pos += made;
            o.room -= made;
            base = upto;
            g = g1;
        }
        __syncthreads();
        const uint32_t from = p;
        p = uni(s->next);
        alone += cnt * (p - from >= 18 * cnt ? kLzSlowCost : kLzFastCost);
        if (p >= W + kLzStep) continue;
        // General steps from p on: one, and more while literal runs that no
        // thread parses follow.
        if (wave == 0) {
            int r = CODAG_E_TRUNCATED;  // p >= end
            if (p < end) {
                const uint32_t team = kLzTurnCost * turns + kLzLinkCost * linked;
                Lz4Step step;
                step.most = 2560;
                lz4_begin(o, step);
                do {
                    if ((general >= 4 && team > (alone + kLzSlowCost * general) / group) ||
                        (group > 1 && lz_huge(in, p, end))) {
                        r = kLzAside;
                        break;
                    }
                    r = lz4_sequence<kTeamH>(in, o, &s->d, step, p, end, cap);
                    general++;
                } while (r == kLz4More && p < end && (in.peek4(p) & 0xfff0) == 0xfff0);
                lz4_end(o, &s->d, step);
            }
            wait_vm();  // what it wrote out is there for the others
            if (l == 0) {
                s->st = (uint32_t)r;
                s->p = p;
                s->pos = o.pos;
                s->wlo = o.wlo;
                s->fa = o.fa;
                s->room = o.room;
            }
        }
        __syncthreads();
        st = (int)uni(s->st);
        p = uni(s->p);
        o.pos = uni(s->pos);
        o.wlo = uni(s->wlo);
        o.fa = uni(s->fa);
        o.room = uni(s->room);
        __syncthreads();
        if (st != kLz4More) break;
        st = CODAG_OK;
    }
    wait_vm();  // a window on its way
    __syncthreads();
    if (wave == 0) o.finish();
    __syncthreads();
    if (st) return st;
    if (made_out) {
        *made_out = o.pos;
        return CODAG_OK;
    }
    return o.pos == cap ? CODAG_OK : CODAG_E_UNDERFLOW;
}

// A block set aside, by the calling wave.
__device__ __forceinline__ int lz_alone(const uint8_t *chunk, uint32_t len, uint8_t *out, uint32_t cap, uint32_t *made,
                                        LzAloneLds *s) {
    LinearIn in;
    in.init(chunk, len, s->in, nullptr);
    return decode_lz4<4096>(in, out, cap, &s->d, made);
}

// Grouped: launches of more blocks than workgroups.
template <bool Grouped>
__global__ void __launch_bounds__(kLzThreads) __attribute__((amdgpu_waves_per_eu(4)))
    lz4_team(const uint8_t *comp, const uint64_t *coff, uint8_t *out, const uint64_t *ooff, uint32_t n,
             int32_t *status, unsigned long long *err) {
    __shared__ __align__(16) LzLds s;
    __shared__ __align__(16) uint32_t s_lin[LinearIn::kLdsWords];
    __shared__ LzDeal s_deal;
    const uint32_t wave = uni(threadIdx.x / kWave);
    if (blockIdx.x >= n) return;
    uint32_t group = 1;
    if constexpr (Grouped)
        group = lz_deal(&s_deal, n, blockIdx.x, [&](uint32_t i) {
            return lz_cost((uint32_t)min(coff[i + 1] - coff[i], (uint64_t)1 << 31),
                           (uint32_t)min(ooff[i + 1] - ooff[i], (uint64_t)1 << 31));
        });
    uint32_t aside = 0;  // a bit per block set aside
    for (uint32_t k = 0; k < group; k++) {
        const uint32_t c = Grouped ? uni(s_deal.mine[k]) : blockIdx.x;
        const uint64_t i0 = coff[c], i1 = coff[c + 1], o0 = ooff[c], o1 = ooff[c + 1];
        int st = CODAG_E_INVALID_ARGUMENT;
        if ((((i1 - i0) | (o1 - o0)) >> 31) == 0)
            st = lz_team_chunk(comp + i0, (uint32_t)(i1 - i0), out + o0, (uint32_t)(o1 - o0), nullptr, &s.t, s_lin, wave,
                               group);
        if (st == kLzAside) aside |= 1u << k;
        else if (wave == 0) report(c, st, status, err);
    }
    if (!aside) return;
    __syncthreads();  // the team's LDS is done with
    if (wave < kLzGroup && ((aside >> wave) & 1)) {
        const uint32_t c = Grouped ? uni(s_deal.mine[wave]) : blockIdx.x;
        const uint64_t i0 = coff[c], o0 = ooff[c];
        report(c, lz_alone(comp + i0, (uint32_t)(coff[c + 1] - i0), out + o0, (uint32_t)(ooff[c + 1] - o0), nullptr,
                           &s.a[wave]), status, err);
    }
}

int launch_lz4_team(const uint8_t *comp, const uint64_t *coff, uint8_t *out, const uint64_t *ooff, uint32_t n,
                    int32_t *status, unsigned long long *err, hipStream_t s) {
    static_assert(kLzGrid * kLzGroup >= kLzTeamMaxChunks && kLzGroup <= kLzTeam, "a wave for every block set aside");
    if (n <= kLzGrid)
        hipLaunchKernelGGL(lz4_team<false>, dim3(n), dim3(kLzThreads), 0, s, comp, coff, out, ooff, n, status, err);
    else
        hipLaunchKernelGGL(lz4_team<true>, dim3(kLzGrid), dim3(kLzThreads), 0, s, comp, coff, out, ooff, n, status, err);
    return hipGetLastError() == hipSuccess ? CODAG_OK : CODAG_E_HIP;
}

// ---- compressed ORC streams

// ORC chunk f into out + f * block, as orc_frame_decode with a team per chunk.
// (Grouped: LZ4 streams that may have more chunks than a launch has workgroups.)
template <int Codec, uint32_t kTeam, bool Grouped = false>
__global__ void __launch_bounds__(kTeam * kWave) __attribute__((amdgpu_waves_per_eu(4)))
    orc_frame_team(const uint8_t *framed, uint32_t block, uint8_t *out, uint64_t out_cap, const OrcFrame *frames,
                   OrcMeta *meta) {
    __shared__ __align__(16) typename std::conditional<Codec == CODAG_LZ4, LzLds, typename Team<kTeam>::Lds>::type s;
    __shared__ __align__(16) uint32_t s_ring[kRoundInWords];
    static_assert(kRoundInWords >= LinearIn::kLdsWords, "wave 0's input");
    const uint32_t wave = uni(threadIdx.x / kWave);
    const uint32_t count = uni(meta->count), complete = uni(meta->complete);
    if (blockIdx.x >= count) return;
    __shared__ LzDeal s_deal;
    uint32_t group = 1;
    if constexpr (Grouped)
        group = lz_deal(&s_deal, count, blockIdx.x, [&](uint32_t i) {
            return frames[i].original ? frames[i].len / 64 : lz_cost(frames[i].len, block);
        });
    auto room_of = [&](uint32_t f) {
        const uint64_t at = (uint64_t)f * block;
        return at >= out_cap ? 0u : (uint32_t)min((uint64_t)block, out_cap - at);
    };
    auto done = [&](uint32_t f, int st, uint32_t made) {  // by one lane
        const bool last = f + 1 == count && complete;     // the chunk that ends the stream
        if (st == CODAG_OK && !last && made != block) st = made < block ? CODAG_E_UNDERFLOW : CODAG_E_OVERFLOW;
        if (st != CODAG_OK) atomicMin(&meta->key, (unsigned long long)error_key(f, st));
        else if (last) meta->last = made;
    };
    uint32_t aside = 0;  // a bit per LZ4 block set aside
    for (uint32_t k = 0; k < group; k++) {
        const uint32_t f = Grouped ? uni(s_deal.mine[k]) : blockIdx.x;
        const uint64_t at = (uint64_t)f * block, src = uni64(frames[f].src);
        const uint32_t len = uni(frames[f].len), original = uni(frames[f].original), room = room_of(f);
        int st = CODAG_OK;
        uint32_t made = 0;
        if (original) {
            if (len > room) {
                st = CODAG_E_OVERFLOW;
            } else {
                const WavePiece mine = wave_piece(len, wave, kTeam);
                wave_stream(out + at + mine.begin, framed + src + mine.begin, mine.size);
                made = len;
            }
        } else if (len >= (1u << 28)) {
            st = CODAG_E_INVALID_ARGUMENT;
        } else {
            if constexpr (Codec == CODAG_LZ4)
                st = lz_team_chunk(framed + src, len, out + at, room, &made, &s.t, s_ring, wave, group);
            else
                st = Team<kTeam>::chunk(framed + src, len, out + at, room, &made, &s, s_ring, wave);
        }
        if (Codec == CODAG_LZ4 && st == kLzAside) aside |= 1u << k;
        else if (threadIdx.x == 0) done(f, st, made);
    }
    if constexpr (Codec == CODAG_LZ4) {
        if (!aside) return;
        __syncthreads();  // the team's LDS is done with
        if (wave < kLzGroup && ((aside >> wave) & 1)) {
            const uint32_t f = Grouped ? uni(s_deal.mine[wave]) : blockIdx.x;
            uint32_t made = 0;
            const int st = lz_alone(framed + uni64(frames[f].src), uni(frames[f].len), out + (uint64_t)f * block,
                                    room_of(f), &made, &s.a[wave]);
            if (lane() == 0) done(f, st, made);
        }
    }
}

void launch_orc_frame_team(int codec, const uint8_t *framed, uint32_t block, uint8_t *out, uint64_t out_cap,
                           const OrcFrame *frames, uint32_t max_frames, OrcMeta *meta, hipStream_t s) {
    if (codec == CODAG_LZ4 && max_frames <= kLzGrid)
        hipLaunchKernelGGL((orc_frame_team<CODAG_LZ4, kLzTeam>), dim3(max_frames), dim3(kLzThreads), 0, s, framed, block,
                           out, out_cap, frames, meta);
    else if (codec == CODAG_LZ4)
        hipLaunchKernelGGL((orc_frame_team<CODAG_LZ4, kLzTeam, true>), dim3(kLzGrid), dim3(kLzThreads), 0, s, framed,
                           block, out, out_cap, frames, meta);
    else if (max_frames <= kBigTeamMaxChunks)
        hipLaunchKernelGGL((orc_frame_team<CODAG_DEFLATE, 16>), dim3(max_frames), dim3(16 * kWave), 0, s, framed, block,
                           out, out_cap, frames, meta);
    else
        hipLaunchKernelGGL((orc_frame_team<CODAG_DEFLATE, 8>), dim3(max_frames), dim3(8 * kWave), 0, s, framed, block,
                           out, out_cap, frames, meta);
}

}  // namespace codag
