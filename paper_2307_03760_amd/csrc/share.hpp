// Index arithmetic of the copies (host code too: no HIP here).
#pragma once

#include <stdint.h>

namespace codag {

struct WavePiece {
    uint32_t begin, size;
};

// The part of len bytes (below 2^31) that wave `wave` of `waves` copies: whole
// kilobytes, one after another, the last wave with bytes left taking the rest.
// Rounded up twice, so that waves * share is never below len.
constexpr WavePiece wave_piece(uint32_t len, uint32_t wave, uint32_t waves) {
    const uint32_t share = ((len + waves - 1) / waves + 1023) & ~1023u;
    const uint64_t from = (uint64_t)wave * share;
    const uint32_t begin = from < len ? (uint32_t)from : len;
    return {begin, len - begin < share ? len - begin : share};
}

// Where a thread reads the 16 bytes that an output window of H bytes moves
// towards its front: x is their place, or, past the window's end (a slide's last
// trip is a full one), the window's last 16 bytes, which are not wanted there.
constexpr uint32_t slide_from(uint32_t x, uint32_t H) { return x < H - 16 ? x : H - 16; }

}  // namespace codag
