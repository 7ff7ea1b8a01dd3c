// ORC byte RLE by one workgroup per chunk.
//
// A byte RLE stream is a chain of groups, each a header byte (0..127: a run
// of header + 3 copies of the next byte; -1..-128: -header literal bytes), and
// what one wave decoding a chunk waits for is the chain: about 700 cycles from
// header to header, for 66 output bytes on average in mixed data.  Here a
// workgroup takes the chunk in windows of 4,096 (2,048) byte positions.  Every thread
// works out, for its positions, where the group that would start there ends
// and how many values it holds; three rounds of link doubling in LDS turn
// that into where eight groups end; the real chain is then one LDS read per
// eight groups, and the groups between are found from the doubled links, all
// at once.  Eight lanes write each group, sixteen bytes a lane.
//
// What is left is some 6 us a window for its eight barriers and dependent
// LDS reads; one chunk of 200,000 values takes 106 us, 833 by one wave.
// Measured against one wave per chunk: 400 chunks of 50,000 values 220 to 36
// us, 1,024 of 10,000 59 to 25, 2,048 of 30,000 160 to 80; at 4,096 chunks the
// two are equal (16,000 values) or the waves ahead (500), hence the limit.
#include <hip/hip_runtime.h>

#include "../../include/codag.h"
#include "decode.hpp"
#include "internal.hpp"
#include "window.hpp"

namespace codag {

constexpr uint32_t kByteLevels = 4;                // links over 1, 2, 4 and 8 groups
constexpr uint32_t kByteAhead = 160;               // a group's bytes and a 16-byte read past its last

// With T threads a window has 4 T byte positions.
template <uint32_t T>
struct ByteLds {
    static constexpr uint32_t kStep = 4 * T, kPieces = (kStep + kByteAhead) / 16;
    static constexpr uint32_t kUnits = kStep / 2 / 8 + 1;  // stretches of eight groups in a window (a group has two bytes or more)
    static_assert(kStep + 8 * 130 < (1u << 16), "links fit 16 bits");
    uint32_t buf[2][kPieces * 4];
    // Position p's link over 2^k groups: where the next group starts (0-15)
    // and the values in between (16-31).  Links stop at the window's end.
    uint32_t link[kByteLevels][kStep];
    uint2 unit[kUnits];      // every eighth group: position, first value
    unsigned long long err;  // first value of the failing group << 4 | -status
    uint32_t pos, n, units;
};

template <uint32_t kByteThreads>
__global__ void __launch_bounds__(kByteThreads)
    byte_rle_blocks(const uint8_t *comp, const uint64_t *coff, uint8_t *out, const uint64_t *ooff, uint32_t n_chunks,
                    int32_t *status, unsigned long long *err) {
    constexpr uint32_t kByteStep = ByteLds<kByteThreads>::kStep, kBytePieces = ByteLds<kByteThreads>::kPieces;
    __shared__ __align__(16) ByteLds<kByteThreads> s;
    const uint32_t t = threadIdx.x, c = blockIdx.x;
    if (c >= n_chunks) return;
    const uint64_t i0 = coff[c], i1 = coff[c + 1], o0 = ooff[c], o1 = ooff[c + 1];
    if ((((i1 - i0) | (o1 - o0)) >> 31) != 0) {
        if (t < kWave) report(c, CODAG_E_INVALID_ARGUMENT, status, err);
        return;
    }
    const uint8_t *chunk = comp + i0;
    const uint32_t skip = (uint32_t)(reinterpret_cast<uintptr_t>(chunk) & 15);
    const uint8_t *gbase = chunk - skip;  // positions are relative to the 16-byte hull
    const uint32_t end = skip + (uint32_t)(i1 - i0), cap = (uint32_t)(o1 - o0);
    uint8_t *dst = out + o0;
    if (t == 0) s.err = ~0ull;
    __syncthreads();

    // Window w's bytes into buffer w & 1, by the last waves, which write the
    // fewest groups (a wait for loads also waits for the wave's stores).
    constexpr uint32_t kLoaders = (kBytePieces + kWave - 1) / kWave * kWave;
    static_assert(kLoaders <= kByteThreads, "one piece a thread");
    auto issue = [&](uint32_t w) {
        const uint32_t q = t - (kByteThreads - kLoaders), at = w * kByteStep + 16 * q;
        if (q < kBytePieces && at < end)
            __builtin_amdgcn_global_load_lds(gbase + at, (lds_void *)(s.buf[w & 1] + 4 * (q & ~63u)), 16, 0, 0);
    };
    uint32_t pos = skip, n = 0;  // the next group and its first value
    issue(0);
    int st = CODAG_OK;
    for (uint32_t w = 0;; w++) {
        // The same on every thread.
        if (s.err != ~0ull) break;  // (set before the barrier that ended the window)
        if (n == cap) {
            if (pos != end) st = CODAG_E_CORRUPT;
            break;
        }
        if (pos >= end) {
            st = CODAG_E_TRUNCATED;
            break;
        }
        const uint32_t W = w * kByteStep;
        const uint32_t lim = min(kByteStep, end - W);  // positions of this window (W < end: pos < end)
        if (t >= kByteThreads - kLoaders) wait_vm();
        __syncthreads();  // window w has landed
        if (W + kByteStep < end) issue(w + 1);
        const uint8_t *bytes = reinterpret_cast<const uint8_t *>(s.buf[w & 1]);
        // Links over one group: four positions a thread.
        {
            const uint32_t v = s.buf[w & 1][t];
            uint32_t e[4];
#pragma unroll
            for (uint32_t i = 0; i < 4; i++) {
                const uint32_t h = (v >> (8 * i)) & 0xff, p = 4 * t + i;
                e[i] = h < 128 ? (p + 2) | ((h + 3) << 16) : (p + 257 - h) | ((256 - h) << 16);
            }
            reinterpret_cast<uint4 *>(s.link[0])[t] = make_uint4(e[0], e[1], e[2], e[3]);
            __syncthreads();
#pragma unroll
            for (uint32_t k = 1; k < kByteLevels; k++) {
#pragma unroll
                for (uint32_t i = 0; i < 4; i++) {
                    const uint32_t to = e[i] & 0xffff;
                    const uint32_t f = s.link[k - 1][min(to, kByteStep - 1)];
                    if (to < lim) e[i] = f + (e[i] & 0xffff0000u);
                }
                reinterpret_cast<uint4 *>(s.link[k])[t] = make_uint4(e[0], e[1], e[2], e[3]);
                __syncthreads();
            }
        }
        // The chain, eight groups a step.
        if (t < kWave) {
            uint32_t p = pos - W, v = n, u = 0;
            while (p < lim) {
                if (t == 0) s.unit[u] = make_uint2(p, v);
                const uint32_t f = uni(s.link[kByteLevels - 1][p]);
                p = f & 0xffff;
                v += f >> 16;
                u++;
            }
            if (t == 0) {
                s.pos = W + p;
                s.n = v;
                s.units = u;
            }
        }
        __syncthreads();
        // Groups: eight lanes each.
        const uint32_t groups = 8 * s.units;
        for (uint32_t g = t / 8; g < groups; g += kByteThreads / 8) {
            const uint2 un = s.unit[g / 8];
            uint32_t p = un.x, v = un.y;
#pragma unroll
            for (uint32_t k = 0; k < 3; k++) {
                if ((g >> (2 - k)) & 1) {
                    const uint32_t f = s.link[2 - k][min(p, kByteStep - 1)];
                    if (p < lim) {
                        v += f >> 16;
                        p = f & 0xffff;
                    }
                }
            }
            if (p >= lim || v > cap) continue;  // past the window, or after an output overflow
            const uint32_t h = bytes[p];
            const bool run = h < 128;
            const uint32_t len = run ? h + 3 : 256 - h, from = p + 1;
            int bad = CODAG_OK;
            if (v == cap) bad = CODAG_E_CORRUPT;  // input left over
            else if (run && W + p + 2 > end) bad = CODAG_E_TRUNCATED;
            else if (v + len > cap) bad = CODAG_E_OVERFLOW;
            else if (!run && W + from + len > end) bad = CODAG_E_TRUNCATED;
            if (bad) {
                atomicMin(&s.err, ((unsigned long long)v << 4) | (unsigned long long)(-bad));
                continue;
            }
            uint8_t *to = dst + v;
            const uint64_t rep = bytes[from] * 0x0101010101010101ull;
            const uint32_t sub = t & 7;
            if (len >= 16) {
                for (uint32_t k = 16 * sub; k < len; k += 128) {
                    const uint32_t j = min(k, len - 16);
                    u128_any x;
                    if (run) {
                        x.x = x.y = x.z = x.w = (uint32_t)rep;
                    } else {
                        x = *reinterpret_cast<const u128_any *>(bytes + from + j);
                    }
                    *reinterpret_cast<u128_any *>(to + j) = x;
                }
            } else {
                // Two bytes a lane.
#pragma unroll
                for (uint32_t k = 0; k < 2; k++) {
                    const uint32_t j = 2 * sub + k;
                    if (j < len) to[j] = run ? (uint8_t)rep : bytes[from + j];
                }
            }
        }
        __syncthreads();
        pos = s.pos;
        n = s.n;
    }
    // A load issued one window ahead may still be landing.
    wait_vm();
    if (t < kWave) {
        const unsigned long long k = s.err;
        report(c, k != ~0ull ? -(int)(k & 15) : st, status, err);
    }
}

int launch_byte_rle_blocks(const uint8_t *comp, const uint64_t *coff, uint8_t *out, const uint64_t *ooff, uint32_t n,
                           int32_t *status, unsigned long long *err, hipStream_t s) {
    // As many threads as let all the workgroups run at once (two of 1,024 on a
    // CU): 400 chunks of 50,000 values take 36 us with 1,024 threads and 45
    // with 512, 1,024 chunks 81 and 69, 2,048 chunks of 30,000 96 and 80.
    if (n <= 512)
        hipLaunchKernelGGL(byte_rle_blocks<1024>, dim3(n), dim3(1024), 0, s, comp, coff, out, ooff, n, status, err);
    else
        hipLaunchKernelGGL(byte_rle_blocks<512>, dim3(n), dim3(512), 0, s, comp, coff, out, ooff, n, status, err);
    return hipGetLastError() == hipSuccess ? CODAG_OK : CODAG_E_HIP;
}

}  // namespace codag
