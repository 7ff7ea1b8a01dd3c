"""The output window's slide, run on the host with the library's own read rule:
every byte of the output kept moves to its new place, and no read or write leaves
the window."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#include "share.hpp"
// One slide of a window of H bytes holding `held` (the rest is free) by T
// threads, for an append of len bytes.
static bool slide(uint32_t H, uint32_t T, uint32_t held, uint32_t len) {
    std::vector<unsigned char> win(H), old;
    for (uint32_t i = 0; i < H; i++) win[i] = (unsigned char)(i * 2654435761u >> 13);
    old = win;
    const uint32_t lo = (held + len - H + 511) & ~511u;  // the new first byte
    std::vector<unsigned char> v(16 * T);
    for (uint32_t i = 0; i < held - lo; i += 16 * T) {
        for (uint32_t t = 0; t < T; t++) {
            const uint32_t from = codag::slide_from(lo + i + 16 * t, H), to = i + 16 * t;
            if (from + 16 > H || to + 16 > H) return false;
            std::memcpy(&v[16 * t], &win[from], 16);
        }
        std::memcpy(&win[i], v.data(), 16 * T);
    }
    return std::memcmp(win.data(), &old[lo], held - lo) == 0;
}
int main(int argc, char **argv) {
    const uint32_t H = std::atoi(argv[1]), T = std::atoi(argv[2]), append = H - 1536;
    unsigned bad = 0;
    for (uint32_t held = 1536; held <= H; held += held % 512 == 511 || held % 512 < 2 ? 1 : 85)
        for (uint32_t len : {H - held + 1, (H - held + 1 + append) / 2, append})
            if (held + len > H && len <= append) bad += !slide(H, T, held, len);
    std::printf("%u\n", bad);
    return bad != 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("slide")
    (d / "slide.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2307_03760_amd", "csrc"),
                    str(d / "slide.cpp"), "-o", str(d / "slide")], check=True)
    return str(d / "slide")


@pytest.mark.parametrize("window,threads", [(4096, 64), (8192, 64), (16384, 64), (32768, 64), (32768, 512),
                                            (32768, 1024)])
def test_slide_stays_in_the_window(exe, window, threads):
    done = subprocess.run([exe, str(window), str(threads)], capture_output=True, text=True)
    assert (done.returncode, done.stdout.strip()) == (0, "0")
