"""The pieces in which the waves of a workgroup copy a run of bytes cover every
byte once, whatever its length (the library's own header, built for the host)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "share.hpp"
static bool covered(uint32_t len, uint32_t waves) {
    uint32_t at = 0;
    for (uint32_t w = 0; w < waves; w++) {
        const codag::WavePiece p = codag::wave_piece(len, w, waves);
        if (p.begin != at) return false;
        at += p.size;
    }
    return at == len;
}
int main() {
    unsigned bad = 0;
    for (uint32_t waves : {8u, 16u}) {
        for (uint32_t len = 0; len < 1u << 23; len++) bad += !covered(len, waves);
        for (uint32_t len = 0x7fffff00u; len < 0x80000000u; len++) bad += !covered(len, waves);
    }
    std::printf("%u\n", bad);
    return bad != 0;
}
"""


def test_pieces_cover_every_length(tmp_path):
    src, exe = tmp_path / "share.cpp", tmp_path / "share"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2307_03760_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert (done.returncode, done.stdout.strip()) == (0, "0")
