"""The per-pixel table's words, compiled for the host from the library's own header: what the passes
keep in a pixel's key maximum (an opaque fragment hides what lies behind it, or not, beside the
largest depth key itself) comes back for every kind of inverse depth, in any order of the tile's
chunks, and the offsets of a tile whose fragments fill 32 bits need no bit for it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>
#include "hair_internal.h"
using namespace hair;

static uint32_t key_of(float iz) {
    uint32_t b;
    memcpy(&b, &iz, 4);
    return 0xFFFFFFFFu - b;
}

int main() {
    const float izs[] = {0.0f, 1e-45f, 1e-38f, 1e-6f, 0.3f, 1.0f, 100.0f, 1e30f, 3.4028235e38f};
    for (float iz : izs)
        if (kmax_key(kmax_seen(key_of(iz))) != key_of(iz)) return printf("key of %g lost\n", iz);
    std::mt19937 rng(1);
    for (int trial = 0; trial < 2000; ++trial) {
        // one pixel: the keys of its stored fragments, in chunks, hidden or not behind the farthest
        const bool hides = rng() & 1u;
        std::vector<uint32_t> keys(1 + rng() % 40);
        for (uint32_t& k : keys) k = key_of(std::uniform_real_distribution<float>(1e-3f, 10.0f)(rng));
        const uint32_t far = *std::max_element(keys.begin(), keys.end());
        uint32_t word = hides ? far : 0u;                     // after k_tile_prep
        for (size_t i = 0; i < keys.size();) {                // each chunk: read the flag, add its maximum
            const size_t e = std::min(keys.size(), i + 1 + rng() % 5);
            if (kmax_hides(word) != hides) return printf("flag lost\n");
            if (hides && word != far) return printf("opaque key lost\n");
            word = std::max(word, kmax_seen(*std::max_element(keys.begin() + i, keys.begin() + e)));
            i = e;
        }
        if (kmax_key(word) != far) return printf("maximum lost\n");
    }
    // an opaque fragment's word hides whatever its key is (a NaN's may lack the top bit): the count
    // and the emit pass then leave out the same fragments
    for (uint32_t key : {0x003FFFFFu, 0x803FFFFFu, 0u, 0x7FFFFFFFu})
        if (!kmax_hides(kmax_key(key)) || kmax_key(key) < key) return printf("word of %08x\n", key);
    // offsets of a tile: 256 pixels of 2^24 - 1 fragments
    uint32_t off = 0;
    for (int p = 0; p < kTilePix; ++p) {
        if (off != (uint32_t)((unsigned long long)p * kMaxListLen)) return printf("offset of pixel %d\n", p);
        off += kMaxListLen;
    }
    static_assert((unsigned long long)kTilePix * kMaxListLen < (1ull << 32), "");
    static_assert((unsigned long long)kTilePix * kMaxListLen > (1ull << 31), "no bit is free");
    puts("ok");
    return 0;
}
"""


def test_key_maxima_and_offsets(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "words.cpp", tmp_path / "words"
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1",
                    "-I", os.path.join(ROOT, "paper_2405_10565_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout


def test_offsets_are_read_whole():
    """No pass masks an offset of the table."""
    text = open(os.path.join(ROOT, "paper_2405_10565_amd", "csrc", "hair_kernels.hip")).read()
    reads = [line for line in text.splitlines() if "pix_off[" in line]
    assert len(reads) >= 6
    assert not [line for line in reads if "&" in line.split("pix_off[", 1)[1].replace("&f.", "")]


def test_the_opaque_pass_stores_words_that_hide():
    text = open(os.path.join(ROOT, "paper_2405_10565_amd", "csrc", "hair_kernels.hip")).read()
    stores = [line for line in text.splitlines() if "atomicMin(&f.pix_kmax[" in line]
    assert stores and all("kmax_key(" in line for line in stores)
