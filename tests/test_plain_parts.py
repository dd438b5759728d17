"""Into how many workgroups whole FP4 chunks are split: no launch of 2^32 threads or more, whatever the number of chunks, and one workgroup per chunk where nothing
else fits or where a workgroup would have fewer rows than 32 (encoder) or about as many as it has wavefronts (decoder)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_19263_amd", "csrc")
PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "zc_internal.h"
int main(int argc, char **argv)
{
    for (int i = 1; i < argc; i++) {
        const uint32_t n = (uint32_t)strtoul(argv[i], nullptr, 10);
        for (uint32_t rows : {1u, 63u, 64u, 127u, 128u, 255u, 256u, 1024u}) printf("%u ", zc::plain_encode_parts(n, rows));
        for (uint32_t fmt : {ZC_FMT_FP4_E2M1_MX, ZC_FMT_FP4_E2M1_NV})
            for (uint32_t rows : {16u, 31u, 32u, 63u, 64u, 1024u}) printf("%u ", zc::plain_decode_parts(fmt, n, rows));
        printf("\\n");
    }
}
"""


def test_launches_stay_below_the_limit(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    source, program = tmp_path / "parts.cpp", str(tmp_path / "parts")
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I" + CSRC, str(source), "-o", program], check=True)
    most = (2 ** 32 - 1) // 256
    # the largest number of chunks that k workgroups each fit, its neighbours, and the ends
    counts = sorted({1, 2, 448, 1024, 1025, 5376, 1 << 20, most, most - 1} | {most // k + d for k in (2, 3, 5, 9) for d in (-1, 0, 1)})
    lines = subprocess.run([program] + [str(n) for n in counts], capture_output=True, text=True, check=True).stdout.split("\n")
    for n, line in zip(counts, lines):
        for parts, usual in zip(map(int, line.split()), (1, 1, 2, 2, 4, 4, 8, 8) + (1, 1, 2, 2, 4, 4) + ((1, 1, 2, 2, 4, 4) if n > 1024 else (1,) * 6)):
            assert parts in (1, usual), (n, line)
            assert n * (parts + 1 if parts > 1 else 1) * 256 < 2 ** 32, (n, line)
            assert parts == usual or n * (usual + 1) * 256 >= 2 ** 32, (n, line)
