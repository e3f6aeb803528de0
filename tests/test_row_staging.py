"""Index arithmetic of the quantizer's row staging (csrc/row_staging.h), run on the host: every 16-byte read of
every lane stays inside the row's LDS buffer, and where the row has the elements, the transfers have put
them there.  All row lengths, bf16 and fp32."""
import os
import subprocess

from paper_2502_05003_amd import build

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <stdio.h>
#include "row_staging.h"

template <int E>
int check()
{
    typedef quest::RowStaging<E> S;
    int bad = 0;
    for (int cols = 64; cols <= 16384; cols += 64) {
        const int row_bytes = cols * E, buffer = S::buffer_bytes(cols);
        if (buffer < row_bytes)
            ++bad;
        for (int at = 0; at < row_bytes; at += 1024)
            for (int lane = 0; lane < 64; ++lane) {
                const int source = S::source(at, lane, row_bytes);
                if (at + 16 * lane + 16 > buffer || source < 0 || source + 16 > row_bytes || source % 16)
                    ++bad;
            }
        for (int t = 0; 1024 * t < cols; ++t)
            for (int m = 0; m < 32; ++m)
                for (int h = 0; h < 2; ++h)
                    for (int i = 0; i < S::kReads; ++i) {
                        const int at = S::read(t, m, h, i, buffer);
                        if (at < 0 || at + 16 > buffer || at % 16)
                            ++bad;
                        const int want = (1024 * t + 32 * m + 16 * h) * E + 16 * i;   // byte of the row
                        if (1024 * t + 32 * m < cols && S::source(at / 1024 * 1024, at % 1024 / 16, row_bytes) != want)
                            ++bad;
                    }
    }
    return bad;
}

int main()
{
    printf("%d %d\n", check<2>(), check<4>());
    return 0;
}
"""


def test_every_read_is_inside_the_buffer_and_finds_its_chunk(tmp_path):
    source, program = tmp_path / "check.hip", str(tmp_path / "check")
    source.write_text(PROGRAM)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", build.CSRC, str(source), "-o", program],
                   check=True, capture_output=True)
    run = subprocess.run([program], check=True, capture_output=True, text=True)
    assert run.stdout.split() == ["0", "0"]
