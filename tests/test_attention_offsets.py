"""The attention kernel's fetch offsets at sizes that no test can allocate: compiled for the host and compared with whole numbers."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_12526_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "sp_attn_offsets.h"
int main()
{
    char what;
    long long a, b, c, d;
    while (scanf(" %c %lld %lld %lld %lld", &what, &a, &b, &c, &d) == 5)
        if (what == 'v') printf("%lld\n", (long long)sp::value_row_offset((int)a, (int)b));
        else printf("%lld\n", (long long)(sp::key_tile_offset((int)a, (int)d) + sp::key_row_offset((int)a, (int)b, (int)c, (int)d)));
}
"""


def test_offsets_are_wide_enough(tmp_path):
    src, exe = tmp_path / "offsets.cpp", tmp_path / "offsets"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    ask, want = [], []
    for rows in (256, 68_174_336, 2**31 - 256):             # 63 rows of the second are the first to pass 2^32 elements
        for d in (0, 1, 31, 32, 63):
            ask.append(f"v {d} {rows} 0 0")
            want.append(d * rows)
    for ld in (384, 3072):
        for length in (1, 60, 65, 2**32 // 384 + 100, 2**31 - 1):
            tiles = {-7, -1, 0, 57, (length - 1) // 64 * 64, (length - 1) // 64 * 64 - 7}
            for kt0 in sorted(t for t in tiles if t < length):
                for i in (0, 6, 7, 31, 32, 63):
                    if kt0 + i >= 2**31:                    # (token counts are 32-bit)
                        continue
                    ask.append(f"k {kt0} {i} {length} {ld}")
                    want.append(min(max(kt0 + i, 0), length - 1) * ld)
    out = subprocess.run([str(exe)], input="\n".join(ask), capture_output=True, text=True, check=True).stdout.split()
    assert [int(v) for v in out] == want
