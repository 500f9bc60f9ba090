"""Divisions by numbers that the host knows, as the attention kernels take them, over the ranges they state (host code, no GPU
needed: the same functions, compiled for the host)."""
import os
import subprocess

from paper_2605_20104_amd import build

PROGRAM = r"""
#include <cstdio>
#include "attn_shared.h"
using namespace graft;
// quotients around multiples of d, where a multiplier that is off shows first: the largest ones, and those in between
template <class Div> static long wrong(uint32_t d, int64_t end, Div&& div) {
    long n = 0;
    const int64_t step = end / d / 4000 + 1;
    for (int64_t q = (end - 1) / d; q >= 0; q -= (q > 200 ? step : 1))
        for (int64_t x = q * d - 1; x <= q * d + 1; ++x)
            if (x >= 0 && x < end && div(static_cast<int>(x)) != x / d) ++n;
    return n;
}
int main() {
    long any = 0, known = 0;
    for (uint32_t d = 1; d <= 2048; ++d) {
        const Magic m = magic_any(d);
        any += wrong(d, int64_t{1} << 31, [&](int x) { return div_any(x, m.m, m.shift); });
        const uint32_t m31 = magic31(d);
        const int64_t end = d == 1 ? int64_t{1} << 31 : ((int64_t{1} << 31) - 1) / (d - 1) + 1;
        known += wrong(d, end, [&](int x) { return div31(x, m31); });
    }
    // the bound of magic31 is needed: a merge of 140 row blocks a (sequence, KV head) has up to 2^28 of them
    const uint32_t m140 = magic31(140);
    std::printf("%ld %ld %ld\n", any, known, wrong(140, int64_t{1} << 28, [&](int x) { return div31(x, m140); }));
}
"""


def test_divisions_are_exact_over_their_ranges(tmp_path):
    src, exe = tmp_path / "division.hip", tmp_path / "division"
    src.write_text(PROGRAM)
    subprocess.check_call([build._hipcc(), *build.HIPCC_FLAGS, str(src), "-o", str(exe)], stderr=subprocess.DEVNULL)
    any_, known, beyond = map(int, subprocess.check_output([str(exe)], text=True, timeout=100).split())
    assert (any_, known) == (0, 0)
    assert beyond > 0, "magic31 would do: this test compares nothing"
    merge = open(os.path.join(build.CSRC, "tree_attn.hip")).read()
    assert "div_any(tile_c / PIECES" in merge                     # the merge's row blocks, which the launch lets grow to 2^28
