"""Where the product's any-K kernel finds a row's scales, on the CPU: a tiled row's are 1 KB a superstage apart, so that the offset
passes 2^31 from K = 2^30 + 512 on."""
import os
import subprocess

import paper_2511_04214_amd as brq

SIZES = (256, 288, 512, 544, 768, 4000, 2 ** 26, 2 ** 30 - 32, 2 ** 30, 2 ** 30 + 32, 2 ** 30 + 512, 2 ** 30 + 800, 2 ** 31 - 512, 2 ** 31 - 32)


def test_scales_of_every_k(tmp_path):
    csrc = os.path.join(os.path.dirname(brq.LIB_PATH), "csrc")
    src, exe = tmp_path / "offsets.cpp", str(tmp_path / "offsets")
    src.write_text('''#include <stdio.h>
#include "brq_launch.h"
int main() {
    for (long long K : {%s})
        for (int tiled = 0; tiled < 2; ++tiled) {
            const int groups = (int)(K / 32), pairs = (groups + 7) / 8;
            for (int t : {0, 1, 2, pairs / 2, pairs - 2, pairs - 1})
                if (t >= 0 && t < pairs) printf("%%lld %%d %%d %%lld\\n", K, tiled, t, (long long)brq::pair_scales(tiled, t, groups));
        }
}''' % ", ".join("%dLL" % k for k in SIZES))
    subprocess.check_call(["g++", "-std=c++17", "-fwrapv", "-D__HIP_PLATFORM_AMD__=1", "-isystem/opt/rocm/include", "-I" + csrc, str(src), "-o", exe])
    seen = 0
    for line in subprocess.check_output([exe], text=True).splitlines():
        K, tiled, t, at = (int(v) for v in line.split())
        first = min(8 * t, K // 32 - 8) if not tiled else 8 * t
        assert at == (first // 16 * 1024 + first % 16 if tiled else first), (K, tiled, t)
        assert 0 <= at and at + 8 <= ((K + 511) // 512 * 1024 if tiled else K // 32), (K, tiled, t)
        seen += 1
    assert seen > 8 * len(SIZES)
