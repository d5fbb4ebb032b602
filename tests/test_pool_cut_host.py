"""How the pool kernels cut a map (pool_cut of csrc/sk_kernels.h), on the CPU: over sizes from one window to long and wide maps every window lies in
exactly one chain, workgroups stay within the kernels' launch bounds, and grids within what a launch takes or the caller's own check."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1509_03371_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <cstddef>
#include <cstdint>
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
enum hipError_t { hipSuccess };
typedef struct Stream *hipStream_t;
"""

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "sk_kernels.h"
int main()
{
    long bad = 0, cuts = 0;
    for (int Ho : {1, 2, 3, 7, 8, 31, 33, 64, 100, 527, 1066, 20000})
        for (int cols : {1, 2, 5, 16, 37, 64, 65, 129, 131, 200, 256, 257, 512, 1058, 5000})
            for (int d : {1, 2, 3, 5, 8, 16, 33})
                for (long planes : {1L, 6L, 48L, 384L})
                    for (long short_waves : {sk::POOL_WAVES, sk::POOL_WAVES / 4})
                        for (int most : {256, 512}) {
                            const sk::PoolCut c = sk::pool_cut(Ho, cols, d, planes, short_waves, most);
                            ++cuts;
                            const dim3 b = c.block(), g = c.grid(cols, planes);
                            bool ok = c.bx >= 1 && c.bp >= 1 && c.bs >= 1 && c.len >= 1 && b.x * b.y * b.z <= (unsigned)most && g.z == planes;
                            ok = ok && (long)g.x * c.bx >= cols && ((long)g.x - 1) * c.bx < cols;
                            // (class, segment) of every thread row of the grid, as the kernels compute them
                            std::vector<int> seen((size_t)d * c.nseg, 0);
                            for (long y = 0; ok && y < c.gy; ++y)
                                for (int ty = 0; ty < c.bp; ++ty)
                                    for (int tz = 0; tz < c.bs; ++tz) {
                                        const int sblock = (int)(y / c.pblocks), phase = (int)(y - (long)sblock * c.pblocks) * c.bp + ty, seg = sblock * c.bs + tz;
                                        if (phase < d && seg < c.nseg) ++seen[(size_t)phase * c.nseg + seg];
                                    }
                            for (int s : seen) ok = ok && s == 1;
                            for (int phase = 0; ok && phase < d && phase < Ho; ++phase) ok = (Ho - phase + d - 1) / d <= c.nseg * c.len;
                            if (!ok && bad++ < 5) printf("%d %d %d %ld: %d %d %d len %d nseg %d\n", Ho, cols, d, planes, c.bx, c.bp, c.bs, c.len, c.nseg);
                        }
    printf("%ld cuts, %ld bad\n", cuts, bad);
    return bad != 0;
}
"""


def test_every_window_in_one_chain(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (tmp_path / "main.cpp").write_text(PROGRAM)
    exe = tmp_path / "cuts"
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", str(tmp_path), "-I", CSRC, "-o", str(exe), str(tmp_path / "main.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
