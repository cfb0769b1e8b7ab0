"""The positions that a workgroup of the front end's kernels reads lie inside its sample, also where it has no positions of
its own.  The kernels' index arithmetic (csrc/hdt_share.h) is compiled for the host and walked through."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_08330_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "hdt_share.h"

// what k_parents_from_levels reads of one sample, workgroup by workgroup, and whether every position has one owner
static int check(int batch, int n)
{
    const int shares = hpe_shares(batch, n);
    int next = 0, bad = 0;
    for (int k = 0; k < shares; k++) {
        const HpeShare s = hpe_share(k, n, shares);
        if (!s.empty()) {
            bad += s.first != next || s.last > n;
            next = s.last;
        }
        if (shares > 1 && s.first > 0)
            for (int end = s.first; end > 0; end -= kBack * kOrdThreads)
                for (int u = 0; u < kBack; u++)
                    for (int tid : {0, 1, 63, 64, 511, 1022, 1023}) {
                        const int j = hpe_position_in_front(s, end, u, tid);
                        bad += j >= n;
                    }
    }
    bad += next != n;
    if (bad) std::printf("batch %d, %d positions, %d shares: %d faults\n", batch, n, shares, bad);
    return bad;
}

int main()
{
    int bad = 0;
    for (int batch : {1, 2, 3, 4, 5, 7, 15, 16, 17, 31, 32, 33, 40, 63, 64, 65, 85, 86, 127, 128, 129, 255, 256, 257, 1000})
        for (int chunks : {1, 2, 3, 4, 5, 6, 7, 8, 9, 13, 31, 33, 63, 64, 65, 66, 96, 127, 129, 191, 193, 511, 512})
            for (int d : {-1023, -512, -1, 0})
                bad += check(batch, chunks * 1024 + d);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_position_a_workgroup_reads_is_inside_its_sample(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I", CSRC, str(src),
                    "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout[-2000:]


PROGRAM_BUILD = r"""
#include <cstdio>
#include <initializer_list>
#include "hdt_share.h"

// entries that a wave of the busiest compute unit takes, in all rounds
static double busiest(int batch, long long entries, int shares)
{
    const long long rounds = ((long long)batch * shares + kOnChip - 1) / kOnChip;
    return (double)rounds * (double)((entries + 16ll * shares - 1) / (16ll * shares));
}

int main()
{
    int bad = 0;
    for (int batch = 1; batch <= 2000; batch += batch < 700 ? 1 : 37)
        for (long long entries : {1, 13, 40, 72, 208, 288, 1152, 5000, 70000, 300000000}) {
            const int shares = cross_build_shares(batch, 8192, entries);
            const double fair = (double)batch * (double)entries / (16. * kOnChip);
            // a scan is worth 2.5 entries: up to a handful of entries nothing can be divided, beyond them little is idle
            if (shares < 1 || (shares - 1) * 16ll >= entries || (fair > 20. && busiest(batch, entries, shares) > 1.4 * fair + 4.)) {
                bad++;
                std::printf("batch %d, %lld entries: %d shares, busiest %g, fair %g\n", batch, entries, shares, busiest(batch, entries, shares), fair);
            }
        }
    for (int batch : {1 << 20, 2147483647})
        for (long long entries : {1ll, 1152ll, 600000000ll}) bad += cross_build_shares(batch, 1 << 19, entries) < 1;
    // a long scan is not repeated for entries that take less time: one round where there can be one
    for (int batch : {1, 3, 10, 24, 40}) bad += batch * cross_build_shares(batch, 1 << 19, 13312) > kOnChip;
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_the_cross_attention_build_leaves_no_half_of_the_chip_idle(tmp_path):
    src, exe = tmp_path / "shares.cpp", tmp_path / "shares"
    src.write_text(PROGRAM_BUILD)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I", CSRC, str(src),
                    "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout[-2000:]
