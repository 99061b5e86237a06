"""The entries of the X-engine's scale table that each thread of an F-engine launch
writes (for_share in corr_internal.h, compiled here for the host): at every grid
the F-engine accepts, up to 2^30 workgroups, each entry once and nothing else."""
import os
import subprocess

from paper_1305_5639_amd.build import CSRC

PROGRAM = r"""
#include "corr_internal.h"
#include <cstdio>
#include <set>
#include <vector>
int main() {
    for (int log2_work : {0, 3, 22, 23, 24, 25, 30})
        for (int less : {0, 1, 7})
            for (int th : {256, 512})
                for (int C : {16, 1024, 8192}) {
                    const int n_work = (1 << log2_work) - less;
                    if (n_work < 1) continue;
                    std::set<int> ws;              // the first workgroups, and some around each power of two
                    for (int w = 0; w < 40; ++w) ws.insert(w);
                    for (int b = 5; b <= 30; ++b)
                        for (int d = -1; d <= 1; ++d) ws.insert((1 << b) + d);
                    ws.insert(n_work - 1);
                    std::vector<int> times(C, 0);
                    for (int w : ws)
                        for (int tid = 0; w < n_work && tid < th; ++tid)
                            corr::for_share(w, n_work, th, tid, C, [&](int k) {
                                if (k < 0 || k >= C) {
                                    std::printf("n_work %d th %d C %d: workgroup %d writes entry %d\n", n_work, th, C, w, k);
                                    std::exit(1);
                                }
                                ++times[k];
                            });
                    for (int k = 0; k < C; ++k)
                        if (times[k] != 1) {
                            std::printf("n_work %d th %d C %d: entry %d written %d times\n", n_work, th, C, k, times[k]);
                            return 1;
                        }
                }
    return 0;
}
"""


def test_every_scale_is_written_once(tmp_path):
    src, exe = tmp_path / "share.cpp", tmp_path / "share"
    src.write_text(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include", f"-I{CSRC}", str(src),
                        "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
