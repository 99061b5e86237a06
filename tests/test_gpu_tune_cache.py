"""The autotuner's saved choices (CORR_TUNE_CACHE): a line of the present kernels is
used by the next process, one of an earlier revision is not.  Each handle is tuned in
a process of its own, for the file is read once."""
import os
import subprocess
import sys

import pytest

from helpers import say

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TUNE = """
import sys, torch
import paper_1305_5639_amd as corr
C, A = 64, 256
for N in map(int, sys.argv[1:]):
    with corr.Correlator(N, 1, C, A, "fp16") as c:
        t = c.autotune_fx(torch.zeros((N, A * C), dtype=torch.complex64, device="cuda:0"), A)
        print("TUNED", t["tile"], int(t["ms_tuned"] > 0))
"""


def tune(cache, *inputs):
    """(tile, whether it was timed) for each number of inputs, in turn."""
    r = subprocess.run([sys.executable, "-c", TUNE, *map(str, inputs)], cwd=ROOT, capture_output=True, text=True,
                       timeout=100, env={**os.environ, "CORR_TUNE_CACHE": str(cache)})
    assert r.returncode == 0, r.stderr
    return [(int(l.split()[1]), l.split()[2] == "1") for l in r.stdout.splitlines() if l.startswith("TUNED")]


def test_saved_choices(tmp_path):
    say("autotuner cache file")
    cache = tmp_path / "tune.txt"
    (tile, timed), = tune(cache, 100)
    assert timed
    line, = cache.read_text().splitlines()
    assert tune(cache, 100) == [(tile, False)]
    # the same choice as the first revision wrote it, and the other block size
    words = line.split()
    assert words[0] == "fx2"
    old = tmp_path / "old.txt"
    old.write_text("# a comment\n" + " ".join(["fx"] + words[1:6] + [str(192 - tile), words[7]]) + "\n")
    (_, timed), = tune(old, 100)
    assert timed
    assert old.read_text().splitlines()[-1].startswith("fx2 ")


def test_one_choice_per_kernel(tmp_path):
    """Up to 32 inputs another kernel runs in the low-precision forms than up to 64:
    a choice timed at one says nothing of the other."""
    say("autotuner cache: 20, 60, 31 and 33 inputs")
    cache = tmp_path / "tune.txt"
    assert [timed for _, timed in tune(cache, 20, 60, 31, 33)] == [True, True, False, False]
    assert [l.split()[3] for l in cache.read_text().splitlines()] == ["0", "1"]
