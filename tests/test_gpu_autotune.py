"""The autotuner where counts without flags run in vertex-relative tables."""
import os
import subprocess
import sys

import pytest

import graphgen as gg
import paper_2009_11665_amd as sg

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
import sys
sys.path.insert(0, %r)
import graphgen as gg, paper_2009_11665_amd as sg
g = sg.Graph.from_csr(gg.rmat(14, 200_000, seed=9))
t = sg.autotune(sg.Plan(gg.CATERPILLAR10), g, "u64", 2)
print("tuned", t.spmm_width, t.ema_rows, t.batch, t.flags, flush=True)
""" % ROOT


def child(cache):
    out = subprocess.run([sys.executable, "-c", CHILD], env=dict(os.environ, SG2V_TUNE_CACHE=str(cache)),
                         capture_output=True, text=True, timeout=100, check=True).stdout
    return [int(x) for x in [ln for ln in out.splitlines() if ln.startswith("tuned")][-1].split()[1:]]


def test_autotune_keeps_relative_tables_and_automatic_passes():
    """Relative tables are about twice as fast here: no flag that leaves them, and the
    automatic colourings per pass, are installed; width and rows are settings of the
    absolute tables."""
    g = sg.Graph.from_csr(gg.rmat(14, 200_000, seed=9))
    p = sg.Plan(gg.CATERPILLAR10)
    old = sg.get_tuning()
    try:
        print("autotune", flush=True)
        t = sg.autotune(p, g, "fp32s", 2)
        assert t.flags == 0 and t.spmm_width in (16, 32, 64, 128)
        c = sg.Colorings(g, 10, 5, 2)
        sg.profile_start()
        sg.count(p, g, c, "fp32s")
        assert sg.profile_stop()["ema_single"]["launches"] == 0
    finally:
        sg.restore_tuning(old)


def test_autotune_cache_of_the_absolute_tables_is_not_taken(tmp_path):
    """A cache file is read back, but not its lines from before the relative tables:
    their keys lack the version, and their flags would keep a caller off them."""
    cache = tmp_path / "cache"
    first = child(cache)
    line = cache.read_text().splitlines()
    assert len(line) == 1 and "/t2 " in line[0]
    key, rest = line[0].split(" ", 1)
    assert child(cache) == first and len(cache.read_text().splitlines()) == 1  # read back
    cache.write_text(key[:-len("/t2")] + " 16 4 77 1 0 0 0 0\n")  # width, rows, batch, flags
    again = child(cache)
    assert again[2] in (0, 1, 2)  # timed anew
    assert len(cache.read_text().splitlines()) == 2
