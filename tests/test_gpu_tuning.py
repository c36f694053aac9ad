"""The autotuner times what a call launches, and takes no entry that an older build wrote."""
import os
import re
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_entries_of_another_format_are_not_used(tmp_path, monkeypatch):
    """A cache file's entries in the old form (seven numbers: their times were those of another
    cut) are passed over; the context's own entry, appended, is read back."""
    from paper_2412_14671_amd import Context
    path = tmp_path / "tiles"
    path.write_text("24 32 40 5 1 0 7\n")
    monkeypatch.setenv("MUSTER_TUNE_CACHE", str(path))
    got = []
    for _ in range(2):
        c = Context(0)
        try:
            got.append(c.sim_tiling((24, 32, 40), 5, "silncc"))
        finally:
            c.close()
    print("tilings", got, path.read_text().splitlines(), flush=True)
    assert got[0][1] in (16, 24) and got[1] == got[0]   # 7 is no candidate
    lines = path.read_text().splitlines()
    assert lines[0] == "24 32 40 5 1 0 7" and len(lines) == 2


@pytest.mark.parametrize("dims,window", [((32, 32, 32), 5), ((64, 48, 40), 7)])
def test_timed_cut_is_the_launched_one(dims, window):
    """The statistics of a candidate walk its chunk or parts of it in multiples of the window, the
    gradient multiples of the window whatever the chunk, as set_sim_parts cuts every launch."""
    code = ("import torch\nfrom paper_2412_14671_amd import Context\nc = Context(0)\n"
            f"print(c.sim_tiling({dims}, {window}, 'silncc'))\nc.close()\n")
    env = dict(os.environ, MUSTER_TUNE_VERBOSE="1")
    env.pop("MUSTER_TUNE_CACHE", None)
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, capture_output=True,
                       text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]
    rows = re.findall(r"shape (\d) zchunk (\d+) parts (\d+) gradient (\d+) ", r.stderr)
    print(rows, flush=True)
    assert len(rows) >= 3
    grad = {}
    for shape, zc, zs, zg in (tuple(map(int, row)) for row in rows):
        assert zs == zc or (zs < zc and zs % window == 0)
        assert zg % window == 0
        assert grad.setdefault(shape, zg) == zg
