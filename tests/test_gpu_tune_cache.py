"""Lines of the autotuner's cache file that another build wrote (no build at the
end of the line, or another one) are not taken: the choice is timed again and
appended.  Each step in a process of its own, since the file is read once."""
import json
import os
import subprocess
import sys

import pytest

from paper_2401_13680_amd import api

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TUNE = (
    "import json, torch\n"
    "from paper_2401_13680_amd import api, synth\n"
    "T = torch.from_numpy(synth.regime_series(8000, 14, len_range=(500, 1500)).x).cuda()\n"
    "code, ms = api.tune_geometry(T, 200, 100)\n"
    "api.set_geometry(101, 0)\n"
    "r = api.select_length(T, [48, 64, 80], 2, autotune=True)\n"
    "print(json.dumps([code, ms, r['m_best'], r['scores']]))\n")


def tune(cache):
    p = subprocess.run([sys.executable, "-c", TUNE], cwd=ROOT, env=dict(os.environ, PST_AUTOTUNE_CACHE=str(cache)),
                       capture_output=True, text=True, timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    return json.loads(p.stdout.strip().splitlines()[-1]), cache.read_text().splitlines()


@pytest.mark.parametrize("build", ["", " 0123456789abcdef"])
def test_lines_of_another_build_are_timed_again(tmp_path, build):
    cache = tmp_path / "tune.txt"
    first, lines = tune(cache)
    geo = [ln.split() for ln in lines if ln.startswith("geo ")]
    grid = [ln.split() for ln in lines if not ln.startswith("geo ")]
    assert len(geo) == 1 and len(grid) == 1 and len(geo[0]) == 6 and len(grid[0]) == 7
    # the same choices as if another build had timed them, the geometry not the built-in one
    other = next(c for c in api.geometry_candidates(101) if c != api.geometry(101))
    cache.write_text(f"geo {geo[0][1]} 101 {other} 0.0001{build}\n" + " ".join(grid[0][:3]) + f" 1 0 0.0001{build}\n")
    again, lines = tune(cache)
    assert again[1] > 0.0001 and len(lines) == 4 and again[2:] == first[2:]
    taken, lines = tune(cache)
    assert len(lines) == 4 and taken[0] == again[0] and abs(taken[1] - again[1]) < 1e-3
