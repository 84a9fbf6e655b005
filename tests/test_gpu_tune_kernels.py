"""A tiling in the tuning cache that was timed with kernels of another generation
is not taken: the plan is timed again, and the older entry stays in the file."""
import json

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def test_tilings_of_older_kernels_are_timed_again(tmp_path, monkeypatch):
    from paper_2001_01583_amd import hpnfft as H
    path = tmp_path / "tune.json"
    monkeypatch.setenv("HPNFFT_TUNE_CACHE", str(path))
    g = W.rng(77)
    x = torch.from_numpy(W.uniform_points(20000, 3, g)).cuda()

    def tuned():
        p = H.Plan((16, 16, 16), 20000, m=8, precision="f64")
        p.set_points(x)
        p.autotune()
        return p.tiles

    tuned()
    (key, _), = json.loads(path.read_text())["entries"].items()
    parts = key.split("|")
    assert parts[0] == "v3" and parts[1].startswith("k")
    older = "|".join(parts[:1] + parts[2:])  # (keys named no generation before)
    path.write_text('{"hpnfft_tune_cache": 3,\n "entries": {\n  "%s": [4, 24, 512]\n }}\n' % older)
    tuned()
    entries = json.loads(path.read_text())["entries"]
    assert entries[older] == [4, 24, 512] and key in entries
