"""Launch shapes kept in the JSON file hold for the kernels they were timed on: entries of another revision,
or of a library that did not write one, are measured again."""
import json
import os
import subprocess
import sys

import pytest
import torch

from test_gpu_batch import _CHILD

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


@pytest.mark.parametrize("revision", [None, 1, 1000])
def test_entries_of_other_kernels_are_measured_again(tmp_path, revision):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    cache = tmp_path / "tune.json"
    env = dict(os.environ, IBDL_TUNE_CACHE=str(cache))

    def run():
        r = subprocess.run([sys.executable, "-c", _CHILD, root], env=env, capture_output=True, text=True, timeout=240)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(cache.read_text())["entries"]

    first = run()
    assert len({e["kernels"] for e in first}) == 1
    lines = []
    for line in cache.read_text().splitlines():
        e = line.strip().rstrip(",")
        if e.startswith('{"kernels"'):
            d = json.loads(e)
            del d["kernels"]
            if revision is not None:
                d = {"kernels": revision, **d}
            d["tile"], d["blocks"] = 8, 7   # no measurement yields these
            line = line.replace(e, json.dumps(d))
        lines.append(line)
    cache.write_text("\n".join(lines) + "\n")
    again = run()
    assert [(e["kernels"], e["key"]) for e in again] == [(e["kernels"], e["key"]) for e in first]
    assert all(e["tile"] != 8 and e["blocks"] != 7 for e in again)
    before = cache.read_text()
    run()
    assert cache.read_text() == before
