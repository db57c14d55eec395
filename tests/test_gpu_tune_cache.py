"""The autotune cache: a line says which sweep it timed; one without (written
when sdq_tune timed the column-pivoted sweeps) or of another sweep is not used
for the sweep that runs now, and stays in the file."""
import json

import pytest
import torch

from paper_2003_05286_amd import binding as sdq
from _gpu import say

pytestmark = pytest.mark.gpu


def test_lines_of_other_kernels_are_not_used(tmp_path):
    path = tmp_path / "tune.jsonl"
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    old = {"arch": arch, "n": 36, "variant": 5, "blocks_per_cu": 1, "ms": 0.1}
    path.write_text(json.dumps(old) + "\n" + json.dumps({**old, "sweep": 2}) + "\n")
    ctx = sdq.Context(0)
    say("[gpu] sdq_tune n = 36 with an older cache")
    ctx.tune([36], str(path))
    lines = [json.loads(x) for x in path.read_text().splitlines()]
    assert lines[:2] == [old, {**old, "sweep": 2}] and len(lines) == 3
    assert lines[2]["n"] == 36 and lines[2]["sweep"] not in (0, 2)
    ctx.tune([36], str(path))  # and that line is read back
    assert len(path.read_text().splitlines()) == 3
    ctx.close()
