"""GPU: the generic row passes for lines that do not fit LDS (gather or epilogue
kernel and a row transform over HBM) at small sizes, in FP32 and FP64, two and
three dimensions, doubled and GaNi grids: HOM_NO_FAST keeps the register passes
out of both runs and HOM_LONG_ROWS selects the long form, whose results are
bitwise those of the fused generic form (the same arithmetic per line).  With
register passes on the row axis HOM_LONG_ROWS changes nothing, also on grids of
more than 65535 rows."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

import homgen
import test_gpu_long_rows as lr

pytestmark = pytest.mark.gpu


def _run(long_rows):
    env = dict(os.environ, HOM_NO_FAST="1")
    env.pop("HOM_LONG_ROWS", None)
    if long_rows:
        env["HOM_LONG_ROWS"] = "1"
    code = lr._SCRIPT % dict(root=lr.ROOT, tests=os.path.join(lr.ROOT, "tests"))
    p = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)
    sys.stderr.write(p.stderr[-2000:])
    assert p.returncode == 0, p.stderr[-2000:]
    return json.loads(p.stdout.strip().splitlines()[-1])


def test_long_rows_are_bitwise_the_fused_generic_ones():
    fused, long_form = _run(False), _run(True)
    for name, *_ in lr.CASES:
        assert fused[name] == long_form[name], name


@pytest.mark.parametrize("dual", [False, True])
@pytest.mark.parametrize("generic", [False, True])
def test_more_than_65535_rows(generic, dual, monkeypatch):
    import torch
    import paper_1404_3614_amd as H
    N, M = (365, 181, 3), (729, 375, 5)
    pb = H.problem_from_cell(homgen.sphere_cell(seed=3, n=4, anisotropic=False), N, precision="mixed", M=M, max_loads=1)
    n = pb.flen[int(dual)]
    rng = np.random.default_rng(1)
    x = torch.tensor(rng.standard_normal(n) + 1j * rng.standard_normal(n), device="cuda")
    if generic:
        monkeypatch.setenv("HOM_NO_FAST", "1")
    monkeypatch.delenv("HOM_LONG_ROWS", raising=False)
    y = pb.apply(x, dual)
    monkeypatch.setenv("HOM_LONG_ROWS", "1")
    z = pb.apply(x, dual)
    assert bool(torch.isfinite(torch.view_as_real(y)).all()) and bool((torch.view_as_real(y) == torch.view_as_real(z)).all())
