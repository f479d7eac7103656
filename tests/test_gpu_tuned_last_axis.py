"""A measured table's choice (MIFFT_TUNE_TABLE) is what multidimensional plans
run along their last axis, also where it equals the built-in one."""
import os
import subprocess
import sys

import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("line,want,batch", [("c32 11 8 256 3", (8, 256, 3), 160),    # the built-in choice of plain plans
                                             ("c32 11 16 128 3", (16, 128, 3), 32),   # and of last axes in streams
                                             ("c32 11 8 256 2", (8, 256, 2), 160),
                                             ("", (16, 128, 3), 129), ("", (8, 256, 3), 128), ("", (8, 256, 2), 24)])
def test_table_reaches_last_axis(tmp_path, line, want, batch):
    need_gpu()
    table = tmp_path / "tune.txt"
    table.write_text(line + "\n")
    code = ("from paper_2203_09384_amd import api\n"
            f"d = api.PlanND((64, 2048), {batch}).describe()\n"
            "print('got', d['ept'], d['wg'], d['variant'])\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=dict(os.environ, MIFFT_TUNE_TABLE=str(table)),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    assert tuple(int(v) for v in r.stdout.split("got ")[1].split()) == want
