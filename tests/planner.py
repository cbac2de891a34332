"""The library's planner (csrc/lopt_plan.h) on the CPU: which tiles, blocks and workspace a tensor list gets."""
from __future__ import annotations

import atexit
import functools
import json
import os
import shutil
import subprocess
import tempfile

from paper_2506_10315_amd.binding import flatten_shape

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
N_CU = 256   # compute units of an MI355X


@functools.lru_cache(maxsize=None)
def _probe():
    where = tempfile.mkdtemp(prefix="lopt_planner_")
    atexit.register(shutil.rmtree, where, ignore_errors=True)
    out = os.path.join(where, "probe")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2506_10315_amd", "csrc"),
                    os.path.join(ROOT, "tests", "planner_probe.cpp"), "-o", out], check=True, capture_output=True, text=True)
    return out


def plan(shapes, kind="small_fc_lopt", hidden=None, lstm_hidden=512, n_bank=256, groups=0):
    """The plan of a list of shapes with the default apply kernels."""
    h = hidden if hidden is not None else 32 if kind == "small_fc_lopt" else 4
    hp = next(x for x in (4, 8, 16, 32) if h <= x)
    p = 29 * h + h + h * h + h + 2 * h + 2
    folded = n_bank >= 4 and lstm_hidden * p <= lstm_hidden * n_bank + n_bank * p
    args = [int(kind == "velo"), hp, p, lstm_hidden, n_bank, int(folded), groups, N_CU,
            0 if kind == "velo" else 1 if hp == 32 else 2]
    r = subprocess.run([_probe(), *map(str, args)], input="\n".join("%d %d" % flatten_shape(s)[1:] for s in shapes), capture_output=True,
                       text=True, check=True)
    return json.loads(r.stdout)
