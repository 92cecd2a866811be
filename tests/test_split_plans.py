"""The split-K workspace is fixed when a surrogate's workspaces are made (a
captured step holds its address, and a call under capture cannot allocate), so
its bound must cover every plan (CPU only).

Builds tests/host/split_plans.cpp against the library's own plan.h and runs it
over the row counts of train steps and prediction passes of many nets.  A second
build sizes the workspace by the train step alone, which a prediction of more
rows than the batch must exceed.
"""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "host", "split_plans.cpp")


def run(tmp_path, *flags):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    exe = os.path.join(str(tmp_path), "plans")
    inc = os.path.join(ROOT, "paper_2309_16743_amd", "csrc")
    res = subprocess.run([gxx, "-std=c++17", "-O2", "-Wall", "-Werror", *flags, f"-I{inc}", SRC, "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return subprocess.run([exe], capture_output=True, text=True, timeout=300)


def test_split_workspace_covers_every_plan(tmp_path):
    res = run(tmp_path)
    assert res.returncode == 0 and res.stdout.endswith("ok\n"), res.stdout[-2000:]


def test_train_step_alone_does_not_bound_predictions(tmp_path):
    res = run(tmp_path, "-DTRAIN_ONLY")
    assert res.returncode == 1 and "of 6 64 64 256 ask for" in res.stdout, res.stdout[-2000:]
