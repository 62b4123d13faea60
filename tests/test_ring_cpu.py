"""The unit encoder's ring of round entries (csrc/gz_ring.h): a host model of a
workgroup whose scheduler lags and whose units are dropped (malformed incoming
superblocks) uses no entry of another round and never stalls."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("ring") / "ring_model")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I",
                    os.path.join(ROOT, "paper_2308_05199_amd", "csrc"),
                    os.path.join(ROOT, "tests", "ring_model.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("workers", [3, 11, 15])
@pytest.mark.parametrize("drop", [0, 90, 100])
@pytest.mark.parametrize("lag", [1, 40])
def test_entries_are_reused_after_the_scheduler(model, workers, drop, lag):
    for seed in range(8):
        r = subprocess.run([model, str(workers), "60", str(drop), str(lag), str(seed)],
                           capture_output=True, text=True, timeout=60)
        assert r.stdout.strip() == "ok", (workers, drop, lag, seed, r.stdout)
