"""What the host decides before a launch (bz_plan.hpp), on the CPU."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_29942_amd", "csrc")


def test_plans(tmp_path):
    exe = os.path.join(str(tmp_path), "plan_checks")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-DBZ_HD=inline", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "plan_checks.cpp"), "-o", exe],
                   check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert all(line.startswith("OK ") for line in out.stdout.splitlines()) and out.stdout


@pytest.mark.gpu
def test_new_lengths_allocate_nothing():
    """A plain call on a length that is new to the library, but whose field,
    rows and words per plane are not, takes no device memory."""
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    o = bz.bz_default_options()
    o.max_codewords = 100

    def call(n, k):
        G = np.zeros((k, n), dtype=np.uint8)
        G[:, :k] = np.eye(k, dtype=np.uint8)
        st, _ = bz.bz_min_distance_ex(3, torch.from_numpy(G).cuda(), o)
        assert st in (bz.OK, bz.ERR_LIMIT)

    for k in range(2, 42):
        call(k + 1, k)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for k in range(2, 42):
        for n in range(k + 2, k + 33):  # one word of processed columns
            call(n, k)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free
