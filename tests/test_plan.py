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


@pytest.mark.gpu
def test_many_small_codes():
    """More codes than compute units: every result is the kernel's without tables."""
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    rng = np.random.default_rng(61)
    codes = []
    for i in range(600):
        p = (3, 7)[i % 2]
        k = int(rng.integers(1, 33 if p == 3 else 13))
        codes.append((p, rng.integers(0, p, size=(k, int(rng.integers(k, k + 14))), dtype=np.uint8)))
    got = bz.min_distance_batch(codes, device="cuda:0")
    for (p, G), r in zip(codes, got):
        ref = bz.min_distance(p, G, pair_tables=-1)
        for key in ("status", "d", "m", "ranks", "stages", "codewords_total"):
            assert r[key] == ref[key], (p, G.shape, key, r[key], ref[key])


@pytest.mark.gpu
def test_server_memory():
    """A server's device memory is what the header says: the slots with their
    pair tables, and at most 3 MiB a slot for triples."""
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    bz.Server(slots=1, max_n=8).stop()  # the context's own memory
    for max_n, tables in ((48, 0.45e6), (64, 0.78e6), (128, 2.26e6)):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        server = bz.Server(max_n=max_n)
        used = free - torch.cuda.mem_get_info()[0]
        server.stop()
        slot = 28e3 + 4096 * max_n + 64 * max_n + tables + 3 * 2**20
        assert used <= 1024 * slot * 1.05 + 64e6, (max_n, used)


@pytest.mark.gpu
def test_server_without_room_for_triples():
    """Four codes that would take triples, and room for one at a time: the
    others run with pair tables, and every result is the plain call's."""
    import time

    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    codes = [np.random.default_rng([62, i]).integers(0, 7, size=(28, 56), dtype=np.uint8) for i in range(12)]
    server = bz.Server(slots=4, max_n=64)
    out = {}
    for tag, G in enumerate(codes):
        server.submit(7, G, tag)
    t0 = time.perf_counter()
    while len(out) < len(codes):
        out.update(server.poll())
        assert time.perf_counter() - t0 < 60
    server.stop()
    took = [bool(out[tag]["info"] & bz.INFO_TRIPLES) for tag in range(len(codes))]
    assert any(took) and not all(took)
    for tag, G in enumerate(codes):
        ref = bz.min_distance(7, G)
        for key in ("status", "d", "m", "ranks", "stages", "terminated_by", "codewords_total"):
            assert out[tag][key] == ref[key], (tag, key)
