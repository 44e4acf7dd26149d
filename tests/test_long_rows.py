"""The list of long rows that the multi-source gather step works from: the host
code that makes it, under sanitizers (CPU), and a graph with more rows above
4,096 in-neighbours than the workgroups hold slots for (GPU)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_05081_amd", "csrc")


def test_long_rows_under_sanitizer(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "long_rows_check")
    r = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-pthread", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-I", CSRC, os.path.join(ROOT, "tests", "sanitize", "long_rows_check.cpp"),
                        os.path.join(CSRC, "host_build.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and " 0 failures" in r.stdout, r.stdout[-4000:] + r.stderr[-4000:]


@pytest.mark.gpu
def test_more_wide_rows_than_slots():
    """64 slots a compute unit for rows cut into pieces; the rows past them go
    to a wave each. Every one of `pool` vertices has an arc to every hub, so a
    hub is at level 1 of each source and nothing else is reached."""
    import torch
    from paper_2606_05081_amd import blest
    slots = 64 * torch.cuda.get_device_properties(0).multi_processor_count
    pool, hubs = 4101, slots + 77
    n = pool + hubs
    rp = np.concatenate([np.arange(pool + 1, dtype=np.int64) * hubs, np.full(hubs, pool * hubs)]).astype(np.int32)
    col = np.tile(np.arange(pool, n, dtype=np.int32), pool)
    assert col.size == pool * hubs < 2 ** 31
    srcs = np.array([0, 1, pool - 1, 2000, 2000] + list(range(64, 128)) + [n - 1], np.int32)
    want = np.full((srcs.size, n), -1, np.int16)
    want[:-1, pool:] = 1
    want[np.arange(srcs.size), srcs] = 0
    with blest.Graph(rp, col, directed=1, reorder=0, msbfs_width=128) as g:
        for policy in (blest.Policy.HEURISTIC, blest.Policy.BOTTOM_UP):
            g.set_policy(policy)
            assert np.array_equal(g.msbfs(srcs).cpu().numpy(), want)
            s, r, _ = g.closeness(srcs)
            assert np.array_equal(s.cpu().numpy(), [hubs] * (srcs.size - 1) + [0])
            assert np.array_equal(r.cpu().numpy(), [hubs + 1] * (srcs.size - 1) + [1])
            far = np.zeros(n, np.int64)
            far[pool:] = srcs.size - 1
            assert np.array_equal(g.far(srcs).cpu().numpy(), far)
