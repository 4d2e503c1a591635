"""Host checks of bench.py: the multi-GPU refusal and the algorithmic bytes
per position it prices each kernel class with (the figures of the kernel
table in the design notes)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def test_more_than_one_gpu_is_refused():
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                         text=True, timeout=120)
    assert res.returncode == 2
    assert "one GPU only" in res.stderr and res.stdout == ""


@pytest.fixture(scope="module")
def bench():
    import bench as B
    return B


@pytest.mark.parametrize("name,op,expected", [
    ("c3", "restore", 4), ("c3", "update", 4), ("c3", "perturb", (6 + 29 * 4) / 30),
    ("c4", "restore", 12), ("c4", "perturb", 12 + 2 / 30), ("c4", "update", 12),
    ("c4u", "restore", 8), ("c4c", "restore", 4),
    ("c5", "perturb", 4), ("c5", "restore", 4), ("c5", "update", 10), ("c5", "stage_master", 6), ("c5", "backup", 4),
    ("c1", "restore", 8), ("c1", "perturb", (12 + 7 * 8) / 8),
    ("c3h", "perturb", 4), ("c3h", "backup_host", 2), ("c3h", "restore_host", 2),
])
def test_bytes_per_position(bench, name, op, expected):
    import synthetic as S
    assert bench.bytes_per_position(S.workload(name), op) == pytest.approx(expected)


@pytest.mark.parametrize("name", ["c1", "c2", "c5", "p0"])
def test_update_normals_counts_the_streams_that_are_generated(bench, name):
    """Normals of one step's updates: every member's own stream where none
    cancels (c1, p0), and without the mirrored pairs of equal rewards (c2, c5:
    a pair contributes only if its two rewards differ)."""
    import oracle as O
    import synthetic as S
    O.build(force=False)
    W = S.workload(name)
    iters = range(1 if W.copes_step else len(W.active))
    rnorm = [O.normalize(W.rewards(t), W.norm_mode)[0] for t in iters]
    if name == "p0":
        assert bench.update_normals(W, rnorm, W.sizes()) == 10 * W.d          # 40 members over 4 subspaces
        return
    want = 0
    for t, k in enumerate(W.active):
        r = W.rewards(t)
        streams = sum(a != b for a, b in zip(r[::2], r[1::2])) if name in ("c2", "c5") else W.n
        assert name == "c1" or 0 < streams < W.n // 2
        want += streams * W.sizes()[k]
    assert bench.update_normals(W, rnorm, W.sizes()) == want


def test_extras_default_to_the_other_benchmark_workloads(bench):
    assert bench.parse([]).extras == ["c1", "c2", "c4", "c5"]
    assert bench.parse(["--workload", "c4"]).extras == []
    assert bench.parse(["--no-extras"]).extras == []
    assert bench.parse(["--extras", "c1,c2"]).extras == ["c1", "c2"]


def test_counter_figures_are_keyed_to_the_kernel_sources(bench):
    sha = bench.sources_sha256()
    assert len(sha) == 64
    assert sha == bench.sources_sha256()          # a pure function of the sources
