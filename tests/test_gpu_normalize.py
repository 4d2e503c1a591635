"""Reward normalisation at the sizes where its kernels change: the waves of the
joint z-score (256 and 1,024 rewards), the 16 rewards per workgroup of the
ranks, groups of one and empty groups, and calls in place."""
import numpy as np
import pytest

import paper_2608_02391_amd as cp
import synthetic as S
from tests.gpu_helpers import to_dev, to_host, torch, zscore_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    t = torch()
    assert t.cuda.is_available(), "GPU tests need an MI355X"
    cp.load()
    return t


def _rewards(n, kind):
    g = np.random.default_rng(n)
    if kind == "signed":                                   # ties across the sign of zero, wide range
        r = (g.normal(size=n) * 10.0 ** g.integers(-30, 30, n)).astype(np.float32)
        r[::5] = 0.0
        r[1::7] = -0.0
        return r
    if kind == "constant":
        return np.full(n, np.float32(0.1))
    return (g.random((n, 8)) < 0.4).mean(axis=1).astype(np.float32)


def _check(orc, T, r, mode, group=None, n_groups=1):
    ref, rst = orc.normalize(r, mode, group)
    for in_place in (False, True):
        dr = to_dev(r)
        out = dr if in_place else T.full((len(r),), 7.0, dtype=T.float32, device="cuda")
        st = T.full((1,), -7, dtype=T.int32, device="cuda")
        cp.cpes_normalize_rewards(dr, out, mode, group=None if group is None else to_dev(group), n_groups=n_groups,
                                  status=st)
        T.cuda.synchronize()
        got = to_host(out)
        assert int(st.item()) == rst
        if mode == S.NORM_RANK or rst != 0:
            assert np.array_equal(got, ref)
        else:
            assert zscore_close(got, ref, r, group)


@pytest.mark.parametrize("n", [1, 2, 3, 15, 16, 17, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 4095, 4096])
@pytest.mark.parametrize("kind", ["signed", "constant", "mean"])
@pytest.mark.parametrize("mode", [S.NORM_Z, S.NORM_RANK])
def test_joint(orc, T, n, kind, mode):
    _check(orc, T, _rewards(n, kind), mode)


@pytest.mark.parametrize("n,K", [(1, 1), (3, 3), (64, 5), (257, 1), (1000, 1000), (1025, 31), (4096, 1024)])
@pytest.mark.parametrize("kind", ["signed", "mean"])
@pytest.mark.parametrize("mode", [S.NORM_Z, S.NORM_RANK])
def test_groups(orc, T, n, K, kind, mode):
    """Random group sizes: some groups empty, some of one reward."""
    g = np.random.default_rng(n + K).integers(0, K, n).astype(np.int32)
    _check(orc, T, _rewards(n, kind), mode, g, K)


@pytest.mark.parametrize("n", [1, 17, 257, 4096])
@pytest.mark.parametrize("mode", [S.NORM_Z, S.NORM_RANK])
def test_failures(orc, T, n, mode):
    """A non-finite last reward or a bad last group id: zeros and a status."""
    r = _rewards(n, "mean")
    r[-1] = np.inf
    g = (np.arange(n) % 2).astype(np.int32) if n > 1 else np.zeros(1, np.int32)
    K = 2 if n > 1 else 1
    bad = g.copy()
    bad[-1] = -1
    for in_place in (False, True):
        for group, expect in ((None, 1), (g, 1), (bad, 2)):
            dr = to_dev(r)
            out = dr if in_place else T.full((n,), 7.0, dtype=T.float32, device="cuda")
            st = T.full((1,), -7, dtype=T.int32, device="cuda")
            cp.cpes_normalize_rewards(dr, out, mode, group=None if group is None else to_dev(group),
                                      n_groups=1 if group is None else K, status=st)
            T.cuda.synchronize()
            assert int(st.item()) == expect and not to_host(out).any()
