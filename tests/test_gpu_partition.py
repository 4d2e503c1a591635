"""The passes of the permutation partition at the sizes where they change:
workgroups that share a tile (small partitions), the round-function tables
(from 2^23 elements; as many rounds at a time as their tables fit the LDS) and
the 64-bit walk (above 2^32)."""
import numpy as np
import pytest

import paper_2608_02391_amd as cp


def test_fp64_bucket_is_the_integer_quotient():
    """y (K / d) + 2^-36 truncated is floor(y K / d) for y < d <= 2^32 and
    K <= 256: checked next to every subspace boundary and at random."""
    rng = np.random.default_rng(5)
    ds = [1, 2, 255, 4095, 2304, (1 << 23) + 1, 4022468096, (1 << 32) - 1, 1 << 32]
    ds += [int(x) for x in rng.integers(256, 1 << 32, 40)]
    for d in ds:
        for K in {1, 2, 3, 7, 8, 16, 31, 64, 255, 256}:
            if K > d:
                continue
            edges = [-(-k * d // K) + o for k in range(K + 1) for o in (-1, 0, 1)]
            y = np.array([v for v in edges if 0 <= v < d] + [int(v) for v in rng.integers(0, d, 200)], dtype=np.uint64)
            got = np.trunc(y.astype(np.float64) * (float(K) / float(d)) + 2.0 ** -36).astype(np.uint64)
            assert np.array_equal(got, y * np.uint64(K) // np.uint64(d)), (d, K)


def _check(T, d, K, wide, shift=0):
    """The whole map against the element-wise permutation: every subspace's
    entries strictly ascending, each in its own bucket, at the exact offsets
    (so every element occurs once)."""
    seed = 1000 + K
    buf = T.full((d + shift,), -1, dtype=T.int64 if wide else T.int32, device="cuda")
    index = buf[shift:]
    ws = T.empty(cp.cpes_partition_workspace_bytes(cp.PART_PERMUTATION, d, K), dtype=T.uint8, device="cuda")
    st = T.full((1,), -7, dtype=T.int32, device="cuda")
    if wide:
        offs = cp.cpes_partition(cp.PART_PERMUTATION, d, K, seed, index=index, workspace=ws, status=st)
    else:
        offs = cp.cpes_partition32(d, K, seed, index, ws, status=st)
    assert offs == [-(-k * d // K) for k in range(K + 1)]
    del ws
    bucket = T.empty(d, dtype=T.uint8, device="cuda")
    step = 1 << 26
    part = T.empty(min(step, d), dtype=T.int32, device="cuda")
    for s in range(0, d, step):
        n = min(step, d - s)
        cp.cpes_debug_prp(seed, d, K, s, n, None, part)
        bucket[s:s + n] = part[:n]
    assert int(st.item()) == 0
    assert bool((buf[:shift] == -1).all())
    for k in range(K):
        for s in range(offs[k], offs[k + 1], step):
            e = min(offs[k + 1], s + step + 1)             # one entry of overlap
            idx = index[s:e].to(T.int64)
            if not wide:
                idx &= 0xFFFFFFFF
            assert bool((idx[1:] > idx[:-1]).all()) and int(idx[0]) >= 0 and int(idx[-1]) < d
            assert bool((bucket[idx] == k).all())


@pytest.mark.gpu
@pytest.mark.parametrize("d,K,wide,shift", [
    (2047, 5, True, 0), (2048, 8, False, 0), (2049, 9, True, 0), (511, 33, False, 0), ((1 << 20) + 3, 64, True, 0),
    ((1 << 23) - 1, 8, True, 0),                                                            # one tile per workgroup
    (1 << 23, 8, True, 0), ((1 << 23) + 1, 3, False, 1), ((1 << 24) + 1, 33, True, 1),     # all rounds' tables in LDS
    (1 << 26, 256, False, 3),                                                               # the last such size
    ((1 << 26) + 1, 8, True, 0), (1 << 28, 16, False, 0),                                   # h = 14: two rounds at a time
    ((1 << 28) + 1, 8, False, 0), (1 << 30, 8, False, 1),                                   # h = 15: one, in half of the LDS
    ((1 << 30) + 3, 7, False, 0), (1 << 32, 8, False, 0),                                   # h = 16: one, undoubled
])
def test_map_matches_the_permutation(d, K, wide, shift):
    import torch as T

    _check(T, d, K, wide, shift)
    if d >= 1 << 30:
        T.cuda.empty_cache()


@pytest.mark.gpu
def test_map_above_2_to_32():
    """Walks on more than 32 bits take the 64-bit kernel and the integer quotient."""
    import torch as T

    _check(T, (1 << 32) + 5, 8, True)
    T.cuda.empty_cache()
