"""The branches of the noise and copy kernels that neither length nor layout
selects: streams whose coefficient is zero, noise blocks above 2^32, and
ranges and side buffers, on the device or the host, that start at no vector
boundary."""
import numpy as np
import pytest

import paper_2608_02391_amd as cp
import synthetic as S
from tests.gpu_helpers import describe_mismatch, f32_close, to_dev, to_host, torch, ulp_bf16, ulp_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    t = torch()
    assert t.cuda.is_available(), "GPU tests need an MI355X"
    cp.load()
    return t


def _members(n, zero):
    """n members with rewards, those in `zero` with a coefficient of exactly
    zero: a reward of 0 or -0, or a mirrored pair with equal rewards."""
    rng = np.random.default_rng(n)
    seeds, signs, r = list(range(50, 50 + n)), [1] * n, rng.normal(size=n).astype(np.float32)
    for i in zero:
        r[i] = -0.0 if i % 2 else 0.0
    if n >= 6:                                            # members 2 and 3 cancel
        seeds[3], signs[3] = seeds[2], -1
        r[3] = r[2]
    return seeds, signs, r


@pytest.mark.parametrize("n,zero", [
    (1, []), (1, [0]), (5, [0, 4]), (6, [0, 5]), (64, [0, 62, 63]), (65, [64]), (66, list(range(66))),
    (130, list(range(60, 70)) + [127, 128, 129]), (256, list(range(0, 256, 3)) + [63, 64, 191, 192, 255])])
@pytest.mark.parametrize("kind", ["contiguous", "map"])
def test_streams_with_zero_coefficients(orc, T, n, zero, kind):
    """An update whose members partly cancel equals the oracle's; one whose
    members all do leaves the weights' bits alone."""
    length = 2 * 512 + 77
    w = S.host_weights(4 * length, S.F32, n)
    index = np.sort(np.random.default_rng(1).permutation(4 * length)[:length]).astype(np.int64) if kind == "map" else None
    dmap = to_dev(index) if kind == "map" else None
    seeds, signs, r = _members(n, zero)
    dw = to_dev(w)
    sub = cp.subspace(0 if kind == "map" else 5, length, dmap)
    cp.cpes_update(dw, sub, seeds, signs, to_dev(r), 0.01, 1.0, cp.SCALE_ALPHA_OVER_N)
    ref = w.copy()
    orc.update(ref, 0 if kind == "map" else 5, length, seeds, signs, r, np.float32(0.01), np.float32(1.0),
               S.SCALE_ALPHA_OVER_N, index=index)
    T.cuda.synchronize()
    got = to_host(dw)
    # the bar of updated fp32 weights
    assert f32_close(got, ref), describe_mismatch(got, ref)
    if len(zero) == n:
        assert np.array_equal(got, w)


def test_step_ranges_cross_the_words_of_the_stream_bits(orc, T):
    """The whole-step update: subspaces whose streams begin inside a 64-bit
    word, end at one, or are all zero, one without members."""
    counts = [63, 2, 0, 64, 65, 1, 61]                    # 256 members
    K, n = len(counts), sum(counts)
    ks = np.repeat(np.arange(K), counts)
    rng = np.random.default_rng(3)
    r = rng.normal(size=n).astype(np.float32)
    r[rng.permutation(n)[:120]] = 0.0
    r[ks == 5] = 0.0                                       # a subspace none of whose streams contributes
    order = rng.permutation(n)
    ks, r = ks[order], r[order]
    seeds, signs = list(range(900, 900 + n)), [1 - 2 * (i % 2) for i in range(n)]
    bounds = [0, 1000, 1777, 2000, 4099, 5000, 6001, 7003]
    w = S.host_weights(7003, S.F32, 8)
    sigmas = [1.0] * K
    dw = to_dev(w)
    cp.cpes_update_step(dw, bounds, seeds, signs, ks.tolist(), to_dev(r), 0.01, sigmas, cp.SCALE_ALPHA_OVER_N)
    ref = w.copy()
    orc.update_step(ref, bounds, seeds, signs, ks, r, np.float32(0.01), sigmas, S.SCALE_ALPHA_OVER_N)
    T.cuda.synchronize()
    got = to_host(dw)
    assert f32_close(got, ref), describe_mismatch(got, ref)
    assert np.array_equal(got[5000:6001], w[5000:6001]) and np.array_equal(got[1777:2000], w[1777:2000])


@pytest.mark.parametrize("noise0", [(1 << 34) - 4096, (1 << 34) - 1024, 1 << 34, (1 << 36) + 8])
@pytest.mark.parametrize("dtype", [S.BF16, S.F32])
@pytest.mark.parametrize("layout", ["contiguous", "map", "map_ascending"])
def test_noise_blocks_around_2_to_32(orc, T, noise0, dtype, layout):
    """A shard whose noise blocks lie below, across or above 2^32 (the kernels
    for short blocks end there)."""
    length = 4096
    w = S.host_weights(2 * length, dtype, 4)
    index = np.arange(0, 2 * length, 2, dtype=np.int64) if layout != "contiguous" else None
    sub = cp.subspace(0, length, None if index is None else to_dev(index), noise_offset=noise0,
                      ascending=layout == "map_ascending")
    dw, ref = to_dev(w), w.copy()
    cp.cpes_perturb(dw, sub, 0.25, 77, -1)
    orc.perturb(ref, 0, length, np.float32(0.25), 77, -1, index=index, j0=noise0)
    T.cuda.synchronize()
    got = to_host(dw)
    assert (ulp_bf16(got, ref) if dtype == S.BF16 else ulp_f32(got, ref)).max() <= 1      # the bar of perturbations
    if dtype == S.F32:
        r = np.array([0.5, -1.25, 0.0], dtype=np.float32)
        dw, ref = to_dev(w), w.copy()
        cp.cpes_update(dw, sub, [1, 2, 3], [1, -1, 1], to_dev(r), 0.01, 1.0, cp.SCALE_ALPHA_OVER_N)
        orc.update(ref, 0, length, [1, 2, 3], [1, -1, 1], r, np.float32(0.01), np.float32(1.0), S.SCALE_ALPHA_OVER_N,
                   index=index, j0=noise0)
        T.cuda.synchronize()
        assert f32_close(to_host(dw), ref)


@pytest.mark.parametrize("length", [1, 7, 8, 9, 2047, 2048, 2049, 70001])
@pytest.mark.parametrize("dtype", [S.BF16, S.F32])
@pytest.mark.parametrize("layout", ["contiguous", "chunk", "map", "ascending", "ascending32"])
def test_any_element_alignment(orc, T, length, dtype, layout):
    """Weights, backup and master each at their own element offset from a
    vector boundary: the same bits as from aligned copies.  Through ascending
    maps (one entry in four: whole-line windows) the map starts at an odd
    entry too."""
    C = 256
    numel = 4 * length + 8 * C
    base = S.host_weights(numel + 8, dtype, length)
    if layout == "contiguous":
        make = lambda off: cp.subspace(off, length)
    elif layout == "chunk":
        chunks = to_dev(np.random.default_rng(2).permutation(numel // C)[:length // C + 1].astype(np.int64))
        make = lambda off: cp.subspace(0, length, chunks, C)
    else:
        index = np.sort(np.random.default_rng(2).permutation(numel)[:length + 3])
        index = to_dev(index.astype(np.int32 if layout == "ascending32" else np.int64))
        make = lambda off: cp.subspace(3, length, index, ascending=layout != "map")
    tdt = T.bfloat16 if dtype == S.BF16 else T.float32
    r = to_dev(np.array([0.5, -1.0], dtype=np.float32))

    def passes(shift, side):
        """Weights `shift` elements past a vector boundary, side buffers `side`."""
        buf = T.zeros(numel + 16, dtype=tdt, device="cuda")
        w = buf[shift:shift + numel]
        w.copy_(to_dev(base)[:numel])
        sub = make(16)
        bak = T.zeros(length + 8, dtype=tdt, device="cuda")[side:side + length]
        out = []
        cp.cpes_perturb(w, sub, 0.5, 3, 1, aux=bak, aux_mode=cp.AUX_SNAPSHOT)
        out += [w.clone(), bak.clone()]
        cp.cpes_perturb(w, sub, 0.5, 4, 1)
        cp.cpes_perturb(w, sub, 0.25, 5, -1, aux=bak, aux_mode=cp.AUX_BACKUP)
        out.append(w.clone())
        cp.cpes_restore(w, sub, aux=bak)
        out.append(w.clone())
        cp.cpes_backup(w, sub, bak)
        master = T.zeros(length + 8, dtype=T.float32, device="cuda")[side:side + length]
        cp.cpes_stage_master(w, sub, master)
        cp.cpes_update(w, sub, [8, 9], [1, 1], r, 0.01, 1.0, master=master if dtype == S.BF16 else None)
        out += [w.clone(), bak.clone(), master.clone()]
        if dtype == S.BF16:
            cp.cpes_perturb(w, sub, 0.5, 6, 1, aux=master, aux_mode=cp.AUX_MASTER)
            out.append(w.clone())
            cp.cpes_restore(w, sub, aux=master, aux_mode=cp.AUX_MASTER)
        cp.cpes_update_step(w, [16, 16 + min(length, 77), 16 + length], [8, 9], [1, 1], [0, 1], r, 0.01, [1.0, 1.0])
        out.append(w.clone())
        assert not bool(buf[:shift].any()) and not bool(buf[shift + numel:].any())        # nothing outside
        return out

    want = passes(0, 0)
    assert not bool(T.equal(want[0], want[3]))
    for shift, side in ((1, 0), (0, 1), (3, 5), (7, 2)):
        for a, b in zip(want, passes(shift, side)):
            assert T.equal(a, b)


@pytest.mark.parametrize("length", [1, 9, 2049, 70001])
@pytest.mark.parametrize("dtype", [S.BF16, S.F32])
@pytest.mark.parametrize("layout", ["contiguous", "chunk", "map", "ascending", "ascending32"])
def test_host_backup_at_any_element(orc, T, length, dtype, layout):
    """Backup to pinned host memory and restore from it with the weights and
    the host buffer each at their own element offset from a vector boundary:
    the host holds the bits that the subspace had, a restore brings them back,
    and nothing around either range is written."""
    C = 256
    numel = 4 * length + 8 * C
    base = S.host_weights(numel, dtype, length)
    rng = np.random.default_rng(4)
    if layout == "contiguous":
        at, sub = np.arange(5, 5 + length), cp.subspace(5, length)
    elif layout == "chunk":
        chunks = rng.permutation(numel // C)[:length // C + 1].astype(np.int64)
        at = (chunks[:, None] * C + np.arange(C)).reshape(-1)[:length]
        sub = cp.subspace(0, length, to_dev(chunks), C)
    else:
        index = np.sort(rng.permutation(numel)[:length + 3])
        at = index[3:]
        sub = cp.subspace(3, length, to_dev(index.astype(np.int32 if layout == "ascending32" else np.int64)),
                          ascending=layout != "map")
    tdt = T.bfloat16 if dtype == S.BF16 else T.float32
    w0 = to_dev(base)
    for shift, side in ((0, 0), (1, 0), (0, 1), (3, 5), (7, 2)):
        buf = T.zeros(numel + 16, dtype=tdt, device="cuda")
        w = buf[shift:shift + numel]
        w.copy_(w0)
        host = T.full((length + 16,), 7, dtype=tdt, pin_memory=True)
        hb = host[side:side + length]
        cp.cpes_backup_to_host(w, sub, hb)
        T.cuda.synchronize()
        assert np.array_equal(to_host(hb), base[at])
        assert bool((host[:side] == 7).all()) and bool((host[side + length:] == 7).all())
        cp.cpes_perturb(w, sub, 0.5, 3, 1)
        assert not bool(T.equal(w, w0))
        cp.cpes_restore_from_host(w, sub, hb)
        T.cuda.synchronize()
        assert bool(T.equal(w, w0))
        assert not bool(buf[:shift].any()) and not bool(buf[shift + numel:].any())


@pytest.mark.parametrize("kind", ["contiguous", "map", "step"])
@pytest.mark.parametrize("dtype,n", [(S.F32, 1), (S.F32, 256), (S.BF16, 256)])
def test_update_sums_in_64_bits(orc, T, kind, dtype, n):
    """From zero weights with a step of 1 the update is the noise sum rounded
    once (twice for bf16): the oracle's 64-bit factors give it, to one rounding
    to fp32 and the 2^-44 of the device's factors.  A sum of 256 terms in fp32
    is some ten roundings off."""
    length = 4 * 515 + 3
    seeds, c = [900 + u for u in range(n)], np.random.default_rng(n).normal(size=n).astype(np.float32)
    want, size = np.zeros(length), np.zeros(length)
    for seed, cu in zip(seeds, c):
        x = orc.blocks(seed, 0, 0, (length + 3) // 4).reshape(-1, 2)
        rho, (co, si) = orc.bm_radius_many(x[:, 0]), orc.bm_angle_many(x[:, 1])
        z = np.stack([rho * co, rho * si], axis=1).reshape(-1)[:length]
        want += float(cu) * z
        size += abs(float(cu)) * np.abs(z)
    w = T.zeros(4 * length, dtype=T.bfloat16 if dtype == S.BF16 else T.float32, device="cuda")
    at = np.arange(length)
    if kind == "map":
        at = np.sort(np.random.default_rng(3).permutation(4 * length)[:length]).astype(np.int64)
    if kind == "step":
        cp.cpes_update_step(w, [0, length], seeds, [1] * n, [0] * n, to_dev(c), float(n), [1.0], cp.SCALE_ALPHA_OVER_N)
    else:
        sub = cp.subspace(0, length, to_dev(at) if kind == "map" else None)
        cp.cpes_update(w, sub, seeds, [1] * n, to_dev(c), float(n), 1.0, cp.SCALE_ALPHA_OVER_N)
    got = w.double().cpu().numpy()
    rounding = 2.0 ** -24 if dtype == S.F32 else 2.0 ** -8 * 1.01
    assert np.all(np.abs(got[at] - want) <= rounding * np.abs(want) + 2.0 ** -44 * size)
    rest = np.ones(4 * length, dtype=bool)
    rest[at] = False
    assert not got[rest].any()
