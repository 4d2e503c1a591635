"""Performance cases of the CoPES parameter-space path, each through the public
entry points of ``paper_2608_02391_amd`` as a training program calls them.

A case is one of six kinds of work:

* ``step``      one whole ES step on one contiguous subspace of a small model:
                every member perturbed and restored, the rewards normalised,
                the update;
* ``member``    the loop body of a member: the previous member's perturbation
                is undone from the backup (or the fp32 master), then this
                member's is applied; the perturbed model is what comes back;
* ``update``    the end of a generation: the last member is undone, the master
                staged if there is one, the rewards normalised, the update;
* ``paper``     one CoPES step as the paper runs it: chunk partition replayed
                from its seed, N / K members per subspace, joint
                standardisation, one composed update;
* ``partition`` an element-level random partition replayed from its seed;
* ``rewards``   the standardisation of a large population's rewards.

``listed()`` has the named ones, ``draw()`` spreads over the sizes, layouts
(contiguous, chunk lists, int64 and uint32 element maps), weight types, sources
and normalisations of the same kinds.  ``exact()`` evaluates a case in 64 bits
with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_02391_amd as cp

SIGMA, ALPHA, INIT_STD = 1e-3, 5e-4, 0.02
LAYER = 100930816                       # parameters of one decoder layer (hidden 2560, intermediate 9728, 32 / 8 heads)
MASK = 0xFFFFFFFF


def listed():
    return [
        # the smallest configuration: an fp32 vector of 2^20 in 4 subspaces, one of them active, 8 members;
        # a step of about twenty small calls, so launches and latency count
        dict(name="tiny_step", kind="step", d=1 << 20, K=4, active=0, dtype="fp32", n=8, mirrored=False,
             rewards="uniform", norm="z"),
        # one member on one sixteenth of 12 transformer layers (hidden 1024): a subspace of 9.4 M bf16 weights
        dict(name="layer_member", kind="member", d=150994944, K=16, active=3, dtype="bf16", layout="contiguous",
             chunk=0, source="in_place"),
        # the end of that configuration's generation: 16 mirrored pairs, success / failure rewards, centred ranks
        dict(name="layer_update", kind="update", d=150994944, K=16, active=3, dtype="bf16", layout="contiguous",
             chunk=0, master=False, n=32, mirrored=True, rewards="bernoulli", norm="rank"),
        # one member on a group of 5 decoder layers of a 4 G model: 504,654,080 bf16 weights
        dict(name="group_member", kind="member", d=10 * LAYER, K=2, active=1, dtype="bf16", layout="contiguous",
             chunk=0, source="in_place"),
        # the update of such a group from 30 members: the largest call
        dict(name="group_update", kind="update", d=10 * LAYER, K=2, active=1, dtype="bf16", layout="contiguous",
             chunk=0, master=False, n=30, mirrored=False, rewards="uniform", norm="z"),
        # one member on one of 8 element-permuted subspaces, through an int64 map
        dict(name="map_member", kind="member", d=10 * LAYER, K=8, active=2, dtype="bf16", layout="map64", chunk=0,
             source="backup"),
        # the update of such a subspace through a uint32 map
        dict(name="map32_update", kind="update", d=10 * LAYER, K=8, active=2, dtype="bf16", layout="map32", chunk=0,
             master=False, n=30, mirrored=False, rewards="uniform", norm="z"),
        # a subspace of 251 M with an fp32 master, 64 mirrored pairs, rewards averaged over 8 rollouts
        dict(name="master_update", kind="update", d=1005617024, K=4, active=1, dtype="bf16", layout="contiguous",
             chunk=0, master=True, n=128, mirrored=True, rewards="mean", norm="z"),
        # the paper's settings (K = 4, N = 40, chunks of 65,536) on the 151 M model: a whole call sequence
        dict(name="paper_step", kind="paper", d=150994944, K=4, dtype="bf16", chunk=65536, n=40),
        # the element-level partition of ten layers, resampled every step from its seed
        dict(name="permutation", kind="partition", d=10 * LAYER, K=8, map="int64"),
        # one member on a third of an odd-sized model: ranges that start at no aligned address
        dict(name="ragged_member", kind="member", d=100000007, K=3, active=1, dtype="bf16", layout="contiguous",
             chunk=0, source="in_place"),
        # the largest population one call standardises
        dict(name="rewards", kind="rewards", n=4096, groups=0, rewards="mean", norm="z"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "member", "member", "member", "update", "update", "paper", "partition", "rewards"])
    rew, norm = rng.choice(["uniform", "bernoulli", "mean"]), rng.choice(["z", "z", "rank"])
    if kind == "rewards":
        n = _log_int(rng, 3, 4096)
        return dict(kind=kind, n=n, groups=rng.choice([0, 0, min(n, rng.randint(2, 64))]), rewards=rew, norm=norm)
    if kind == "partition":
        d = _log_int(rng, 1 << 16, 1 << 28) | rng.randint(0, 1)
        return dict(kind=kind, d=d, K=rng.choice([2, 4, 8, 8, 16, rng.randint(2, 64)]), map=rng.choice(["int64", "int32"]))
    if kind == "paper":
        K = rng.choice([2, 4, 8])
        return dict(kind=kind, d=_log_int(rng, 1 << 21, 1 << 27) | rng.randint(0, 1), K=K, dtype="bf16",
                    chunk=1 << rng.randint(12, 16), n=K * rng.randint(2, 10))
    K = rng.choice([1, 2, 4, 8, 8, 16, rng.randint(3, 12)])
    active = rng.randint(0, K - 1)
    dtype = rng.choice(["bf16", "bf16", "fp32"])
    mirrored = rng.random() < 0.5
    if kind == "step":
        return dict(kind=kind, d=_log_int(rng, 1 << 16, 1 << 24) | rng.randint(0, 1), K=K, active=active, dtype=dtype,
                    n=2 * rng.randint(2, 16), mirrored=mirrored, rewards=rew, norm=norm)
    layout = rng.choice(["contiguous", "contiguous", "chunk", "map64", "map32"])
    if layout != "contiguous" and K == 1:
        K = 4
        active = rng.randint(0, 3)
    chunk = 1 << rng.randint(10, 16) if layout == "chunk" else 0
    if kind == "member":
        d = _log_int(rng, 1 << 20, 1 << (29 if layout in ("contiguous", "chunk") else 28)) | rng.randint(0, 1)
        source = rng.choice(["in_place", "backup", "master"] if dtype == "bf16" else ["in_place", "backup"])
        return dict(kind=kind, d=d, K=K, active=active, dtype=dtype, layout=layout, chunk=chunk, source=source)
    n = 2 * rng.randint(2, 64)
    d = min(_log_int(rng, 1 << 20, 1 << 28), K * 10000000000 // n) | rng.randint(0, 1)
    return dict(kind=kind, d=d, K=K, active=active, dtype=dtype, layout=layout, chunk=chunk,
                master=dtype == "bf16" and rng.random() < 0.3, n=n, mirrored=mirrored, rewards=rew, norm=norm)


# ------------------------------------------------------------------- inputs --

def _dtype(case):
    return torch.float32 if case["dtype"] == "fp32" else torch.bfloat16


def _weights(case, seed):
    """N(0, 0.02^2) weights of the whole model."""
    d, dt = case["d"], _dtype(case)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    w = torch.empty(d, dtype=dt, device="cuda")
    for s in range(0, d, 1 << 28):
        e = min(d, s + (1 << 28))
        w[s:e] = torch.randn(e - s, generator=g, device="cuda").mul_(INIT_STD)
    return w


def _rewards(case, seed):
    g = np.random.default_rng(seed)
    n, kind = case["n"], case["rewards"]
    if kind == "uniform":
        r = g.random(n, dtype=np.float32)
    elif kind == "bernoulli":
        r = (g.random(n) < 0.4).astype(np.float32)
    else:
        r = (g.random((n, 8)) < 0.4).mean(axis=1).astype(np.float32)
    return torch.from_numpy(r).cuda()


def _members(case, seed):
    """(seeds, signs) of the generation's members."""
    base, n = 1000 * (seed % (1 << 40)), case["n"]
    if case.get("mirrored"):
        return [base + i // 2 + 1 for i in range(n)], [1 - 2 * (i % 2) for i in range(n)]
    return [base + i + 1 for i in range(n)], [1] * n


def _sigma(d, length):
    """sigma_k = sigma sqrt(d / d_k)."""
    return float(np.float32(SIGMA * math.sqrt(d / length)))


def _norm(case):
    return cp.NORM_RANK if case["norm"] == "rank" else cp.NORM_Z


def _partition_seed(seed):
    return 33 + seed


def _element_map(d, K, seed, wide):
    index = torch.empty(d, dtype=torch.int64 if wide else torch.int32, device="cuda")
    ws = torch.empty(cp.cpes_partition_workspace_bytes(cp.PART_PERMUTATION, d, K), dtype=torch.uint8, device="cuda")
    if wide:
        return cp.cpes_partition(cp.PART_PERMUTATION, d, K, seed, index=index, workspace=ws), index
    return cp.cpes_partition32(d, K, seed, index, ws), index


def _subspace(case, seed):
    """The active subspace as a program holds it: its descriptor and length."""
    d, K, k, layout = case["d"], case["K"], case["active"], case.get("layout", "contiguous")
    if layout == "contiguous":
        offs = cp.cpes_partition(cp.PART_CONTIGUOUS, d, K)
        return cp.subspace(offs[k], offs[k + 1] - offs[k]), offs[k + 1] - offs[k]
    if layout == "chunk":
        C = case["chunk"]
        chunks = torch.empty(-(-d // C), dtype=torch.int64, device="cuda")
        ws = torch.empty(cp.cpes_partition_chunks_workspace_bytes(d, C, K), dtype=torch.uint8, device="cuda")
        offs, lens = cp.cpes_partition_chunks(d, C, K, _partition_seed(seed), chunks, ws)
        return cp.subspace(offs[k], lens[k], chunks, C), lens[k]
    offs, index = _element_map(d, K, _partition_seed(seed), layout == "map64")
    return cp.subspace(offs[k], offs[k + 1] - offs[k], index, ascending=True), offs[k + 1] - offs[k]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "rewards":
        r = _rewards(case, seed)
        group = None
        if case["groups"]:
            g = np.random.default_rng(seed + 1).permutation(np.arange(case["n"]) % case["groups"]).astype(np.int32)
            group = torch.from_numpy(g).cuda()
        return dict(case=case, r=r, group=group, out=torch.empty_like(r),
                    status=torch.empty(1, dtype=torch.int32, device="cuda"))
    if kind == "partition":
        d, K = case["d"], case["K"]
        nbytes = cp.cpes_partition_workspace_bytes(cp.PART_PERMUTATION, d, K)
        return dict(case=case, seed=_partition_seed(seed),
                    index=torch.empty(d, dtype=getattr(torch, case["map"]), device="cuda"),
                    ws=torch.empty(nbytes, dtype=torch.uint8, device="cuda"),
                    status=torch.empty(1, dtype=torch.int32, device="cuda"))
    w, dt = _weights(case, seed), _dtype(case)
    if kind == "paper":
        d, C, K = case["d"], case["chunk"], case["K"]
        r = _rewards(dict(n=case["n"], rewards="uniform"), seed)
        seeds, signs = _members(case, seed)
        nbytes = cp.cpes_partition_chunks_workspace_bytes(d, C, K)
        return dict(case=case, w=w, r=r, rnorm=torch.empty_like(r), seeds=seeds, signs=signs,
                    partition_seed=_partition_seed(seed),
                    chunks=torch.empty(-(-d // C), dtype=torch.int64, device="cuda"),
                    ws=torch.empty(nbytes, dtype=torch.uint8, device="cuda"),
                    backup=torch.empty(-(-d // K) + 2 * C, dtype=dt, device="cuda"))
    if kind == "step":
        length = -(-case["d"] // case["K"])
        r = _rewards(case, seed)
        seeds, signs = _members(case, seed)
        return dict(case=case, w=w, r=r, rnorm=torch.empty_like(r), seeds=seeds, signs=signs,
                    backup=torch.empty(length, dtype=dt, device="cuda"))
    sub, length = _subspace(case, seed)
    sigma = _sigma(case["d"], length)
    state = dict(case=case, w=w, sub=sub, sigma=sigma)
    previous = 1000 * (seed % (1 << 40)) + 900
    if kind == "member" and case["source"] == "master":
        state["master"] = torch.empty(length, dtype=torch.float32, device="cuda")
        cp.cpes_stage_master(w, sub, state["master"])
        cp.cpes_perturb(w, sub, sigma, previous, 1, aux=state["master"], aux_mode=cp.AUX_MASTER)
    else:
        state["backup"] = torch.empty(length, dtype=dt, device="cuda")
        cp.cpes_perturb(w, sub, sigma, previous, 1, aux=state["backup"], aux_mode=cp.AUX_SNAPSHOT)
    if kind == "member":
        state.update(seed=previous + 1, sign=1 - 2 * (seed & 1))
        return state
    r = _rewards(case, seed)
    seeds, signs = _members(case, seed)
    state.update(r=r, rnorm=torch.empty_like(r), seeds=seeds, signs=signs)
    if case["master"]:
        state["master"] = torch.empty(length, dtype=torch.float32, device="cuda")
    return state


# ---------------------------------------------------------------- one pass --

def _run_member(st):
    w, sub, source = st["w"], st["sub"], st["case"]["source"]
    if source == "master":
        cp.cpes_restore(w, sub, aux=st["master"], aux_mode=cp.AUX_MASTER)
        cp.cpes_perturb(w, sub, st["sigma"], st["seed"], st["sign"], aux=st["master"], aux_mode=cp.AUX_MASTER)
        return {"w": w}
    cp.cpes_restore(w, sub, aux=st["backup"], aux_mode=cp.AUX_SNAPSHOT)
    if source == "backup":
        cp.cpes_perturb(w, sub, st["sigma"], st["seed"], st["sign"], aux=st["backup"], aux_mode=cp.AUX_BACKUP)
    else:
        cp.cpes_perturb(w, sub, st["sigma"], st["seed"], st["sign"])
    return {"w": w}


def _run_update(st):
    w, sub, master = st["w"], st["sub"], st.get("master")
    cp.cpes_restore(w, sub, aux=st["backup"], aux_mode=cp.AUX_SNAPSHOT)
    if master is not None:
        cp.cpes_stage_master(w, sub, master)
    cp.cpes_normalize_rewards(st["r"], st["rnorm"], _norm(st["case"]))
    cp.cpes_update(w, sub, st["seeds"], st["signs"], st["rnorm"], ALPHA, st["sigma"], master=master)
    return {"w": w, "rnorm": st["rnorm"]} if master is None else {"w": w, "rnorm": st["rnorm"], "master": master}


def _members_pass(w, sub, sigma, seeds, signs, backup):
    for m, (seed, sign) in enumerate(zip(seeds, signs)):
        cp.cpes_perturb(w, sub, sigma, seed, sign, aux=backup if m == 0 else None,
                        aux_mode=cp.AUX_SNAPSHOT if m == 0 else cp.AUX_NONE)
        # the perturbed model would be evaluated here
        cp.cpes_restore(w, sub, aux=backup, aux_mode=cp.AUX_SNAPSHOT)


def _run_step(st):
    case, w = st["case"], st["w"]
    k, offs = case["active"], cp.cpes_partition(cp.PART_CONTIGUOUS, case["d"], case["K"])
    length = offs[k + 1] - offs[k]
    sub, sigma = cp.subspace(offs[k], length), _sigma(case["d"], length)
    _members_pass(w, sub, sigma, st["seeds"], st["signs"], st["backup"])
    cp.cpes_normalize_rewards(st["r"], st["rnorm"], _norm(case))
    cp.cpes_update(w, sub, st["seeds"], st["signs"], st["rnorm"], ALPHA, sigma)
    return {"w": w, "rnorm": st["rnorm"], "backup": st["backup"][:length]}


def _run_paper(st):
    case, w = st["case"], st["w"]
    d, K, C, n = case["d"], case["K"], case["chunk"], case["n"]
    offs, lens = cp.cpes_partition_chunks(d, C, K, st["partition_seed"], st["chunks"], st["ws"])
    per = n // K
    sigmas = [_sigma(d, length) for length in lens]
    for k in range(K):
        sub = cp.subspace(offs[k], lens[k], st["chunks"], C)
        _members_pass(w, sub, sigmas[k], st["seeds"][k * per:(k + 1) * per], st["signs"][k * per:(k + 1) * per],
                      st["backup"])
    cp.cpes_normalize_rewards(st["r"], st["rnorm"], cp.NORM_Z)
    cp.cpes_update_step(w, offs, st["seeds"], st["signs"], [i // per for i in range(n)], st["rnorm"], ALPHA, sigmas,
                        cp.SCALE_ALPHA_OVER_N, index=st["chunks"], chunk=C, lengths=lens)
    return {"w": w, "rnorm": st["rnorm"], "chunks": st["chunks"]}


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "member":
        return _run_member(st)
    if kind == "update":
        return _run_update(st)
    if kind == "step":
        return _run_step(st)
    if kind == "paper":
        return _run_paper(st)
    if kind == "partition":
        if case["map"] == "int64":
            offs = cp.cpes_partition(cp.PART_PERMUTATION, case["d"], case["K"], st["seed"], index=st["index"],
                                     workspace=st["ws"], status=st["status"])
        else:
            offs = cp.cpes_partition32(case["d"], case["K"], st["seed"], st["index"], st["ws"], status=st["status"])
        return {"index": st["index"], "status": st["status"], "offsets": np.array(offs, dtype=np.int64)}
    cp.cpes_normalize_rewards(st["r"], st["out"], _norm(case), group=st["group"], n_groups=case["groups"] or 1,
                              status=st["status"])
    return {"out": st["out"], "status": st["status"]}


# -------------------------------------------------------------------- costs --

#: Operations one normal cannot do without: a quarter of a Philox4x32-10 block
#: (20 multiplies, 20 three-way xors) and half of a Box-Muller pair (ln, sqrt,
#: cos, sin and two products).
NORMAL_OPS = 13


def work(case):
    """Each buffer of a call read once and written once, and the operations of the noise."""
    kind = case["kind"]
    if kind == "rewards":
        n = case["n"]
        return {"bytes": (12 if case["groups"] else 8) * n, "flops": 6 * n}
    if kind == "partition":
        # eight Philox blocks of the permutation per element; the map is written once
        return {"bytes": (8 if case["map"] == "int64" else 4) * case["d"], "flops": 8 * 40 * case["d"]}
    e = 4 if case.get("dtype") == "fp32" else 2
    entry = {"map64": 8, "map32": 4}.get(case.get("layout"), 0)
    length = case["d"] // case["K"]
    if kind == "member":
        if case["source"] == "master":
            per = 2 * (4 + 2 + entry)             # two passes: master read, weights written
        else:
            per = 2 * (2 * e + entry)             # backup (or weights) read, weights written, twice
        return {"bytes": per * length, "flops": (NORMAL_OPS + 2) * length}
    streams = case["n"] // 2 if case.get("mirrored") else case["n"]
    if kind == "update":
        restore, stage, update = 2 * e + entry, 4 + e + entry, (4 + 4 + e if case["master"] else 2 * e) + entry
        per = restore + update + (stage if case["master"] else 0)
        return {"bytes": per * length, "flops": (NORMAL_OPS + 2) * streams * length}
    if kind == "step":
        n = case["n"]
        return {"bytes": ((3 + 4 * n - 2) + 2) * e * length, "flops": (NORMAL_OPS + 2) * (n + streams) * length}
    n, K, d = case["n"], case["K"], case["d"]
    per = n // K
    return {"bytes": ((1 + 4 * per) + 2) * 2 * d, "flops": (NORMAL_OPS + 2) * 2 * per * d}


def tolerance(case):
    kind = case["kind"]
    if kind == "partition":
        return "exact"                            # whole numbers
    if kind == "rewards":
        return {"rel": 1.2e-7, "max": 5e-7}       # fp64 sums in another order, one rounding to fp32
    # four times the difference from exact() rounded to the weights' type, measured over the listed cases
    if case.get("dtype") == "fp32":
        return {"rel": 5e-7, "max": 6e-6}         # fp32 accumulation: 1.2e-7 and 1.5e-6 measured
    # bf16: a sum next to a rounding boundary may fall on its other side, one ulp (2^-7) off: 2e-5 and 7.8e-3 measured
    return {"rel": 8e-5, "max": 3.2e-2}


# ------------------------------------------------------------------- 64 bits --

def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors (or ints) holding 32-bit words."""
    k0, k1 = seed & MASK, (seed >> 32) & MASK
    for _ in range(10):
        pa, pb = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((pb >> 32) & MASK) ^ c1 ^ k0, pb & MASK, ((pa >> 32) & MASK) ^ c3 ^ k1, pa & MASK
        k0, k1 = (k0 + 0x9E3779B9) & MASK, (k1 + 0xBB67AE85) & MASK
    return c0, c1, c2, c3


def _normals(seed, j0, n):
    """Noise indices j0 .. j0 + n - 1 (j0 a multiple of 4) of a member, in 64 bits."""
    q = torch.arange(j0 // 4, (j0 + n + 3) // 4, dtype=torch.int64, device="cuda")
    zero = torch.zeros_like(q)
    x = _philox(q & MASK, q >> 32, zero, zero, seed)
    out = torch.empty(q.numel(), 4, dtype=torch.float64, device="cuda")
    for h in (0, 2):
        u, v = ((x[h] >> 8) + 1).double() * 2.0 ** -24, ((x[h + 1] >> 8) + 1).double() * (math.pi * 2.0 ** -23)
        rho = (-2.0 * u.log()).sqrt()
        out[:, h], out[:, h + 1] = rho * v.cos(), rho * v.sin()
    return out.view(-1)[:n]


def _buckets(d, K, seed):
    """Subspace of every element of [0, d): floor(E(i) K / d), E the keyed permutation."""
    bits = max(2, (d - 1).bit_length())
    h = (bits + 1) // 2

    def feistel(x):
        L, R = x >> h, x & ((1 << h) - 1)
        zero = torch.zeros_like(x)
        for r in range(8):
            y = _philox(R, zero + r, zero + 3, zero, seed)[0]
            L, R = R, L ^ (y & ((1 << h) - 1))
        return (L << h) | R

    out = torch.empty(d, dtype=torch.uint8, device="cuda")
    for s in range(0, d, 1 << 23):
        y = feistel(torch.arange(s, min(d, s + (1 << 23)), dtype=torch.int64, device="cuda"))
        while True:
            over = (y >= d).nonzero().view(-1)
            if over.numel() == 0:
                break
            y[over] = feistel(y[over])
        out[s:s + (1 << 23)] = (y * K // d).to(torch.uint8)
    return out


def _positions(bucket, k):
    return (bucket == k).nonzero().view(-1)


def _exact_rewards(r, norm, group=None):
    r = r.double()
    out = torch.zeros_like(r)
    for g in ([None] if group is None else range(int(group.max()) + 1)):
        at = slice(None) if g is None else (group == g).nonzero().view(-1)
        x = r[at]
        if norm == "z":
            sd = (x - x.mean()).square().mean().sqrt()
            if x.numel() and x.max() > x.min():
                out[at] = (x - x.mean()) / sd
        elif x.numel() > 1:
            s = x.sort().values
            lo, hi = torch.searchsorted(s, x), torch.searchsorted(s, x, right=True)
            out[at] = (lo + hi - 1).double() / 2 / (x.numel() - 1) - 0.5
    return out


def _coefficients(seeds, signs, rhat):
    c = {}
    for s, g, r in zip(seeds, signs, rhat.tolist()):
        c[s] = c.get(s, 0.0) + g * r
    return c


def _exact_subspace(case, seed):
    """(length, position -> parameter): a range start or an index tensor."""
    d, K, k, layout = case["d"], case["K"], case["active"], case.get("layout", "contiguous")
    if layout == "contiguous":
        return d * (k + 1) // K - d * k // K, d * k // K
    if layout == "chunk":
        at = _chunk_positions(d, case["chunk"], _positions(_buckets(-(-d // case["chunk"]), K, _partition_seed(seed)), k))
    else:
        at = _positions(_buckets(d, K, _partition_seed(seed)), k)
    return at.numel(), at


def _chunk_positions(d, C, chunks):
    at = (chunks.view(-1, 1) * C + torch.arange(C, device="cuda")).view(-1)
    return at[at < d]


def _add_noise(w, at, length, terms, base=None):
    """w[p(j)] (+)= sum of c eps_j(seed) over terms (and the same into ``base``)."""
    step = 1 << 24
    for s in range(0, length, step):
        n = min(step, length - s)
        acc = torch.zeros(n, dtype=torch.float64, device="cuda")
        for sd, c in terms:
            acc += c * _normals(sd, s, n)
        if isinstance(at, int):
            w[at + s:at + s + n] += acc
        else:
            w[at[s:s + n]] += acc
        if base is not None:
            base[s:s + n] += acc


def exact(case, seed):
    kind = case["kind"]
    if kind == "rewards":
        st = prepare(case, seed)
        return {"out": _exact_rewards(st["r"], case["norm"], st["group"]), "status": None}
    if kind == "partition":
        d, K = case["d"], case["K"]
        bucket = _buckets(d, K, _partition_seed(seed))
        index = torch.cat([_positions(bucket, k).to(getattr(torch, case["map"])) for k in range(K)])
        return {"index": index, "status": torch.zeros(1, dtype=torch.int32),
                "offsets": np.array([-(-k * d // K) for k in range(K + 1)], dtype=np.int64)}
    w0 = _weights(case, seed)
    w = w0.double()
    if kind == "paper":
        d, K, C, n = case["d"], case["K"], case["chunk"], case["n"]
        seeds, signs = _members(case, seed)
        rhat = _exact_rewards(_rewards(dict(n=n, rewards="uniform"), seed), "z")
        bucket, per = _buckets(-(-d // C), K, _partition_seed(seed)), n // K
        chunks = []
        for k in range(K):
            chunks.append(_positions(bucket, k))
            at = _chunk_positions(d, C, chunks[k])
            c = _coefficients(seeds[k * per:(k + 1) * per], signs[k * per:(k + 1) * per], rhat[k * per:(k + 1) * per])
            _add_noise(w, at, at.numel(), [(s, ALPHA / per * x) for s, x in c.items()])
        return {"w": w, "rnorm": rhat, "chunks": torch.cat(chunks)}
    length, at = _exact_subspace(case, seed)
    sigma = _sigma(case["d"], length)
    if kind == "member":
        member = 1000 * (seed % (1 << 40)) + 901
        _add_noise(w, at, length, [(member, sigma * (1 - 2 * (seed & 1)))])
        return {"w": w}
    seeds, signs = _members(case, seed)
    rhat = _exact_rewards(_rewards(case, seed), case["norm"])
    step = ALPHA / (case["n"] * sigma)
    terms = [(s, step * c) for s, c in _coefficients(seeds, signs, rhat).items()]
    old = (w0[at:at + length] if isinstance(at, int) else w0[at]) if kind == "step" or case["master"] else None
    master = old.double() if kind == "update" and case["master"] else None
    _add_noise(w, at, length, terms, master)
    out = {"w": w, "rnorm": rhat}
    if kind == "step":
        out["backup"] = old.double()
    if master is not None:
        out["master"] = master
    return out
