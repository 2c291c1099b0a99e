"""Workloads of the GEEK data pass for timing: what a program that clusters
data with this package has it do, from one small call to the full workloads.

``listed()`` gives the named cases, ``draw(rng)`` one more case of the same
ranges, ``prepare(case, seed)`` the state a program holds before the call
(device inputs made from the seed, and buffers it would keep), ``run(state)``
one pass through the public entry points, ``work(case)`` the bytes and
operations of a pass, and ``exact(case, seed)`` the floating outputs in
float64 from plain torch.

Cases of many large outputs go through the C ABI's job descriptors with output
buffers and a workspace that the caller keeps, as the ABI intends; the others
through the torch-facing wrappers, which allocate their outputs.  The
assignment's ``counters`` (how many rows each internal pass settled) are not
among the outputs: they say how the work was split, not what came out.
"""

from __future__ import annotations

import math
import random

import torch

from paper_2106_10515_amd import _lib as L
from paper_2106_10515_amd import api

DEV = "cuda:0"
PRECISION = {"fp32": L.GEEK_PREC_FP32, "bf16": L.GEEK_PREC_BF16, "fp8": L.GEEK_PREC_FP8}
VOCAB = 1_000_000      # token vocabulary of the sets
PER_SEED = 32          # members of a planted seed
SILK_K, SILK_L, SILK_DELTA = 3, 20, 10
SET_K, SET_BANDS = 4, 64   # MinHash rows per band and bands of the sets
HET_K, HET_BANDS, HET_CODES, HET_NUM, HET_CAT = 4, 32, 20, 20, 10


# ------------------------------------------------------------------- the cases
def listed():
    return [
        # one small problem through the wrappers with their defaults: latency,
        # launches and host work (the smallest job of the batched workload)
        dict(name="small_call", kind="call", n=1_000, d=16, clusters=10, m=8, L=16),
        # the small dense configuration, every step of the method by default
        # options: hash, buckets, SILK, float32 assignment to SILK's seeds
        dict(name="pass_20k", kind="pass", n=20_000, d=32, clusters=50, spread=10.0, sizes="equal",
             m=8, L=16, w=4.0, precision="fp32"),
        # the whole pass with SILK at 10^6 points: about 90,000 close seeds
        dict(name="pass_1m", kind="pass", n=1_000_000, d=128, clusters=1_000, spread=50.0, sizes="zipf",
             m=10, L=32, w=8.0, precision="bf16"),
        # the data transformation of the large dense workload (10^7 x 128,
        # 32 tables of 10 codes): hash with fingerprints, then buckets
        dict(name="buckets_10m", kind="buckets", n=10_000_000, d=128, clusters=10_000, m=10, L=32,
             w=8.0, scaled=False),
        # its assignment to 10^4 planted seeds on the bf16 matrix cores
        dict(name="assign_bf16_10m", kind="assign", n=10_000_000, d=128, k=10_000, sizes="zipf",
             precision="bf16"),
        # an ordinary assignment at the wrapper's default precision; ragged
        # row count, width and seed count
        dict(name="assign_fp32_500k", kind="assign", n=500_009, d=100, k=3_001, sizes="equal",
             precision="fp32"),
        # a further assignment pass: an assignment's clusters become the seeds
        dict(name="refine_2m", kind="refine", n=2_000_003, d=128, k=2_000, precision="bf16"),
        # sparse sets: MinHash 4 x 64, bands to buckets, modes and assignment
        dict(name="sets_1m", kind="sets", n=1_000_000, k=2_000, hash="minhash", F=SET_K * SET_BANDS),
        # sparse sets through densified one-permutation hashing, D = 400
        dict(name="sets_doph_300k", kind="sets", n=300_007, k=1_000, hash="doph", F=400),
        # heterogeneous rows at the wrapper's default precision
        dict(name="hetero_fp8_2m", kind="hetero", n=2_000_000, k=1_000, precision="fp8"),
        # Algorithm 1's buckets of equal size on the large dense rows
        dict(name="quantile_10m", kind="quantile", n=10_000_000, d=128, m=40, t=10_000),
        # many independent dense problems in one call per step
        dict(name="batch_64", kind="batch", jobs=64, layout=7, n_lo=1_000, n_hi=300_000, k_hi=3_000,
             m=8, L=16, w=4.0, precision="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["call", "pass", "buckets", "assign", "assign", "refine", "sets", "sets", "hetero",
                       "quantile", "batch"])
    if kind == "call":
        return dict(kind=kind, n=_log(rng, 200, 20_000), d=rng.randint(2, 64), clusters=rng.randint(2, 60),
                    m=8, L=rng.choice([4, 8, 16]))
    if kind == "pass":
        n = _log(rng, 10_000, 300_000)
        m, w = rng.choice([(8, 4.0), (10, 8.0)])
        return dict(kind=kind, n=n, d=rng.randint(16, 128), clusters=max(10, n // rng.randint(300, 1000)),
                    spread=rng.choice([10.0, 50.0]), sizes="equal", m=m, L=rng.choice([16, 32]), w=w,
                    precision=rng.choice(["fp32", "bf16"]))
    if kind == "buckets":
        return dict(kind=kind, n=_log(rng, 50_000, 5_000_000), d=rng.randint(8, 256),
                    clusters=_log(rng, 50, 5_000), m=rng.choice([4, 8, 10, 12]), L=rng.randint(4, 32),
                    w=8.0, scaled=rng.random() < 0.5)
    if kind == "assign":
        precision = rng.choice(["fp32", "bf16", "fp8"])
        n, d, k = _log(rng, 10_000, 3_000_000), rng.randint(8, 256), _log(rng, 50, 8_000)
        if precision != "bf16":
            k = max(50, min(k, int(1.5e12 / n / d)))
        return dict(kind=kind, n=n, d=d, k=k, sizes=rng.choice(["equal", "zipf"]), precision=precision)
    if kind == "refine":
        return dict(kind=kind, n=_log(rng, 50_000, 2_000_000), d=rng.randint(16, 256), k=_log(rng, 100, 2_000),
                    precision=rng.choice(["fp32", "bf16"]))
    if kind == "sets":
        how = rng.choice(["minhash", "doph"])
        return dict(kind=kind, n=_log(rng, 20_000, 900_000 if how == "minhash" else 300_000),
                    k=_log(rng, 50, 2_000 if how == "minhash" else 1_000), hash=how,
                    F=SET_K * SET_BANDS if how == "minhash" else rng.randint(SET_K * SET_BANDS, 400))
    if kind == "hetero":
        return dict(kind=kind, n=_log(rng, 50_000, 2_000_000), k=_log(rng, 50, 1_000),
                    precision=rng.choice(["fp8", "bf16"]))
    if kind == "quantile":
        return dict(kind=kind, n=_log(rng, 100_000, 8_000_000), d=rng.randint(8, 256), m=rng.randint(4, 40),
                    t=_log(rng, 100, 10_000))
    return dict(kind="batch", jobs=rng.randint(16, 64), layout=rng.randint(8, 1 << 30), n_lo=1_000, n_hi=200_000,
                k_hi=_log(rng, 500, 3_000), m=8, L=16, w=4.0, precision="bf16")


# ------------------------------------------------------------------ the inputs
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1_000_003 + stream)
    return g


def _labels(n, clusters, sizes, g):
    """Cluster of every row: equal or Zipf(1) shares, every cluster used,
    shuffled."""
    if sizes == "equal":
        lab = torch.arange(n, device=DEV) % clusters
    else:
        share = 1.0 / torch.arange(1, clusters + 1, device=DEV, dtype=torch.float64)
        cdf = torch.cumsum(share, 0) / share.sum()
        rest = (torch.arange(max(n - clusters, 0), device=DEV) + 0.5) / max(n - clusters, 1)
        lab = torch.cat([torch.arange(min(n, clusters), device=DEV),
                         torch.searchsorted(cdf, rest.double()).clamp_(max=clusters - 1)])
    return lab[torch.randperm(n, device=DEV, generator=g)]


def _mixture(n, d, clusters, spread, sizes, seed, stream=0):
    """Rows of an isotropic Gaussian mixture (sigma 1, centres uniform in
    [-spread, spread]^d) and their clusters."""
    g = _gen(seed, stream)
    lab = _labels(n, clusters, sizes, g)
    centers = (torch.rand((clusters, d), generator=g, device=DEV) * 2 - 1) * spread
    X = torch.empty((n, d), device=DEV)
    step = 1 << 21
    for s in range(0, n, step):
        part = X[s:s + step]
        part.normal_(generator=g)
        part += centers[lab[s:s + step]]
    return X, lab


def _planted(lab, clusters, per_seed=PER_SEED):
    """Seed j = the first ids (ascending, at most per_seed) of cluster j;
    every cluster is used."""
    order = torch.sort(lab, stable=True).indices
    sizes = torch.bincount(lab, minlength=clusters)
    start = torch.cumsum(sizes, 0) - sizes
    take = sizes.clamp(max=per_seed)
    off = torch.zeros(clusters + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(take, 0)
    at = torch.arange(int(off[-1]), device=DEV) - torch.repeat_interleave(off[:-1] - start, take)
    return off.int(), order[at].int()


def _projections(count, d, w, g):
    A = torch.randn((count, d), generator=g, device=DEV)
    return A, torch.rand(count, generator=g, device=DEV) * (w * 0.999)


def _key_words(count, g):
    return torch.randint(-2**31, 2**31, (count, 2), generator=g, device=DEV, dtype=torch.int64).int()


def _zipf(vocab, s):
    p = torch.arange(1, vocab + 1, device=DEV, dtype=torch.float64) ** (-s)
    return torch.cumsum(p, 0) / p.sum()


def _sets(n, clusters, seed):
    """Sparse sets over the vocabulary: lognormal sizes, Zipf(1.1) tokens, 60 %
    of a set's draws from its cluster's prototype; repeats within a set
    dropped, tokens ascending."""
    g = _gen(seed, 0)
    cdf = _zipf(VOCAB, 1.1)

    def sizes(count):
        z = torch.randn(count, generator=g, device=DEV, dtype=torch.float64)
        return torch.exp(4.5 + 0.6 * z).round().clamp(5, 2000).long()

    def zipf(count):
        u = torch.rand(count, generator=g, device=DEV, dtype=torch.float64)
        return torch.searchsorted(cdf, u).clamp_(max=VOCAB - 1)

    proto = sizes(clusters)
    proto_off = torch.cumsum(proto, 0) - proto
    proto_tok = zipf(int(proto.sum()))
    lab = _labels(n, clusters, "equal", g)
    row = torch.repeat_interleave(torch.arange(n, device=DEV), sizes(n))
    count = row.numel()
    c = lab[row]
    u = torch.rand(count, generator=g, device=DEV, dtype=torch.float64)
    tok = proto_tok[proto_off[c] + (u * proto[c]).long()]
    own = torch.rand(count, generator=g, device=DEV) >= 0.6
    tok = torch.where(own, zipf(count), tok)
    key = torch.unique_consecutive(torch.sort((row << 20) | tok).values)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.bincount(key >> 20, minlength=n), 0)
    return off, (key & (2**20 - 1)).int(), lab


def _hetero(n, clusters, seed):
    """Numeric attributes of a mixture and categorical ones with 10..1000
    values, Zipf(1.2) with an offset per (attribute, cluster)."""
    X, lab = _mixture(n, HET_NUM, clusters, 10.0, "equal", seed)
    g = _gen(seed, 1)
    cat = torch.empty((n, HET_CAT), dtype=torch.int32, device=DEV)
    for a in range(HET_CAT):
        values = int(round(10 ** (1 + 2 * (a + 0.5) / HET_CAT)))
        z = torch.searchsorted(_zipf(values, 1.2), torch.rand(n, generator=g, device=DEV, dtype=torch.float64))
        shift = torch.randint(0, values, (clusters,), generator=g, device=DEV)
        cat[:, a] = ((z + shift[lab]) % values).int()
    return X, cat, lab


def _layout(case):
    """(n, d, clusters) of every job of a batch."""
    r = random.Random(case["layout"])
    jobs = []
    for _ in range(case["jobs"]):
        n = _log(r, case["n_lo"], case["n_hi"])
        jobs.append((n, r.choice([16, 32, 64, 128, 256]), min(n // 8, _log(r, 10, case["k_hi"]))))
    return jobs


# --------------------------------------------------- buffers a caller may keep
def _words(*shape):
    return torch.zeros(shape, dtype=torch.int32, device=DEV)


def _bucket_out(T, n):
    return dict(members=_words(T, n), offsets=_words(T, n + 1), nbuckets=_words(T), bucket_of=_words(T, n))


def _bucket_job(keys, n, T, words, table_stride, row_stride, out, key_fp=None):
    return L.BucketizeJob(n=n, T=T, key_words=words, keys=keys.data_ptr(), table_stride=table_stride,
                          row_stride=row_stride, members=out["members"].data_ptr(),
                          offsets=out["offsets"].data_ptr(), nbuckets=out["nbuckets"].data_ptr(),
                          bucket_of=out["bucket_of"].data_ptr(),
                          key_fp=None if key_fp is None else key_fp.data_ptr())


class _Chain:
    """Calls of the C ABI in order, with the workspace and status word that
    the caller keeps."""

    def __init__(self, *calls):
        self.calls = calls
        need = max(L.workspace_size(op, jobs) for op, _, jobs in calls)
        self.ws = torch.empty(need + 256, dtype=torch.uint8, device=DEV)
        self.status = torch.zeros(1, dtype=torch.int32, device=DEV)

    def __call__(self):
        stream = torch.cuda.current_stream().cuda_stream
        for _, fn, jobs in self.calls:
            fn(jobs, self.ws.data_ptr(), self.ws.numel(), self.status.data_ptr(), stream)


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return state["pass"](state)


def _result(out):
    return {name: value for name, value in out.items() if name != "counters" and value is not None}


# one small problem: hash, buckets and assignment with default options
def _prepare_call(case, seed):
    X, lab = _mixture(case["n"], case["d"], case["clusters"], 10.0, "equal", seed)
    w = 4.0 * math.sqrt(case["d"])
    A, b = _projections(case["m"] * case["L"], case["d"], w, _gen(seed, 1))
    so, sm = _planted(lab, case["clusters"])
    return dict(case, X=X, A=A, b=b, w=w, so=so, sm=sm, **{"pass": _run_call})


def _run_call(s):
    n = s["n"]
    keys, _ = api.hash_dense(s["X"], s["A"], s["b"], s["m"], s["L"], s["w"])
    members, _, nbuckets, bucket_of = api.bucketize(keys, n, s["L"], 4, n * 4, 4)
    out = api.assign_euclid(s["X"], s["so"], s["sm"], s["clusters"])
    # (the wrapper's offsets hold nothing defined past a table's bucket count;
    # members and bucket_of determine them)
    return dict(keys=keys, members=members, nbuckets=nbuckets, bucket_of=bucket_of, **_result(out))


# the whole pass: hash, buckets, SILK's seeds, assignment to them; the program
# reads the status and the seed count before the assignment
def _prepare_pass(case, seed):
    n, d, m, T, dev = case["n"], case["d"], case["m"], case["L"], torch.device(DEV)
    X, _ = _mixture(n, d, case["clusters"], case["spread"], case["sizes"], seed)
    g = _gen(seed, 1)
    w = case["w"] * math.sqrt(d)
    A, b = _projections(m * T, d, w, g)
    silk = _key_words((SILK_L + 1) * SILK_K, g)
    cap_k, cap_members = max(1024, n // 4), max(4096, 16 * n)
    keys, out = _words(T, n, 4), _bucket_out(T, n)
    seeds = dict(seed_offsets=_words(cap_k + 1), seed_members=_words(cap_members), k_out=_words(1),
                 needed=torch.zeros(3, dtype=torch.int64, device=DEV),
                 silk_counts=torch.zeros(4, dtype=torch.int64, device=DEV))
    own = dict(assign=_words(n), centroids=torch.zeros((cap_k, d), dtype=torch.float64, device=DEV),
               dist=torch.zeros(n, dtype=torch.float64, device=DEV),
               sse=torch.zeros(1, dtype=torch.float64, device=DEV),
               radius=torch.zeros(cap_k, dtype=torch.float64, device=DEV))
    hj = L.HashJob(kind=L.GEEK_HASH_DENSE, d=d, n=n, X=X.data_ptr(), ldx=d, A=A.data_ptr(), b=b.data_ptr(),
                   m=m, L=T, w=w, keys=keys.data_ptr())
    bj = _bucket_job(keys, n, T, 4, n * 4, 4, out)
    sj = L.SilkJob(n=n, T=T, K=SILK_K, members=out["members"].data_ptr(), offsets=out["offsets"].data_ptr(),
                   nbuckets=out["nbuckets"].data_ptr(), L=SILK_L, delta=SILK_DELTA, silk_keys=silk.data_ptr(),
                   cap_k=cap_k, cap_members=cap_members, cap_c=32 * n,
                   seed_offsets=seeds["seed_offsets"].data_ptr(), seed_members=seeds["seed_members"].data_ptr(),
                   k_out=seeds["k_out"].data_ptr(), needed=seeds["needed"].data_ptr(),
                   counters=seeds["silk_counts"].data_ptr())
    chain = _Chain((L.GEEK_OP_HASH, L.geek_hash, [hj]), (L.GEEK_OP_BUCKETIZE, L.geek_bucketize, [bj]),
                   (L.GEEK_OP_SILK, L.geek_silk_seeds, [sj]))
    return {"pass": _run_pass, "chain": chain, "kept": (A, b, silk), "X": X, "own": own, "seeds": seeds,
            "precision": PRECISION[case["precision"]], "device": dev, "out": dict(keys=keys, **out, **seeds, **own)}


def _run_pass(s):
    X, own, seeds, chain = s["X"], s["own"], s["seeds"], s["chain"]
    chain()
    api.check_status(chain.status, "hash, buckets and seeds")
    job = L.AssignJob(metric=L.GEEK_METRIC_EUCLID, precision=s["precision"], n=X.shape[0], d=X.shape[1],
                      k=int(seeds["k_out"]), X=X.data_ptr(), ldx=X.stride(0),
                      seed_offsets=seeds["seed_offsets"].data_ptr(), seed_members=seeds["seed_members"].data_ptr(),
                      **{name: t.data_ptr() for name, t in own.items()})
    ws = api.workspace(L.workspace_size(L.GEEK_OP_ASSIGN, [job]), s["device"])
    L.geek_assign([job], ws.data_ptr(), ws.numel(), chain.status.data_ptr(), api.stream_ptr(s["device"]))
    return s["out"]


# hash with fingerprints, then buckets, into buffers that the caller keeps
def _prepare_buckets(case, seed):
    n, d, m, T = case["n"], case["d"], case["m"], case["L"]
    X, _ = _mixture(n, d, case["clusters"], 50.0, "zipf", seed)
    w = case["w"] * (math.sqrt(d) if case["scaled"] else 1.0)
    A, b = _projections(m * T, d, w, _gen(seed, 1))
    keys, fp, out = _words(T, n, 4), _words(T, n), _bucket_out(T, n)
    hj = L.HashJob(kind=L.GEEK_HASH_DENSE, d=d, n=n, X=X.data_ptr(), ldx=d, A=A.data_ptr(), b=b.data_ptr(),
                   m=m, L=T, w=w, keys=keys.data_ptr(), key_fp=fp.data_ptr())
    bj = _bucket_job(keys, n, T, 4, n * 4, 4, out, fp)
    chain = _Chain((L.GEEK_OP_HASH, L.geek_hash, [hj]), (L.GEEK_OP_BUCKETIZE, L.geek_bucketize, [bj]))
    return {"pass": _run_chain, "chain": chain, "kept": (X, A, b), "out": dict(keys=keys, key_fp=fp, **out)}


def _run_chain(s):
    s["chain"]()
    return s["out"]


# assignment of dense rows to planted seeds
def _prepare_assign(case, seed):
    X, lab = _mixture(case["n"], case["d"], case["k"], 50.0, case["sizes"], seed)
    so, sm = _planted(lab, case["k"])
    status = api.new_status(torch.device(DEV))
    return dict(case, X=X, so=so, sm=sm, status=status, **{"pass": _run_assign})


def _run_assign(s):
    return _result(api.assign_euclid(s["X"], s["so"], s["sm"], s["k"], PRECISION[s["precision"]],
                                     status=s["status"], check=False))


# a further pass: the last assignment's clusters as seeds (three labels unused)
def _prepare_refine(case, seed):
    X, lab = _mixture(case["n"], case["d"], case["k"], 50.0, "zipf", seed)
    return dict(case, X=X, before=lab.int(), **{"pass": _run_refine})


def _run_refine(s):
    return _result(api.assignment_pass(s["X"], s["before"], s["k"] + 3, PRECISION[s["precision"]]))


# sets: signatures, buckets of the bands, modes and assignment
def _prepare_sets(case, seed):
    n, F, k = case["n"], case["F"], case["k"]
    off, tok, lab = _sets(n, k, seed)
    mh = _key_words(F if case["hash"] == "minhash" else 1, _gen(seed, 2))
    so, sm = _planted(lab, k)
    sig, out = _words(n, F), _bucket_out(SET_BANDS, n)
    own = dict(assign=_words(n), modes=_words(k, F), dist=torch.zeros(n, dtype=torch.float64, device=DEV),
               sse=torch.zeros(1, dtype=torch.float64, device=DEV),
               radius=torch.zeros(k, dtype=torch.float64, device=DEV))
    hj = L.HashJob(kind=L.GEEK_HASH_SETS if case["hash"] == "minhash" else L.GEEK_HASH_DOPH, n=n, F=F,
                   offsets=off.data_ptr(), tokens=tok.data_ptr(), mh_keys=mh.data_ptr(), sig=sig.data_ptr())
    bj = _bucket_job(sig, n, SET_BANDS, SET_K, SET_K, F, out)
    aj = L.AssignJob(metric=L.GEEK_METRIC_SIG, n=n, k=k, sig=sig.data_ptr(), F=F, n_members=sm.numel(),
                     seed_offsets=so.data_ptr(), seed_members=sm.data_ptr(),
                     **{name: t.data_ptr() for name, t in own.items()})
    chain = _Chain((L.GEEK_OP_HASH, L.geek_hash, [hj]), (L.GEEK_OP_BUCKETIZE, L.geek_bucketize, [bj]),
                   (L.GEEK_OP_ASSIGN, L.geek_assign, [aj]))
    return {"pass": _run_chain, "chain": chain, "kept": (off, tok, mh, so, sm), "out": dict(sig=sig, **out, **own)}


# heterogeneous rows: signatures, buckets of the bands, mixed assignment
def _prepare_hetero(case, seed):
    n, k, F = case["n"], case["k"], HET_K * HET_BANDS
    X, cat, lab = _hetero(n, k, seed)
    g = _gen(seed, 2)
    A, b = _projections(HET_CODES, HET_NUM, 4.0, g)
    so, sm = _planted(lab, k)
    out = _bucket_out(HET_BANDS, n)
    return dict(case, X=X, cat=cat, A=A, b=b, mh=_key_words(F, g), so=so, sm=sm, out=out,
                status=api.new_status(torch.device(DEV)), **{"pass": _run_hetero})


def _run_hetero(s):
    n, F, out = s["n"], HET_K * HET_BANDS, s["out"]
    sig = api.hash_hetero(s["X"], s["cat"], s["A"], s["b"], HET_CODES, 1, 4.0, s["mh"], status=s["status"],
                          check=False)
    job = _bucket_job(sig, n, HET_BANDS, HET_K, HET_K, F, out)
    ws = api.workspace(L.workspace_size(L.GEEK_OP_BUCKETIZE, [job]), sig.device)
    L.geek_bucketize([job], ws.data_ptr(), ws.numel(), s["status"].data_ptr(), api.stream_ptr(sig.device))
    got = api.assign_hetero(s["X"], s["cat"], s["so"], s["sm"], s["k"], 1.0, PRECISION[s["precision"]],
                            status=s["status"], check=False)
    return dict(sig=sig, **out, **_result(got))


# Algorithm 1: ranks along each projection split evenly
def _prepare_quantile(case, seed):
    X, _ = _mixture(case["n"], case["d"], min(case["n"] // 100, 10_000), 50.0, "zipf", seed)
    A, _ = _projections(case["m"], case["d"], 1.0, _gen(seed, 1))
    return dict(case, X=X, A=A, status=api.new_status(torch.device(DEV)), **{"pass": _run_quantile})


def _run_quantile(s):
    members, offsets, bucket_of = api.quantile_buckets(s["X"], s["A"], s["t"], status=s["status"], check=False)
    return dict(members=members, offsets=offsets, bucket_of=bucket_of)


# many dense problems, one call per step; the results of all jobs lie in one
# buffer per kind, each job's part at a multiple of 16 bytes
def _prepare_batch(case, seed):
    m, T, prec = case["m"], case["L"], PRECISION[case["precision"]]
    specs = _layout(case)
    g = _gen(seed, 1)
    hashes = {d: _projections(m * T, d, case["w"], g) for d in sorted({d for _, d, _ in specs})}
    problems = []
    for j, (n, d, k) in enumerate(specs):
        X, lab = _mixture(n, d, k, 10.0, "equal", seed, 10 + j)
        problems.append((X, *_planted(lab, k)))

    up = lambda v: -(-v // 4) * 4  # noqa: E731
    sizes = dict(keys=[T * n * 4 for n, _, _ in specs], members=[T * n for n, _, _ in specs],
                 offsets=[T * (n + 1) for n, _, _ in specs], nbuckets=[T] * len(specs),
                 bucket_of=[T * n for n, _, _ in specs], assign=[n for n, _, _ in specs])
    wide = dict(centroids=[k * d for _, d, k in specs], dist=[n for n, _, _ in specs], sse=[1] * len(specs),
                radius=[k for _, _, k in specs])
    out, part = {}, {}
    for group, dtype in ((sizes, torch.int32), (wide, torch.float64)):
        for name, counts in group.items():
            buf = torch.zeros(sum(map(up, counts)), dtype=dtype, device=DEV)
            at, part[name], out[name] = 0, [], buf
            for c in counts:
                part[name].append(buf.data_ptr() + at * buf.element_size())
                at += up(c)
    hj, bj, aj = [], [], []
    for j, ((n, d, k), (X, so, sm)) in enumerate(zip(specs, problems)):
        A, b = hashes[d]
        p = {name: v[j] for name, v in part.items()}
        hj.append(L.HashJob(kind=L.GEEK_HASH_DENSE, d=d, n=n, X=X.data_ptr(), ldx=d, A=A.data_ptr(),
                            b=b.data_ptr(), m=m, L=T, w=case["w"], keys=p["keys"]))
        bj.append(L.BucketizeJob(n=n, T=T, key_words=4, keys=p["keys"], table_stride=n * 4, row_stride=4,
                                 members=p["members"], offsets=p["offsets"], nbuckets=p["nbuckets"],
                                 bucket_of=p["bucket_of"]))
        aj.append(L.AssignJob(metric=L.GEEK_METRIC_EUCLID, precision=prec, n=n, d=d, k=k, X=X.data_ptr(), ldx=d,
                              n_members=sm.numel(), seed_offsets=so.data_ptr(), seed_members=sm.data_ptr(),
                              assign=p["assign"], centroids=p["centroids"], dist=p["dist"], sse=p["sse"],
                              radius=p["radius"]))
    chain = _Chain((L.GEEK_OP_HASH, L.geek_hash, hj), (L.GEEK_OP_BUCKETIZE, L.geek_bucketize, bj),
                   (L.GEEK_OP_ASSIGN, L.geek_assign, aj))
    return {"pass": _run_chain, "chain": chain, "kept": (problems, hashes), "out": out}


# ------------------------------------------------------------- the work it takes
def _dense_work(n, d, P, T):
    """Hash and buckets: rows and projections in, keys, members, offsets and
    bucket_of out."""
    return 4 * n * d + 4 * P * (d + 1) + T * n * (16 + 12), 2 * n * d * P


def _assign_work(n, d, k):
    """Rows in (their seed members' rows are among them), assignment,
    distance, centroids and radius out."""
    return 4 * n * d + 12 * n + 8 * k * d + 8 * k + 4 * k * (PER_SEED + 1), 2 * n * d * k


def work(case):
    kind, n = case["kind"], case.get("n", 0)
    if kind in ("call", "pass", "buckets"):
        b, f = _dense_work(n, case["d"], case["m"] * case["L"], case["L"])
        if kind == "call":
            b2, f2 = _assign_work(n, case["d"], case["clusters"])
            b, f = b + b2 - 4 * n * case["d"], f + f2
        if kind == "pass":
            # plus the rows' assignment to at least one seed a cluster (how
            # many seeds SILK finds is known only afterwards)
            b, f = b + 12 * n, f + 2 * n * case["d"] * case["clusters"]
    elif kind == "assign":
        b, f = _assign_work(n, case["d"], case["k"])
    elif kind == "refine":
        b, f = _assign_work(n, case["d"], case["k"])
        b += 4 * n + 4 * n  # labels in, the clusters' members
    elif kind == "sets":
        mean = 100  # tokens of a set, about
        b = n * (4 * mean + 8 + 4 * case["F"] + SET_BANDS * 12 + 12) + 4 * case["k"] * case["F"]
        f = 2 * n * mean * (case["F"] if case["hash"] == "minhash" else 1)
    elif kind == "hetero":
        F = HET_K * HET_BANDS
        b = n * (4 * HET_NUM + 4 * HET_CAT + 4 * F + HET_BANDS * 12 + 12)
        f = 2 * n * (HET_NUM * HET_CODES + (HET_CODES + HET_CAT) * F + HET_NUM * case["k"] + HET_CAT * case["k"])
    elif kind == "quantile":
        b = 4 * n * case["d"] + 8 * case["m"] * n
        f = 2 * n * case["d"] * case["m"]
    else:
        b = f = 0
        for n, d, k in _layout(case):
            b1, f1 = _dense_work(n, d, case["m"] * case["L"], case["L"])
            b2, f2 = _assign_work(n, d, k)
            b, f = b + b1 + b2 - 4 * n * d, f + f1 + f2
    return {"bytes": float(b), "flops": float(f)}


# -------------------------------------------------- the floating outputs, plainly
def _centers(X, so, sm):
    """Means of the seeds' members in float64."""
    k = so.numel() - 1
    size = (so[1:] - so[:-1]).long()
    of = torch.repeat_interleave(torch.arange(k, device=DEV), size)
    C = torch.zeros((k, X.shape[1]), dtype=torch.float64, device=DEV)
    step = 1 << 21
    for s in range(0, sm.numel(), step):
        C.index_add_(0, of[s:s + step], X[sm[s:s + step].long()].double())
    return C / size[:, None].double()


def _modes(V, so, sm):
    """Most frequent value (the smallest on ties) of every column over each
    seed's members; V holds non-negative int64 values."""
    k, F = so.numel() - 1, V.shape[1]
    size = (so[1:] - so[:-1]).long()
    most = int(size.max())
    pad = torch.iinfo(torch.int64).max
    M = torch.empty((k, F), dtype=torch.int64, device=DEV)
    slot = torch.arange(most, device=DEV)
    for s in range(0, k, 256):
        sz = size[s:s + 256]
        at = so[:-1][s:s + 256].long()[:, None] + torch.minimum(slot[None, :], sz[:, None] - 1)
        v = V[sm[at].long()]                                     # [seeds, most, F]
        v = torch.where((slot[None, :] < sz[:, None])[:, :, None], v, pad)
        v = torch.sort(v, dim=1).values
        idx = slot[None, :, None].expand_as(v)
        new = torch.ones_like(v, dtype=torch.bool)
        new[:, 1:] = v[:, 1:] != v[:, :-1]
        run_len = idx - torch.cummax(torch.where(new, idx, 0), dim=1).values + 1
        run_len = torch.where(v == pad, 0, run_len)
        best = run_len.max(dim=1, keepdim=True).values
        first = torch.where(run_len == best, idx, most).min(dim=1, keepdim=True).values
        M[s:s + 256] = torch.gather(v, 1, first)[:, 0]
    return M


def _nearest(X, C, extra=None):
    """Smallest squared distance (plus extra(first row, last row), if any) of
    every row, and its centre."""
    n = X.shape[0]
    dist = torch.empty(n, dtype=torch.float64, device=DEV)
    own = torch.empty(n, dtype=torch.int64, device=DEV)
    c2 = (C * C).sum(1)
    step = max(256, (1 << 28) // C.shape[0])
    for s in range(0, n, step):
        x = X[s:s + step].double()
        v = torch.addmm(c2, x, C.t(), alpha=-2.0)
        e = None if extra is None else extra(s, min(n, s + step))
        a = (v if e is None else v + e).argmin(1)
        own[s:s + step] = a
        got = ((x - C[a]) ** 2).sum(1)
        dist[s:s + step] = got if e is None else got + e.gather(1, a[:, None])[:, 0]
    return dist, own


def _radius(dist, own, k, root=True):
    far = torch.zeros(k, dtype=torch.float64, device=DEV).scatter_reduce_(0, own, dist, "amax")
    return far.sqrt() if root else far


def _exact_euclid(X, so, sm):
    C = _centers(X, so, sm)
    dist, own = _nearest(X, C)
    return dict(assign=None, centroids=C, dist=dist, sse=dist.sum().reshape(1), radius=_radius(dist, own, C.shape[0]))


def _mix32(x):
    """MurmurHash3's 32-bit finalizer on int64 tensors holding 32-bit words."""
    x = x ^ (x >> 16)
    x = (x * 0x85EBCA6B) & 0xFFFFFFFF
    x = x ^ (x >> 13)
    x = (x * 0xC2B2AE35) & 0xFFFFFFFF
    return x ^ (x >> 16)


def _signatures(case, off, tok, mh):
    n, F, count = case["n"], case["F"], off[1:] - off[:-1]
    row = torch.repeat_interleave(torch.arange(n, device=DEV), count)
    mixed = _mix32(tok.long() & 0xFFFFFFFF)
    a, b = (mh[:, 0].long() & 0xFFFFFFFF) | 1, mh[:, 1].long() & 0xFFFFFFFF
    top = 1 << 32
    if case["hash"] == "minhash":
        sig = torch.empty((n, F), dtype=torch.int64, device=DEV)
        for f in range(F):
            v = (mixed * a[f] + b[f]) & 0xFFFFFFFF
            sig[:, f] = torch.full((n,), top, device=DEV).scatter_reduce_(0, row, v, "amin")
        return sig
    v = (mixed * a[0] + b[0]) & 0xFFFFFFFF
    sig = torch.full((n * F,), top, device=DEV).scatter_reduce_(0, row * F + ((v * F) >> 32), v, "amin").view(n, F)
    # an empty bin takes the first filled bin to its right, cyclically
    twice = torch.cat([sig, sig], 1)
    at = torch.where(twice < top, torch.arange(2 * F, device=DEV)[None, :], 2 * F)
    at = torch.flip(torch.cummin(torch.flip(at, [1]), 1).values, [1])[:, :F]
    return torch.gather(twice, 1, at)


def _exact_sets(case, seed):
    n, F, k = case["n"], case["F"], case["k"]
    off, tok, lab = _sets(n, k, seed)
    so, sm = _planted(lab, k)
    sig = _signatures(case, off, tok, _key_words(F if case["hash"] == "minhash" else 1, _gen(seed, 2)))
    M = _modes(sig, so, sm)
    S, M = (sig - (1 << 31)).int(), (M - (1 << 31)).int()  # order kept, half the bytes
    best = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    own = torch.zeros(n, dtype=torch.int64, device=DEV)
    for j in range(k):
        same = (S == M[j]).sum(1)
        own = torch.where(same > best, j, own)
        best = torch.maximum(best, same)
    dist = 1.0 - best.double() / F
    return dict(dist=dist, sse=dist.sum().reshape(1), radius=_radius(dist, own, k, root=False))


def _exact_hetero(case, seed):
    X, cat, lab = _hetero(case["n"], case["k"], seed)
    so, sm = _planted(lab, case["k"])
    M = _modes(cat.long(), so, sm).int()
    C = _centers(X, so, sm)

    def mismatches(s, e):
        v = torch.zeros((e - s, case["k"]), dtype=torch.float64, device=DEV)
        for a in range(HET_CAT):
            v += cat[s:e, a, None] != M[None, :, a]
        return v

    dist, own = _nearest(X, C, mismatches)
    # (the radius of heterogeneous clusters is the largest D itself, no root)
    return dict(centroids=C, dist=dist, sse=dist.sum().reshape(1), radius=_radius(dist, own, case["k"], root=False))


def exact(case, seed):
    kind = case["kind"]
    if kind == "call":
        X, lab = _mixture(case["n"], case["d"], case["clusters"], 10.0, "equal", seed)
        return _exact_euclid(X, *_planted(lab, case["clusters"]))
    if kind == "assign":
        X, lab = _mixture(case["n"], case["d"], case["k"], 50.0, case["sizes"], seed)
        return _exact_euclid(X, *_planted(lab, case["k"]))
    if kind == "refine":
        X, lab = _mixture(case["n"], case["d"], case["k"], 50.0, "zipf", seed)
        return _exact_euclid(X, *_planted(lab, case["k"], case["n"]))
    if kind == "sets":
        return _exact_sets(case, seed)
    if kind == "hetero":
        return _exact_hetero(case, seed)
    if kind == "batch":
        up = lambda t: torch.cat([t.reshape(-1), t.new_zeros(-t.numel() % 4)])  # noqa: E731
        parts = []
        for j, (n, d, k) in enumerate(_layout(case)):
            X, lab = _mixture(n, d, k, 10.0, "equal", seed, 10 + j)
            parts.append(_exact_euclid(X, *_planted(lab, k)))
        return {name: torch.cat([up(p[name]) for p in parts]) for name in ("centroids", "dist", "sse", "radius")}
    return None  # whole numbers (buckets, quantiles), or seeds that SILK itself finds (pass)
