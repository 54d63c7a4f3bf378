"""The work that a user of this library has it do, case by case.

Every case is one pass of a serving program through the public entry points
(``paper_2401_14021_amd.binding``), on the synthetic inputs of
``paper_2401_14021_amd.inputs`` (clustered datastores with about 320 rows per
cluster, 1200 for neighbour language models; queries near datastore rows; caches that
hold a query's source row half of the time).  Four kinds of work:

* ``speculate``  the per-request cache lookup alone: a speculation step, run once
                 per decoded chunk and by far the most frequent call.
* ``round``      a verification round: cache lookup of all recorded queries, batched exact
                 retrieval, first-mismatch compare, cache update.
* ``retrieve``   exact retrieval alone: plain iterative serving (one query), the
                 prefetch that fills a cache, and batches without speculation.
* ``simple``     the same from the caller's fp32 rows, with no prepared copy.
* ``knnlm``      a round of a neighbour language model: k entries from the cache and their
                 token distribution, retrieval and its distribution, compare on
                 tokens, next-n cache update.
* ``build``      the low-precision scan copy of a datastore (index build).
"""
from __future__ import annotations

import math

import torch

from paper_2401_14021_amd import binding as B
from paper_2401_14021_amd import inputs

_TORCH = {"bf16": torch.bfloat16, "f16": torch.float16}


def listed():
    return [
        # a decoding step of a modest serving batch: every request asks its own cache once
        dict(name="speculate_64", kind="speculate", N=1_000_000, d=768, R=64, s_lo=1, s_hi=1, C=1024),
        # one user, a small corpus, stride 3: all launches and latency
        dict(name="round_tiny", kind="round", N=100_000, d=768, scan="bf16", R=1, s_lo=3, s_hi=3, k=1, C=64,
             order="iid"),
        # sixteen concurrent requests over a million passages
        dict(name="round_medium", kind="round", N=1_000_000, d=768, scan="bf16", R=16, s_lo=1, s_hi=8, k=5,
             C=1024, order="iid"),
        # an odd embedding width and row count, fp16 copy, ragged strides, corpus-ordered rows
        dict(name="round_odd", kind="round", N=777_001, d=392, scan="f16", R=33, s_lo=1, s_hi=5, k=10, C=500,
             order="corpus"),
        # plain iterative serving / prefetch of one request over a large corpus: a read of the whole copy
        dict(name="retrieve_one", kind="retrieve", N=8_000_000, d=768, scan="bf16", Q=1, k=20, order="iid"),
        # a batch between the memory-bound and the matrix-bound end, ragged
        dict(name="retrieve_200", kind="retrieve", N=6_000_000, d=768, scan="bf16", Q=200, k=20, order="iid"),
        # a large verification batch: 256 requests with stride 4, top-20 cache update
        dict(name="round_large", kind="round", N=10_000_000, d=768, scan="bf16", R=256, s_lo=4, s_hi=4, k=20,
             C=1024, order="iid"),
        # the stress loop: 512 requests, ragged strides, caches of 4096
        dict(name="round_stress", kind="round", N=4_000_000, d=768, scan="bf16", R=512, s_lo=1, s_hi=8, k=20,
             C=4096, order="iid"),
        # neighbour language model, inner product: fp16 keys, 32 requests x 8 tokens, k = 1024
        dict(name="knnlm_ip", kind="knnlm", N=10_000_000, d=1024, metric="ip", R=32, s=8, k=1024, C=2048, n_next=10,
             order="iid"),
        # the same by squared distance, smaller: 16 requests x 4 tokens, k = 256, corpus-ordered keys
        dict(name="knnlm_l2", kind="knnlm", N=2_000_000, d=1024, metric="l2", R=16, s=4, k=256, C=1000, n_next=10,
             order="corpus"),
        # a first try-out: the caller's fp32 matrix, no copy, synchronous
        dict(name="simple_16", kind="simple", N=500_000, d=384, Q=16, k=10),
        # index build of a store that fits neither cache
        dict(name="build_copy", kind="build", N=4_000_000, d=768, metric="ip", scan="bf16"),
    ]


def _spread(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["speculate", "round", "round", "round", "retrieve", "retrieve", "knnlm", "knnlm", "simple",
                       "build"])
    order = rng.choice(["iid", "corpus"])
    d = rng.choice([768, 768, 1024, 384, 8 * rng.randint(16, 128)])
    scan = rng.choice(["bf16", "bf16", "f16"])
    if kind == "speculate":
        return dict(kind=kind, N=_spread(rng, 50_000, 2_000_000), d=d, R=_spread(rng, 1, 512), s_lo=1,
                    s_hi=rng.choice([1, 1, 4]), C=_spread(rng, 64, 4096))
    if kind == "round":
        R, s_hi = _spread(rng, 1, 512), rng.randint(1, 8)
        s_lo = rng.choice([1, s_hi])
        # the largest: about as much as a thousand queries over ten million rows of 768
        most = 7.0e12 / (R * (s_lo + s_hi) / 2 * d)
        N = _spread(rng, 50_000, max(60_000, min(8_000_000, most)))
        k = rng.choice([1, 5, 10, 20, rng.randint(1, 32)])
        return dict(kind=kind, N=N, d=d, scan=scan, R=R, s_lo=s_lo, s_hi=s_hi, k=k, C=_spread(rng, 64, 4096),
                    order=order)
    if kind == "retrieve":
        Q = _spread(rng, 1, 1000)
        N = _spread(rng, 50_000, max(60_000, min(8_000_000, 7.0e12 / (Q * d))))
        return dict(kind=kind, N=N, d=d, scan=scan, Q=Q, k=rng.choice([1, 20, rng.randint(1, 100)]), order=order)
    if kind == "knnlm":
        R, s, metric = _spread(rng, 1, 32), rng.randint(1, 8), rng.choice(["ip", "l2"])
        k = _spread(rng, 16, 1024)
        return dict(kind=kind, N=_spread(rng, 100_000, 6_000_000), d=rng.choice([1024, 512, 768]), metric=metric, R=R, s=s,
                    k=k, C=max(k, _spread(rng, 256, 2048)), n_next=10, order=order)
    if kind == "simple":
        return dict(kind=kind, N=_spread(rng, 20_000, 2_000_000), d=d, Q=_spread(rng, 1, 300), k=rng.randint(1, 32))
    return dict(kind="build", N=_spread(rng, 100_000, 4_000_000), d=d, metric=rng.choice(["ip", "l2"]), scan=scan)


def _strides(case):
    if case["kind"] == "knnlm":
        return [case["s"]] * case["R"]
    # part of the case and not of the seed, so that work() is that of every state
    return inputs.uniform_strides(case["R"], case["s_lo"], case["s_hi"], seed=7)


def _rows(case, seed, device="cuda"):
    N, d = case["N"], case["d"]
    X, _ = inputs.clustered_datastore(N, d, max(8, N // 320), seed, device=device, order=case.get("order", "iid"))
    return X


def prepare(case, seed):
    kind, N, d = case["kind"], case["N"], case["d"]
    dev = "cuda"
    st = dict(case=case)
    if kind == "build":
        st["X"] = _rows(case, seed)
        return st
    if kind == "knnlm":
        l2 = case["metric"] == "l2"
        # fp16 keys are their own scan copy; by squared distance the copy carries the norms
        keys, st["values"] = inputs.knnlm_datastore(N, d, max(8, N // 1200), seed, device=dev, order=case["order"])
        st["ds"] = B.Datastore.for_l2(keys) if l2 else B.Datastore(keys)
        st["T"] = 10.0 if l2 else 1.0
        sigma = 0.5
    elif kind == "simple":
        st["X"] = _rows(case, seed)
        Q = case["Q"]
        st["q"] = inputs.queries_near_rows(st["X"], inputs.pick_rows(N, Q, seed + 1), seed + 2)
        return st
    elif kind == "speculate":
        st["ds"] = B.Datastore(_rows(case, seed))
        sigma = 0.05
    else:
        st["ds"] = B.Datastore.from_fp32(_rows(case, seed), _TORCH[case["scan"]])
        sigma = 0.05
    ds = st["ds"]
    if kind == "retrieve":
        Q = case["Q"]
        st["q"] = inputs.queries_near_rows(ds.exact, inputs.pick_rows(N, Q, seed + 1), seed + 2, sigma=sigma)
        st["ws"] = B.alloc_workspace(Q, ds, case["k"])
        return st
    off = inputs.stride_offsets(_strides(case))
    Q, R, C = int(off[-1]), case["R"], case["C"]
    src = inputs.pick_rows(N, Q, seed + 1)
    st["q"] = inputs.queries_near_rows(ds.exact, src, seed + 2, sigma=sigma)
    # caches near the end of a generation: filled, half of the queries' source rows among the ids
    cids, clen = inputs.speculation_caches(N, R, C, off, src, None, seed + 3)
    st.update(off=off.to(dev), cids=cids.to(dev), clen=clen.to(dev))
    if kind == "knnlm":
        n = int(B.lib().ralm_cache_lookup_topk_workspace_bytes(Q, C))
        st["spec_ws"] = torch.empty(n + 256, dtype=torch.uint8, device=dev)
    else:
        st["spec_ws"] = torch.empty(max(Q, 1), dtype=torch.int64, device=dev)
    if kind != "speculate":
        st["head"] = torch.zeros(R, dtype=torch.int32, device=dev)
        st["ws"] = B.alloc_workspace(Q, ds, case["k"])
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "build":
        if case["metric"] == "l2":
            return B.Datastore.for_l2(st["X"], _TORCH[case["scan"]]).scan
        return B.Datastore.from_fp32(st["X"], _TORCH[case["scan"]]).scan
    if kind == "simple":
        return B.ralm_retrieve_topk(st["q"], st["X"], case["k"])
    ds = st["ds"]
    if kind == "retrieve":
        return B.ralm_retrieve_topk_ex(st["q"], ds, case["k"], workspace=st["ws"])
    cids, clen, q, off = st["cids"], st["clen"], st["q"], st["off"]
    if kind == "speculate":
        return B.ralm_cache_lookup(cids, clen, q, off, ds, workspace=st["spec_ws"])
    k, head = case["k"], st["head"]
    if kind == "round":
        spec, spec_sc = B.ralm_cache_lookup(cids, clen, q, off, ds, workspace=st["spec_ws"])
        ids, sc = B.ralm_retrieve_topk_ex(q, ds, k, workspace=st["ws"])
        miss = B.ralm_verify(spec, ids, off, true_stride=k)
        B.ralm_cache_insert(cids, clen, head, ids, off, ds.N, p=k, first_mismatch=miss)
        return spec, spec_sc, ids, sc, miss, cids, clen, head
    # neighbour language model: what is compared is the most probable token
    s_ids, s_sc = B.ralm_cache_lookup_topk(cids, clen, q, off, ds, min(k, case["C"]), workspace=st["spec_ws"])
    _, _, s_tok, s_p = B.ralm_knnlm_probs(s_ids, s_sc, st["values"], st["T"])
    ids, sc = B.ralm_retrieve_topk_ex(q, ds, k, workspace=st["ws"])
    tok, w, top, p = B.ralm_knnlm_probs(ids, sc, st["values"], st["T"])
    miss = B.ralm_verify(s_tok, top, off)
    B.ralm_cache_insert(cids, clen, head, ids, off, ds.N, p=min(8, k), n_next=case["n_next"], first_mismatch=miss)
    return s_ids, s_sc, s_tok, s_p, ids, sc, tok, w, top, p, miss, cids, clen, head


def work(case):
    """Every row that is scored read once, results written once; 2 flops per element and pair."""
    kind, N, d = case["kind"], case["N"], case["d"]
    if kind == "build":
        return {"bytes": N * d * 6 + (N * 16 if case["metric"] == "l2" else 0), "flops": 2 * N * d if case["metric"] == "l2" else 0}
    if kind == "simple":
        return {"bytes": N * d * 4 + case["Q"] * (d * 4 + case["k"] * 8), "flops": 2 * case["Q"] * N * d}
    if kind == "retrieve":
        return {"bytes": N * d * 2 + case["Q"] * (d * 4 + case["k"] * (8 + d * 4)), "flops": 2 * case["Q"] * N * d}
    strides = _strides(case)
    Q, R, C, es = sum(strides), case["R"], case["C"], 2 if kind == "knnlm" else 4
    b, f = R * min(C, N) * (d * es + 4) + Q * (d * 4 + 8), 2 * Q * C * d
    if kind != "speculate":
        b += N * d * 2 + Q * case["k"] * (8 + d * es) + R * C * 4
        f += 2 * Q * N * d
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Scores are double sums rounded once to fp32: another order of the sums flips a last bit (1.2e-7
    of the value at most) about once in 1e8 scores, and an id only where two scores then tie.
    Against torch's float64 products of the same rows all scores of the listed cases were equal, so
    the bounds are those of a few flipped last bits."""
    if case["kind"] == "build":
        # rounding is exact; by squared distance the sum of squares may round the other way
        return "exact" if case["metric"] == "ip" else {"rel": 1e-6, "max": 1e-2}
    if case["kind"] == "knnlm":
        # a last bit of a score near 1000 is 6e-5 in the exponent of its weight
        return {"rel": 2e-5, "max": 5e-4, "differ": 1e-5}
    return {"rel": 1.2e-7, "max": 2.4e-7, "differ": 1e-5}
