"""The calls that a speculative-decoding program makes of this library, as
cases to be timed: every retrieval path (exact scans of long and of PCA-short
keys, one query and batches, the inverted file), verification of retrieved
drafts (dense and through the loose trie), the steps of SEN between them, and
the datastore build.

A case is a dict of plain values; ``prepare`` makes the inputs and keeps what
a serving program keeps (the index handle, the workspace and the output
buffers), ``run`` is one pass through the public entry points of
``paper_2606_00021_amd.sense``.
"""
from __future__ import annotations

import math

import torch

from paper_2606_00021_amd import sense, synth

DEV = "cuda:0"
DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
MAX_KEY_BYTES = 1 << 34          # the largest listed store: 1M x 8192, 16-bit
MAX_LOGIT_BYTES = 16 * 64 * 8 * 32_000 * 4


def listed():
    return [
        # One decoding stream over a small datastore: the smallest retrieval,
        # where launches and latency count.
        dict(name="retrieve-1q-16k-d4096", kind="retrieve", n=16_384, d=4096, key="f16", nq=1,
             k=8, span=8, metric="cosine", query="f32", ragged=False),
        # The headline: one stream over a million hidden states.
        dict(name="retrieve-1q-1m-d4096", kind="retrieve", n=1_048_576, d=4096, key="bf16", nq=1,
             k=64, span=8, metric="cosine", query="f32", ragged=False),
        # A small server: 13 streams, an odd store size below the size where
        # batches are filtered, inner product, key-typed queries.
        dict(name="retrieve-13q-100k-d3584", kind="retrieve", n=100_003, d=3584, key="bf16",
             nq=13, k=32, span=10, metric="ip", query="bf16", ragged=True),
        # A loaded server with the keys of the largest model.
        dict(name="retrieve-64q-1m-d8192", kind="retrieve", n=1_048_576, d=8192, key="bf16",
             nq=64, k=128, span=12, metric="cosine", query="f32", ragged=False),
        # The paper's key geometry (4096 -> 64), exact search: each step
        # projects the batch's hidden states and searches their projections.
        dict(name="short-64q-1m-d64", kind="short", n=1_048_576, d=64, hidden=4096, key="bf16",
             nq=64, k=64, span=8, metric="cosine"),
        # The paper's retriever (IVF-PQ, 4096 lists, 32 probed, 16 codes) in
        # one decoding stream, the query projected in the step.
        dict(name="ivfpq-1q-1m-d64", kind="ivf", n=1_048_576, d=64, hidden=4096, nlist=4096,
             nprobe=32, m=16, nq=1, k=64, span=8, metric="cosine"),
        # The same on a loaded server.
        dict(name="ivfpq-64q-1m-d64", kind="ivf", n=1_048_576, d=64, hidden=4096, nlist=4096,
             nprobe=32, m=16, nq=64, k=64, span=8, metric="cosine"),
        # Verification of one stream's drafts, 16-bit logits, large vocabulary.
        dict(name="verify-64x8-v152k-bf16", kind="verify", groups=1, cand=64, m=8, vocab=152_064,
             logits="bf16", ragged=False),
        # Verification of 16 streams' drafts, fp32 logits, ragged drafts.
        dict(name="verify-16x64x8-v32k-f32", kind="verify", groups=16, cand=64, m=8,
             vocab=32_000, logits="f32", ragged=True),
        # SEN's steps after the static search: dynamic search over the
        # generated context, candidate selection, loose trie with the tree
        # attention mask, verification through the trie.
        dict(name="sen-64+16-v152k", kind="sen", ctx=4096, d=4096, nq=1, ks=64, kd=16, top=64,
             m=8, vocab=152_064, logits="bf16", cache=2048),
        # Datastore build: hidden states projected to the stored short keys.
        dict(name="project-store-262k-d4096", kind="project", n=262_144, din=4096, dout=64,
             x="bf16", out="bf16"),
        # Datastore build: list assignment and PQ encoding of short keys.
        dict(name="ivf-build-262k-d64", kind="build", n=262_144, d=64, nlist=4096, m=16,
             metric="cosine"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["retrieve", "retrieve", "short", "ivf", "verify", "sen", "project",
                       "build"])
    metric = rng.choice(["cosine", "cosine", "ip"])
    span = rng.randint(4, 16)
    if kind == "retrieve":
        d = 8 * _log(rng, 64, 1024)
        n = _log(rng, 16_384, min(4_194_304, MAX_KEY_BYTES // (2 * d)))
        key = rng.choice(["bf16", "f16"])
        return dict(kind=kind, n=n, d=d, key=key, nq=rng.choice([1, _log(rng, 1, 64)]),
                    k=_log(rng, 4, 128), span=span, metric=metric,
                    query=rng.choice(["f32", key]), ragged=rng.random() < 0.5)
    if kind == "short":
        return dict(kind=kind, n=_log(rng, 16_384, 1_048_576), d=8 * rng.randint(2, 8),
                    hidden=512 * rng.randint(2, 16), key=rng.choice(["bf16", "f16"]),
                    nq=_log(rng, 1, 64), k=_log(rng, 4, 128), span=span, metric=metric)
    if kind == "ivf":
        d = rng.choice([32, 64, 64, 128])
        # 256-entry codebooks are taken up to d = 64.
        m = rng.choice([0, d // 8, d // 4, d // 4]) if d <= 64 else 0
        return dict(kind=kind, n=_log(rng, 65_536, 1_048_576), d=d,
                    hidden=512 * rng.randint(2, 16), nlist=_log(rng, 256, 4096),
                    nprobe=_log(rng, 4, 64), m=m, nq=_log(rng, 1, 64), k=_log(rng, 4, 64),
                    span=span, metric=metric)
    if kind == "verify":
        logits = rng.choice(["f32", "f16", "bf16"])
        vocab = rng.choice([32_000, 128_256, 152_064, _log(rng, 32_000, 152_064)])
        m = rng.randint(4, 16)
        most = MAX_LOGIT_BYTES // (vocab * m * (4 if logits == "f32" else 2))
        groups = _log(rng, 1, min(16, most // 4))
        return dict(kind=kind, groups=groups, cand=_log(rng, 4, min(128, most // groups)), m=m,
                    vocab=vocab, logits=logits, ragged=rng.random() < 0.5)
    if kind == "sen":
        m = rng.randint(4, 12)
        ks, kd = _log(rng, 8, 128), _log(rng, 4, 32)
        vocab = rng.choice([32_000, 128_256, 152_064])
        nq = rng.randint(1, max(1, min(4, 256 // ks)))
        return dict(kind=kind, ctx=_log(rng, 64, 4096), d=8 * _log(rng, 64, 1024), nq=nq, ks=ks,
                    kd=kd, top=rng.randint(4, min(ks + kd, 64)), m=m, vocab=vocab,
                    logits=rng.choice(["bf16", "f16"]), cache=_log(rng, 1024, 4096))
    if kind == "project":
        din = 512 * rng.randint(1, 16)
        x = rng.choice(["bf16", "f16"])
        return dict(kind=kind, n=_log(rng, 64, min(262_144, (1 << 31) // (2 * din))), din=din,
                    dout=8 * rng.randint(2, 16), x=x, out=rng.choice([x, "f32"]))
    d = rng.choice([32, 64, 64])
    return dict(kind=kind, n=_log(rng, 16_384, 262_144), d=d,
                nlist=_log(rng, 256, 4096), m=rng.choice([d // 8, d // 4]), metric=metric)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV)


def _clustered(g, n, d, dtype, n_clusters, noise, outliers, normalize=False):
    """Stored keys: clusters of near rows; hidden states with a few channels
    of large magnitude (outliers > 0), projections L2-normalised.  Cluster
    sizes are skewed, as those of retrieved text are.  Returns the keys, each
    row's cluster and the cluster centres."""
    cen = _randn(g, n_clusters, d)
    weight = torch.exp(0.5 * _randn(g, n_clusters))
    edges = torch.cumsum(weight / weight.sum(), 0)
    label = torch.searchsorted(edges, torch.rand(n, generator=g, device=DEV)).clamp_(
        max=n_clusters - 1)
    channels = torch.randperm(d, generator=g, device=DEV)[:outliers]
    keys = torch.empty((n, d), dtype=dtype, device=DEV)
    step = max(1, (1 << 28) // d)
    for r in range(0, n, step):
        x = cen[label[r:r + step]]
        x.add_(_randn(g, *x.shape), alpha=noise)
        x[:, channels] *= 20.0
        if normalize:
            x /= x.norm(dim=1, keepdim=True)
        keys[r:r + step] = x.to(dtype)
    return keys, label, cen


def _spans(g, n, span, ragged):
    spans = torch.randint(0, 152_064, (n, span), generator=g, device=DEV, dtype=torch.int32)
    if not ragged:
        return spans, None
    return spans, torch.randint(0, span + 1, (n,), generator=g, device=DEV, dtype=torch.int32)


def _near(g, keys, nq, noise):
    rows = torch.randint(0, keys.shape[0], (nq,), generator=g, device=DEV)
    x = keys[rows].float()
    return (x + noise * _randn(g, *x.shape)).contiguous()


def _workspace(nbytes):
    return torch.empty(max(nbytes, 1), dtype=torch.uint8, device=DEV)


def _hits(nq, k, span):
    return (torch.empty((nq, k), dtype=torch.int64, device=DEV),
            torch.empty((nq, k), dtype=torch.float32, device=DEV),
            torch.empty((nq, k, span), dtype=torch.int32, device=DEV),
            torch.empty((nq, k), dtype=torch.int32, device=DEV))


def _basis(g, d_out, d_in):
    """Orthonormal principal directions and a mean, as a PCA fit gives them."""
    q, _ = torch.linalg.qr(_randn(g, d_in, d_out).cpu())
    return q.T.contiguous().to(DEV), (0.1 * _randn(g, d_in)).contiguous()


def _hidden(basis, mean, target):
    """Hidden states whose projections are `target` (plus what the basis does
    not span): what a decoder holds before it projects."""
    g = _gen(int(target.shape[0]))
    rest = 0.3 * _randn(g, target.shape[0], basis.shape[1])
    return (mean + target @ basis + rest - rest @ basis.T @ basis).contiguous()


def _logits(g, shape, vocab, dtype, tokens):
    """Rows ~ N(0, 2^2) with the draft token raised at 60 % of the positions,
    by an amount that takes the row from flat to nearly certain."""
    out = torch.empty((*shape, vocab), dtype=dtype, device=DEV).view(-1, vocab)
    tok = tokens.reshape(-1).long()
    up = (torch.rand(tok.numel(), generator=g, device=DEV) < 0.6) * (
        6.0 + 10.0 * torch.rand(tok.numel(), generator=g, device=DEV))
    step = max(1, (1 << 28) // vocab)
    for r in range(0, out.shape[0], step):
        x = _randn(g, min(step, out.shape[0] - r), vocab).mul_(2.0)
        x.scatter_add_(1, tok[r:r + step, None], up[r:r + step, None])
        out[r:r + step] = x.to(dtype)
    return out.view(*shape, vocab)


def prepare(case, seed):
    g = _gen(seed)
    c = dict(case)
    s = {"case": c}
    kind = c["kind"]
    if kind in ("retrieve", "short"):
        short = kind == "short"
        keys, _, _ = _clustered(g, c["n"], c["d"], DT[c["key"]], max(16, c["n"] // 256), 0.3,
                                0 if short else 4, normalize=short)
        spans, lens = _spans(g, c["n"], c["span"], c.get("ragged", False))
        s["index"] = sense.sense_build_index(keys, spans, lens, metric=c["metric"])
        s["keys"] = keys
        near = _near(g, keys, c["nq"], 0.02 if short else 0.05)
        if short:
            s["basis"], s["mean"] = _basis(g, c["d"], c["hidden"])
            s["x"] = _hidden(s["basis"], s["mean"], near)
            s["q"] = torch.empty((c["nq"], c["d"]), dtype=torch.float32, device=DEV)
            s["pws"] = _workspace(sense.sense_project_workspace_size(
                s["basis"], torch.float32, c["nq"], s["mean"]))
        else:
            s["q"] = near.to(DT[c["query"]])
        s["ws"] = _workspace(sense.sense_retrieve_workspace_size(s["index"], c["nq"], c["k"]))
        s["out"] = _hits(c["nq"], c["k"], c["span"])
    elif kind == "ivf":
        keys, label, cen = _clustered(g, c["n"], c["d"], torch.bfloat16, c["nlist"], 0.3, 0,
                                      normalize=True)
        cen = (cen / cen.norm(dim=1, keepdim=True)).contiguous()
        spans, _ = _spans(g, c["n"], c["span"], False)
        near = _near(g, keys, c["nq"], 0.02)
        lists = label.to(torch.int32)
        books = codes = None
        if c["m"]:
            # Residuals of unit keys around unit centres: about N(0, 0.3^2 / d) each.
            books = (0.3 / math.sqrt(c["d"]) * _randn(g, c["m"], 256, c["d"] // c["m"])).contiguous()
            codes = torch.randint(0, 256, (c["n"], c["m"]), generator=g, device=DEV,
                                  dtype=torch.uint8)
        s["index"] = sense.sense_build_ivf_index(
            None if c["m"] else keys, spans, cen, lists, metric=c["metric"], codebooks=books,
            codes=codes, key_dtype=torch.bfloat16)
        s["truth"] = (None if c["m"] else keys, lists, cen, books, codes)
        s["basis"], s["mean"] = _basis(g, c["d"], c["hidden"])
        s["x"] = _hidden(s["basis"], s["mean"], near)
        s["q"] = torch.empty((c["nq"], c["d"]), dtype=torch.float32, device=DEV)
        s["pws"] = _workspace(sense.sense_project_workspace_size(
            s["basis"], torch.float32, c["nq"], s["mean"]))
        s["ws"] = _workspace(sense.sense_ivf_search_workspace_size(
            s["index"], c["nq"], c["k"], c["nprobe"]))
        s["out"] = _hits(c["nq"], c["k"], c["span"])
    elif kind == "verify":
        n = c["groups"] * c["cand"]
        s["drafts"] = torch.randint(0, c["vocab"], (n, c["m"]), generator=g, device=DEV,
                                    dtype=torch.int32)
        s["len"] = torch.randint(0, c["m"] + 1, (n,), generator=g, device=DEV,
                                 dtype=torch.int32) if c["ragged"] else None
        s["logits"] = _logits(g, (n, c["m"]), c["vocab"], DT[c["logits"]], s["drafts"])
        s["ws"] = _workspace(sense.sense_soft_gate_verify_workspace_size(n, c["m"], c["vocab"]))
        s["out"] = _gate_out(n, c["m"], c["groups"])
    elif kind == "sen":
        _prepare_sen(g, c, s, seed)
    elif kind == "project":
        # Hidden states of n_clusters contexts with a few large channels.
        x, _, _ = _clustered(g, c["n"], c["din"], DT[c["x"]], 256, 0.3, 4)
        s["x"] = x
        s["basis"], s["mean"] = _basis(g, c["dout"], c["din"])
        s["out"] = torch.empty((c["n"], c["dout"]), dtype=DT[c["out"]], device=DEV)
        s["ws"] = _workspace(sense.sense_project_workspace_size(s["basis"], x.dtype, c["n"],
                                                                s["mean"]))
    else:
        keys, _, cen = _clustered(g, c["n"], c["d"], torch.bfloat16, c["nlist"], 0.5, 0,
                                  normalize=True)
        s["keys"], s["cen"] = keys, (cen / cen.norm(dim=1, keepdim=True)).contiguous()
        s["books"] = (0.5 / math.sqrt(c["d"]) * _randn(g, c["m"], 256,
                                                       c["d"] // c["m"])).contiguous()
        s["lists"] = torch.empty(c["n"], dtype=torch.int32, device=DEV)
        s["codes"] = torch.empty((c["n"], c["m"]), dtype=torch.uint8, device=DEV)
    return s


def _gate_out(n, m, groups):
    return {"accept_len": torch.empty(n, dtype=torch.int32, device=DEV),
            "best": torch.empty(groups, dtype=torch.int32, device=DEV),
            "gate_score": torch.empty((n, m), dtype=torch.float32, device=DEV),
            "masks": torch.empty((n, m), dtype=torch.uint8, device=DEV),
            "rank": torch.empty((n, m), dtype=torch.int32, device=DEV)}


def _prepare_sen(g, c, s, seed):
    nq, m, top, vocab = c["nq"], c["m"], c["top"], c["vocab"]
    # The dynamic cache after ctx generated positions, which revisit topics.
    hidden, _, _ = _clustered(g, c["ctx"], c["d"], torch.float32, 64, 0.3, 4)
    tokens = torch.randint(0, vocab, (c["ctx"],), generator=g, device=DEV, dtype=torch.int32)
    dyn = sense.sense_build_dynamic_index(c["d"], c["ctx"], m, torch.bfloat16, "cosine")
    sense.sense_index_append(dyn, hidden, tokens)
    s["dyn"], s["hidden"] = dyn, hidden
    s["q"] = _near(g, hidden, nq, 0.05)
    s["dws"] = _workspace(sense.sense_retrieve_workspace_size(dyn, nq, c["kd"]))
    s["dout"] = _hits(nq, c["kd"], m)
    # The static search's hits: continuations that share prefixes, as those of
    # neighbouring rows do, similarities that fall with the rank.
    drafts, lens = synth.make_drafts(seed, nq * c["ks"], m, vocab, DEV, ragged=False,
                                     n_groups=nq)
    score = torch.sort(0.6 + 0.4 * torch.rand((nq, c["ks"]), generator=g, device=DEV), dim=1,
                       descending=True).values
    s["static"] = (score.contiguous(), drafts.view(nq, c["ks"], m), lens.view(nq, c["ks"]))
    s["anchors"] = drafts.view(nq, c["ks"], m)[:, 0, 0].contiguous()
    s["sel"] = (torch.empty((nq, top, m), dtype=torch.int32, device=DEV),
                torch.empty((nq, top), dtype=torch.int32, device=DEV),
                torch.empty((nq, top), dtype=torch.int32, device=DEV),
                torch.empty((nq, top), dtype=torch.float32, device=DEV))
    nodes = top * m
    s["full"] = {"dtype": torch.bfloat16, "prefix_len": c["cache"] - nodes, "cache_len": c["cache"]}
    dyn_hits = sense.sense_retrieve(dyn, s["q"], c["kd"], workspace=s["dws"], out=s["dout"])
    sel = _select(s, dyn_hits)
    s["trie"] = sense.sense_build_loose_trie(sel[0].view(nq * top, m), sel[1].view(-1),
                                             n_groups=nq, full_mask=s["full"])
    # The target model's rows for this tree: row 1 + parent(u) judges node u.
    tree = s["trie"]
    judged = torch.zeros((nq, 1 + nodes), dtype=torch.int64, device=DEV)
    judged.scatter_reduce_(1, 1 + tree["tree_parent"].long(),
                           tree["tree_tokens"].long().clamp_(min=0), "amax")
    s["logits"] = _logits(g, (nq, 1 + nodes), vocab, DT[c["logits"]], judged)
    s["rows"] = int(tree["tree_len"].sum())
    s["ws"] = _workspace(sense.sense_soft_gate_verify_tree_workspace_size(nq * top, m, vocab, nq))
    s["out"] = _gate_out(nq * top, m, nq)


def _select(s, dyn_hits):
    return sense.sense_select_candidates(
        s["static"], (dyn_hits[1], dyn_hits[2], dyn_hits[3]), s["anchors"], s["case"]["top"],
        100.0, 1.0, 0.05, out=s["sel"])


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "retrieve":
        return sense.sense_retrieve(s["index"], s["q"], c["k"], workspace=s["ws"], out=s["out"])
    if kind == "short":
        q = sense.sense_project(s["x"], s["basis"], s["mean"], out=s["q"], workspace=s["pws"])
        return sense.sense_retrieve(s["index"], q, c["k"], workspace=s["ws"], out=s["out"])
    if kind == "ivf":
        q = sense.sense_project(s["x"], s["basis"], s["mean"], out=s["q"], workspace=s["pws"])
        return sense.sense_ivf_search(s["index"], q, c["k"], c["nprobe"], workspace=s["ws"],
                                      out=s["out"])
    if kind == "verify":
        return sense.sense_soft_gate_verify(s["logits"], s["drafts"], s["len"],
                                            n_groups=c["groups"], workspace=s["ws"],
                                            out=s["out"])
    if kind == "sen":
        nq, m, top = c["nq"], c["m"], c["top"]
        hits = sense.sense_retrieve(s["dyn"], s["q"], c["kd"], workspace=s["dws"], out=s["dout"])
        sel = _select(s, hits)
        trie = sense.sense_build_loose_trie(sel[0].view(nq * top, m), sel[1].view(-1),
                                            n_groups=nq, full_mask=s["full"], out=s["trie"])
        gate = sense.sense_soft_gate_verify_tree(s["logits"], trie, n_groups=nq,
                                                 workspace=s["ws"], out=s["out"])
        return [hits, sel, trie, gate]
    if kind == "project":
        return sense.sense_project(s["x"], s["basis"], s["mean"], out=s["out"],
                                   workspace=s["ws"])
    lists = sense.sense_ivf_assign(s["keys"], s["cen"], c["metric"], out=s["lists"])
    codes = sense.sense_pq_encode(s["keys"], s["cen"], lists, s["books"], out=s["codes"])
    return lists, codes


def work(case):
    c = case
    kind = c["kind"]
    if kind in ("retrieve", "short"):
        hits = c["nq"] * c["k"] * (8 + 4 + 4 + 2 * 4 * c["span"])
        b = c["n"] * (2 * c["d"] + (4 if c["metric"] == "cosine" else 0)) + hits
        f = 2 * c["nq"] * c["n"] * c["d"]
        if kind == "short":
            b += 4 * c["hidden"] * (c["nq"] + c["d"] + 1)
            f += 2 * c["nq"] * c["hidden"] * c["d"]
        else:
            b += c["nq"] * c["d"] * (4 if c["query"] == "f32" else 2)
        return {"bytes": b, "flops": f}
    if kind == "ivf":
        # A probed list is read once for the batch: at most every row.
        rows = min(c["n"], c["nq"] * c["nprobe"] * c["n"] // c["nlist"])
        each = c["m"] + 4 if c["m"] else 2 * c["d"] + 8
        hits = c["nq"] * c["k"] * (8 + 4 + 4 + 2 * 4 * c["span"])
        b = rows * each + 4 * c["nlist"] * (c["d"] + 1) + hits + (1024 * c["d"] if c["m"] else 0)
        b += 4 * c["hidden"] * (c["nq"] + c["d"] + 1)
        per = c["m"] if c["m"] else 2 * c["d"]
        f = c["nq"] * (2 * c["nlist"] * c["d"] + c["nprobe"] * c["n"] // c["nlist"] * per
                       + 2 * c["hidden"] * c["d"])
        return {"bytes": b, "flops": f}
    if kind == "verify":
        rows = c["groups"] * c["cand"] * c["m"] / (2 if c["ragged"] else 1)
        e = 4 if c["logits"] == "f32" else 2
        return {"bytes": int(rows * (c["vocab"] * e + 13)), "flops": int(rows * c["vocab"] * 5)}
    if kind == "sen":
        # About seven tenths of the drafts' tokens are nodes of the trie.
        rows = int(0.7 * c["nq"] * c["top"] * c["m"])
        b = c["ctx"] * (2 * c["d"] + 4) + 4 * c["nq"] * c["d"]
        b += rows * (2 * c["vocab"] + 2 * c["cache"] + 40)
        b += c["nq"] * (c["ks"] + c["kd"] + 2 * c["top"]) * (4 * c["m"] + 8)
        return {"bytes": b, "flops": 2 * c["nq"] * c["ctx"] * c["d"] + 5 * rows * c["vocab"]}
    if kind == "project":
        b = c["n"] * (2 * c["din"] + c["dout"] * (4 if c["out"] == "f32" else 2))
        return {"bytes": b + 4 * c["din"] * (c["dout"] + 1),
                "flops": 2 * c["n"] * c["din"] * c["dout"]}
    b = 2 * c["n"] * 2 * c["d"] + 2 * 4 * c["nlist"] * c["d"] + 1024 * c["d"]
    b += c["n"] * (4 + 4 + c["m"])
    return {"bytes": b, "flops": 2 * c["n"] * c["d"] * (c["nlist"] + 256)}


def tolerance(case):
    """Scores are 32-bit sums (1e-7 to 2e-6 off their 64-bit values).  Two rows
    whose scores differ by less than that may change places, which moves whole
    values (ids, drafts)."""
    kind = case["kind"]
    if kind == "project":
        # One rounding of the output type where it has 16 bits.
        # 32-bit results of 16-bit rows: the basis in two halves of the row type.
        return {"rel": {"bf16": 3e-3, "f16": 4e-4, "f32": 2e-5}[case["out"]], "max": 0.02}
    if kind == "build":
        return {"rel": 8e-6, "differ": 1e-3}
    return {"rel": 8e-6, "differ": 1e-2}


def _scores64(keys, q, cosine):
    """nq x n fp64 similarities, the keys taken in pieces."""
    q = q.double()
    if cosine:
        q = q / q.norm(dim=1, keepdim=True)
    out = torch.empty((q.shape[0], keys.shape[0]), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // keys.shape[1])
    for r in range(0, keys.shape[0], step):
        x = keys[r:r + step].double()
        y = q @ x.T
        out[:, r:r + step] = y / x.norm(dim=1) if cosine else y
    return out


def _project64(x, basis, mean):
    y = (x.double() - mean.double()) @ basis.double().T
    return y / y.norm(dim=1, keepdim=True)


def _gate64(rows, normalize):
    out = []
    for r in range(0, rows.shape[0], 512):
        p = torch.log_softmax(rows[r:r + 512].double(), dim=1)
        out.append(-(p.exp() * p).sum(dim=1) / normalize)
    return torch.cat(out)


def exact(case, seed):
    s = prepare(case, seed)
    c = s["case"]
    kind = c["kind"]
    cosine = c.get("metric") == "cosine"
    if kind in ("retrieve", "short"):
        q = _project64(s["x"], s["basis"], s["mean"]) if kind == "short" else s["q"]
        return None, torch.topk(_scores64(s["keys"], q, cosine), c["k"]).values, None, None
    if kind == "ivf":
        keys, lists, cen, books, codes = s["truth"]
        q = _project64(s["x"], s["basis"], s["mean"])
        probe = torch.topk(_scores64(cen, q, cosine), c["nprobe"]).indices
        if c["m"]:
            keys = cen[lists.long()].double()
            for j in range(c["m"]):
                w = c["d"] // c["m"]
                keys[:, j * w:(j + 1) * w] += books[j].double()[codes[:, j].long()]
        if c["m"] and cosine:
            q = q / q.norm(dim=1, keepdim=True)
        sc = q @ keys.T if c["m"] else _scores64(keys, q, cosine)
        hit = torch.zeros((c["nq"], c["nlist"]), dtype=torch.bool, device=DEV)
        hit.scatter_(1, probe, True)
        for i in range(c["nq"]):
            sc[i].masked_fill_(~hit[i][lists.long()], -math.inf)
        best = torch.topk(sc, c["k"]).values
        return None, torch.where(torch.isinf(best), math.nan, best), None, None
    if kind == "verify":
        n, m = s["drafts"].shape
        e = _gate64(s["logits"].view(n * m, -1), math.log(c["vocab"])).view(n, m)
        if c["ragged"]:
            e = e * (torch.arange(m, device=DEV)[None, :] < s["len"][:, None])
        return {"accept_len": None, "best": None, "gate_score": e, "masks": None, "rank": None}
    if kind == "sen":
        near = torch.topk(_scores64(s["hidden"].bfloat16(), s["q"], True), c["kd"]).values
        return [[None, near, None, None], None, None, None]
    if kind == "project":
        return _project64(s["x"], s["basis"], s["mean"])
    return None
