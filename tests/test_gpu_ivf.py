"""GPU parity of the inverted file (the ANN retriever of Sec. 3.2 Eq. 7 as
the implementation details configure it: IVF with nprobe lists searched,
PQ-coded residuals).

Assignment and encoding: identical to the oracle except where the oracle's
two best choices are within a relative 1e-5 (then the GPU's choice must be
one of those near ties).  Search: the GPU index is built from the oracle's
own list ids and codes, so both sides search the same index; probes are the
oracle's up to near ties of the coarse scores, and results follow the
retrieval rules over the candidates' oracle scores.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_00021_amd import sense, synth
from parity import check_topk, host_bits

pytestmark = pytest.mark.gpu

DEV = "cuda"


def store(n, d, kdt, seed, clusters=64):
    w = synth.scaled(synth.WORKLOADS["tiny-16k-d4096"], n=n, d=d, key_dtype=kdt,
                     n_clusters=clusters, n_outliers=2)
    ds = synth.make_datastore(w, seed, DEV)
    return w, ds


def decoded(keys):
    return keys.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("n,d,kdt,nlist,metric", [
    (20000, 64, "bf16", 256, "cosine"),
    (7001, 32, "f16", 100, "ip"),
    (3000, 128, "bf16", 37, "cosine"),
])
def test_assign_matches_oracle(n, d, kdt, nlist, metric):
    print(f"[ivf-assign] n={n} d={d} nlist={nlist} {metric}", flush=True)
    w, ds = store(n, d, kdt, 3)
    cen, _ = synth.fit_ivf(ds.keys, 3, nlist, iters=2)
    got = sense.sense_ivf_assign(ds.keys, cen, metric).cpu().numpy()
    torch.cuda.synchronize()
    lists, best = oracle.ivf_assign(host_bits(ds.keys), kdt, cen.cpu().numpy(), metric)
    x = decoded(ds.keys)
    c = cen.cpu().numpy().astype(np.float64)
    s = x @ c.T
    if metric == "cosine":
        s = s / (np.linalg.norm(x, axis=1, keepdims=True) * np.linalg.norm(c, axis=1))
    diff = np.flatnonzero(got != lists)
    for i in diff:
        assert s[i, got[i]] >= best[i] - 1e-5 * abs(best[i]), f"row {i}: not a near tie"
    assert diff.size <= max(3, n // 1000)


@pytest.mark.parametrize("d,m,ksub", [(64, 16, 256), (32, 8, 64), (128, 8, 16)])
def test_pq_encode_matches_oracle(d, m, ksub):
    print(f"[pq-encode] d={d} m={m} ksub={ksub}", flush=True)
    w, ds = store(6000, d, "bf16", 4)
    cen, books = synth.fit_ivf(ds.keys, 4, 64, pq_m=m, ksub=ksub, iters=2)
    lists = sense.sense_ivf_assign(ds.keys, cen, "cosine")
    got = sense.sense_pq_encode(ds.keys, cen, lists, books).cpu().numpy()
    torch.cuda.synchronize()
    lh = lists.cpu().numpy()
    want = oracle.pq_encode(host_bits(ds.keys), "bf16", cen.cpu().numpy(), lh, books.cpu().numpy())
    x = decoded(ds.keys)
    r = x - cen.cpu().numpy().astype(np.float64)[lh]
    cb = books.cpu().numpy().astype(np.float64)
    dsub = d // m
    for i, j in zip(*np.nonzero(got != want)):
        sl = r[i, j * dsub:(j + 1) * dsub]
        dg = np.sum((sl - cb[j, got[i, j]]) ** 2)
        dw = np.sum((sl - cb[j, want[i, j]]) ** 2)
        assert dg <= dw + 1e-5 * max(dw, 1e-12), f"({i},{j}) not a near tie"
    assert (got != want).sum() <= max(3, got.size // 2000)


def candidate_scores(x, lists, probe, q, metric, cen=None, codes=None, books=None):
    """Oracle-side score of every row for the given probe set (-inf outside),
    the same formulas as the oracle's search, in numpy."""
    inside = np.isin(lists, probe)
    if codes is None:
        s = x @ q
        if metric == "cosine":
            s = s / (np.linalg.norm(x, axis=1) * np.linalg.norm(q))
    else:
        m = books.shape[0]
        rec = cen[lists] + np.concatenate([books[j][codes[:, j]] for j in range(m)], axis=1)
        u = q / np.linalg.norm(q) if metric == "cosine" else q
        s = rec @ u
    return np.where(inside, s, -np.inf)


IVF_CASES = [
    # n, d, key dtype, nlist, nprobe, k, n_queries, metric, pq (m, ksub) or None
    (30000, 64, "bf16", 256, 16, 32, 3, "cosine", None),
    (30000, 64, "bf16", 256, 32, 64, 2, "cosine", (16, 256)),
    (12000, 32, "f16", 64, 8, 16, 5, "ip", None),
    (12000, 32, "f16", 64, 8, 16, 4, "ip", (8, 64)),
    (5000, 128, "bf16", 50, 50, 20, 1, "cosine", None),      # nprobe = nlist
    (4000, 64, "bf16", 400, 2, 100, 2, "cosine", None),       # fewer candidates than k
    # enough queries that a PQ scan block takes several probes of its query
    # (16, 32 and 64 codes per row in 16-byte words; 8 codes, byte loads)
    (30000, 64, "bf16", 256, 32, 64, 40, "cosine", (16, 256)),
    (20000, 128, "bf16", 128, 64, 32, 24, "ip", (32, 128)),
    (12000, 64, "f16", 64, 48, 16, 16, "ip", (64, 256)),
    (12000, 32, "f16", 64, 40, 16, 20, "cosine", (8, 64)),
]


@pytest.mark.parametrize("case", IVF_CASES, ids=[str(i) for i in range(len(IVF_CASES))])
def test_ivf_search_matches_oracle(case):
    n, d, kdt, nlist, nprobe, k, nq, metric, pq = case
    print(f"[ivf-search] case={case}", flush=True)
    w, ds = store(n, d, kdt, 7)
    q, _ = synth.make_queries(w, ds, 7, n_queries=nq)
    cen, books = synth.fit_ivf(ds.keys, 7, nlist, pq_m=pq[0] if pq else 0,
                               ksub=pq[1] if pq else 256, iters=3)
    kb = host_bits(ds.keys)
    cen_h = cen.cpu().numpy().astype(np.float64)
    lists, _ = oracle.ivf_assign(kb, kdt, cen_h, metric)
    codes = books_h = None
    if pq:
        books_h = books.cpu().numpy().astype(np.float64)
        codes = oracle.pq_encode(kb, kdt, cen_h, lists, books_h)
    index = sense.sense_build_ivf_index(
        ds.keys if not pq else None, ds.spans, cen, torch.from_numpy(lists).to(DEV),
        metric=metric, codebooks=books if pq else None,
        codes=torch.from_numpy(codes).to(DEV) if pq else None, key_dtype=ds.keys.dtype)
    ids, sc, dr, dl, probe = sense.sense_ivf_search(index, q, k, nprobe, want_probe=True)
    torch.cuda.synchronize()
    x = decoded(ds.keys)
    qh = q.cpu().numpy().astype(np.float64)
    spans = ds.spans.cpu().numpy()
    for qq in range(nq):
        o_probe, coarse, o_ids, o_sc = oracle.ivf_search(
            qh[qq], cen_h, lists, nprobe, k, metric, keys=None if pq else kb, key_dtype=kdt,
            codes=codes, codebooks=books_h)
        g_probe = probe[qq].cpu().numpy()
        # probes: the oracle's top-nprobe lists up to near ties of the coarse score
        kth = coarse[o_probe[-1]]
        assert len(set(g_probe.tolist())) == nprobe
        for l in set(g_probe.tolist()) - set(o_probe.tolist()):
            assert coarse[l] >= kth - 1e-5 * abs(kth), f"query {qq}: list {l} is not a near tie"
        cs = candidate_scores(x, lists, g_probe, qh[qq], metric, cen_h, codes, books_h)
        g_ids = ids[qq].cpu().numpy()
        n_cand = int(np.isfinite(cs).sum())
        real = min(k, n_cand)
        if real < k:                              # fewer candidates than k
            assert (g_ids[real:] == -1).all() and np.isnan(sc[qq, real:].cpu().numpy()).all()
            assert (dl[qq, real:].cpu().numpy() == 0).all()
        if real > 0:
            check_topk(g_ids[:real], sc[qq, :real].cpu().numpy(), cs, real)
            if set(g_probe.tolist()) == set(o_probe.tolist()):
                assert set(g_ids[:real].tolist()) <= set(
                    np.flatnonzero(np.isfinite(cs)).tolist())
                np.testing.assert_allclose(np.sort(o_sc[:real]), np.sort(cs[o_ids[:real]]),
                                           rtol=1e-12)
            assert np.array_equal(dr[qq, :real].cpu().numpy(), spans[g_ids[:real]])
    index.close()


def exact_per_query(flat, q, k):
    """The exact retrieval one query at a time: the single-query scan sums a
    row in fp32 like the inverted file's list scan (a batch would take the
    matrix cores, whose hi + lo split rounds differently)."""
    parts = [sense.sense_retrieve(flat, q[i:i + 1].contiguous(), k) for i in range(q.shape[0])]
    torch.cuda.synchronize()
    return (torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts]),
            torch.cat([p[2] for p in parts]))


def test_ivf_flat_probing_everything_equals_exact_retrieval():
    w, ds = store(8000, 64, "bf16", 9)
    q, _ = synth.make_queries(w, ds, 9, n_queries=2)
    cen, _ = synth.fit_ivf(ds.keys, 9, 32, iters=2)
    lists = sense.sense_ivf_assign(ds.keys, cen, "cosine")
    index = sense.sense_build_ivf_index(ds.keys, ds.spans, cen, lists)
    ids, sc, dr, _ = sense.sense_ivf_search(index, q, 40, 32)
    flat = sense.sense_build_index(ds.keys, ds.spans)
    e_ids, e_sc, e_dr = exact_per_query(flat, q, 40)
    assert torch.equal(ids, e_ids)
    assert torch.allclose(sc, e_sc, rtol=1e-6, atol=0)
    assert torch.equal(dr, e_dr)
    index.close()
    flat.close()


@pytest.mark.parametrize("k", [200, 1024])
def test_ivf_flat_probing_everything_many_rounds(k):
    """40000 candidates per query: the candidate selection walks them in
    several rounds (running top k plus the next keys); the result must still
    be the exact retrieval, order, scores and drafts."""
    w, ds = store(40000, 32, "bf16", 13)
    q, _ = synth.make_queries(w, ds, 13, n_queries=3)
    cen, _ = synth.fit_ivf(ds.keys, 13, 64, iters=2)
    lists = sense.sense_ivf_assign(ds.keys, cen, "cosine")
    index = sense.sense_build_ivf_index(ds.keys, ds.spans, cen, lists)
    ids, sc, dr, _ = sense.sense_ivf_search(index, q, k, 64)
    flat = sense.sense_build_index(ds.keys, ds.spans)
    e_ids, e_sc, e_dr = exact_per_query(flat, q, k)
    assert torch.equal(ids, e_ids)
    assert torch.allclose(sc, e_sc, rtol=1e-6, atol=0)
    assert torch.equal(dr, e_dr)
    index.close()
    flat.close()


@pytest.mark.parametrize("n", [4096, 4097, 8192, 8193, 16384, 16385, 20000])
def test_ivf_candidate_counts_at_selection_boundaries(n):
    """Probing every list makes the candidate count n: the candidate
    selection takes 4, 8 or 16 keys per thread by the count (one round up to
    16384, then several); each must equal the exact retrieval."""
    w, ds = store(n, 32, "bf16", 17)
    q, _ = synth.make_queries(w, ds, 17, n_queries=2)
    cen, _ = synth.fit_ivf(ds.keys, 17, 16, iters=2)
    lists = sense.sense_ivf_assign(ds.keys, cen, "cosine")
    index = sense.sense_build_ivf_index(ds.keys, ds.spans, cen, lists)
    ids, sc, dr, _ = sense.sense_ivf_search(index, q, 100, 16)
    flat = sense.sense_build_index(ds.keys, ds.spans)
    e_ids, e_sc, e_dr = exact_per_query(flat, q, 100)
    assert torch.equal(ids, e_ids)
    assert torch.allclose(sc, e_sc, rtol=1e-6, atol=0)
    assert torch.equal(dr, e_dr)
    index.close()
    flat.close()


def test_full_size_ivf_pq_bench_shape():
    """IVF-PQ at the bench's shape: 1M x 64 bf16 keys, nlist 4096, nprobe 32,
    pq_m 16 (ksub 256), k = 64, searched with one query and with a batch of
    64 (the launch configurations timed), on an index built from the
    oracle's own list ids and codes; each query as in the small cases."""
    n, d, nlist, nprobe, m, k = 1 << 20, 64, 4096, 32, 16, 64
    print(f"[ivf] full size n={n} d={d} nlist={nlist} nprobe={nprobe} pq_m={m}", flush=True)
    w, ds = store(n, d, "bf16", 23, clusters=4096)
    q, _ = synth.make_queries(w, ds, 23, n_queries=64)
    cen, books = synth.fit_ivf(ds.keys, 23, nlist, pq_m=m)
    kb = host_bits(ds.keys)
    cen_h = cen.cpu().numpy().astype(np.float64)
    books_h = books.cpu().numpy().astype(np.float64)
    lists, _ = oracle.ivf_assign(kb, "bf16", cen_h, "cosine")
    codes = oracle.pq_encode(kb, "bf16", cen_h, lists, books_h)
    print("[ivf] oracle assignment and codes done", flush=True)
    index = sense.sense_build_ivf_index(None, ds.spans, cen, torch.from_numpy(lists).to(DEV),
                                        codebooks=books, codes=torch.from_numpy(codes).to(DEV),
                                        key_dtype=ds.keys.dtype)
    qh = q.cpu().numpy().astype(np.float64)
    spans = ds.spans.cpu().numpy()
    # reconstructed keys (centroid + codewords), the PQ scores' row vectors
    rec = cen_h[lists] + np.concatenate([books_h[j][codes[:, j]] for j in range(m)], axis=1)
    for nq in (1, 64):
        ids, sc, dr, dl, probe = sense.sense_ivf_search(index, q[:nq], k, nprobe,
                                                        want_probe=True)
        torch.cuda.synchronize()
        for qq in range(nq):
            o_probe, coarse, o_ids, o_sc = oracle.ivf_search(
                qh[qq], cen_h, lists, nprobe, k, "cosine", codes=codes, codebooks=books_h)
            g_probe = probe[qq].cpu().numpy()
            kth = coarse[o_probe[-1]]
            assert len(set(g_probe.tolist())) == nprobe
            for l in set(g_probe.tolist()) - set(o_probe.tolist()):
                assert coarse[l] >= kth - 1e-5 * abs(kth), f"query {qq}: list {l} not a near tie"
            inside = np.isin(lists, g_probe)
            u = qh[qq] / np.linalg.norm(qh[qq])
            cs = np.where(inside, rec @ u, -np.inf)
            g_ids = ids[qq].cpu().numpy()
            check_topk(g_ids, sc[qq].cpu().numpy(), cs, k)
            if set(g_probe.tolist()) == set(o_probe.tolist()):
                np.testing.assert_allclose(np.sort(o_sc), np.sort(cs[o_ids]), rtol=1e-12)
            assert np.array_equal(dr[qq].cpu().numpy(), spans[g_ids])
        print(f"[ivf] {nq} queries ok", flush=True)
    index.close()


def test_ivf_rejects_bad_list_ids():
    w, ds = store(1000, 64, "bf16", 2)
    cen, _ = synth.fit_ivf(ds.keys, 2, 16, iters=1)
    bad = torch.zeros(1000, dtype=torch.int32, device=DEV)
    bad[17] = 16
    with pytest.raises(sense.SenseError):
        sense.sense_build_ivf_index(ds.keys, ds.spans, cen, bad)


def test_ivf_skewed_lists_with_fewer_candidates_than_k():
    """One list holds most rows and is not probed, so the candidate buffer
    (sized for the largest lists) is mostly padding: every real candidate
    must come back, then padding (a chunk of the buffer can hold more than k
    entries but fewer than k real ones)."""
    n, d, nlist = 12000, 64, 40
    w, ds = store(n, d, "bf16", 11)
    g = torch.Generator(device=DEV).manual_seed(11)
    cen = torch.randn(nlist, d, generator=g, device=DEV)
    q = cen[5:6].clone().contiguous()
    cen[0] = -q[0]                                   # the big list points away from the query
    lists = torch.zeros(n, dtype=torch.int32, device=DEV)
    small = torch.arange(10000, n, device=DEV)
    lists[small] = (1 + (small - 10000) % (nlist - 1)).to(torch.int32)
    index = sense.sense_build_ivf_index(ds.keys, ds.spans, cen, lists)
    ids, sc, _, _, probe = sense.sense_ivf_search(index, q, 100, 1, want_probe=True)
    torch.cuda.synchronize()
    kb = host_bits(ds.keys)
    o_probe, coarse, o_ids, o_sc = oracle.ivf_search(q[0].cpu().numpy(), cen.cpu().numpy(),
                                                      lists.cpu().numpy(), 1, 100, "cosine",
                                                      keys=kb, key_dtype="bf16")
    assert 0 not in probe[0].cpu().tolist()
    real = int((o_ids >= 0).sum())
    assert 0 < real < 100
    g_ids = ids[0].cpu().numpy()
    assert (g_ids[real:] == -1).all()
    x = decoded(ds.keys)
    cs = candidate_scores(x, lists.cpu().numpy(), probe[0].cpu().numpy(), q[0].cpu().numpy()
                          .astype(np.float64), "cosine")
    check_topk(g_ids[:real], sc[0, :real].cpu().numpy(), cs, real)
    index.close()


# Edges of the build kernels' tiles: one key, one under and over a 16-key tile
# and a block, lists under and over a staged centroid tile, dims that leave a
# 32-dim step ragged, sub-vectors of every length class, codebooks around the
# eight entries compared at once.
BUILD_CASES = [
    # n, d, key dtype, nlist, metric, m, ksub, key stride, centroid scale
    (1, 8, "bf16", 1, "cosine", 8, 1, 8, 1.0),
    (127, 64, "f16", 31, "ip", 16, 7, 64, 1.0),
    (129, 64, "bf16", 33, "cosine", 32, 8, 72, 1e-15),
    (2049, 40, "f16", 65, "cosine", 8, 9, 48, 1e6),
    (35_000, 128, "bf16", 130, "ip", 8, 128, 128, 1e10),
    (70_001, 24, "f16", 64, "cosine", 8, 256, 24, 1.0),
    (140_003, 64, "bf16", 97, "cosine", 16, 256, 64, 1.0),
    (270_001, 32, "bf16", 63, "ip", 4, 200, 40, 1e-4),
    # the shapes that share the centroids, by rounds of blocks
    (77_001, 64, "f16", 97, "ip", 8, 16, 64, 1.0),
    (100_001, 64, "f16", 97, "cosine", 8, 16, 64, 1.0),
    (140_001, 64, "f16", 66, "cosine", 8, 16, 64, 1.0),
    (150_001, 128, "f16", 70, "ip", 8, 16, 128, 1.0),
    (180_001, 128, "bf16", 70, "cosine", 8, 16, 128, 1.0),
]


@pytest.mark.parametrize("case", BUILD_CASES, ids=[str(i) for i in range(len(BUILD_CASES))])
def test_build_kernel_edges(case):
    n, d, kdt, nlist, metric, m, ksub, ld, scale = case
    print(f"[ivf-build-edges] case={case}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(n + d)
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[kdt]
    cen = torch.randn(nlist, d, generator=g, device=DEV)
    if nlist > 40:
        cen[40] = cen[7]                                   # a tie: the lower list wins
    lab = torch.randint(0, nlist, (n,), generator=g, device=DEV)
    keys = torch.full((n, ld), 7.0, dtype=dt, device=DEV)[:, :d]
    keys.copy_(cen[lab] + 0.5 * torch.randn(n, d, generator=g, device=DEV))
    odd = {}
    if n > 100:
        keys[3] = 0.0
        keys[50, 1] = float("nan")
        odd = {3: 0, 50: 0}                                # no centroid is better than the first
    cen *= scale
    got = sense.sense_ivf_assign(keys, cen, metric)
    torch.cuda.synchronize()
    x, c = keys.double(), cen.double()
    s, weight = x @ c.T, x.norm(dim=1, keepdim=True) * c.norm(dim=1)
    if metric == "cosine":
        s = s / weight
        weight = torch.ones_like(s)
    gl = got.long()
    assert int(gl.min()) >= 0 and int(gl.max()) < nlist
    off = float((gl != s.nan_to_num(-1e300).argmax(dim=1)).float().mean())
    print(f"[ivf-build-edges] {off:.2e} of the lists are not the 64-bit choice", flush=True)
    # Two fp32 sums of d products each, and the norms' and scale's roundings.
    bound = 2 * (d + 8) * 2.0 ** -23 * weight.max(dim=1).values
    sel = s.gather(1, gl[:, None])[:, 0]
    ok = sel >= s.max(dim=1).values - bound
    for row, want in odd.items():
        assert int(gl[row]) == want
        ok[row] = True
    assert bool(ok.all()), f"rows {torch.nonzero(~ok).flatten()[:5].tolist()}"
    if nlist > 40:
        assert not bool((gl == 40).any())

    books = 0.5 * scale * torch.randn(m, ksub, d // m, generator=g, device=DEV)
    if ksub > 8:
        books[:, 8] = books[:, 2]
    lists = got.clone()
    if n > 100:
        lists[10], lists[11] = -1, nlist                   # no such list: code 0 throughout
    codes = sense.sense_pq_encode(keys, cen, lists, books).long()
    torch.cuda.synchronize()
    if n > 100:
        assert not bool(codes[10:12].any()) and not bool(codes[50, 1 * m // d]), "code 0"
    rows = torch.ones(n, dtype=torch.bool, device=DEV)
    if n > 100:
        rows[10] = rows[11] = rows[50] = False
    r = (keys.float() - cen[lists.clamp(0, nlist - 1).long()]).double().view(n, m, d // m)
    for j in range(m):
        for i0 in range(0, n, 1 << 15):
            rj = r[i0:i0 + (1 << 15), j]
            dist = ((rj[:, None, :] - books[j].double()[None]) ** 2).sum(dim=2)
            mine = dist.gather(1, codes[i0:i0 + (1 << 15), j:j + 1])[:, 0]
            best = dist.min(dim=1).values
            near = mine <= best * (1 + 2 * (d // m + 3) * 2.0 ** -23) + 1e-37
            assert bool((near | ~rows[i0:i0 + (1 << 15)]).all()), f"slice {j} from row {i0}"
        if ksub > 8:
            assert not bool((codes[:, j] == 8).any())


def _special_keys(n, d, dt, g, cen):
    """Ordinary keys with rows that a norm or a product cannot serve: zero,
    infinite, NaN, and squared norms that overflow or vanish in fp32 (bf16)."""
    lab = torch.randint(0, cen.shape[0], (n,), generator=g, device=DEV)
    keys = cen[lab] + 0.5 * torch.randn(n, d, generator=g, device=DEV)
    kind = torch.randint(0, 60, (n,), generator=g, device=DEV)
    kind[0], kind[n - 1] = 0, 1                        # the first and the last row among them
    keys[kind == 0] = 0.0
    keys[kind == 1, 1] = float("inf")
    keys[kind == 2, d - 1] = float("-inf")
    keys[kind == 3, 0] = float("nan")
    keys[kind == 4, 0] = float("inf")
    keys[kind == 4, 1] = float("inf")
    if dt == torch.bfloat16:
        keys[kind == 5] *= 1e25
        keys[kind == 6] *= 1e-30
        keys[kind == 7] *= 1e18
        keys[kind == 8] *= 1e-18
    return keys.to(dt), kind


@pytest.mark.parametrize("metric", ["cosine", "ip"])
@pytest.mark.parametrize("inf_centroid", [False, True])
@pytest.mark.parametrize("n,d,nlist,kdt", [(2_000, 64, 130, "bf16"), (2_000, 8, 70, "f16"),
                                           (300_001, 32, 65, "bf16"), (80_001, 128, 100, "f16")])
def test_assign_rows_without_an_ordinary_norm(n, d, nlist, kdt, inf_centroid, metric):
    """The list of a key is the first centroid whose fp32 score no other exceeds;
    list 0 where no score is a number above -inf.  With infinite centroid elements
    (of both signs) the infinite scores of ordinary keys count."""
    print(f"[ivf-assign-special] n={n} d={d} nlist={nlist} {kdt} {metric} {inf_centroid}",
          flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(n + d)
    cen = torch.randn(nlist, d, generator=g, device=DEV)
    clean = cen.clone()
    if inf_centroid:
        cen[20, 3], cen[41, 6], cen[0, 2] = float("inf"), float("-inf"), float("nan")
    keys, kind = _special_keys(n, d, {"bf16": torch.bfloat16, "f16": torch.float16}[kdt], g, clean)
    got = sense.sense_ivf_assign(keys, cen, metric).cpu().long()
    rows = torch.nonzero(kind < 10).view(-1).cpu()
    x, c = keys[rows.to(DEV)].float().cpu(), cen.cpu()
    s = torch.empty((len(rows), nlist))
    for i in range(0, len(rows), 512):
        s[i:i + 512] = (x[i:i + 512, None, :] * c[None]).sum(dim=2)
    wide = x.double() @ c.double().T
    plain = torch.isfinite(x).all(dim=1)[:, None] & (torch.isfinite(wide) == torch.isfinite(s))
    if metric == "cosine":
        xn = (x * x).sum(dim=1)
        s = s * (1.0 / c.norm(dim=1)) * torch.where(xn > 0, 1.0 / xn.sqrt(), torch.zeros(()))[:, None]
    best = s.nan_to_num(nan=-float("inf"), posinf=float("inf"), neginf=-float("inf"))
    top = best.max(dim=1).values
    want = (best == top[:, None]).int().argmax(dim=1)
    mine = best.gather(1, got[rows][:, None])[:, 0]
    # Ordinary scores may change places within the sums' rounding (see
    # test_build_kernel_edges); the others are exact.
    exact = ~(plain.all(dim=1) & (top != 0) & torch.isfinite(top))
    assert torch.equal(got[rows][exact], want[exact])
    near = top - mine <= 2 * (d + 8) * 2.0 ** -23 * (
        (x.norm(dim=1) * clean.cpu().norm(dim=1).max()) if metric == "ip" else torch.ones(len(rows)))
    assert bool((near | exact).all())


def test_assign_time_with_zero_keys():
    """Zero keys (padding rows, empty embeddings) take the lists' ordinary path:
    a store with one in a hundred of them is assigned in about the time of a
    store without (one lane walking all centroids for each took 180 times it)."""
    n, d, nlist = 262_144, 64, 4096
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    cen = torch.randn(nlist, d, generator=g, device=DEV)
    plain = torch.randn(n, d, generator=g, device=DEV).to(torch.bfloat16)
    zeros = plain.clone()
    zeros[torch.rand(n, generator=g, device=DEV) < 0.01] = 0.0
    out = torch.empty(n, dtype=torch.int32, device=DEV)
    best = {}
    for name, keys in (("plain", plain), ("zeros", zeros)):
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            sense.sense_ivf_assign(keys, cen, "cosine", out=out)
            b.record()
            b.synchronize()
            best[name] = min(best.get(name, 1e9), a.elapsed_time(b))
    print(f"[ivf-assign-zeros] {best['plain']:.3f} ms, {best['zeros']:.3f} with zero keys", flush=True)
    assert best["zeros"] < 3 * best["plain"]


@pytest.mark.parametrize("metric", ["cosine", "ip"])
@pytest.mark.parametrize("kdt", ["bf16", "f16"])
@pytest.mark.parametrize("small", [2.0 ** -12, 2.0 ** -30])
def test_assign_keys_in_small_coordinates(small, kdt, metric):
    """Centroids with one large coordinate, keys that are zero there: the choice
    rests on coordinates far below the centroids' largest, which count with all
    their bits.  The list's 64-bit score is the best one but for the rounding of
    fp32 sums, d + 8 roundings of the terms' magnitudes for either side (norm,
    scale and sum)."""
    for n in (3_000, 140_000):                         # both ways to share the centroids
        d, nlist = 64, 2048
        print(f"[ivf-assign-small] n={n} small={small:.1e} {kdt} {metric}", flush=True)
        g = torch.Generator(device=DEV)
        g.manual_seed(n)
        cen = small * torch.randn(nlist, d, generator=g, device=DEV)
        cen[:, 5] = 1.0
        keys = torch.randn(n, d, generator=g, device=DEV)
        keys[:, 5] = 0.0
        keys = keys.to({"bf16": torch.bfloat16, "f16": torch.float16}[kdt])
        got = sense.sense_ivf_assign(keys, cen, metric).long()
        torch.cuda.synchronize()
        c = cen.double() / (cen.double().norm(dim=1, keepdim=True) if metric == "cosine" else 1.0)
        off = 0
        for i in range(0, n, 1 << 14):
            x = keys[i:i + (1 << 14)].double()
            s, terms = x @ c.T, x.abs() @ c.abs().T
            best = s.argmax(dim=1, keepdim=True)
            mine = got[i:i + (1 << 14), None]
            off += int((best != mine).sum())
            bound = (d + 8) * 2.0 ** -24 * (terms.gather(1, best) + terms.gather(1, mine))
            assert bool((s.gather(1, mine) >= s.gather(1, best) - bound).all())
        print(f"[ivf-assign-small] {off} of {n} lists are not the 64-bit choice", flush=True)


def test_assign_time_past_a_round():
    """A fourteenth more fp16 keys than fill a round of four-tile blocks take 1.45
    times as long (a second, near empty round of them made it 1.9 times)."""
    d, nlist, us = 64, 4096, {}
    for n in (131_072, 140_000):
        g = torch.Generator(device=DEV)
        g.manual_seed(n)
        cen = torch.randn(nlist, d, generator=g, device=DEV)
        keys = torch.randn(n, d, generator=g, device=DEV).to(torch.float16)
        out = torch.empty(n, dtype=torch.int32, device=DEV)
        us[n] = 1e9
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(4):
                sense.sense_ivf_assign(keys, cen, "cosine", out=out)
            b.record()
            b.synchronize()
            us[n] = min(us[n], a.elapsed_time(b) * 250)
    print(f"[ivf-assign-time] {us}", flush=True)
    assert us[140_000] < 1.7 * us[131_072]
