"""The work whose speed this repository answers for, as callable cases.

Every case is one thing that a program using the library does, through the public binding:

  step      one decode step of one layer (or of a batch's sequences in one launch): score the pages,
            pick the best ones, attend to them, optionally together with a window of recent tokens
  reuse     an anchor layer's step followed by two layers that attend to the anchor's tokens (a three
            layer stretch of a decode step under selection reuse)
  hier      the same step with the staged selection (clusters first, then their pages)
  build     clustering and paging of a prefilled layer
  turn      a saved prompt is resumed: its index is loaded, the tokens of the new turn are inserted in
            one call, and the first answer step runs
  generate  a saved prompt is resumed and a few tokens are generated one by one (insert, then step)

Keys come from a Gaussian mixture (one component per two clusters, 0.3 around its centre), values are
N(0, 1), queries lie around centres: the distributions of this repository's benchmark.  Indexes that
a case only reads are laid out here from the mixture's labels and handed over with import_arrays, so
that the 64-bit results in exact() need none of the library's code.
"""
import math

import torch

from paper_2604_10539_amd import IceIndex
from paper_2604_10539_amd.binding import ICE_GEOMETRY_RAW, ICE_GEOMETRY_TRANSFORMED, IMPORT_FIELDS

D = 128
SIGMA = 0.3
DEV = "cuda"
UNIT_TOKENS = 1 << 20  # (unit, token) pairs that the input makers touch at a time


def _case(name, kind, batch, heads, group, n, page, clusters, **more):
    c = {"kind": kind, "batch": batch, "heads": heads, "group": group, "n": n, "page": page, "clusters": clusters}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: a short chat on a model with two KV heads on this GPU
        _case("step_4k_2heads", "step", 1, 2, 4, 4096, 16, 64, budget=256, window=0),
        # the ordinary one: one layer of an 8-KV-head model at 32k, one sequence
        _case("step_32k_8heads", "step", 1, 8, 4, 32768, 16, 512, budget=256, window=0),
        # long context, larger budget, and the window of recent tokens that the decode loop keeps beside the pages
        _case("step_131k_window", "step", 1, 8, 4, 131072, 16, 2048, budget=1024, window=512),
        # a serving batch (or all layers of one sequence at once): one unit per compute unit
        _case("step_32k_batch32", "step", 32, 8, 4, 32768, 16, 512, budget=256, window=0),
        # a batch that does not divide the chip, odd lengths, larger pages, 64 query heads over 8 KV heads
        _case("step_ragged_batch39", "step", 39, 8, 8, 11777, 32, 184, budget=700, window=131),
        # selection reuse: an anchor layer and the two layers behind it, four sequences
        _case("reuse_32k_batch4", "reuse", 4, 8, 4, 32768, 16, 512, budget=512),
        # the staged selection on a serving batch
        _case("hier_32k_batch16", "hier", 16, 8, 4, 32768, 16, 512, budget=256, probe=64),
        # prefill of one layer
        _case("build_32k_8heads", "build", 1, 8, 4, 32768, 16, 512, iters=10, transformed=False, outliers=0.0),
        # two prompts of an odd length, larger pages, distances on the transformed keys
        _case("build_ragged_batch2", "build", 2, 8, 4, 23457, 32, 366, iters=6, transformed=True, outliers=0.0),
        # the longest prefill: 131k tokens with outliers
        _case("build_131k_8heads", "build", 1, 8, 4, 131072, 16, 2048, iters=10, transformed=False, outliers=0.05),
        # a new turn of 200 tokens on four saved prompts
        _case("turn_8k_batch4", "turn", 4, 8, 4, 8192, 16, 128, new=200, budget=256),
        # sixteen generated tokens on one saved prompt
        _case("generate_16k_8heads", "generate", 1, 8, 4, 16384, 16, 256, new=16, budget=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "reuse", "hier", "build", "build", "turn", "generate"])
    heads = rng.choice([1, 2, 4, 8, 8])
    group = rng.choice([1, 2, 4, 4, 8])
    page = rng.choice([16, 16, 32, 64])
    if kind == "build":
        batch = _log(rng, 1, 4)
        n = _log(rng, 1000, min(131072, 600000 // (batch * heads)))
        clusters = max(8, n // rng.choice([64, 64, 100]))
        iters = rng.randint(3, 10)
        while 2.0 * batch * heads * n * clusters * D * iters > 5.0e12:  # (the longest listed prefill: 5.5e12)
            clusters = clusters * 2 // 3
        return _case(None, kind, batch, heads, group, n, page, clusters, iters=iters, transformed=rng.random() < 0.3,
                     outliers=rng.choice([0.0, 0.05]))
    if kind in ("turn", "generate"):
        batch = _log(rng, 1, 8 if kind == "turn" else 4)
        n = _log(rng, 1000, 16384)
        return _case(None, kind, batch, heads, group, n, page, max(8, n // 64), new=_log(rng, 16, 300) if kind == "turn" else rng.randint(4, 24),
                     budget=page * rng.randint(4, 16))
    if kind == "reuse":
        batch = _log(rng, 1, 8)
        n = _log(rng, 2000, 65536)
        return _case(None, kind, batch, heads, group, n, page, max(8, n // 64), budget=_log(rng, 128, 1024))
    if kind == "hier":
        batch = _log(rng, 1, 32)
        n = _log(rng, 2000, 65536)
        clusters = max(8, n // 64)
        return _case(None, kind, batch, heads, group, n, page, clusters, budget=_log(rng, 128, 1024), probe=max(4, clusters // 8))
    batch = _log(rng, 1, 48)
    n = _log(rng, 1000, min(131072, (8 << 20) // (batch * heads)))
    return _case(None, kind, batch, heads, group, n, page, max(8, n // 64), budget=_log(rng, 128, 2048),
                 window=rng.choice([0, 0, _log(rng, 16, 1024)]))


# ---------------------------------------------------------------------------------------- inputs
def _bits(x):
    return x.to(torch.bfloat16).view(torch.int16)


def _f(x, dtype=torch.float64):
    return x.view(torch.bfloat16).to(dtype)


def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEV)


def _around(gen, cen, comp):
    """Rows around the centres `comp` [U, m] of cen [U, M, D]: fp32 rows and their offset's first coordinate."""
    noise = SIGMA * _normal(gen, comp.shape[0], comp.shape[1], D)
    side = noise[..., 0] > 0
    return noise.add_(torch.gather(cen, 1, comp[..., None].expand(-1, -1, D))), side


def _prefill(case, gen, outliers=0.0):
    """Keys, values (bf16 bits [U, n, D]), cluster labels [U, n] and the centres [U, M, D]."""
    U, n, C = case["batch"] * case["heads"], case["n"], case["clusters"]
    M = max(1, C // 2)
    cen = _normal(gen, U, M, D)
    K = torch.empty(U, n, D, dtype=torch.int16, device=DEV)
    V = torch.empty_like(K)
    label = torch.empty(U, n, dtype=torch.int64, device=DEV)
    step = max(1, UNIT_TOKENS // n)
    for u in range(0, U, step):
        c = cen[u:u + step]
        comp = torch.randint(M, (c.shape[0], n), generator=gen, device=DEV)
        x, side = _around(gen, c, comp)
        if outliers:
            far = torch.rand(c.shape[0], n, generator=gen, device=DEV) < outliers
            y = torch.rand(c.shape[0], n, D, generator=gen, device=DEV) * 6 - 3
            x = torch.where(far[..., None], y, x)
        K[u:u + step], V[u:u + step] = _bits(x), _bits(_normal(gen, c.shape[0], n, D))
        label[u:u + step] = (2 * comp + side).clamp_(max=C - 1)
    return K, V, label, cen


def _queries(case, gen, cen):
    G = case["group"]
    comp = torch.randint(cen.shape[1], (cen.shape[0], G), generator=gen, device=DEV)
    return _bits(_around(gen, cen, comp)[0]).view(case["batch"], case["heads"] * G, D)


def _snapshot(case, K, V, label, max_tokens):
    """The arrays of an index over these tokens (import_arrays' names and layouts): clusters in id order, members in
    ascending position, cut into pages."""
    U, n, s, C = K.shape[0], case["n"], case["page"], case["clusters"]
    MP = max_tokens // s + C
    i32 = dict(dtype=torch.int32, device=DEV)
    a = {"Kp": torch.zeros(U, MP, s, D, dtype=torch.int16, device=DEV), "Vp": torch.zeros(U, MP, s, D, dtype=torch.int16, device=DEV),
         "page_cluster": torch.full((U, MP), -1, **i32), "page_fill": torch.zeros(U, MP, **i32), "page_pos": torch.full((U, MP, s), -1, **i32),
         "cluster_tail": torch.empty(U, C, **i32), "cluster_cnt": torch.empty(U, C, **i32),
         "cluster_sum": torch.zeros(U, C, D, device=DEV), "centroid": torch.empty(U, C, D, device=DEV),
         "page_sum": torch.zeros(U, MP, D, device=DEV), "rep": torch.zeros(U, MP, D, dtype=torch.int16, device=DEV),
         "n_pages": torch.empty(U, **i32)}
    step = max(1, UNIT_TOKENS // n)
    for u0 in range(0, U, step):
        lab = label[u0:u0 + step]
        m = lab.shape[0]
        cl, order = torch.sort(lab, dim=1, stable=True)
        cnt = torch.zeros(m, C, dtype=torch.int64, device=DEV).scatter_add_(1, lab, torch.ones_like(lab))
        pages = (cnt + s - 1) // s
        pbase, start = torch.cumsum(pages, 1) - pages, torch.cumsum(cnt, 1) - cnt
        r = torch.arange(n, device=DEV)[None] - torch.gather(start, 1, cl)
        page = torch.gather(pbase, 1, cl) + r // s
        uu = torch.arange(m, device=DEV)[:, None].expand(-1, n)
        k, v = torch.gather(K[u0:u0 + step], 1, order[..., None].expand(-1, -1, D)), torch.gather(V[u0:u0 + step], 1, order[..., None].expand(-1, -1, D))
        sub = {x: y[u0:u0 + step] for x, y in a.items()}
        sub["Kp"][uu, page, r % s] = k
        sub["Vp"][uu, page, r % s] = v
        sub["page_pos"][uu, page, r % s] = order.int()
        sub["page_cluster"][uu, page] = cl.int()
        sub["page_fill"].copy_((sub["page_pos"] >= 0).sum(2))
        sub["cluster_tail"].copy_(torch.where(cnt > 0, pbase + pages - 1, -1))
        sub["cluster_cnt"].copy_(cnt)
        sub["n_pages"].copy_(pages.sum(1))
        for t in range(s):  # (empty slots are zero rows)
            sub["page_sum"] += _f(sub["Kp"][:, :, t], torch.float32)
        sub["rep"].copy_(_bits(sub["page_sum"] / sub["page_fill"].clamp(min=1)[..., None]))
        # the clusters' sums, page by page in id order (at most as many additions as a cluster has pages)
        for t in range(int(pages.max())):
            own = t < pages
            p = (pbase + t).clamp(max=MP - 1)
            sub["cluster_sum"] += torch.gather(sub["page_sum"], 1, p[..., None].expand(-1, -1, D)) * own[..., None]
        sub["centroid"].copy_(sub["cluster_sum"] / cnt.clamp(min=1)[..., None])
    return a


def _make(case, seed):
    """Everything a case works on, from the seed alone (no library code)."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    b, h, U, n = case["batch"], case["heads"], case["batch"] * case["heads"], case["n"]
    if case["kind"] == "build":
        K, V, _, _ = _prefill(case, gen, case["outliers"])
        pick = torch.argsort(torch.rand(U, n, generator=gen, device=DEV), dim=1)[:, :case["clusters"]]
        return {"K": K, "V": V, "init": torch.sort(pick, dim=1)[0].int().contiguous()}
    new = case.get("new", 0)
    K, V, label, cen = _prefill(case, gen)
    m = {"arrays": _snapshot(case, K, V, label, n + new), "q": _queries(case, gen, cen)}
    del K, V, label
    if case.get("window"):
        comp = torch.randint(cen.shape[1], (U, case["window"]), generator=gen, device=DEV)
        m["wk"] = _bits(_around(gen, cen, comp)[0]).view(b, h, -1, D)
        m["wv"] = _bits(_normal(gen, U, case["window"], D)).view(b, h, -1, D)
    if case["kind"] == "reuse":
        m["layers"] = []
        for _ in range(2):
            k2, v2, _, c2 = _prefill(case, gen)
            m["layers"].append((_queries(case, gen, c2), k2.view(b, h, n, D), v2.view(b, h, n, D)))
    if new:
        comp = torch.randint(cen.shape[1], (U, new), generator=gen, device=DEV)
        m["k"] = _bits(_around(gen, cen, comp)[0]).view(b, h, new, D)
        m["v"] = _bits(_normal(gen, U, new, D)).view(b, h, new, D)
    if case["kind"] == "generate":
        m["steps"] = [(m["k"][:, :, t].contiguous(), m["v"][:, :, t].contiguous(), _queries(case, gen, cen)) for t in range(new)]
    return m


def prepare(case, seed):
    m = _make(case, seed)
    st = dict(case)
    st.update(m)
    if case["kind"] == "build":
        ix = IceIndex(case["batch"], case["heads"], case["group"], case["n"], case["page"], case["clusters"], kmeans_iters=case["iters"],
                      init_idx=m["init"], geometry=ICE_GEOMETRY_TRANSFORMED if case["transformed"] else ICE_GEOMETRY_RAW)
        ix.workspace.zero_()  # (a page's unused tail slots are not written by a build)
        st["ix"] = ix
        return st
    ix = IceIndex(case["batch"], case["heads"], case["group"], case["n"] + case.get("new", 0), case["page"], case["clusters"])
    ix.import_arrays(m["arrays"], case["n"])
    st["ix"] = ix
    if case["kind"] not in ("turn", "generate"):  # (only these load the saved arrays again)
        torch.cuda.synchronize()
        del st["arrays"]
    return st


def run(st):
    ix, kind = st["ix"], st["kind"]
    if kind == "step":
        if st["window"]:
            return ix.select_attend_resident(st["q"], st["budget"], st["wk"], st["wv"])
        return ix.select_attend(st["q"], st["budget"])
    if kind == "reuse":
        ids, n_sel, out = ix.select_attend(st["q"], st["budget"])
        pos, n_tok = ix.selected_tokens(ids, n_sel)
        return [ids, n_sel, out, pos, n_tok] + [ix.attend_tokens(q, K, V, pos, n_tok) for q, K, V in st["layers"]]
    if kind == "hier":
        ids, n_sel, scores, clusters, out = ix.select_hier(st["q"], st["budget"], st["probe"])
        return ids, n_sel, scores, clusters, out
    if kind == "build":
        ix.build_index(st["K"].view(st["batch"], st["heads"], st["n"], D), st["V"].view(st["batch"], st["heads"], st["n"], D))
        return _state(st, with_assign=True)
    ix.import_arrays(st["arrays"], st["n"])
    if kind == "turn":
        ix.insert_batch(st["k"], st["v"])
        return {"step": ix.select_attend(st["q"], st["budget"]), "state": _state(st)}
    steps = []
    for k, v, q in st["steps"]:
        ix.insert(k, v)
        steps.append(ix.select_attend(q, st["budget"]))
    return {"outs": [s[2] for s in steps], "ids": [s[0] for s in steps], "state": _state(st)}


def _state(st, with_assign=False):
    """The whole index, as views of the workspace (they stay valid: the layout is the index's for life)."""
    if "state" not in st:
        ex = st["ix"].export()
        st["state"] = {name: ex[name] for name in IMPORT_FIELDS + (("assign",) if with_assign else ())}
    return st["state"]


# ------------------------------------------------------------------------------------ accounting
def _pages(case):
    """Live pages per unit, on average: every cluster's last page is about half full."""
    return min(case["n"] / case["page"] + case["clusters"] / 2, case["n"] // case["page"] + case["clusters"])


def _step_work(case, pages, rows):
    U, G = case["batch"] * case["heads"], case["group"]
    return {"bytes": U * (pages * 2 * D + G * 2 * D + 4 * case["budget"] // case["page"] + rows * 4 * D + G * 4 * D),
            "flops": U * G * (pages * 2 * D + rows * 4 * D)}


def work(case):
    U, G, n, s, C = case["batch"] * case["heads"], case["group"], case["n"], case["page"], case["clusters"]
    if case["kind"] == "build":
        pages, T = _pages(case), case["iters"]
        # keys and values in; tiles, sums, representatives, positions, centroids and the assignment out
        return {"bytes": U * (2 * n * 2 * D + pages * (s * (4 * D + 4) + 6 * D + 8) + n * 4 + C * 8 * D),
                "flops": U * T * 2.0 * n * C * (D + (1 if case["transformed"] else 0)) + U * T * n * D}
    pages, fill = _pages(case), n / _pages(case)
    rows = min(case["budget"] // s, pages) * fill
    if case["kind"] == "hier":
        cand = pages * min(1.0, case["probe"] / C)
        w = _step_work(case, cand, rows)
        w["bytes"] += U * (C * 2 * D + pages * 4)
        w["flops"] += U * G * C * 2 * D
        return w
    w = _step_work(case, pages, rows + case.get("window", 0))
    if case["kind"] == "reuse":
        w["bytes"] += U * (rows * 8 + 2 * (rows * 4 * D + G * 6 * D))
        w["flops"] += 2 * U * G * rows * 4 * D
    if case["kind"] in ("turn", "generate"):
        steps = 1 if case["kind"] == "turn" else case["new"]
        MP = (n + case["new"]) // s + C
        load = 2 * U * (MP * (s * (4 * D + 4) + 6 * D + 8) + C * (8 * D + 8))  # the saved arrays, read and written
        insert = U * (C * 2 * D * steps + case["new"] * (8 * D + 4) + min(C, case["new"]) * 16 * D)
        w = {"bytes": steps * w["bytes"] + load + insert, "flops": steps * w["flops"] + U * case["new"] * C * 2.0 * D}
    return w


def tolerance(case):
    # A build and an insertion follow a stated order of additions, and one flipped near-tie would renumber every
    # page behind it: their states are the same bits.  Outputs of the attention are fp32 sums with weights in two bf16
    # terms (2^-16 each): measured 1e-5 from the 64-bit result, four times that allowed between two orders.
    if case["kind"] == "build":
        return "exact"
    return {"rel": 4e-5, "max": 4e-4, "differ": 0.0}


# ------------------------------------------------------------------------------------ 64-bit results
def _top(score, k):
    """The k best of each row, ids ascending (lower id on equal scores)."""
    return torch.sort(torch.sort(score, dim=1, descending=True, stable=True)[1][:, :k], dim=1)[0]


def _scores(q, rows):
    """max over the group of q_h . row / ||q_h||: q [U, G, D], rows [U, m, D], both 64-bit."""
    return (rows @ (q / q.norm(dim=2, keepdim=True).clamp(min=1e-20)).transpose(1, 2).contiguous()).amax(2)


def _softmax_rows(q, k, v, ok):
    z = (k @ q.transpose(1, 2).contiguous()).transpose(1, 2) / math.sqrt(D)
    p = torch.softmax(z.masked_fill(~ok[:, None], -math.inf), dim=2)
    return p @ v


def _attend(case, a, q, ids, wk=None, wv=None):
    """Attention over pages ids [U, P] of the arrays `a` (and the window), q [U, G, D] 64-bit."""
    U = ids.shape[0]
    uu = torch.arange(U, device=DEV)[:, None]
    k, v = _f(a["Kp"][uu, ids]).reshape(U, -1, D), _f(a["Vp"][uu, ids]).reshape(U, -1, D)
    ok = (torch.arange(case["page"], device=DEV) < a["page_fill"][uu, ids][..., None]).reshape(U, -1)
    if wk is not None:
        k, v = torch.cat([k, _f(wk).view(U, -1, D)], 1), torch.cat([v, _f(wv).view(U, -1, D)], 1)
        ok = torch.cat([ok, torch.ones(U, wk.shape[2], dtype=torch.bool, device=DEV)], 1)
    return _softmax_rows(q, k, v, ok).view(case["batch"], -1, D)


def _select(case, a, q, allowed=None):
    """The flat selection: page ids [U, P] (every unit has at least P pages here) or None where one has not."""
    MP, P = a["rep"].shape[1], case["budget"] // case["page"]
    sc = torch.empty(q.shape[0], MP, dtype=torch.float64, device=DEV)
    for u in range(0, q.shape[0], 32):
        sc[u:u + 32] = _scores(q[u:u + 32], _f(a["rep"][u:u + 32]))
    live = torch.arange(MP, device=DEV) < a["n_pages"][:, None]
    if allowed is not None:
        live &= allowed
    if int(live.sum(1).min()) < P:
        return None, None
    sc.masked_fill_(~live, -math.inf)
    return _top(sc, P), sc


def _insert(case, a, k, v, at):
    """One token per unit into the arrays `a` (64-bit sums): nearest bf16 centroid, tail page, running means."""
    U, s = k.shape[0], case["page"]
    uu = torch.arange(U, device=DEV)
    kk = _f(k)
    cb = _f(_bits(a["centroid"]))
    c = ((cb * cb).sum(2) - 2 * (cb @ kk[:, :, None])[..., 0]).argmin(1)
    tail = a["cluster_tail"][uu, c].long()
    fresh = (tail < 0) | (a["page_fill"][uu, tail.clamp(min=0)] >= s)
    p = torch.where(fresh, a["n_pages"].long(), tail)
    a["n_pages"] += fresh.int()
    slot = a["page_fill"][uu, p].long()
    a["Kp"][uu, p, slot], a["Vp"][uu, p, slot] = k, v
    a["page_pos"][uu, p, slot] = at
    a["page_fill"][uu, p] += 1
    a["page_cluster"][uu, p] = c.int()
    a["cluster_tail"][uu, c] = p.int()
    a["page_sum"][uu, p] += kk
    a["rep"][uu, p] = _bits(a["page_sum"][uu, p] / a["page_fill"][uu, p][:, None])
    a["cluster_cnt"][uu, c] += 1
    a["cluster_sum"][uu, c] += kk
    a["centroid"][uu, c] = a["cluster_sum"][uu, c] / a["cluster_cnt"][uu, c][:, None]


def _lloyd(case, m):
    """Means and sums after the stated rounds: assignment to bf16 centroids, everything else in 64 bits."""
    U, C = m["K"].shape[0], case["clusters"]
    cen, tot = torch.empty(U, C, D, dtype=torch.float64, device=DEV), torch.empty(U, C, D, dtype=torch.float64, device=DEV)
    for u in range(U):
        k = _f(m["K"][u])
        if case["transformed"]:
            n2 = (k * k).sum(1)
            k = torch.cat([k, (n2.max() - n2).clamp(min=0).sqrt().to(torch.bfloat16).double()[:, None]], 1)
        mu = k[m["init"][u].long()]
        for _ in range(case["iters"]):
            b = mu.to(torch.bfloat16).double()
            h = (b * b).sum(1) / 2
            lab = torch.cat([(k[i:i + 65536] @ b.t() - h).argmax(1) for i in range(0, k.shape[0], 65536)])
            cnt = torch.bincount(lab, minlength=C).double()[:, None]
            tsum = torch.zeros(C, k.shape[1], dtype=torch.float64, device=DEV).index_add_(0, lab, k)
            mu = torch.where(cnt > 0, tsum / cnt.clamp(min=1), mu)
        cen[u], tot[u] = mu[:, :D], tsum[:, :D]
    return cen, tot


def exact(case, seed):
    m = _make(case, seed)
    U, G = case["batch"] * case["heads"], case["group"]
    none = {name: None for name in IMPORT_FIELDS}
    if case["kind"] == "build":
        cen, tot = _lloyd(case, m)
        return dict(none, assign=None, centroid=cen, cluster_sum=tot)
    a, q = m["arrays"], _f(m["q"]).view(U, G, D)
    if case["kind"] in ("turn", "generate"):
        a["centroid"], a["cluster_sum"], a["page_sum"] = a["centroid"].double(), a["cluster_sum"].double(), a["page_sum"].double()
        outs = []
        for t in range(case["new"]):
            _insert(case, a, m["k"][:, :, t].reshape(U, D), m["v"][:, :, t].reshape(U, D), case["n"] + t)
            if case["kind"] == "generate":
                qt = _f(m["steps"][t][2]).view(U, G, D)
                ids, _ = _select(case, a, qt)
                outs.append(None if ids is None else _attend(case, a, qt, ids))
        state = dict(none, centroid=a["centroid"], cluster_sum=a["cluster_sum"], page_sum=a["page_sum"])
        if case["kind"] == "generate":
            return {"outs": outs, "ids": [None] * len(outs), "state": state}
        ids, _ = _select(case, a, q)
        return {"step": (None, None, None if ids is None else _attend(case, a, q, ids)), "state": state}
    if case["kind"] == "hier":
        kept = _top(_scores(q, _f(_bits(a["centroid"]))), min(case["probe"], case["clusters"]))
        is_kept = torch.zeros(U, case["clusters"], dtype=torch.bool, device=DEV).scatter_(1, kept, True)
        own = torch.gather(is_kept, 1, a["page_cluster"].long().clamp(min=0)) & (a["page_cluster"] >= 0)
        ids, sc = _select(case, a, q, own)
        if ids is None:
            return None
        return None, None, torch.gather(sc, 1, ids).view(case["batch"], case["heads"], -1), None, _attend(case, a, q, ids)
    ids, _ = _select(case, a, q)
    if ids is None:
        return None
    if case["kind"] == "step":
        return None, None, _attend(case, a, q, ids, m.get("wk"), m.get("wv"))
    outs = []
    uu = torch.arange(U, device=DEV)[:, None]
    pos = a["page_pos"][uu, ids].long().view(U, -1)
    for q2, K2, V2 in m["layers"]:
        rows = pos.clamp(min=0)[..., None].expand(-1, -1, D)
        k, v = (_f(torch.gather(x.view(U, -1, D), 1, rows)) for x in (K2, V2))
        outs.append(_softmax_rows(_f(q2).view(U, G, D), k, v, pos >= 0).view(case["batch"], -1, D))
    return [None, None, _attend(case, a, q, ids), None, None] + outs
