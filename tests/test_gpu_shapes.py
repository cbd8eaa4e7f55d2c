"""GPU tests at the sizes where a kernel's split of the work can go wrong: edges of tiles and ranges,
remainders, the smallest and largest counts of a launch rule."""
import numpy as np
import pytest

import datagen
from datagen import bf16_bits_to_f32 as widen, f32_to_bf16_bits as narrow
from tests.util import D, down, up

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,at", [(1, 0), (255, 254), (256, 0), (257, 256), (1025, 511), (66000, 65999)])
def test_radius_of_transformed_keys_is_the_largest_norm(n, at):
    """The squared radius is the largest squared norm wherever that key sits: first or last workgroup, first or
    last row of one, and with more workgroups than a workgroup has threads (66000 keys: 258)."""
    from paper_2604_10539_amd import IceIndex
    from paper_2604_10539_amd.binding import ICE_GEOMETRY_TRANSFORMED
    rng = np.random.default_rng(n)
    K = narrow(rng.standard_normal((1, 2, n, D)).astype(np.float32))
    K[0, 1, at] = narrow(widen(K[0, 1, at]) * np.float32(2.0))
    ix = IceIndex(1, 2, 4, n, 16, 1, kmeans_iters=1, geometry=ICE_GEOMETRY_TRANSFORMED)
    ix.build_index(up(K), up(K))
    geo = ix.export_geometry()
    n2 = (widen(K[0]).astype(np.float64) ** 2).sum(2)
    c2 = down(geo["radius_sq"])
    # a squared norm is a chain of at most 8 + 4 fp32 additions of non-negative terms, each rounded product included
    np.testing.assert_allclose(c2, n2.max(1), rtol=13 * 2.0 ** -24)
    extra = widen(down(geo["key_extra"]))
    a = np.sqrt(np.maximum(c2[:, None].astype(np.float64) - n2, 0.0))
    # one bf16 rounding (2^-9) of a square root whose argument carries an absolute error of 14 * 2^-24 * c2
    bound = 2.0 ** -8 * a + np.sqrt(14 * 2.0 ** -24 * c2[:, None])
    assert np.all(np.abs(extra - a) <= bound)


@pytest.mark.parametrize("tiles,n", [(1, 256), (2, 257), (3, 700), (5, 1000), (6, 511), (7, 2049), (9, 1300), (12, 2600), (13, 777),
                                     (16, 4097), (17, 900), (25, 3000)])
def test_assignment_at_every_share_of_a_centroid_slice(tiles, n):
    """Centroid tiles of 32 that do not fill a slice of 16 (or fill a second one in part) are dealt unevenly to the
    waves, and runs of key tiles end anywhere: every key gets its nearest centroid, raw and transformed."""
    from paper_2604_10539_amd import IceIndex
    from paper_2604_10539_amd.binding import ICE_GEOMETRY_TRANSFORMED
    C, U = 32 * tiles - 3, 3
    n = max(n, C)
    w = datagen.small(n_tokens=n, n_clusters=C, n_kv_heads=U, n_components=max(4, C // 3))
    K, V = datagen.keys_values(w)
    ix = IceIndex(1, U, 4, n, 16, C, kmeans_iters=1, init_idx=up(datagen.init_indices(w)), geometry=ICE_GEOMETRY_TRANSFORMED)
    ix.build_index(up(K), up(V))
    ex, geo = ix.export(), ix.export_geometry()
    got = down(ex["assign"])
    mu = widen(down(ex["assign_centroid_bf16"])[:, :C]).astype(np.float64)
    mu = np.concatenate([mu, widen(down(geo["assign_centroid_extra_bf16"])[:, :C])[..., None]], axis=2)
    k = widen(K[0]).astype(np.float64)
    kx = np.concatenate([k, widen(down(geo["key_extra"]))[..., None]], axis=2)
    ix2 = IceIndex(1, U, 4, n, 16, C, kmeans_iters=1)
    got2 = down(ix2.debug_assign(up(K), ex["assign_centroid_bf16"][:, :C].contiguous(), with_best=False)[0])
    for u in range(U):
        for a, keys, cen in ((got[u], kx[u], mu[u]), (got2[u], k[u], mu[u][:, :D])):
            obj = (cen ** 2).sum(1)[None] - 2.0 * keys @ cen.T
            best = obj.min(1)
            # both candidates' fp32 chains (129 or 128 products and the seed), halved objective doubled again
            mag = 0.5 * (cen ** 2).sum(1).max() + np.linalg.norm(keys, axis=1) * np.linalg.norm(cen, axis=1).max()
            assert np.all(obj[np.arange(n), a] - best <= 4.0 * (D + 3) * 2.0 ** -24 * mag)


@pytest.mark.parametrize("U,n,C,s,lump,fused,R,L", [
    # fused: the assignment sorts its own runs; ranges R of L tokens and what the members are read by; lump: tokens in a row of
    # one cluster (and the transformed keys, whose extra coordinate is summed over the same members)
    (1, 1, 1, 16, 0, 1, 1, 256),             # one token
    (2, 256, 1, 16, 9, 1, 1, 256), (2, 257, 1, 16, 9, 1, 2, 256), (2, 1024, 1, 16, 9, 1, 4, 256),  # one wave adds the coordinates, four of them do
    (2, 1023, 7, 16, 0, 1, 4, 256), (2, 1024, 7, 16, 0, 1, 4, 256), (2, 1025, 7, 64, 0, 1, 5, 256),
    (1, 2048, 100, 16, 0, 1, 8, 256),        # the most pieces that are picked per member
    (1, 2049, 100, 16, 0, 1, 9, 256),        # ... and the first that are listed in LDS
    (60, 9000, 40, 32, 0, 1, 4, 2304),       # nine tiles per run
    (32, 32768, 40, 16, 0, 1, 8, 4096),      # sixteen, the longest
    (3, 2500, 4, 16, 600, 1, 10, 256),       # more members than are listed: searched
    (1, 8000, 100, 16, 0, 1, 32, 256),
    (1, 12000, 300, 16, 600, 1, 47, 256),    # a cluster longer than the list beside listed ones
    (1, 16384, 40, 16, 900, 1, 64, 256),     # the most pieces that a wave holds
    (1, 16640, 100, 16, 900, 1, 65, 256),    # ... and one more
    (1, 20000, 60, 64, 5000, 1, 79, 256),
    (1, 32768, 100, 16, 3000, 1, 128, 256),  # the most ranges
    (1, 32768, 16, 16, 600, 0, 32, 1024),    # as many tokens, clusters too large for so many
    (2, 1000, 600, 16, 0, 0, 1, 1024), (2, 1024, 600, 16, 0, 0, 1, 1024), (2, 1025, 600, 64, 0, 0, 2, 1024),  # a sort by itself around one range
    (1, 8192, 600, 16, 0, 0, 8, 1024), (1, 8193, 600, 16, 0, 0, 9, 1024),  # ... picked, listed
    (60, 9000, 600, 32, 0, 0, 3, 4096),      # the longest range that ranks in four groups
    (1, 40000, 200, 16, 0, 0, 40, 1024),     # most clusters listed in LDS
    (1, 66000, 900, 16, 0, 0, 33, 2048),     # two centroid slices
    (1, 270000, 64, 64, 5000, 0, 33, 8192),  # lane masks; clusters longer than the list
    (1, 70000, 8192, 16, 0, 0, 35, 2048),    # four segments, no lane masks
    (1, 530000, 8192, 16, 0, 0, 65, 8192),   # more than one wave holds; the longest of four segments
    (1, 9000, 8192, 16, 0, 0, 9, 1024),      # four segments, one token per cluster or none
    (300, 1100, 24, 16, 0, 0, 1, 2048),      # more units than CUs
    (260, 4100, 40, 16, 0, 0, 1, 8192),
    (1, 1050000, 64, 64, 0, 0, 33, 32768),   # the longest
])
def test_pages_hold_the_members_in_ascending_position(U, n, C, s, lump, fused, R, L):
    """The page layout is the stable sort of the assignment, whatever the sort's ranges and segments are, and the
    means are the members' means."""
    from paper_2604_10539_amd import IceIndex, ice_debug_build_plan, make_config
    plan = ice_debug_build_plan(make_config(1, U, 4, n), n, C)
    assert (plan["fused"], plan["ranges"], plan["range_len"]) == (fused, R, L)
    w = datagen.small(n_tokens=min(n, 300000), n_clusters=C, n_kv_heads=U, n_components=max(2, C // 3))
    K, V = datagen.keys_values(w)
    if n > 300000:  # (rows of a shorter draw, in another order)
        at = np.random.default_rng(n).integers(0, 300000, n)
        K, V = K[:, :, at], V[:, :, at[::-1]]
    if lump:
        K[0, 0, n // 3:n // 3 + lump] = K[0, 0, n // 3]
    tk = int(lump > 0)  # (the transformed keys' extra coordinate is summed over the same members)
    ix = IceIndex(1, U, 4, n, s, C, kmeans_iters=2, init_idx=up(datagen.init_indices(w)), geometry=tk)
    ix.build_index(up(K), up(V))
    ex = {k: down(v) for k, v in ix.export().items() if k != "view"}
    geo = {k: down(v) for k, v in ix.export_geometry().items()} if tk else None
    for u in range(U):
        a = ex["assign"][u, :n]
        order = np.argsort(a, kind="stable")
        cnt = np.bincount(a, minlength=C)
        pages = (cnt + s - 1) // s
        base, start = np.cumsum(pages) - pages, np.cumsum(cnt) - cnt
        npg = int(pages.sum())
        assert ex["n_pages"][u] == npg and np.array_equal(ex["cluster_cnt"][u], cnt)
        assert np.array_equal(ex["cluster_tail"][u], np.where(cnt > 0, base + pages - 1, -1))
        want = np.full((ex["page_pos"].shape[1], s), -1)
        r = np.arange(n) - start[a[order]]
        want[base[a[order]] + r // s, r % s] = order
        assert np.array_equal(ex["page_pos"][u], want)
        assert np.array_equal(ex["page_fill"][u], (want >= 0).sum(1))
        assert np.array_equal(ex["page_cluster"][u], np.concatenate([np.repeat(np.arange(C), pages), np.full(len(want) - npg, -1)]))
        live = want[:npg] >= 0
        assert np.array_equal(ex["Kp"][u, :npg][live], K[0, u][want[:npg][live]])
        assert np.array_equal(ex["Vp"][u, :npg][live], V[0, u][want[:npg][live]])
        by_cluster = widen(K[0, u])[order].astype(np.float64)
        sums, mags = np.zeros((C, D)), np.zeros((C, D))
        for c in np.flatnonzero(cnt)[:200]:
            part = by_cluster[start[c]:start[c] + cnt[c]]
            sums[c], mags[c] = part.sum(0), np.abs(part).sum(0)
        # at most cnt + 8 roundings of partial sums bounded by the sum of magnitudes
        seen = np.flatnonzero(cnt)[:200]
        assert np.all(np.abs(ex["cluster_sum"][u] - sums)[seen] <= ((cnt[:, None] + 8) * 2.0 ** -24 * mags)[seen])
        if tk:
            extra = np.bincount(a, weights=widen(geo["key_extra"][u, :n]).astype(np.float64), minlength=C)
            assert np.all(np.abs(geo["cluster_sum_extra"][u] - extra) <= (cnt + 8) * 2.0 ** -24 * extra)  # (none is negative)
    # an insertion finds the tail pages' state beside the clusters
    k1 = narrow(np.random.default_rng(5).standard_normal((1, U, D)).astype(np.float32))
    ix2 = IceIndex(1, U, 4, n + 1, s, C, kmeans_iters=2, init_idx=up(datagen.init_indices(w)), geometry=tk)
    ix2.build_index(up(K), up(V))
    ix2.insert(up(k1), up(k1))
    e2 = {k: down(v) for k, v in ix2.export().items() if k != "view"}
    for u in range(U):
        p, t = np.argwhere(e2["page_pos"][u] == n)[0]
        c = e2["page_cluster"][u, p]
        cnt0 = int(ex["cluster_cnt"][u, c])
        assert t == cnt0 % s and e2["page_fill"][u, p] == t + 1 and e2["cluster_cnt"][u, c] == cnt0 + 1
        old = ex["page_sum"][u, p] if t else np.zeros(D, np.float32)
        assert np.array_equal(e2["page_sum"][u, p], old + widen(k1[0, u]))


@pytest.mark.parametrize("C,tk", [(1, 0), (10, 0), (10, 1), (33, 0), (40, 0), (600, 1)])
def test_keys_that_are_not_finite_keep_their_pages(C, tk):
    """A key whose scores do not compare (infinities, NaN) is nearest to nothing; its token still sits in a page of a
    cluster, as every other one does."""
    from paper_2604_10539_amd import IceIndex
    n, U, s = 2000, 2, 16
    w = datagen.small(n_tokens=n, n_clusters=C, n_kv_heads=U, n_components=max(2, C // 3))
    K, V = datagen.keys_values(w)
    init = datagen.init_indices(w)
    odd = [t for t in range(100, 1900, 150) if t not in init[0, 1]]
    for i, t in enumerate(odd):
        K[0, 1, t, i % D:] = [0x7FC0, 0x7F80, 0xFF80, 0xFFC0][i % 4]  # NaN, inf, -inf, -NaN
    ix = IceIndex(1, U, 4, n, s, C, kmeans_iters=2, init_idx=up(init), geometry=tk)
    ix.build_index(up(K), up(V))
    ex = {k: down(v) for k, v in ix.export().items() if k != "view"}
    for u in range(U):
        a = ex["assign"][u, :n]
        assert a.min() >= 0 and a.max() < C
        assert np.array_equal(ex["cluster_cnt"][u], np.bincount(a, minlength=C))
        pos = ex["page_pos"][u]
        assert np.array_equal(np.sort(pos[pos >= 0]), np.arange(n))
        assert int(ex["page_fill"][u].sum()) == n and np.array_equal(ex["page_cluster"][u, :ex["n_pages"][u]], a[pos[:ex["n_pages"][u], 0]])


def test_a_prefill_of_thousands_of_ranges():
    """Nothing in the build is sized by the number of ranges the sort cuts a unit into: 25.3 million tokens in ranges of
    8192 (the longest beside 4640 clusters) are 3089 of them, and the pages still hold the clusters' members in order."""
    import torch
    from paper_2604_10539_amd import IceIndex
    n, C, s = 25_300_000, 4640, 64
    gen = torch.Generator(device="cuda").manual_seed(3)
    K = torch.empty(1, 1, n, D, dtype=torch.int16, device="cuda")
    for i in range(0, n, 1 << 20):
        part = K[0, 0, i:i + (1 << 20)]
        part.copy_(torch.randn(part.shape, generator=gen, device="cuda").to(torch.bfloat16).view(torch.int16))
    ix = IceIndex(1, 1, 4, n, s, C, kmeans_iters=1)
    ix.build_index(K, K)
    ex = ix.export()
    assign = ex["assign"][0, :n].long()
    a, order = torch.sort(assign, stable=True)
    cnt = torch.bincount(assign, minlength=C)
    pages = (cnt + s - 1) // s
    base, start = torch.cumsum(pages, 0) - pages, torch.cumsum(cnt, 0) - cnt
    assert int(ex["n_pages"][0]) == int(pages.sum()) and torch.equal(ex["cluster_cnt"][0].long(), cnt)
    want = torch.full_like(ex["page_pos"][0], -1)
    r = torch.arange(n, device="cuda") - start[a]
    want[base[a] + r // s, r % s] = order.int()
    assert torch.equal(ex["page_pos"][0], want)
    assert torch.equal(ex["page_fill"][0], (want >= 0).sum(1).int())
    tail = ex["page_pos"][0, int(ex["cluster_tail"][0, 17])]
    live = tail[tail >= 0].long()
    assert torch.equal(ex["Kp"][0, int(ex["cluster_tail"][0, 17]), :len(live)], K[0, 0, live])
    # a mean of thousands of rows, from pieces in every range: at most cnt + 8 roundings of partial sums
    rows = K[0, 0, torch.nonzero(assign == 17)[:, 0]].view(torch.bfloat16).double()
    bound = (len(rows) + 8) * 2.0 ** -24 * rows.abs().sum(0)
    assert bool(((ex["cluster_sum"][0, 17].double() - rows.sum(0)).abs() <= bound).all())


def _attention_rows(q, k, v):
    """softmax(q k^T / sqrt(d)) v in 64 bits: q [G, D], k, v [m, D]."""
    z = q @ k.T / np.sqrt(D)
    p = np.exp(z - z.max(1, keepdims=True))
    return (p / p.sum(1, keepdims=True)) @ v


def _listed_rows(ex, u, ids, n):
    """Keys and values of the tokens of a unit's first n listed pages."""
    ks, vs = [np.empty((0, D))], [np.empty((0, D))]
    for p in ids[:max(n, 0)]:
        f = ex["page_fill"][u, p]
        ks.append(widen(ex["Kp"][u, p, :f]).astype(np.float64))
        vs.append(widen(ex["Vp"][u, p, :f]).astype(np.float64))
    return np.concatenate(ks), np.concatenate(vs)


# The output is a mean of N(0, 1) values: weights in two bf16 terms (2^-16 relative each, at most a few hundred tokens of
# weight below one) and fp32 sums stay below 2e-4 of a value of magnitude about 4.
ATTEND_TOL = 2e-4


@pytest.mark.parametrize("U,G,s,budget,n_res", [
    (2, 4, 16, 512, 512),     # split: pages' and rows' shares, none of them ragged
    (2, 4, 16, 560, 497),     # ragged shares of both
    (1, 8, 64, 64, 800),      # one page, many row shares
    (3, 2, 32, 1600, 16),     # many pages, one row share
    (2, 4, 64, 64 * 50, 0),   # pages of 64 alone, shares of four and fewer
    (4, 1, 64, 1024, 500),    # ... and beside rows
    (33, 1, 16, 512, 700),    # too many units to split
    (4, 4, 16, 256, 1),       # too little to split
    (130, 4, 16, 640, 0),     # fills fetched ahead, no rows
])
def test_attention_split_over_workgroups_with_rows_beside_the_pages(U, G, s, budget, n_res):
    """select_attend_resident and attend_resident on both sides of the rules that split the attention, whole lists
    and lists cut short."""
    from paper_2604_10539_amd import IceIndex
    w = datagen.small(n_tokens=2600, n_clusters=40, n_kv_heads=U, group_size=G, page_size=s, n_components=16)
    K, V = datagen.keys_values(w)
    ix = IceIndex(1, U, G, 2600, s, 40, kmeans_iters=1, init_idx=up(datagen.init_indices(w)))
    ix.build_index(up(K), up(V))
    rng = np.random.default_rng(U + n_res)
    rk = narrow(rng.standard_normal((1, U, max(n_res, 1), D)).astype(np.float32))[:, :, :n_res].copy()
    rv = narrow(rng.standard_normal((1, U, max(n_res, 1), D)).astype(np.float32))[:, :, :n_res].copy()
    q = datagen.queries(w)
    if n_res:
        ids, n_sel, out = ix.select_attend_resident(up(q), budget, up(rk), up(rv))
    else:
        ids, n_sel, out = ix.select_attend(up(q), budget)
    ex = {k: down(v) for k, v in ix.export().items() if k != "view"}
    n_cut = n_sel.clone()
    n_cut[0, ::2] = 3
    n_cut[0, U // 2] = 0 if n_res else 1
    cut = ix.attend_resident(up(q), ids, n_cut, up(rk), up(rv)) if n_res else ix.attend(up(q), ids, n_cut)
    qf = widen(q).astype(np.float64).reshape(U, G, D)
    for u in range(U):
        for got, n in ((out, n_sel), (cut, n_cut)):
            k, v = _listed_rows(ex, u, down(ids)[0, u], int(n[0, u]))
            k = np.concatenate([k, widen(rk[0, u]).astype(np.float64)])
            v = np.concatenate([v, widen(rv[0, u]).astype(np.float64)])
            assert np.abs(down(got).reshape(U, G, D)[u] - _attention_rows(qf[u], k, v)).max() <= ATTEND_TOL


@pytest.mark.parametrize("U,G,s,budget,tops", [(23, 4, 16, 256, 0), (24, 4, 16, 640, 0), (24, 1, 64, 256, 0), (40, 2, 32, 256, 8), (40, 8, 16, 640, 0)])
def test_attention_behind_a_staged_selection(U, G, s, budget, tops):
    """Both forms of the attention that follow the staged selection in its launch, over its own pages."""
    from paper_2604_10539_amd import IceIndex
    w = datagen.small(n_tokens=2600, n_clusters=40, n_kv_heads=U, group_size=G, page_size=s, n_components=16)
    K, V = datagen.keys_values(w)
    ix = IceIndex(1, U, G, 2600, s, 40, kmeans_iters=1, init_idx=up(datagen.init_indices(w)))
    ix.build_index(up(K), up(V))
    q = datagen.queries(w)
    if tops:
        ix.build_top_level(tops)
        ids, n_sel, out = (ix.select_hier3(up(q), budget, tops // 2, 30)[i] for i in (0, 1, -1))
    else:
        ids, n_sel, out = (ix.select_hier(up(q), budget, 30)[i] for i in (0, 1, -1))
    ex = {k: down(v) for k, v in ix.export().items() if k != "view"}
    qf = widen(q).astype(np.float64).reshape(U, G, D)
    for u in range(U):
        k, v = _listed_rows(ex, u, down(ids)[0, u], int(n_sel[0, u]))
        assert len(k) and np.abs(down(out).reshape(U, G, D)[u] - _attention_rows(qf[u], k, v)).max() <= ATTEND_TOL


@pytest.mark.parametrize("U,G,max_tok,built", [(1, 4, 1, True), (2, 8, 512, True), (8, 4, 513, True), (5, 1, 250, True), (40, 2, 300, True),
                                                (2, 4, 600, False)])
def test_attention_by_position(U, G, max_tok, built):
    """Gathered rows: lists that end anywhere (also at once), and on an index that was laid out but never built (whose
    workspace holds anything).  The workspace is left as it is: such calls may overlap."""
    from paper_2604_10539_amd import IceIndex
    n = 1500
    w = datagen.small(n_tokens=n, n_clusters=24, n_kv_heads=U, group_size=G)
    K, V = datagen.keys_values(w)
    ix = IceIndex(1, U, G, n, 16, 24, kmeans_iters=1, init_idx=up(datagen.init_indices(w)))
    ix.workspace.fill_(0x5A)
    if built:
        ix.build_index(up(K), up(V))
    else:
        ix.debug_assign(up(K), up(K[0, :, :24]))
    rng = np.random.default_rng(max_tok)
    pos = np.stack([rng.permutation(n)[:max_tok] for _ in range(U)])[None].astype(np.int32)
    n_tok = rng.integers(0, max_tok + 1, (1, U)).astype(np.int32)
    n_tok[0, 0] = max_tok
    if U > 1:
        n_tok[0, 1] = 0
    for u in range(U):
        pos[0, u, n_tok[0, u]:] = -1
    q = datagen.queries(w)
    qf = widen(q).astype(np.float64).reshape(U, G, D)
    before = ix.workspace.clone()
    for _ in range(2):
        out = down(ix.attend_tokens(up(q), up(K), up(V), up(pos), up(n_tok))).reshape(U, G, D)
        for u in range(U):
            p = pos[0, u, :n_tok[0, u]]
            ref = _attention_rows(qf[u], widen(K[0, u, p]).astype(np.float64), widen(V[0, u, p]).astype(np.float64)) if len(p) else np.zeros((G, D))
            assert np.abs(out[u] - ref).max() <= ATTEND_TOL
    assert bool((ix.workspace == before).all())


def test_attention_by_position_on_several_streams_at_once():
    """Layers that reuse one anchor's selection may attend side by side through the anchor's index."""
    import torch
    from paper_2604_10539_amd import IceIndex
    U, G, n, m = 4, 4, 6000, 2000
    w = datagen.small(n_tokens=n, n_clusters=24, n_kv_heads=U, group_size=G)
    K, V = datagen.keys_values(w)
    ix = IceIndex(1, U, G, n, 16, 24, kmeans_iters=1, init_idx=up(datagen.init_indices(w)))
    ix.build_index(up(K), up(V))
    gen = torch.Generator(device="cuda").manual_seed(1)
    layers = []
    for _ in range(4):
        rows = torch.randn(3, 1, U, n, D, generator=gen, device="cuda").to(torch.bfloat16).view(torch.int16)
        pos = torch.argsort(torch.rand(1, U, n, generator=gen, device="cuda"), dim=2)[:, :, :m].int().contiguous()
        layers.append((rows[2, :, :, :G].reshape(1, U * G, D).contiguous(), rows[0], rows[1], pos, torch.full((1, U), m, dtype=torch.int32, device="cuda")))
    want = [ix.attend_tokens(*x) for x in layers]
    streams = [torch.cuda.Stream() for _ in layers]
    torch.cuda.synchronize()
    for _ in range(5):
        got = []
        for s, x in zip(streams, layers):
            with torch.cuda.stream(s):
                got.append([ix.attend_tokens(*x) for _ in range(4)])
        torch.cuda.synchronize()
        assert all(torch.equal(g, y) for gs, y in zip(got, want) for g in gs)


def test_unit_whose_selection_failed_gets_zeros_with_a_window_too():
    """The attention of a selection call that moved to a launch of its own leaves the failed unit's output zero, as the
    fused one does, although there are rows to attend to."""
    from paper_2604_10539_amd import IceIndex
    from paper_2604_10539_amd.binding import ice_debug_select_fault
    w = datagen.small(n_tokens=8000, n_clusters=100, n_kv_heads=2)
    K, V = datagen.keys_values(w)
    ix = IceIndex(1, 2, 4, 8000, 16, 100, kmeans_iters=1, init_idx=up(datagen.init_indices(w)))
    ix.build_index(up(K), up(V))
    q, rows = up(datagen.queries(w)), up(K[:, :, :600])
    for budget, n_res in ((256, 16), (512, 600)):  # fused, split
        ids, n_sel, good = ix.select_attend_resident(q, budget, rows[:, :, :n_res].contiguous(), rows[:, :, :n_res].contiguous())
        assert int(n_sel.min()) == budget // 16 and float(good.abs().max()) > 0
    ids, n_sel = ix._sel_buffers(256)
    ice_debug_select_fault(ix.handle, q, 256, ids, n_sel, None, 0, 2)
    for budget, n_res in ((256, 16), (512, 600)):
        ids, n_sel, out = ix.select_attend_resident(q, budget, rows[:, :, :n_res].contiguous(), rows[:, :, :n_res].contiguous())
        assert int(n_sel.max()) == -1 and int(ids.max()) == -1 and float(out.abs().max()) == 0.0


@pytest.mark.parametrize("m,C,s,tk", [(2, 20, 16, 0), (16, 20, 16, 0), (17, 20, 16, 1), (33, 300, 64, 0), (100, 20, 16, 1), (21, 5000, 16, 0),
                                       (3, 8192, 16, 0), (3, 8192, 16, 1), (5, 6000, 16, 1)])
def test_insertions_in_rounds_equal_single_ones(m, C, s, tk):
    """A call takes as many tokens at a time as its tables hold (16, fewer with many clusters) and reads back what it
    stored: remainders of one token, rows moved and pages opened in one round and used in the next."""
    from paper_2604_10539_amd import IceIndex
    n, U = max(700, C), 3
    w = datagen.small(n_tokens=n, n_clusters=C, n_kv_heads=U, n_components=6, page_size=s)
    K, V = datagen.keys_values(w)
    new = narrow((widen(K[:, :, :1]) + 0.4 * np.random.default_rng(m).standard_normal((1, U, m, D))).astype(np.float32))  # they crowd
    new[:, :, 1::3] = K[:, :, 5:5 + len(range(1, m, 3))]
    state = []
    for batch in (True, False):
        ix = IceIndex(1, U, 4, n + m, s, C, kmeans_iters=1, init_idx=up(datagen.init_indices(w)), geometry=tk)
        ix.workspace.zero_()
        ix.build_index(up(K), up(V))
        if batch:
            ix.insert_batch(up(new), up(new[:, :, ::-1]))
        else:
            for t in range(m):
                ix.insert(up(new[:, :, t]), up(new[:, :, ::-1][:, :, t]))
        ex = {k: down(v).copy() for k, v in ix.export().items() if k not in ("view", "assign")}
        if tk:
            ex.update({k: down(v).copy() for k, v in ix.export_geometry().items()})
        state.append(ex)
    for name in state[0]:
        if name not in ("assign_centroid_bf16", "assign_centroid_extra_bf16"):
            assert np.array_equal(state[0][name], state[1][name]), name


@pytest.mark.parametrize("P,s", [(1, 16), (2, 64), (63, 16), (128, 16), (129, 32), (1024, 64)])
def test_positions_of_listed_pages(P, s):
    """The positions in list and slot order, padded with -1: lists up to the longest, cut short, empty, with entries that
    are not page ids."""
    from paper_2604_10539_amd import IceIndex
    w = datagen.small(n_tokens=5000, n_clusters=60, n_kv_heads=3, page_size=s)
    K, V = datagen.keys_values(w)
    ix = IceIndex(1, 3, 4, 5000, s, 60, kmeans_iters=1, init_idx=up(datagen.init_indices(w)))
    ix.build_index(up(K), up(V))
    ex = {k: down(v) for k, v in ix.export().items() if k != "view"}
    rng = np.random.default_rng(P)
    ids = np.stack([rng.integers(0, ex["n_pages"][u], P) for u in range(3)])[None].astype(np.int32)
    ids[0, 0, P // 2] = ex["page_fill"].shape[1] + 5
    n_sel = np.array([[P, max(P - 1, 0), 0]], np.int32)
    pos, n_tok = ix.selected_tokens(up(ids), up(n_sel))
    pos, n_tok = down(pos), down(n_tok)
    for u in range(3):
        want = [t for p in ids[0, u, :n_sel[0, u]] if 0 <= p < ex["page_fill"].shape[1] for t in ex["page_pos"][u, p, :ex["page_fill"][u, p]]]
        assert n_tok[0, u] == len(want)
        assert np.array_equal(pos[0, u], np.array(want + [-1] * (P * s - len(want))))


@pytest.mark.parametrize("kw,odd", [(dict(n_tokens=1000, n_clusters=33), False), (dict(n_tokens=1000, n_clusters=33), True),
                                    (dict(n_tokens=70, n_clusters=3, n_kv_heads=1, page_size=64), False)])
def test_imports_in_one_launch_and_through_copies(kw, odd):
    """Both forms of an import (odd: one array at an address the single launch does not take) leave the caller's arrays,
    and insertion and selection work on what they derived."""
    from paper_2604_10539_amd import IceIndex
    from paper_2604_10539_amd.binding import IMPORT_FIELDS
    import torch
    w = datagen.small(**kw)
    U, s, C, n = w.n_kv_heads, w.page_size, w.n_clusters, w.n_tokens
    K, V = datagen.keys_values(w)
    make = lambda: IceIndex(1, U, 4, n + 40, s, C, kmeans_iters=2, init_idx=up(datagen.init_indices(w)))
    a = make()
    a.build_index(up(K), up(V))
    arrays = {f: a.export()[f].clone() for f in IMPORT_FIELDS}
    if odd:
        t = arrays["n_pages"]
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        buf[1:] = t
        arrays["n_pages"] = buf[1:]
    b = make()
    b.workspace.fill_(0x33)
    b.import_arrays(arrays, n)
    for f in IMPORT_FIELDS:
        assert torch.equal(b.export()[f], arrays[f]), f
    k1, q = up(K[:, :, :20].copy()), up(datagen.queries(w))
    for ix in (a, b):
        ix.insert_batch(k1, k1)
    (ia, na, oa), (ib, nb, ob) = (ix.select_attend(q, 4 * s) for ix in (a, b))
    assert torch.equal(ia, ib) and torch.equal(na, nb) and torch.equal(oa, ob)
    ea, eb = a.export(), b.export()
    for f in ("page_fill", "page_pos", "cluster_cnt", "cluster_sum", "centroid", "cluster_tail", "n_pages"):
        assert torch.equal(ea[f], eb[f]), f


def _every_stage_again(Kd, Vd, init, C, tk, T):
    """The state of a build of T rounds, the same after every stage of the last round has been done again in full."""
    import torch
    from paper_2604_10539_amd import IceIndex, ice_debug_rerun_stage
    from paper_2604_10539_amd.binding import ICE_GEOMETRY_RAW, ICE_GEOMETRY_TRANSFORMED
    U, n = Kd.shape[1], Kd.shape[2]
    ix = IceIndex(1, U, 4, n, 16, C, kmeans_iters=T, init_idx=init, geometry=ICE_GEOMETRY_TRANSFORMED if tk else ICE_GEOMETRY_RAW)
    ix.build_index(Kd, Vd)

    def state():
        ex = dict(ix.export())
        out = {f: ex[f] for f in ("assign", "cluster_cnt", "cluster_sum", "centroid", "Kp", "page_pos", "page_sum", "n_pages")}
        geo = ix.export_geometry()
        if geo:
            out.update({f: geo[f] for f in ("centroid_extra", "cluster_sum_extra")})
        torch.cuda.synchronize()
        return {f: (x.view(torch.int32) if x.dtype == torch.float32 else x).clone() for f, x in out.items()}
    had = state()
    for stage in range(4):
        ice_debug_rerun_stage(ix.handle, Kd, Vd, stage)
    now = state()
    for f in had:
        if f == "Kp":  # (live pages)
            for u in range(U):
                p = int(had["n_pages"][u])
                assert torch.equal(had[f][u, :p], now[f][u, :p]), (T, f, u)
        else:
            assert torch.equal(had[f], now[f]), (T, f)
    return had


@pytest.mark.parametrize("U,n,C,tk,odd", [(3, 700, 40, 0, False), (2, 3000, 130, 1, False), (2, 4100, 520, 0, False), (1, 1500, 1100, 1, False),
                                          (5, 2600, 500, 0, False), (2, 5000, 16, 1, False), (1, 9000, 250, 0, True), (2, 2000, 700, 1, True)])
def test_later_rounds_do_again_what_changed_and_leave_what_all_of_it_would(U, n, C, tk, odd):
    """A build's later rounds leave out units of which no centroid moved and sum only clusters whose members
    changed.  Every stage of the last round once more, over everything, leaves the same bits, after two rounds, three, ...
    nine (each of them started from the state that the one before found right), twelve and thirty.  Few and many centroid tiles, several
    slices of 512, clusters of one key; `odd`: among keys without a comparable score and equal keys.  Builds this small score
    all centroids in every round; the next test's do not."""
    import torch
    from paper_2604_10539_amd import ice_debug_build_plan, make_config
    assert ice_debug_build_plan(make_config(1, U, 4, n), n, C)["reassign_from"] == 0
    w = datagen.small(n_tokens=n, n_clusters=C, n_kv_heads=U, n_components=max(4, C // 2), outlier_frac=0.05)
    K, V = datagen.keys_values(w)
    if odd:
        K[0, :, 100:400] = K[0, :, 100:101]
        for i, t in enumerate(range(5, n, 211)):
            K[0, :, t, i % D:] = [0x7FC0, 0x7F80, 0xFF80, 0xFFC0][i % 4]  # NaN, inf, -inf, -NaN
    Kd, Vd, init = up(K), up(V), up(datagen.init_indices(w))
    settled = False
    for T in (2, 3, 4, 5, 6, 7, 8, 9, 12, 30):
        had = _every_stage_again(Kd, Vd, init, C, tk, T)
        if T == 12:
            last = had
        if T == 30 and not odd:
            settled = torch.equal(last["assign"], had["assign"])
    assert settled or odd or n > 100 * C  # (rounds in which nothing moves were among them, unless clusters are large)


@pytest.mark.parametrize("U,n,C,tk,odd,slices,run,fused", [
    (8, 32768, 512, 0, "", 1, 4, 1),       # one slice, its sort inside, four key tiles per workgroup
    (16, 23457, 366, 1, "", 1, 6, 1),      # ... transformed, a slice not full, a ragged last tile
    (16, 9000, 700, 0, "", 2, 3, 0),       # two slices (and one at a time for few moved centroids)
    (24, 3000, 1100, 1, "", 3, 2, 0),
    (32, 2060, 2048, 0, "", 4, 2, 0),      # clusters of one key
    (4, 40000, 600, 1, "few", 2, 3, 0),    # components far fewer than clusters: centroids go on moving
    (16, 9000, 700, 0, "none", 2, 3, 0),   # no components at all
    (8, 34000, 400, 0, "none", 1, 5, 1),
    (16, 9000, 700, 1, "odd", 2, 3, 0),    # equal keys, and units of which some keys are not finite beside units of which all are
    (8, 32768, 512, 0, "odd", 1, 4, 1),
    (8, 32768, 512, 1, "odd", 1, 4, 1),
])
def test_later_rounds_that_score_what_moved_leave_what_all_centroids_would(U, n, C, tk, odd, slices, run, fused):
    """The same, after three rounds to nine and after twelve, where later rounds score only the centroids that moved and then the
    keys that lost theirs: from the third round on, over one slice of 512 centroids and several, with the sort inside and after it, from rounds in which most
    centroids moved (those are done in full) to rounds in which few did and none."""
    import torch
    from paper_2604_10539_amd import ice_debug_build_plan, make_config
    p = ice_debug_build_plan(make_config(1, U, 4, n), n, C)
    assert (p["reassign_from"], p["slices"], p["run"], p["fused"]) == (2, slices, run, fused)
    gen = torch.Generator(device="cuda").manual_seed(U * n + C)
    K = torch.randn(1, U, n, D, generator=gen, device="cuda")
    if odd != "none":
        M = C // 20 if odd == "few" else C // 2
        centers = torch.randn(U, M, D, generator=gen, device="cuda")
        at = torch.randint(M, (U, n), generator=gen, device="cuda")
        K = 0.3 * K + torch.gather(centers, 1, at[..., None].expand(-1, -1, D))[None]
    K = K.to(torch.bfloat16).view(torch.int16)
    if odd == "odd":
        K[0, :, 100:400] = K[0, :, 100:101]
        for i, t in enumerate(range(5, n, 211)):
            # NaN, inf, -inf, -NaN, 2^64, -2^64 (whose products overflow)
            K[0, ::2, t, i % D:] = [0x7FC0, 0x7F80, 0xFF80 - 65536, 0xFFC0 - 65536, 0x5F80, 0xDF80 - 65536][i % 6]
    V = torch.randint(-16000, 16000, K.shape, generator=gen, device="cuda", dtype=torch.int16)
    init = torch.stack([torch.sort(torch.randperm(n, generator=gen, device="cuda")[:C])[0] for _ in range(U)]).int()[None].contiguous()
    for T in (3, 4, 5, 6, 7, 8, 9, 12):
        _every_stage_again(K, V, init, C, tk, T)


@pytest.mark.parametrize("U,n,C,tk,data,ranges,fused", [
    (256, 19300, 600, 0, "mix", 1, 0),     # a cluster is one piece; two slices, the second hardly begun; a ragged last tile
    (300, 16500, 300, 1, "mix", 1, 0),     # more units than workgroups of a round, transformed keys
    (32, 32768, 512, 0, "out", 8, 1),      # eight pieces, one full slice with the sort inside
    (33, 28000, 417, 1, "mix", 7, 1),      # ... transformed, a slice that is not full, a last block of few centroids
    (6, 65000, 1100, 0, "out", 32, 0),     # more pieces than a member is picked from directly
    (2, 131072, 1600, 1, "out", 64, 0),
    (1, 262144, 2112, 0, "mix", 64, 0),    # five slices; one tile of rows at a time
    (1, 1100000, 3000, 0, "mix", 68, 0),   # more pieces than a wave holds
    (8, 65536, 1024, 0, "lump", 32, 0),    # a cluster of a third of the keys, equal keys, centroids that are the same
    (8, 65536, 1024, 1, "lump", 32, 0),
    (8, 65536, 1024, 0, "few", 32, 0),     # components far fewer than clusters: lists that come out too long, centroids that go on moving
    (8, 65536, 1024, 0, "half", 32, 0),    # every other unit without structure: those take all in every round
    (8, 65536, 1024, 1, "odd", 32, 0),     # units with keys that are not finite beside units of which all are
    (8, 65536, 1024, 0, "tiny", 32, 0),    # products and squared distances that end among the subnormal numbers
    (8, 65536, 1024, 1, "tiny", 32, 0),
    (8, 65536, 1024, 0, "wide", 32, 0),    # components too wide: units that turn to the moved centroids in the second round
    (32, 32768, 512, 1, "wide", 8, 1),
    (8, 65536, 1024, 0, "late", 32, 0),    # ... that turn in the third: every second cluster is narrow, the others hold most keys
    (32, 32768, 512, 0, "late", 8, 1),
    (4, 131072, 1100, 1, "late", 64, 0),
    (1, 262144, 2112, 0, "late", 64, 0),
    (520, 16500, 450, 0, "half", 1, 0),    # many units, which turn one by one
    (520, 16500, 450, 1, "odd", 1, 0),
    (520, 16500, 450, 0, "late", 1, 0),
    (1, 200000, 2500, 1, "mix", 49, 0),    # transformed keys where one tile of rows fits and a list is two words to a lane
    (8, 65536, 1024, 0, "offset 5", 32, 0),    # a common offset: distances out of cancelled squares, the margin of many times what
    (8, 65536, 1024, 1, "offset 5", 32, 0),    # they are without it
    (8, 65536, 1024, 0, "offset 8", 32, 0),    # ... where it leaves part of the keys open
    (8, 65536, 1024, 0, "offset 20", 32, 0),   # ... nearly all of them
    (8, 65536, 1024, 1, "offset 100", 32, 0),
])
def test_later_rounds_by_the_centroids_near_a_keys_own_leave_what_all_would(U, n, C, tk, data, ranges, fused):
    """The same where every later round takes the keys of a cluster to the centroids near its own and only the keys that this
    leaves open to more of them, from the second round on until hardly any centroid moves; every round is looked at.  Builds of
    so few rounds that they go another way stand for none of them: the shortest build that goes this way leaves then what its units
    leave by themselves."""
    import torch
    from paper_2604_10539_amd import ice_debug_build_plan, make_config
    plan_of = lambda U, T: ice_debug_build_plan(make_config(1, U, 4, n, kmeans_iters=T), n, C)
    p = plan_of(U, 10)
    assert (p["reassign_from"], p["ranges"], p["fused"]) == (1, ranges, fused)
    gen = torch.Generator(device="cuda").manual_seed(U * n + C)
    K = torch.empty(1, U, n, D, dtype=torch.int16, device="cuda")
    M = C // 20 if data == "few" else C // 2
    broad = torch.zeros(U, n, dtype=torch.bool, device="cuda")
    for u in range(U):
        x = torch.randn(n, D, generator=gen, device="cuda")
        if data == "late":
            broad[u] = torch.rand(n, generator=gen, device="cuda") < (0.8 if u % 3 < 2 else 0.1)  # (every third unit does not turn)
            at = torch.randint(M // 2, (n,), generator=gen, device="cuda") + broad[u] * (M // 2)
            x = (0.1 + 0.7 * broad[u].float())[:, None] * x + torch.randn(M, D, generator=gen, device="cuda")[at]
        elif data != "half" or u % 2 == 0:
            x = (0.6 if data == "wide" else 0.3) * x + torch.randn(M, D, generator=gen, device="cuda")[torch.randint(M, (n,), generator=gen, device="cuda")]
        if data == "out":
            far = torch.rand(n, generator=gen, device="cuda") < 0.05
            x = torch.where(far[:, None], 6 * torch.rand(n, D, generator=gen, device="cuda") - 3, x)
        if data == "lump":
            x[n // 2: n // 2 + n // 3] = 0.01 * x[n // 2: n // 2 + n // 3]
            x[100:400] = x[100:101]
        if data.startswith("offset"):  # (so many times the components' spread)
            x = x + float(data.split()[1]) * torch.randn(D, generator=gen, device="cuda")
        if data == "tiny":
            x = torch.ldexp(x, torch.tensor(-50 if u == 0 else -60 - 2 * u, device="cuda"))
        K[0, u] = x.to(torch.bfloat16).view(torch.int16)
    if data == "odd":
        for i, t in enumerate(range(5, n, 2111)):
            K[0, ::2, t, i % D:] = [0x7FC0, 0x7F80, 0xFF80 - 65536, 0xFFC0 - 65536, 0x5F80, 0xDF80 - 65536][i % 6]
    V = torch.randint(-16000, 16000, K.shape, generator=gen, device="cuda", dtype=torch.int16)
    init = torch.stack([torch.sort(torch.randperm(n, generator=gen, device="cuda")[:C])[0] for _ in range(U)])
    if data == "late":
        for u in range(U):
            for first in (0, 1):  # (even clusters start at narrow keys)
                init[u, first::2] = torch.nonzero(broad[u] == bool(first))[:(C + 1 - first) // 2, 0]
    if data == "lump":
        init[:, 10:50] = torch.arange(100, 140, device="cuda")  # (centroids on equal keys)
    init = init.int()[None].contiguous()
    shortest = next(T for T in range(2, 10) if plan_of(U, T)["reassign_from"] == 1)
    for T in range(2, 10):
        had = _every_stage_again(K, V, init, C, tk, T)
        if T == shortest > 2:
            for u in {0, 1, U // 2, U - 1}:
                assert plan_of(1, T)["reassign_from"] != 1
                alone = _every_stage_again(K[:, u:u + 1], V[:, u:u + 1], init[:, u:u + 1], C, tk, T)
                for f in ("assign", "cluster_cnt", "cluster_sum", "centroid", "n_pages"):
                    assert torch.equal(had[f][u], alone[f][0]), (T, f, u)


def test_later_rounds_where_scores_stop_comparing():
    """A cluster that takes in an infinite key in the third round has a mean with which most scores do not compare in the
    fourth.  With eight NaN rows around it since the start, the full contraction finds nine NaN side by side, which hide the
    other rows held beside them; a round that looks only at the centroids that moved has to come to the same."""
    import torch
    from paper_2604_10539_amd import IceIndex
    from paper_2604_10539_amd import ice_debug_build_plan, ice_debug_rerun_stage, make_config
    C, first, j, U = 2048, 64, 127, 32   # rows 64..95 are a tile
    a, b = first + 16, first + 17        # the ninth row of the tile's first half, and the row that loses a key to it
    rng = np.random.default_rng(3)
    K = rng.standard_normal((C, D))      # clusters of one key, far apart
    K *= 100.0 / np.linalg.norm(K, axis=1, keepdims=True)
    K[a] = K[b] = 0.0
    K[b, 0] = 10.0
    K[:, j] = np.where(np.arange(C) > b, 1.0, -2.0 ** -10)
    more = np.zeros((12, D))
    more[:10, 0], more[:10, j] = 30.0, -2.0 ** -10  # row b follows them after the first round
    more[10, 0], more[10, j] = 6.0, 1.0  # goes to b first, then to a, whose coordinate j is positive from then on
    K = narrow(np.concatenate([K, more]).astype(np.float32))
    K[first + np.r_[0:4, 8:12]] = 0x7FC0
    K[C + 11, j] = 0x7F80                # nearest, at +inf, to the first row with a positive coordinate j: b + 1, then b, then a
    Kd, init = up(np.stack([K] * U)[None]), up(np.stack([np.arange(C, dtype=np.int32)] * U)[None])
    assert ice_debug_build_plan(make_config(1, U, 4, len(K)), len(K), C)["reassign_from"] == 2
    for T in (3, 4, 6):
        ix = IceIndex(1, U, 4, len(K), 16, C, kmeans_iters=T, init_idx=init)
        ix.build_index(Kd, Kd)
        ex = ix.export()
        had = {f: ex[f].clone() for f in ("assign", "cluster_cnt", "page_pos")}
        for stage in range(4):
            ice_debug_rerun_stage(ix.handle, Kd, Kd, stage)
        torch.cuda.synchronize()
        for f in had:
            assert torch.equal(had[f], ex[f]), (T, f)
        if T == 3:
            assert had["assign"][0, C + 11] == a
        lost = int((had["assign"][0, :C] != torch.arange(C, device="cuda")).sum())
        assert lost < 16 if T == 3 else lost > 30  # (rows 64..127 of the same lanes)


@pytest.mark.parametrize("U,G", [(3, 4), (2, 8), (256, 1), (256, 8)])
def test_pages_of_one_cluster_side_by_side_at_every_budget(U, G):
    """Pages that score alike sit beside each other, so whole clusters fall into one group of the selection's threshold; the
    budgets are those where its groups, the list behind it and the order of the returned ids change (and kept clusters of the
    staged selection beside them): several workgroups per unit and one."""
    import torch
    from paper_2604_10539_amd import IceIndex
    n, C, s = (4096, 64, 16) if U < 256 else (1500, 40, 16)
    w = datagen.small(n_tokens=n, n_clusters=C, n_kv_heads=min(U, 8), n_components=C // 2, group_size=G)
    K, V = datagen.keys_values(w)
    K, V = (np.ascontiguousarray(np.resize(x[0], (U,) + x.shape[2:]))[None] for x in (K, V))
    q = np.ascontiguousarray(np.resize(datagen.queries(w)[0], (U * G, D)))[None]
    ix = IceIndex(1, U, G, n, s, C, kmeans_iters=3, init_idx=up(np.resize(datagen.init_indices(w)[0], (U, C))[None]))
    ix.build_index(up(K), up(V))
    ex = ix.export()
    torch.cuda.synchronize()
    npg, rep = down(ex["n_pages"]), widen(down(ex["rep"])).astype(np.float64)
    qf = widen(q[0]).astype(np.float64).reshape(U, G, D)
    qf /= np.linalg.norm(qf, axis=2, keepdims=True)
    units = range(U) if U < 256 else (0, 1, 100, 255)
    for P in (1, 2, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 200, 256, 257, int(npg.min()) - 1):
        if P < 1 or P >= npg.min():
            continue
        ids, n_sel, out = (down(x) for x in ix.select_attend(up(q), P * s))
        for u in units:
            got = ids[0, u]
            assert n_sel[0, u] == P and np.all(np.diff(got) > 0)
            sc = (rep[u, :npg[u]] @ qf[u].T).max(1)
            kth = np.sort(sc)[::-1][P - 1]
            # fp32 scores of unit-length rows: chains of 128 additions on values of at most a few units
            assert np.all(sc[got] >= kth - 1e-5 * max(1.0, abs(kth))), (P, u)
        if P in (2, 64, 65, 129, 256, 257):  # (the scores beside their ids, and the staged selection when it keeps every cluster)
            ids2, n2, scores = (down(x) for x in ix.select(up(q), P * s))
            ids3, n3, scores3 = (down(x) for x in ix.select_hier(up(q), P * s, C, attend=False)[:3])
            for i, k, x in ((ids2, n2, scores), (ids3, n3, scores3)):
                assert np.array_equal(i, ids) and np.array_equal(k, n_sel)
                for u in units:
                    sc = (rep[u, :npg[u]] @ qf[u].T).max(1)
                    assert np.all(np.abs(x[0, u] - sc[i[0, u]]) <= 1e-5 * np.maximum(1.0, np.abs(sc[i[0, u]])))
    for probe in (1, 31, C - 1):
        ids, n_sel, _, cl, _ = ix.select_hier(up(q), 64, probe)
        cl = down(cl)[0]
        pc = down(ex["page_cluster"])
        for u in units:
            assert np.all(np.diff(cl[u]) > 0) and 0 <= cl[u, 0] and cl[u, -1] < C
            k = int(down(n_sel)[0, u])
            assert set(pc[u, down(ids)[0, u, :k]]) <= set(cl[u])


@pytest.mark.parametrize("m,C,s,tk", [(18, 16, 16, 0), (40, 17, 16, 1), (50, 430, 16, 1), (50, 470, 16, 0), (48, 225, 32, 0),
                                       (64, 225, 32, 0), (180, 64, 16, 0), (200, 64, 16, 1), (200, 63, 16, 0),
                                       (50, 448, 16, 0), (70, 448, 16, 1), (50, 449, 16, 0), (70, 449, 16, 1)])
def test_insertions_scored_a_round_ahead_equal_single_ones(m, C, s, tk):
    """In long calls, where LDS holds a second table of scores, a round's scores come from the round before, put right for the
    rows it moved: fewer tiles of centroids than scanning waves and more, calls on both sides of the lengths from which it is
    done, the largest count that fits (448 clusters; transformed keys fill LDS to its last byte with it) and the first that
    does not, four and five rounds of them."""
    test_insertions_in_rounds_equal_single_ones(m, C, s, tk)


@pytest.mark.parametrize("G", [4, 8])
@pytest.mark.parametrize("C", [140, 520, 1100])
def test_staged_selection_at_the_edges_of_its_threshold_groups(C, G):
    """The kept clusters and pages at counts where the threshold changes its groups (half the 32, 64 or 128 of them) or goes by
    histograms (above 64), and where the list behind it is ranked in another form: they are the best of 64-bit scores."""
    import torch
    from paper_2604_10539_amd import IceIndex
    n, U, s = 8 * C, 2, 16
    w = datagen.small(n_tokens=n, n_clusters=C, n_kv_heads=U, n_components=C // 2, group_size=G)
    K, V = datagen.keys_values(w)
    ix = IceIndex(1, U, G, n, s, C, kmeans_iters=2, init_idx=up(datagen.init_indices(w)))
    ix.build_index(up(K), up(V))
    ex = ix.export()
    torch.cuda.synchronize()
    npg, pc = down(ex["n_pages"]), down(ex["page_cluster"])
    rep, cen = widen(down(ex["rep"])).astype(np.float64), widen(narrow(down(ex["centroid"]))).astype(np.float64)
    qb = datagen.queries(w)
    qf = widen(qb[0]).astype(np.float64).reshape(U, G, D)
    qf /= np.linalg.norm(qf, axis=2, keepdims=True)
    ahead = 1e-5  # fp32 scores of unit-length queries: chains of 128 additions on values of at most a few units
    for k in (1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 200):
        if k >= C:
            continue
        ids, n_sel, scores, cl, _ = ix.select_hier(up(qb), k * s, k, attend=False)
        ids, n_sel, cl = down(ids)[0], down(n_sel)[0], down(cl)[0]
        for u in range(U):
            sc = (cen[u, :C] @ qf[u].T).max(1)
            kth = np.sort(sc)[::-1][k - 1]
            assert np.all(np.diff(cl[u]) > 0) and np.all(sc[cl[u]] >= kth - ahead * max(1.0, abs(kth))), (k, u)
            cand = np.nonzero(np.isin(pc[u, :npg[u]], cl[u]))[0]
            P = min(k, len(cand))
            assert n_sel[u] == P and np.all(np.diff(ids[u, :P]) > 0) and np.all(ids[u, P:] == -1)
            assert np.all(np.isin(ids[u, :P], cand))
            ps = (rep[u] @ qf[u].T).max(1)
            kth = np.sort(ps[cand])[::-1][P - 1]
            assert np.all(ps[ids[u, :P]] >= kth - ahead * max(1.0, abs(kth))), (k, u)


@pytest.mark.parametrize("G", [4, 8])
def test_staged_selection_among_more_equal_scores_than_its_list_holds(G):
    """700 clusters with the same centroid and 700 pages with the same representative: more of them pass the threshold than are ranked
    by counting, and the lowest ids are kept."""
    import torch
    from paper_2604_10539_amd import IceIndex
    same, C, s, U = 700, 1100, 16, 2
    n = s * same + 8 * (C - same)
    rng = np.random.default_rng(5)
    K = rng.standard_normal((1, U, n, D))
    K[:, :, :s * same] = 3.0 * rng.standard_normal((1, U, 1, D))
    K = narrow(K.astype(np.float32))
    init = np.concatenate([s * np.arange(same), s * same + 8 * np.arange(C - same)]).astype(np.int32)  # (the first keeps all equal keys)
    ix = IceIndex(1, U, G, n, s, C, kmeans_iters=2, init_idx=up(np.ascontiguousarray(np.broadcast_to(init, (1, U, C)))))
    ix.build_index(up(K), up(K))
    ex = ix.export()
    torch.cuda.synchronize()
    cen, pc = down(ex["centroid"])[:, :same], down(ex["page_cluster"])
    assert np.all(cen == cen[:, :1]) and np.all(pc[:, :same] == 0)
    q = np.ascontiguousarray(np.repeat(K[:, :, :1], G, axis=2)).reshape(1, U * G, D)
    for k in (15, 17, 33, 64, 65, 200):
        for P in (15, 17, 33, 64, 65, 200):
            ids, n_sel, _, cl, _ = ix.select_hier(up(q), P * s, k, attend=False)
            assert np.all(down(n_sel) == P), (k, P)
            assert np.array_equal(down(cl)[0], np.tile(np.arange(k), (U, 1))), (k, P)
            assert np.array_equal(down(ids)[0], np.tile(np.arange(P), (U, 1))), (k, P)
