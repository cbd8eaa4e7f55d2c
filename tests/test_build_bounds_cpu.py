"""The bounds behind a large build's later rounds, on the host: where they say that a key need not be scored against a centroid,
that centroid loses to the best one known in fp32, in whatever order the products are added, and the bound on a distance lies
below it.  The keys sit where the rounding of the scores decides: just short of half way to the centroid that is left out, far
from the origin (the distances come out of cancelled squares) and so close to it that products and sums are subnormal.  And which builds
go that way."""
import numpy as np
import pytest

from datagen import bf16_bits_to_f32 as widen, f32_to_bf16_bits as narrow
from paper_2604_10539_amd import ice_debug_build_plan, ice_debug_near_bounds, make_config

D = 128
TINY = np.float32(2.0 ** -126)


def _products(a, b, flush):
    with np.errstate(under="ignore"):
        p = a * b
    return np.where(np.abs(p) < TINY, np.float32(0), p) if flush else p


def _sum32(start, p, order, flush):
    """start + the products in fp32, one after the other in the given order, or in blocks of 16 summed in pairs first."""
    s = start.copy()
    if order == "blocks":
        while p.shape[-1] > D // 16:
            p = p[..., 0::2] + p[..., 1::2]
            p = np.where(np.abs(p) < TINY, np.float32(0), p) if flush else p
    for i in range(p.shape[-1]) if order != "reversed" else range(p.shape[-1] - 1, -1, -1):
        s = s + p[..., i]
        if flush:
            s = np.where(np.abs(s) < TINY, np.float32(0), s)
    return s


def _score(k, c, order, flush):
    c2 = _sum32(np.zeros(c.shape[:-1], np.float32), _products(c, c, flush), order, flush)
    return _sum32(np.float32(-0.5) * c2, _products(k, c, flush), order, flush)


def _cases(spread, large, scale, seed):
    """Own centroid a, centroid c left out, keys at up to half of the way from a to c, all bf16.  spread 0: about the origin, and
    the keys somewhat beside the way; else they share a quarter of large coordinates and are at most so many steps of bf16 apart in
    the others, and half of the keys are exactly half way."""
    rng = np.random.default_rng(seed)
    m = 4000
    if spread:
        sign = rng.choice([-1.0, 1.0], D)
        a, d = sign * (1 + rng.integers(48, 80, (m, D)) / 128), rng.integers(-spread, spread + 1, (m, D)) / 128
        a[:, ::4] *= large
        d[:, ::4] = 0
        part = np.where(np.arange(m) % 2 == 0, 1.0, rng.uniform(0.0, 1.0, m))[:, None]
        k, c = a + part * d, a + 2 * d
    else:
        a, c = rng.standard_normal((m, D)), rng.standard_normal((m, D))
        way = np.where(np.arange(m) % 4 == 0, rng.uniform(0.3, 0.5, m), rng.uniform(0.47, 0.5, m))[:, None]
        k = a + way * (c - a) + rng.standard_normal((m, D)) * rng.choice([0.0, 1e-3, 0.02], m)[:, None]
    return [widen(narrow((scale * x).astype(np.float32))) for x in (a, c, k)]


@pytest.mark.parametrize("flush", [False, True])
@pytest.mark.parametrize("order", ["ascending", "reversed", "blocks"])
@pytest.mark.parametrize("spread,large,scale", [(0, 1, 1.0), (0, 1, 2.0 ** -46), (0, 1, 2.0 ** -50), (0, 1, 2.0 ** -56), (0, 1, 2.0 ** -62), (0, 1, 2.0 ** -68), (0, 1, 2.0 ** -72), (0, 1, 2.0 ** -75),
                                                (32, 1, 1.0), (32, 2, 1.0), (32, 16, 1.0), (32, 64, 1.0), (8, 64, 1.0), (2, 64, 1.0), (32, 256, 1.0), (8, 256, 2.0 ** 46), (32, 1, 2.0 ** -70), (32, 16, 2.0 ** -70)])
def test_a_centroid_that_the_bounds_leave_out_loses(spread, large, scale, order, flush):
    a, c, k = _cases(spread, large, scale, 7 + spread)
    with np.errstate(under="ignore"):
        zero = np.zeros(len(a), np.float32)
        k2 = _sum32(zero, _products(k, k, flush), order, flush)
        a2 = _sum32(zero, _products(a, a, flush), order, flush)
        sa, sc, ac = _score(k, a, order, flush), _score(k, c, order, flush), _score(a, c, order, flush)
    need, _ = ice_debug_near_bounds(k2, a2, sa, sa)      # (the own centroid is the best one known)
    _, dist2 = ice_debug_near_bounds(k2, a2, sa, ac)
    true2 = ((a.astype(np.float64) - c) ** 2).sum(1)
    # (an absolute part of 2^-117 is what near_need's floor stands for)
    assert np.all(dist2 <= true2 * (1 + 2.0 ** -20) + 2.0 ** -117)
    settled = np.sqrt(dist2.astype(np.float64)) > need
    assert np.all(sa[settled] > sc[settled]), int((settled & ~(sa > sc)).sum())
    # without a margin the same test settles keys that it must not: these inputs are such that rounding decides
    bare = np.sqrt(np.maximum(k2.astype(np.float64) - 2.0 * sa, 0.0)) * 2 < np.sqrt(np.maximum(a2.astype(np.float64) - 2.0 * ac, 0.0))
    if (large > 2 and scale >= 1) or (2.0 ** -62 if flush else 2.0 ** -75) <= scale <= (2.0 ** -60 if flush else 2.0 ** -72):
        assert np.any(bare & ~(sa > sc))
    if (spread == 0 or large < 4) and scale >= 2.0 ** -46:
        assert settled.sum() > len(a) // 50, settled.sum()
    if scale <= 2.0 ** -56:  # (distances below the floor: everything is left open)
        assert not settled.any()


def test_bounds_leave_open_what_is_not_a_number_and_settle_zero_keys():
    """Keys of zeros beside others (padding) are settled by the distance of their centroid from the rest."""
    inf, nan = np.float32(np.inf), np.float32(np.nan)
    need, _ = ice_debug_near_bounds([nan, 1, inf, 1], [1, nan, 1, inf], [0, 0, 0, 0], [0, 0, 0, 0])
    assert not any(need < 1e30)
    need, _ = ice_debug_near_bounds([0], [0], [0], [0])
    _, dist2 = ice_debug_near_bounds([0], [0], [0], [-0.5])  # (the nearest other centroid, of norm 1)
    assert 0 < need[0] < 2.0 ** -40 and 0.99 < dist2[0] <= 1


@pytest.mark.parametrize("U,n,C,near", [
    (256, 16384, 512, True), (256, 16384, 513, False), (256, 16383, 300, False),  # 16384 keys, 32 per cluster
    (64, 32768, 1638, True), (64, 32768, 1639, False), (64, 32767, 1638, False),  # 20 from 32768 keys on
    (600, 4000, 450, False), (300, 6100, 300, False), (32, 16384, 2048, False),
])
def test_builds_of_few_keys_per_cluster_make_no_lists_of_near_centroids(U, n, C, near):
    """They took 1.02 to 1.37 times as long with them (600 units x 4000 keys x 450 clusters: 3630 and 4970 us)."""
    assert ice_debug_build_plan(make_config(1, U, 4, n), n, C)["reassign_from"] == (1 if near else 2)


@pytest.mark.parametrize("U,n,C,rounds", [(512, 16384, 260, 6), (256, 24576, 384, 6), (256, 24576, 385, 4), (256, 32768, 512, 4), (256, 32768, 513, 2), (8, 131072, 2048, 2)])
def test_builds_of_few_rounds_and_clusters_make_no_lists_of_near_centroids(U, n, C, rounds):
    """The first round with them costs more than a full one there (512 units x 16384 keys x 260 clusters, three rounds: 4625 and 4980 us)."""
    first = lambda T: ice_debug_build_plan(make_config(1, U, 4, n, kmeans_iters=T), n, C)["reassign_from"]
    assert [first(T) for T in (1, 2, 3, 4, 5, 6, 10)] == [1 if T >= rounds else 2 if T > 2 else 0 for T in (1, 2, 3, 4, 5, 6, 10)]
