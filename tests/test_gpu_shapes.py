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
