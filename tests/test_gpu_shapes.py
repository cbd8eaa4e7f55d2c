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
