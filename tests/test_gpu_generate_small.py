"""Both generation kernels around the size where one takes over from the
other, and the small kernel's remainders: whole grids against the oracle, and
the two kernels' values at the same nodes bit for bit."""
import dataclasses

import numpy as np
import pytest

from paper_2204_02585_amd import scenes
from tests.test_gpu_generate import _full_compare, _generate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_p,n_theta,n_phi", [(5, 2, 3), (33, 6, 11), (97, 3, 33), (98, 31, 2)])
def test_sizes_around_the_rule(n_p, n_theta, n_phi):
    """3 ceil(n_p^2 / 32) = 885 at 97 (the small kernel), 903 at 98."""
    cfg = dataclasses.replace(scenes.GEN_CONFIGS["gen_tiny"], pos_layers=3, dir_layers=2)
    _full_compare(scenes.make_gen_scene(cfg), f"around {n_p}", n_p=n_p, n_theta=n_theta, n_phi=n_phi)


@pytest.mark.parametrize("D,layers", [(8, 6), (32, 2), (1, 1), (13, 16)])
def test_both_kernels_give_the_same_bits(D, layers):
    """Node (i, i') of an 61-node grid is node (2i, 2i') of a 121-node one on a
    box whose node coordinates are exact in binary64."""
    cfg = dataclasses.replace(scenes.GEN_CONFIGS["gen_tiny"], D=D, pos_layers=layers, dir_layers=min(layers, 16))
    g = scenes.make_gen_scene(cfg)
    g.bbox_min, g.bbox_max = (-1.875,) * 3, (1.875,) * 3      # steps of 1/16 and 1/32
    sig_s, uvw_s, beta_s = _generate(g, n_p=61, n_theta=4, n_phi=6)
    sig_l, uvw_l, beta_l = _generate(g, n_p=121, n_theta=4, n_phi=6)
    for j in range(3):
        assert np.array_equal(sig_s[j], sig_l[j][::2, ::2])
        assert np.array_equal(uvw_s[j], uvw_l[j][::2, ::2])
    assert np.array_equal(beta_s, beta_l)
