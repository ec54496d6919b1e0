"""Gradients of a low-rank hypernetwork at the lines of what its two large launches do.  dA and dB of as many blocks as the chip
holds, in front of those of dW0, and of more, behind or among them in rows of eight.  dA and dB where a row of weights is no
multiple of four values, or the last rows and columns do not fill a tile: the values a tile is short of are requested at its edge
and zeroed.  Chunks of stacked rows on both sides of the rule for their requests.  Against the oracle with the bounds of the
parity tests."""
import pytest

import test_gpu_parity as parity
from paper_2603_09237_amd.configs import scaled
from test_gpu_parity import RAGGED, _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [scaled(RAGGED, name=f"r{r}-O{O}-W{W}-A{A}", rank=r, obs_dim=O, width=W, act_dim=A, P=3, N=6, n_hidden=2)
         for r, O, W, A in ((4, 1, 16, 1), (1, 2, 48, 3), (8, 3, 64, 2), (16, 63, 80, 5), (17, 65, 64, 4), (5, 127, 144, 3), (32, 129, 32, 16),
                            (8, 131, 208, 7), (3, 190, 128, 1))]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_factor_gradients_at_the_edges_of_tiles(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_bwd_matches_oracle(cfg, torch, binding)


# blocks of dA / dB (four column runs and more to a preference): 892, 896, 900 of many preferences, 1152 and 1168 of few; dW0 in few
# blocks and in 9, 44, 256, 258, 555
SHARE_CASES = [scaled(RAGGED, name=f"P{P}-L{L}-W{W}-O{O}", rank=2, obs_dim=O, width=W, P=P, N=2 * P, n_hidden=L, hyper_width=4)
               for P, L, W, O in ((223, 3, 16, 5), (224, 3, 16, 5), (225, 3, 48, 24), (290, 3, 48, 76), (173, 3, 144, 17), (72, 3, 528, 17), (73, 3, 528, 17), (130, 2, 400, 250), (130, 2, 400, 256))]


@pytest.mark.parametrize("cfg", SHARE_CASES, ids=lambda c: c.name)
def test_blocks_of_both_kinds_are_all_there(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_bwd_matches_oracle(cfg, torch, binding)


# chunks of rows that a workgroup requests as a whole or tile by tile: 256 and 258 workgroups of 32 features, and of 33, more of them
BRIEF_CASES = [scaled(RAGGED, name=f"P{P}-F{F}-O{O}-W{W}", rank=-1, obs_dim=O, width=W, P=P, N=2 * P, n_hidden=2, hyper_width=F)
               for P, F, O, W in ((3, 32, 61, 160), (3, 32, 63, 160), (3, 33, 63, 160), (33, 32, 61, 160), (33, 32, 63, 160), (33, 40, 63, 160),
                                  (64, 32, 45, 256), (64, 40, 45, 256))]


@pytest.mark.parametrize("cfg", BRIEF_CASES, ids=lambda c: c.name)
def test_chunks_as_a_whole_and_tile_by_tile(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_bwd_matches_oracle(cfg, torch, binding)
