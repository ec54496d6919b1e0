"""How the one-launch forwards take their observations: pieces of eight (fp32 tiles of 16 rows: four) values, the last one of a row
requested as the values that end with the row and moved down, zeros behind it; rows shorter than a piece element by element;
one batch of pieces a thread and several.  Against the oracle with the bounds of the parity tests, and, where the observations are
saved for the first layer's dW, the backward pass that reads them."""
import pytest

import test_gpu_parity as parity
from test_gpu_forward_tiles import case
from test_gpu_parity import _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [case(1, W, 3, 34, 2, obs_dim=o, n_hidden=1) for W in (64, 192, 512) for o in (1, 7, 8, 13, 64, 65, 250)]   # 32-row tiles
CASES += [case(1, W, 90, 37, 5, obs_dim=o, n_hidden=2) for W in (256, 512) for o in (44, 130)]                       # 64-row ones
CASES += [case(1, W, 128, 77, 5, obs_dim=o, n_hidden=1) for W in (256, 512) for o in (3, 11, 14, 64, 127, 255)]      # 128-row ones
CASES += [case(0, 32, 3, 18, 2, obs_dim=o, n_hidden=1) for o in (1, 3, 4, 6, 31, 33, 200)]                           # fp32, 16 rows
CASES += [case(0, W, 10, 37, 6, obs_dim=o, n_hidden=2) for W in (160, 256) for o in (5, 9, 12, 33, 100, 300)]        # split operands
BACKWARD = [case(wd, W, 3, 31, 3, obs_dim=o, n_hidden=2) for wd, W in ((0, 160), (0, 32), (1, 192), (1, 256)) for o in (33, 38, 71)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_forward_at_the_edges_of_pieces(cfg, torch, binding):  # noqa: F811
    parity.test_policy_fwd_matches_oracle(cfg, None, torch, binding)


@pytest.mark.parametrize("cfg", BACKWARD, ids=lambda c: c.name)
def test_saved_observations_at_the_edges_of_pieces(cfg, torch, binding):  # noqa: F811
    parity.test_policy_bwd_matches_oracle(cfg, None, torch, binding)
