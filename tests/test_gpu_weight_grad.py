"""Weight gradients at the edges of the padded rows and of the ranges the contraction is cut into, against the oracle with
the bounds of the parity tests.

Rows around multiples of 32 (a contraction step) and 64 (a range's granule), ranges of unequal length (fp32), the two
splits bf16 takes (equal ranges of a hidden layer, the first layer from 4096 rows on), observation widths around the eight
columns their compact rows are padded to, and a forward that goes layer by layer (width 528) or by tall tiles."""
import pytest

import test_gpu_parity as parity
from test_gpu_forward_tiles import case
from test_gpu_parity import _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [case(wd, 64, 3, n, 1, obs_dim=33) for wd in (0, 1) for n in (63, 64, 65, 95, 96, 97, 127, 129, 257)]
CASES += [case(wd, 144, 4, 131, 5, obs_dim=o, n_hidden=2) for wd in (0, 1) for o in (39, 40, 41, 96, 137)]
CASES += [case(0, 64, 2, 331, 5, obs_dim=45), case(0, 256, 3, 307, 3, obs_dim=19)]       # 16 and 2 ranges, unequal
CASES += [case(1, 64, 2, 128, 8, obs_dim=45), case(1, 64, 2, 823, 5, obs_dim=45)]        # 4 equal ranges; 2 of the first layer
CASES += [case(wd, 528, 3, 37, 3, obs_dim=o, n_hidden=2) for wd in (0, 1) for o in (19, 45, 64)]
CASES += [case(1, 256, 90, 83, 7, obs_dim=45, n_hidden=2)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_weight_gradients_at_row_and_range_edges(cfg, torch, binding):  # noqa: F811
    parity.test_policy_fwd_matches_oracle(cfg, None, torch, binding)
    parity.test_policy_bwd_matches_oracle(cfg, None, torch, binding)
