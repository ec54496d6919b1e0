"""Gradient of the stacked hypernet rows at the edges of its preference groups, against the oracle with the
bounds of the parity tests.

Preferences around multiples of 16 and 32 (a wave's share of df, waves without any), with a last row tile that is not full."""
import pytest

import test_gpu_parity as parity
from paper_2603_09237_amd.configs import scaled
from test_gpu_parity import RAGGED, _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [scaled(RAGGED, name=f"P{p}", P=p, N=2 * p) for p in (2, 15, 16, 17, 32, 33, 64, 65, 97, 127, 128)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_stacked_row_gradients_at_group_and_tile_edges(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_bwd_matches_oracle(cfg, torch, binding)
