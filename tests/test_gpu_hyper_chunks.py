"""Chunks of the stacked hypernet rows: those that a workgroup requests as a whole (up to 32 and up to 64 preferences, both feature
widths, a last chunk of fewer tiles), and chunks of more than eight tiles, whose row offsets are made eight tiles at a time.
Against the oracle with the bounds of the parity tests."""
import pytest

import test_gpu_parity as parity
from paper_2603_09237_amd.configs import scaled
from test_gpu_parity import RAGGED, _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [scaled(RAGGED, name=f"P{P}-F{F}-r{r}-W{W}", P=P, N=2 * P, hyper_width=F, rank=r, width=W, n_hidden=3)
         for P, F, r, W in ((3, 32, 4, 48), (32, 40, 3, 64), (33, 33, 5, 48), (64, 20, 3, 80), (64, 64, 2, 32), (65, 48, 3, 48), (31, 32, -1, 16))]
CASES += [scaled(RAGGED, name=f"eleven-tiles-P{P}", hyper_width=3, rank=-1, obs_dim=61, width=400, n_hidden=5, P=P, N=2 * P) for P in (3, 33)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_gradients_of_rows_in_whole_chunks_and_long_ones(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_fwd_matches_oracle(cfg, torch, binding)
    parity.test_hypernet_bwd_matches_oracle(cfg, torch, binding)
