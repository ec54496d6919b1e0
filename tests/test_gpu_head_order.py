"""The output layer's backward on both sides of the rule for its dW workgroups: up to one a CU they start ahead of everything else, more
of them each ahead of its own preference's dZ ones.  Both types, one and two column tiles, against the oracle with the bounds of
the parity tests."""
import pytest

import test_gpu_parity as parity
from test_gpu_forward_tiles import case
from test_gpu_parity import _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CASES = [case(wd, W, P, 23, 3, n_hidden=L) for wd in (0, 1) for W, P in ((64, 64), (64, 65), (144, 32), (144, 33)) for L in (1, 2)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_output_layer_gradients_however_its_workgroups_are_dealt(cfg, torch, binding):  # noqa: F811
    parity.test_policy_bwd_matches_oracle(cfg, None, torch, binding)
