"""How the loss call moves its cells: run by run and piece by piece, in 16-byte and in single-float pieces, on both sides of the rule
between them, runs of one cell and longer than a group; kernels for up to 4, 8, 12 and 16 action components; statistics of one
block and of more blocks than the closing launch has threads.  Against the oracle with the bounds of the parity tests."""
import pytest

import test_gpu_parity as parity
from paper_2603_09237_amd.configs import scaled
from test_gpu_parity import _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def case(A, K, P, n_g, T, **over):
    return scaled(parity.RAGGED, name=f"loss-A{A}-K{K}-P{P}-n{n_g}-T{T}", act_dim=A, K=K, P=P, N=P * n_g, T=T, obs_dim=3, minibatches=1, **over)


CASES = [case(A, 3, 3, 50, 11) for A in (1, 4, 5, 8, 9, 12, 13, 16)]                   # single floats, runs of 50
CASES += [case(A, 4, 3, 48, 11) for A in (4, 8, 12, 16)]                              # 16-byte pieces
CASES += [case(5, 3, 3, n, 1200 // n + 2) for n in (1, 3, 31, 32, 33, 111, 112, 113, 127, 129, 300)]
CASES += [case(4, 4, 3, n, 1200 // n + 2) for n in (4, 108, 112, 128, 260)]
CASES += [case(3, 2, 40, 61, 90), case(3, 1, 2, 300, 1), case(2, 4, 33, 36, 300)]      # beyond 200 000 cells; one block or two a preference


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
@pytest.mark.parametrize("norm", (0, 1))
def test_loss_however_its_cells_are_moved(cfg, norm, torch, binding):  # noqa: F811
    parity.test_ppo_loss_grad_matches_oracle(cfg, 0, norm, torch, binding)


@pytest.mark.parametrize("cfg", [case(A, 3, 3, n, 12) for A in (2, 6, 8) for n in (37, 120)], ids=lambda c: c.name)
def test_state_dependent_sigma_however_its_cells_are_moved(cfg, torch, binding):  # noqa: F811
    parity.test_ppo_loss_grad_state_sigma_matches_oracle(scaled(cfg, sigma_state=1), torch, binding)
