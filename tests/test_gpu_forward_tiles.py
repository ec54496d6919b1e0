"""The one-launch forward at the edges of its tiles and dispatch, against the oracle with the bounds of the parity tests.

Row counts around the 16-, 32-, 64- and 128-row tiles, widths around the waves' 64 features and around the widths where
the launcher turns to another kernel, observations wider than the network and of odd width, one hidden layer, networks
too narrow for it; each both plain and saving, followed where there are enough rows by the backward pass that reads what
was saved (its bound is a share of the RMS of a sum over the rows, which grows with their root: over 17 rows the re-rounded
bf16 inputs of the layers above alone come to it; and it is meant for as many elements as a few preferences have, not for
the extremes of tens of millions)."""
import pytest

import test_gpu_parity as parity
from test_gpu_parity import _float32_default, binding, torch  # noqa: F401  (fixtures)
from paper_2603_09237_amd.configs import scaled

pytestmark = pytest.mark.gpu

BASE = scaled(parity.RAGGED, name="fwd-tiles", P=3, K=3, act_dim=5, obs_dim=19, n_hidden=3, rank=4)


def case(wd, W, P, n_g, T=1, **over):
    tag = "-".join(f"{k}{v}" for k, v in over.items())
    return scaled(BASE, name=f"fwd-{'bf16' if wd else 'fp32'}-W{W}-P{P}-M{n_g}x{T}-{tag}", wdtype=wd, width=W, P=P, N=P * n_g,
                  T=T, **over)


CASES = [case(wd, W, 3, 17, 1) for wd in (0, 1) for W in (32, 64, 80, 128, 192, 256, 320, 384, 448, 512)]
CASES += [case(wd, W, 3, 66, 1) for wd in (0, 1) for W in (32, 80, 256, 448)]
CASES += [case(wd, 160, 3, n_g, 1) for wd in (0, 1) for n_g in (1, 15, 16, 33)]
CASES += [case(1, 384, 90, 37, 11), case(0, 128, 80, 97, 5), case(1, 128, 80, 67, 6), case(1, 512, 90, 37, 4),
          case(0, 48, 180, 45, 3), case(1, 64, 200, 45, 3)]                   # two and four row tiles a workgroup
CASES += [case(1, 512, 90, 37, 11), case(1, 256, 180, 37, 11), case(0, 512, 70, 37, 7)]  # beyond it: the tall kernels
CASES += [case(wd, 32, 3, 20, 2, obs_dim=121) for wd in (0, 1)] + [case(wd, 96, 3, 20, 2, obs_dim=513, n_hidden=2) for wd in (0, 1)]
CASES += [case(wd, 48, 3, 20, 2, n_hidden=1, obs_dim=45) for wd in (0, 1)] + [case(1, 16, 3, 20, 2, K=1, n_hidden=2)]
CASES += [case(wd, 144, 5, 30, 2, act=0, sigma_state=1) for wd in (0, 1)]
# the narrowest network, output layers of 1, 2 and 3 columns: behind its last matrix comes less than a whole request
# (test_forward_shapes.py walks them)
CASES += [case(wd, 16, 3, 33, 2, K=o, act_dim=o, n_hidden=2, obs_dim=8) for wd in (0, 1) for o in (1, 2, 3)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_forward_and_backward_at_tile_edges(cfg, torch, binding):  # noqa: F811
    parity.test_policy_fwd_matches_oracle(cfg, None, torch, binding)
    if cfg.n_g * cfg.T >= 60 and cfg.P <= 5:
        parity.test_policy_bwd_matches_oracle(cfg, None, torch, binding)


# what the saving forwards of many preferences leave for the backward pass, on three of the preferences: 64-row tiles of four,
# six and eight waves (185 rows), and the layer-by-layer forward on the persistent GEMM with a cut row tile and, at 528, a cut
# column tile (384: 407 rows, beyond the one-launch forward; 528: too wide for it)
@pytest.mark.parametrize("cfg", [case(1, 256, 90, 37, 5), case(1, 384, 90, 37, 5), case(1, 448, 90, 37, 5), case(1, 512, 90, 37, 5),
                                 case(1, 384, 90, 37, 11), case(1, 528, 90, 37, 5)], ids=lambda c: c.name)
def test_backward_on_what_wide_forwards_save(cfg, torch, binding, monkeypatch):  # noqa: F811
    monkeypatch.setattr(parity, "sample_prefs", lambda c: [0, c.P // 3 + 1, c.P - 1])
    parity.test_policy_bwd_matches_oracle(cfg, None, torch, binding)
