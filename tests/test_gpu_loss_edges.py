"""The loss call where a preference has few cells: one, one group of 128 less one, a whole one, one more, two -- one or two blocks a
preference and no more for the closing launch --, in runs as long as all of them and in runs of one cell, in single-float and in
16-byte pieces; and selections that leave out environments and time steps.  Against the oracle with the bounds of the parity tests."""
import numpy as np
import pytest

import test_gpu_parity as parity
from gpu_util import assert_close32, dev, to_np
from paper_2603_09237_amd.configs import scaled
from test_gpu_parity import _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def case(A, K, P, n_g, T, **over):
    name = f"loss-A{A}-K{K}-P{P}-n{n_g}-T{T}" + "".join(f"-{k}{v}" for k, v in over.items())
    return scaled(parity.RAGGED, **{**dict(name=name, act_dim=A, K=K, P=P, N=P * n_g, T=T, obs_dim=3, minibatches=1), **over})


CASES = [case(A, 3, 40, n, T) for A in (3, 13) for n, T in ((1, 1), (127, 1), (128, 1), (129, 1), (256, 1), (1, 127), (1, 128), (1, 129), (32, 8))]
CASES += [case(A, 4, 40, n, T) for A in (4, 16) for n, T in ((4, 1), (4, 32), (128, 1), (132, 1), (64, 4))]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
@pytest.mark.parametrize("norm", (0, 1))
def test_few_cells_a_preference(cfg, norm, torch, binding):  # noqa: F811
    parity.test_ppo_loss_grad_matches_oracle(cfg, 0, norm, torch, binding)


MB_CASES = [(case(5, 3, 7, 63, 9, minibatches=3), 1), (case(5, 3, 7, 63, 9, minibatches=3), 2), (case(13, 2, 7, 44, 11, minibatches=4), 3),
            (case(4, 4, 7, 48, 11, minibatches=3), 1), (case(16, 4, 7, 48, 11, minibatches=2), 1), (case(8, 4, 5, 464, 3, minibatches=4), 2)]


@pytest.mark.parametrize("cfg, mb", MB_CASES, ids=lambda c: getattr(c, "name", str(c)))
def test_a_part_of_the_environments(cfg, mb, torch, binding):  # noqa: F811
    parity.test_ppo_loss_grad_matches_oracle(cfg, mb, 1, torch, binding)


@pytest.mark.parametrize("rows", [(3, 5, 0, 50), (3, 5, 7, 9), (8, 3, 49, 1), (0, 1, 0, 1), (2, 9, 12, 32), (10, 1, 4, 40)], ids=str)
@pytest.mark.parametrize("A, K", [(5, 3), (14, 2), (4, 4)])
def test_a_part_of_the_time_steps(rows, A, K, torch, binding):  # noqa: F811
    """Gradients of the selected cells and statistics; nothing is written outside them."""
    cfg = case(A, K, 6, 50 if A != 4 else 52, 11)
    mu, logsig, act, logp_old, adv_s, v, vtarg = parity.loss_inputs(cfg)
    ctx = binding.Context.from_config(cfg)
    full = lambda t: torch.full(t.shape, 3.25, device="cuda")  # noqa: E731
    dmu, dv, dls, stats = full(mu), full(v), full(logsig), torch.zeros(8, device="cuda")
    ws = torch.empty(ctx.workspace_bytes(rows), dtype=torch.uint8, device="cuda")
    ctx.ppo_loss_grad(rows, dev(mu), dev(logsig), A, dev(act), dev(logp_old), dev(adv_s), dev(v), dev(vtarg), cfg.clip_eps, 0, dmu, dls, dv,
                      stats, ws)
    o_dmu, o_dls, o_dv, o_st = parity.orc.ppo_loss_grad(cfg, rows, mu, logsig, act, logp_old, adv_s, v, vtarg, cfg.clip_eps, False)
    mask = parity.orc.row_mask(cfg, rows, cfg.T)
    g_dmu, g_dv, B = to_np(dmu), to_np(dv), float(mask.sum())
    assert np.all(g_dmu[~mask] == 3.25) and np.all(g_dv[~mask] == 3.25)
    gidx = parity.orc.env_pref_index(cfg.N, cfg.P)
    logp = parity.orc.gaussian_logp(act.astype(np.float64), mu.astype(np.float64), logsig[gidx][None].astype(np.float64))
    rho = np.exp(logp - logp_old)   # (a ratio within rounding of an edge of the clip range may fall on either side of it)
    edge = (np.abs(rho - (1 + cfg.clip_eps)) < 1e-5) | (np.abs(rho - (1 - cfg.clip_eps)) < 1e-5)
    assert_close32(g_dmu * B, o_dmu * B, "dmu*B", mask=(mask & ~edge)[..., None] & np.ones_like(o_dmu, bool))
    assert_close32(g_dv * B, o_dv * B, "dv*B", mask=mask[..., None] & np.ones_like(o_dv, bool))
    if not edge[mask].any():
        assert_close32(to_np(dls), o_dls, "dlogsig")
    st = to_np(stats)
    assert_close32(st[[0, 1, 3, 4, 5, 6]], o_st[[0, 1, 3, 4, 5, 6]], "stats")
    assert st[7] == B
