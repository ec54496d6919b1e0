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


# feature widths at the edges of the contraction steps, factor and output widths that leave runs of four rows across
# segment ends and row ends at odd offsets, more than 64 preferences beside them, and enough rows (strictly affine, more
# than 4096 tiles of 64) for chunks of more than four tiles
ROW_CASES = [scaled(RAGGED, name=f"F{F}-r{r}-A{A}-O{O}-W{W}-P{P}", hyper_width=F, rank=r, act_dim=A, obs_dim=O, width=W, P=P, N=2 * P)
             for F, r, A, O, W, P in ((1, 3, 3, 5, 16, 3), (7, 1, 1, 7, 48, 5), (31, 5, 3, 9, 32, 66), (32, 4, 2, 8, 32, 70),
                                      (33, 3, 5, 11, 16, 4), (64, 7, 3, 13, 80, 129), (32, -1, 3, 5, 48, 6), (33, -1, 5, 7, 16, 67))]
ROW_CASES += [scaled(RAGGED, name=f"many-rows-bf16-{b}", hyper_width=3, rank=-1, obs_dim=61, width=272, n_hidden=5, P=3, N=6, wdtype=b)
              for b in (0, 1)]


@pytest.mark.parametrize("cfg", ROW_CASES, ids=lambda c: c.name)
def test_stacked_rows_and_their_gradients_at_odd_sizes(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_fwd_matches_oracle(cfg, torch, binding)
    parity.test_hypernet_bwd_matches_oracle(cfg, torch, binding)


# the weights themselves: ranks around the contraction steps, rows and columns around the 64 x 128 tiles, observation widths
# that are no multiple of 8, many preferences
MAT_CASES = [scaled(RAGGED, name=f"r{r}-O{O}-W{W}-P{P}-{b}", rank=r, obs_dim=O, width=W, P=P, N=2 * P, n_hidden=L, hyper_width=4, wdtype=b)
             for b in (0, 1)
             for r, O, W, L, P in ((0, 5, 16, 1, 2), (1, 8, 64, 2, 3), (8, 127, 80, 2, 5), (9, 129, 144, 1, 4), (16, 64, 272, 2, 3),
                                   (17, 11, 48, 2, 2), (32, 136, 128, 1, 3), (4, 13, 32, 4, 1025), (12, 24, 256, 3, 301))]


@pytest.mark.parametrize("cfg", MAT_CASES, ids=lambda c: c.name)
def test_weights_at_tile_and_rank_edges(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_fwd_matches_oracle(cfg, torch, binding)


# dA added up from column runs: two to five runs of 128 columns beside layers of one, factors whose element counts are no
# multiple of four, and more than one block of 1024 elements
DA_CASES = [scaled(RAGGED, name=f"dA-r{r}-A{A}-O{O}-W{W}-P{P}", rank=r, act_dim=A, obs_dim=O, width=W, P=P, N=2 * P)
            for r, A, O, W, P in ((1, 3, 129, 16, 2), (3, 5, 40, 272, 3), (5, 1, 513, 144, 2), (17, 7, 200, 96, 3))]


@pytest.mark.parametrize("cfg", DA_CASES, ids=lambda c: c.name)
def test_factor_gradients_from_several_column_runs(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_bwd_matches_oracle(cfg, torch, binding)


# more than 128 preferences: every tile of 64 rows summed by itself, in chunks of four tiles, of five where there are more than 4096
MANY_P = [scaled(RAGGED, name=f"F{F}-P{P}", P=P, N=2 * P, rank=-1, hyper_width=F, obs_dim=16, width=16, n_hidden=1, act_dim=2,
                 wdtype=0) for P, F in ((129, 32), (130, 64), (257, 5))]
MANY_P += [scaled(RAGGED, name="F3-P129-many-rows", P=129, N=258, hyper_width=3, rank=-1, obs_dim=61, width=272, n_hidden=5)]


@pytest.mark.parametrize("cfg", MANY_P, ids=lambda c: c.name)
def test_feature_gradient_of_many_preferences_is_summed_by_tiles(cfg, torch, binding):  # noqa: F811
    """df of a strictly affine network with f = 0, where dbh2 = sum_p df: 64 rows that add up to 2^26, as many that add up to
    32, as many that take the first away.  Every sum of one tile and the sum of the tiles are exact in fp32; a sum that runs
    on from row to row across the tiles loses the small one whole."""
    ctx = binding.Context.from_config(cfg)
    net = parity.ACTOR
    lay = parity.orc.hparam_layout(cfg, net)
    ml, vl = ctx.theta_mat_len(net), ctx.theta_vec_len(net)
    hp = torch.zeros(ctx.hparam_count(net), device="cuda")
    M = torch.zeros(ml, cfg.hyper_width, device="cuda")
    M[:64], M[64:128], M[128:192] = 2.0 ** 20, 0.5, -2.0 ** 20
    at = 0
    for (o, i), l in zip(parity.inputs.layer_shapes(cfg, net), range(cfg.n_hidden + 1)):
        off = lay[f"MW_{l}"][0]
        hp[off:off + o * i * cfg.hyper_width] = M[at:at + o * i].reshape(-1)
        at += o * i
    assert at == ml
    dtm = torch.zeros(cfg.P, ml, device="cuda")
    dtm[:, :192] = 1.0
    dtv, w = torch.zeros(cfg.P, vl, device="cuda"), torch.full((cfg.P, cfg.K), 1.0 / cfg.K, device="cuda")
    dhp = torch.full_like(hp, 9.0)
    ws = torch.empty(ctx.workspace_bytes((0, 1, 0, 1)), dtype=torch.uint8, device="cuda")
    ctx.hypernet_bwd(net, hp, w, dtm, dtv, dhp, ws)
    off = lay["bh2"][0]
    assert (dhp[off:off + cfg.hyper_width] == cfg.P * 32).all(), dhp[off:off + cfg.hyper_width]


# few preferences on both sides of the numbers of stacked rows up to which the trunk shares a launch: workgroups of 64 rows
# (1024, 512 above 32 features) forward, chunks of 256 rows backward
TRUNK_CASES = [scaled(RAGGED, name=f"trunk-F{F}-P{P}-r{r}-O{O}-W{W}", P=P, N=2 * P, rank=r, hyper_width=F, obs_dim=O, width=W, n_hidden=2)
               for F, P, r, O, W in ((32, 16, -1, 11, 128), (32, 16, -1, 40, 144), (32, 2, -1, 11, 240), (32, 2, -1, 40, 256),
                                     (64, 8, -1, 30, 160), (64, 8, -1, 60, 160), (8, 64, 32, 300, 96), (20, 25, 16, 11, 272))]


@pytest.mark.parametrize("cfg", TRUNK_CASES, ids=lambda c: c.name)
def test_trunk_beside_few_and_many_rows(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_fwd_matches_oracle(cfg, torch, binding)
    parity.test_hypernet_bwd_matches_oracle(cfg, torch, binding)
    parity.test_hypernet_bwd_kept_equals_hypernet_bwd(cfg, torch, binding)


def test_few_preferences_of_a_wide_affine_network_take_no_longer_than_more(torch, binding):  # noqa: F811
    """hypernet_fwd of 16 preferences against 17 of a strictly affine 4 x 512 network: 17 weight sets are more to write, so
    the call with 16 is the shorter one (a quarter is left for the clock)."""
    def passes(P):
        cfg = scaled(RAGGED, name=f"affine-4x512-P{P}", P=P, N=2 * P, rank=-1, hyper_width=32, obs_dim=64, width=512, n_hidden=4, wdtype=1)
        ctx, net = binding.Context.from_config(cfg), parity.ACTOR
        hp, w = torch.zeros(ctx.hparam_count(net), device="cuda"), torch.zeros(P, cfg.K, device="cuda")
        tm = torch.empty(P, ctx.theta_mat_len(net), dtype=torch.bfloat16, device="cuda")
        tv = torch.empty(P, ctx.theta_vec_len(net), device="cuda")
        ws = torch.empty(ctx.workspace_bytes((0, 1, 0, 1)), dtype=torch.uint8, device="cuda")

        def once():
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                ctx.hypernet_fwd(net, hp, w, tm, tv, ws)
            b.record()
            b.synchronize()
            return a.elapsed_time(b)
        return once
    few, more = passes(16), passes(17)
    few(), more()
    best = [min(t) for t in zip(*((few(), more()) for _ in range(9)))]
    assert best[0] < 1.25 * best[1], best


# feature widths on both sides of the contraction steps of the stacked map, with the trunk inside its launch and in front
STEP_CASES = [scaled(RAGGED, name=f"steps-F{F}-P{P}", P=P, N=2 * P, hyper_width=F, width=32)
              for F in (8, 9, 12, 13, 16, 17, 21, 24, 25, 28, 29, 36, 40, 41, 48, 49) for P in (5, 520 // F + 1)]


@pytest.mark.parametrize("cfg", STEP_CASES, ids=lambda c: c.name)
def test_stacked_rows_at_every_number_of_steps(cfg, torch, binding):  # noqa: F811
    parity.test_hypernet_fwd_matches_oracle(cfg, torch, binding)


def test_narrow_trunk_takes_less_time_than_a_wide_one(torch, binding):  # noqa: F811
    """hypernet_fwd of 4 preferences of a strictly affine 4 x 512 network with 8 features against 32: a quarter of M to read."""
    def passes(F):
        cfg = scaled(RAGGED, name=f"affine-4x512-F{F}", P=4, N=8, rank=-1, hyper_width=F, obs_dim=16, width=512, n_hidden=4, wdtype=1)
        ctx, net, z = binding.Context.from_config(cfg), parity.ACTOR, lambda *s: torch.zeros(*s, device="cuda")
        hp, w, tm, tv = z(ctx.hparam_count(net)), z(4, cfg.K), z(4, ctx.theta_mat_len(net)).to(torch.bfloat16), z(4, ctx.theta_vec_len(net))
        ws = torch.empty(ctx.workspace_bytes((0, 1, 0, 1)), dtype=torch.uint8, device="cuda")

        def once():
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                ctx.hypernet_fwd(net, hp, w, tm, tv, ws)
            b.record()
            b.synchronize()
            return a.elapsed_time(b)
        return once
    narrow, wide = passes(8), passes(32)
    narrow(), wide()
    best = [min(t) for t in zip(*((narrow(), wide()) for _ in range(9)))]
    assert best[0] < 0.65 * best[1], best


def test_gradient_of_fewer_affine_rows_takes_no_longer(torch, binding):  # noqa: F811
    """hypernet_bwd of 32 preferences of a strictly affine 3 x 512 network against 4 x 512, which has half as many rows again."""
    def passes(L):
        cfg = scaled(RAGGED, name=f"affine-{L}x512", P=32, N=64, rank=-1, hyper_width=32, obs_dim=11, width=512, n_hidden=L, wdtype=1)
        ctx, net, z = binding.Context.from_config(cfg), parity.ACTOR, lambda *s: torch.zeros(*s, device="cuda")
        hp, w, dtm, dtv = z(ctx.hparam_count(net)), z(32, cfg.K), z(32, ctx.theta_mat_len(net)), z(32, ctx.theta_vec_len(net))
        dhp, ws = torch.empty_like(hp), torch.empty(ctx.workspace_bytes((0, 1, 0, 1)), dtype=torch.uint8, device="cuda")

        def once():
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                ctx.hypernet_bwd(net, hp, w, dtm, dtv, dhp, ws)
            b.record()
            b.synchronize()
            return a.elapsed_time(b)
        return once
    few, more = passes(3), passes(4)
    few(), more()
    best = [min(t) for t in zip(*((few(), more()) for _ in range(9)))]
    assert best[0] < best[1], best
