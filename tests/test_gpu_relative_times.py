"""Calls that take about as long as their neighbours of nearly the same work: an odd size beside the next even one, one size more
beside one less.  Both sides are graphs of the same call, replayed in turn; the shortest of either counts."""
import pytest

import test_gpu_parity as parity
from paper_2603_09237_amd.configs import scaled
from test_gpu_parity import RAGGED, _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def case(P, L, W, O, **over):
    return scaled(RAGGED, **{**dict(name=f"P{P}-{L}x{W}-O{O}", P=P, N=2 * P, n_hidden=L, width=W, obs_dim=O, hyper_width=32, wdtype=1), **over})


def hyper(torch, binding, cfg):  # noqa: F811
    """(hypernet_fwd, hypernet_bwd) of the actor's hypernetwork as calls without arguments."""
    ctx, net, z = binding.Context.from_config(cfg), parity.ACTOR, lambda *s: torch.zeros(*s, device="cuda")
    hp, w, dtm, dtv = z(ctx.hparam_count(net)), z(cfg.P, cfg.K), z(cfg.P, ctx.theta_mat_len(net)), z(cfg.P, ctx.theta_vec_len(net))
    tm, tv, dhp = dtm.to(torch.bfloat16 if cfg.wdtype else torch.float32), torch.empty_like(dtv), torch.empty_like(hp)
    ws = torch.empty(ctx.workspace_bytes((0, 1, 0, 1)), dtype=torch.uint8, device="cuda")
    return (lambda: ctx.hypernet_fwd(net, hp, w, tm, tv, ws)), (lambda: ctx.hypernet_bwd_kept(net, hp, w, dtm, dtv, dhp, ws))


def ratio(torch, one, other, calls=20, turns=9):  # noqa: F811
    def graph(call):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            call()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            for _ in range(calls):
                call()
        g.replay()
        return g

    def once(g):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        return a.elapsed_time(b)
    gs = graph(one), graph(other)
    best = [min(t) for t in zip(*((once(gs[0]), once(gs[1])) for _ in range(turns)))]
    return best[0] / best[1]


def test_gradient_of_odd_rows_takes_little_more_than_of_even_ones(torch, binding):  # noqa: F811
    """hypernet_bwd with 190 observations against 192, whose rows are whole four-value pieces: a quarter for the pieces and the clock."""
    odd, even = (hyper(torch, binding, case(13, 2, 512, o, rank=16))[1] for o in (190, 192))
    assert ratio(torch, odd, even) < 1.25


def test_gradient_takes_no_longer_for_another_number_of_base_blocks(torch, binding):  # noqa: F811
    """hypernet_bwd of 9 preferences of 3 x 768 with 57 observations against 60: the less work, so the shorter call (a tenth is left for
    the clock).  Spread block by block, every eighth block of the former was one of dA / dB: all of them on one die."""
    fewer, more = (hyper(torch, binding, case(9, 3, 768, o, rank=16))[1] for o in (57, 60))
    assert ratio(torch, fewer, more) < 1.1


def test_features_beyond_32_cost_little_more_than_32(torch, binding):  # noqa: F811
    """hypernet_fwd of 40 preferences of 2 x 64 with 40 features against 32: a fourth more of M to read and to multiply by, an eighth of
    the call at most (the launches and the trunk are its larger part)."""
    more, fewer = (hyper(torch, binding, case(40, 2, 64, 45, rank=4, hyper_width=F, wdtype=0))[0] for F in (40, 32))
    assert ratio(torch, more, fewer, turns=25) < 1.125


def test_rows_shorter_than_a_piece_take_no_longer_than_a_piece(torch, binding):  # noqa: F811
    """Acting with 7 observations against 8, 106 preferences x 870 rows of 1 x 512: an input less (a thirtieth is left for the clock)."""
    def act(O):
        cfg = case(106, 1, 512, O, N=106 * 87, T=10, rank=4)
        ctx, z = binding.Context.from_config(cfg), lambda *s: torch.zeros(*s, device="cuda")
        tm, tv = z(cfg.P, ctx.theta_mat_len(0)).to(torch.bfloat16), z(cfg.P, ctx.theta_vec_len(0))
        x, out, rows = z(cfg.T + 1, cfg.N, O), z(cfg.T + 1, cfg.N, cfg.act_dim), (0, cfg.T, 0, cfg.n_g)
        ws = torch.empty(ctx.workspace_bytes(rows), dtype=torch.uint8, device="cuda")
        return lambda: ctx.policy_fwd(0, tm, tv, x, rows, out, ws=ws)
    assert ratio(torch, act(7), act(8), turns=25) < 1.033
