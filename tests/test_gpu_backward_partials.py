"""Backward of the target networks at the edges of what its launches leave as partial sums, against the oracle with the
bounds of the parity tests: rows around the 64-row blocks of the output layer's sums, the 128-row tiles and the four blocks
to a 256-row group, columns around the 128 of a workgroup, observation widths around the 16 and 32 columns of the narrow
first layer, the smallest and the largest output layers, split and unsplit contractions side by side."""
import pytest

import test_gpu_parity as parity
from paper_2603_09237_amd.configs import scaled
from test_gpu_parity import RAGGED, _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def case(M, W, O, A, K, L, P, **over):
    return scaled(RAGGED, name=f"M{M}-W{W}-O{O}-A{A}-K{K}-L{L}-P{P}" + "".join(f"-{k}{v}" for k, v in over.items()), T=1, N=P * M,
                  P=P, K=K, obs_dim=O, act_dim=A, n_hidden=L, width=W, **over)


CASES = [case(M, W, O, A, K, L, P, wdtype=b)
         for b in (0, 1)
         for M, W, O, A, K, L, P in ((1, 16, 1, 1, 1, 1, 2), (63, 48, 16, 2, 3, 2, 3), (64, 128, 17, 16, 5, 2, 2), (65, 144, 31, 4, 16, 3, 2),
                                     (255, 112, 32, 3, 2, 2, 4), (256, 272, 33, 5, 4, 2, 2), (257, 64, 5, 8, 2, 3, 2),
                                     (513, 32, 11, 9, 7, 2, 5), (1025, 128, 8, 3, 3, 2, 2))]
CASES += [case(300, 256, 40, 7, 6, 3, 2, wdtype=1, act=0), case(770, 512, 64, 10, 6, 2, 2, wdtype=1),
          case(130, 96, 9, 4, 2, 2, 3, wdtype=1, sigma_state=1), case(130, 96, 9, 4, 2, 2, 3, wdtype=0, mean_tanh=0)]

# weight gradients on small tiles whose contraction is split, evenly and unevenly, beside layers that are not split
CASES += [case(512, 128, 40, 3, 2, 2, 2, wdtype=1), case(2048, 64, 40, 3, 2, 3, 2, wdtype=1), case(4224, 80, 33, 3, 2, 2, 2, wdtype=1),
          case(20, 48, 40, 3, 2, 3, 2, wdtype=0), case(700, 160, 40, 3, 2, 2, 2, wdtype=0),
          case(333, 192, 70, 3, 2, 2, 3, wdtype=0), case(96, 32, 36, 3, 2, 4, 7, wdtype=0)]
# bf16 first layers on small tiles whose last range is the shorter one (padded rows 2112 + 2016 and 2112 + 2048)
CASES += [case(4115, 80, 33, 3, 2, 2, 2, wdtype=1), case(4160, 144, 70, 3, 2, 1, 2, wdtype=1)]

# terms requested together at the end of the backward pass: 32 sums of 64 rows of the output layer's bias (31, 32, 33 and 65 of them), 8
# row blocks of an eighth of a layer's bias sums, 16 ranges of the first layer's dW (16, 17 and more), 2, 4, 8 and 16 ranges of a split one
CASES += [case(M, 64, O, 3, 2, 2, 2, wdtype=b) for b in (0, 1) for M, O in ((1984, 11), (2048, 16), (2049, 17), (4097, 3))]
CASES += [case(M, 128, 40, 3, 2, 2, 2, wdtype=0) for M in (129, 257, 512, 1024, 1030)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_backward_at_the_edges_of_its_partial_sums(cfg, torch, binding):  # noqa: F811
    parity.test_policy_bwd_matches_oracle(cfg, None, torch, binding)


# fp32 weight gradients on both sides of the line between 64 x 64 and 128 x 128 tiles: 7 and 8 rounds of small tiles in the
# place of two
LINE = [case(512, 1824, 34, 2, 2, 2, 2, wdtype=0, rank=2), case(512, 1952, 34, 2, 2, 2, 2, wdtype=0, rank=2)]


@pytest.mark.parametrize("cfg", LINE, ids=lambda c: c.name)
def test_backward_of_wide_fp32_networks(cfg, torch, binding):  # noqa: F811
    parity.test_policy_bwd_matches_oracle(cfg, None, torch, binding)


def test_fp32_weight_gradients_of_a_narrower_network_take_no_longer(torch, binding):  # noqa: F811
    """dW of 2 preferences x 4096 rows x 1952 x 1952 against 2048 x 2048, which is as many 128 x 128 tiles and a tenth more
    weights (a tenth is left for the clock)."""
    def passes(W):
        cfg = case(4096, W, 16, 2, 2, 2, 2, wdtype=0, rank=2)
        ctx, net, rows = binding.Context.from_config(cfg), parity.ACTOR, (0, 1, 0, 4096)
        z = lambda *s: torch.zeros(*s, device="cuda")
        tm, tv = z(2, ctx.theta_mat_len(net)), z(2, ctx.theta_vec_len(net))
        x, mu, dls = z(2, 8192, 16), z(1, 8192, 2), z(2, 2)
        saved, ws = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (ctx.saved_bytes(net, rows), ctx.workspace_bytes(rows)))
        dtm, dtv = torch.empty_like(tm), torch.empty_like(tv)
        ctx.policy_fwd(net, tm, tv, x, rows, mu, saved=saved, ws=ws)

        def once():
            ctx.profile_begin()
            for _ in range(3):
                ctx.policy_bwd(net, tm, tv, x, rows, saved, mu, dls, dtm, dtv, ws)
            ms, n, _ = ctx.profile_end()["dw_hidden"]
            return ms / n
        return once
    narrow, wide = passes(1952), passes(2048)
    narrow(), wide()
    best = [min(t) for t in zip(*((narrow(), wide()) for _ in range(7)))]
    assert best[0] < 1.1 * best[1], best


@pytest.mark.parametrize("M,W,O,P", ((97, 256, 34, 33), (300, 80, 130, 129)))
def test_bf16_weight_gradients_on_small_and_large_tiles_are_the_same_bits(M, W, O, P, torch, binding):  # noqa: F811
    """P - 1 preferences make 512 tiles of 64 x 64 and run on those, P preferences more and run on 128 x 128: every sum keeps
    its order, so the gradients of the first P - 1 are equal."""
    g = torch.Generator(device="cuda").manual_seed(3)
    n = lambda *s: torch.randn(*s, device="cuda", generator=g)
    net, rows, grads, data = parity.ACTOR, (0, 1, 0, M), [], None
    for q in (P, P - 1):
        ctx = binding.Context.from_config(case(M, W, O, 2, 2, 2, q, wdtype=1, rank=2))
        if data is None:
            data = (n(P, ctx.theta_mat_len(net)) * W ** -0.5, n(P, ctx.theta_vec_len(net)) * 0.1, n(2, P * M, O), n(1, P * M, 2), n(P, 2))
        tm, tv, x, dout, dls = data[0][:q].to(torch.bfloat16), data[1][:q], data[2][:, :q * M].contiguous(), data[3][:, :q * M].contiguous(), data[4][:q]
        saved, ws = (torch.empty(b, dtype=torch.uint8, device="cuda") for b in (ctx.saved_bytes(net, rows), ctx.workspace_bytes(rows)))
        dtm, dtv = torch.empty(q, tm.shape[1], device="cuda"), torch.empty(q, tv.shape[1], device="cuda")
        ctx.policy_fwd(net, tm, tv, x, rows, torch.empty_like(dout), saved=saved, ws=ws)
        ctx.policy_bwd(net, tm, tv, x, rows, saved, dout, dls, dtm, dtv, ws)
        grads.append((dtm[:P - 1], dtv[:P - 1]))
    for a, b in zip(*grads):
        assert torch.equal(a, b)


def test_bf16_weight_gradients_of_fewer_preferences_take_no_longer(torch, binding):  # noqa: F811
    """dW of 60 preferences x 6838 rows x 256 x 256 against 64, which is more of the same work (a tenth is left for the clock)."""
    def passes(P):
        cfg = case(6838, 256, 16, 2, 2, 2, P, wdtype=1, rank=2)
        ctx, net, rows, N = binding.Context.from_config(cfg), parity.ACTOR, (0, 1, 0, 6838), 6838 * P
        z = lambda *s, **k: torch.zeros(*s, device="cuda", **k)
        tm, tv = z(P, ctx.theta_mat_len(net), dtype=torch.bfloat16), z(P, ctx.theta_vec_len(net))
        x, mu, dls = z(2, N, 16), z(1, N, 2), z(P, 2)
        saved, ws = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (ctx.saved_bytes(net, rows), ctx.workspace_bytes(rows)))
        dtm, dtv = z(P, ctx.theta_mat_len(net)), z(P, ctx.theta_vec_len(net))
        ctx.policy_fwd(net, tm, tv, x, rows, mu, saved=saved, ws=ws)

        def once():
            ctx.profile_begin()
            for _ in range(3):
                ctx.policy_bwd(net, tm, tv, x, rows, saved, mu, dls, dtm, dtv, ws)
            ms, n, _ = ctx.profile_end()["dw_hidden"]
            return ms / n
        return once
    few, more = passes(60), passes(64)
    few(), more()
    best = [min(t) for t in zip(*((few(), more()) for _ in range(7)))]
    assert best[0] < 1.1 * best[1], best
