"""fp32 products on the bf16 matrix instructions (operands as sums of three bf16 values): as exact as the fp32 instructions, the
same infinite and undefined results."""
import pytest

from paper_2603_09237_amd.configs import CONFIGS, scaled
from test_gpu_forward_bits import ACTOR, layers, make_theta, out_dim
from test_gpu_parity import _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

BASE = scaled(CONFIGS[1], name="split", K=3, act_dim=5, wdtype=0, T=1)


def reference(cfg, tm, tv, x, dout, torch):
    """Outputs [P, M, A] and gradients of the matrices and biases by layer, in float64 on the host."""
    tm, tv = tm.double().cpu(), tv.double().cpu()
    x, dout = (t.double().cpu().view(cfg.P, cfg.n_g, -1) for t in (x, dout))
    outs, dws, dbs = [], [], []
    for p in range(cfg.P):
        hs, zs, voff = [x[p]], [], 0
        W = [tm[p, off:off + do * di].view(do, di) for do, di, off in layers(cfg, ACTOR)]
        for l, w in enumerate(W):
            z = hs[-1] @ w.t() + tv[p, voff:voff + len(w)]
            voff += len(w)
            zs.append(z)
            hs.append(torch.tanh(z) if cfg.act == 0 or l == cfg.n_hidden else z * torch.sigmoid(z))
        outs.append(hs[-1])
        dz, dw, db = dout[p] * (1 - hs[-1] ** 2), [], []
        for l in reversed(range(len(W))):
            dw.insert(0, dz.t() @ hs[l])
            db.insert(0, dz.sum(0))
            if l:
                s = torch.sigmoid(zs[l - 1])
                dz = (dz @ W[l]) * (1 - hs[l] ** 2 if cfg.act == 0 else s * (1 + zs[l - 1] * (1 - s)))
        dws.append(torch.cat([d.reshape(-1) for d in dw]))
        dbs.append(torch.cat(db))
    return torch.stack(outs), torch.stack(dws), torch.stack(dbs)


def device(cfg, ctx, tm, tv, x, dout, torch):
    rows = (0, 1, 0, cfg.n_g)
    ws = torch.empty(ctx.workspace_bytes(rows), dtype=torch.uint8, device="cuda")
    saved = torch.zeros(ctx.saved_bytes(ACTOR, rows), dtype=torch.uint8, device="cuda")
    outs = [torch.zeros(1, cfg.N, out_dim(cfg, ACTOR), device="cuda") for _ in range(2)]
    ctx.policy_fwd(ACTOR, tm, tv, x, rows, outs[0], ws=ws)
    ctx.policy_fwd(ACTOR, tm, tv, x, rows, outs[1], saved=saved, ws=ws)
    dm, dv = torch.empty_like(tm), torch.empty_like(tv)
    ctx.policy_bwd(ACTOR, tm, tv, x, rows, saved, dout, None, dm, dv, ws)
    torch.cuda.synchronize()
    n = sum(do for do, _, _ in layers(cfg, ACTOR))
    return [o.double().cpu().view(cfg.P, cfg.n_g, -1) for o in outs], dm.double().cpu(), dv[:, :n].double().cpu()


def inputs_of(cfg, torch, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(1, cfg.N, cfg.obs_dim, device="cuda", generator=g),
            torch.randn(1, cfg.N, out_dim(cfg, ACTOR), device="cuda", generator=g) / cfg.N)


LARGEST, BF16_LARGEST = 3.4028234663852886e38, 3.3895313892515355e38


# (preferences, width, observation width, rows, hidden layers): tiles of 128 and of 64 with remainders, contractions that end
# inside a step of 16, split and unsplit; a width that goes layer by layer, its first layer from aligned and from odd rows
SHAPES = [(3, 32, 9, 65, 2), (3, 48, 33, 131, 2), (3, 128, 45, 257, 3), (3, 160, 100, 331, 2), (3, 256, 19, 512, 3),
          (3, 272, 37, 97, 2), (3, 528, 44, 129, 2), (3, 528, 45, 40, 1)]
# the one-launch forward on split operands: every number of waves, tiles of 32, 64 and 96 rows with remainders, widths between two
# multiples of 32, observations of one and of many super-steps
SHAPES += [(24, 32, 9, 950, 2), (24, 48, 33, 2070, 2), (24, 64, 8, 2050, 3), (8, 80, 45, 525, 2), (8, 96, 12, 1100, 2),
           (8, 128, 19, 1100, 2), (3, 144, 100, 33, 3), (10, 160, 20, 1850, 2), (8, 176, 130, 545, 2), (10, 192, 45, 1890, 2),
           (8, 208, 65, 1090, 2), (8, 256, 27, 545, 2), (8, 256, 300, 1090, 2)]
SHAPES += [(24, 48, 33, 2070, 3)]
# one hidden layer on it: no ring of weights
SHAPES += [(40, 32, 20, 950, 1), (24, 64, 20, 2070, 1), (8, 144, 45, 2900, 1), (8, 208, 65, 1090, 1)]
# many rows of networks of one and two split waves whose observations are too wide for it: tiles of 16 rows
SHAPES += [(64, 48, 65, 1025, 2), (16, 64, 100, 4096, 2), (16, 64, 100, 4100, 3), (16, 32, 129, 1450, 2)]


@pytest.mark.parametrize("P,W,O,M,L", SHAPES)
@pytest.mark.parametrize("act", (0, 1))
def test_fp32_networks_against_64_bits(P, W, O, M, L, act, torch, binding):  # noqa: F811
    """Error of a whole tensor, 2-norm over 2-norm, in roundings of fp32 (2^-24).  The running sums of k products each take a
    rounding on average half as large as the sum's share of them: sqrt(k) / 4 in all; an activation, its derivative and the
    product with it three more; the 2 L + 1 products an output gradient goes through add up independently.  A product of
    parts left out shows: 3.5e-6 for a missing middle one."""
    cfg = scaled(BASE, name=f"split-P{P}-W{W}-O{O}-M{M}-L{L}", width=W, obs_dim=O, n_hidden=L, act=act, P=P, N=P * M)
    ctx = binding.Context.from_config(cfg)
    tm, tv = make_theta(cfg, ctx, ACTOR, torch, 11)
    x, dout = inputs_of(cfg, torch, 12)
    ref = reference(cfg, tm, tv, x, dout, torch)
    outs, dm, dv = device(cfg, ctx, tm, tv, x, dout, torch)
    bound = 2.0 ** -24 * (max(O, W, M) ** 0.5 / 4 + 3) * (2 * L + 1) ** 0.5
    err = lambda got, want: float((got - want).norm() / want.norm())
    pairs = [("out", outs[0], ref[0]), ("out saving", outs[1], ref[0]), ("db", dv, ref[2])]
    pairs += [(f"dW{l}", dm[:, off:off + do * di], ref[1][:, off:off + do * di]) for l, (do, di, off) in enumerate(layers(cfg, ACTOR))]
    got = {n: err(a, b) for n, a, b in pairs}
    print(f"[gpu-split] {cfg.name} act={act}: " + " ".join(f"{n} {e:.2e}" for n, e in got.items()) + f" bound {bound:.2e}", flush=True)
    assert all(e < bound for e in got.values()), got


@pytest.mark.parametrize("W,O,M,L", [(64, 33, 70, 2), (160, 20, 131, 2), (272, 40, 33, 2)])
@pytest.mark.parametrize("where", ("weight", "observation", "gradient", "largest", "largest observation"))
def test_fp32_infinite_and_undefined_results(where, W, O, M, L, torch, binding):  # noqa: F811
    """An infinite weight, observation or output gradient, and a weight that no bf16 value reaches, show in the same gradients
    as in float64, with the same sign; every other preference and element is as without it.  The largest observation beside a weight
    of zero is a zero."""
    cfg = scaled(BASE, name=f"inf-{where}-W{W}-O{O}-M{M}", width=W, obs_dim=O, n_hidden=L, act=0, P=2, N=2 * M)
    ctx = binding.Context.from_config(cfg)
    tm, tv = make_theta(cfg, ctx, ACTOR, torch, 21)
    x, dout = inputs_of(cfg, torch, 22)
    off1 = layers(cfg, ACTOR)[1][2]
    if where == "weight":
        tm[1, off1 + 7 * W + 3] = float("inf")       # saturates feature 7 of the second layer, spoils dH's column 3
    elif where == "largest":
        tm[1, off1 + 7 * W + 3] = 3.4e38
    elif where == "observation":
        x[0, M + 5, 2] = float("-inf")               # a row of the second preference
    elif where == "largest observation":
        x[0, M + 5, 2], x[0, M + 6, 2] = LARGEST, -LARGEST
        tm[1, 9 * O + 2] = 0.0                       # feature 9 of the first layer
    else:
        dout[0, M + 5, 1] = float("inf")
    ref = reference(cfg, tm, tv, x, dout, torch)
    outs, dm, dv = device(cfg, ctx, tm, tv, x, dout, torch)
    for name, got, want in (("out", outs[0], ref[0]), ("out saving", outs[1], ref[0]), ("dW", dm, ref[1]), ("db", dv, ref[2])):
        want32 = want.float().double()               # a sum beyond fp32's range is infinite
        same = bool((got.isnan() == want32.isnan()).all()) and bool(((got == want32) | ~want32.isinf()).all())
        n = int((got.isnan() != want32.isnan()).sum())
        print(f"[gpu-split] {cfg.name} {name}: NaN {int(want32.isnan().sum())} inf {int(want32.isinf().sum())} wrong {n}", flush=True)
        assert same, (name, n)
        ok = want32.isfinite()
        assert bool(((got - want32).abs() <= 1e-5 + 1e-4 * want32.abs())[ok].all()), name   # (the bounds of the parity tests)


@pytest.mark.parametrize("P,W,O,M,L", [(2, 160, 20, 131, 2), (24, 32, 9, 950, 2), (8, 256, 45, 545, 3), (8, 208, 65, 1090, 1), (2, 64, 33, 70, 2)])
def test_fp32_finite_results_of_the_largest_values(P, W, O, M, L, torch, binding):  # noqa: F811
    """SiLU networks whose features reach the largest float, which no bf16 value does, and a product whose leading parts alone
    overflow: finite in float64 and in fp32, on split operands as well (all but the last shape)."""
    cfg = scaled(BASE, name=f"large-P{P}-W{W}-O{O}-M{M}-L{L}", width=W, obs_dim=O, n_hidden=L, act=1, mean_tanh=0, P=P, N=P * M)
    ctx = binding.Context.from_config(cfg)
    tm, tv = make_theta(cfg, ctx, ACTOR, torch, 31)
    x, _ = inputs_of(cfg, torch, 32)
    p, row = 1, M + 5
    Ws = [tm[p, off:off + do * di].view(do, di) for do, di, off in layers(cfg, ACTOR)]
    Ws[0][:, 1], Ws[0][:, 4] = 0.01, 0.0
    Ws[0][7, 1], Ws[0][9, 1], Ws[0][11, 4] = 1.0, 0.0, 1.00391   # (its leading part is 1.0078)
    for w in Ws[1:]:
        w[:, 7] *= 1e-3
        w[:, 11] *= 1e-3
    Ws[1][3, 7] = 0.0
    tv[p, 7] = tv[p, 11] = 0.0
    x[0, row], x[0, row + 1], x[0, row + 2] = 0.0, 0.0, 0.0
    x[0, row, 1], x[0, row + 1, 1], x[0, row + 2, 4] = LARGEST, -LARGEST, BF16_LARGEST
    rows = (0, 1, 0, cfg.n_g)
    ws = torch.empty(ctx.workspace_bytes(rows), dtype=torch.uint8, device="cuda")
    saved = torch.zeros(ctx.saved_bytes(ACTOR, rows), dtype=torch.uint8, device="cuda")
    h, voff = x.view(P, M, O)[p].double().cpu(), 0
    for l, w in enumerate(Ws):
        z = h @ w.double().cpu().t() + tv[p, voff:voff + len(w)].double().cpu()
        voff += len(w)
        h = z * torch.sigmoid(z) if l < L else z
        assert bool((h.abs() <= LARGEST).all())
    for sv in (None, saved):
        out = torch.zeros(1, cfg.N, out_dim(cfg, ACTOR), device="cuda")
        ctx.policy_fwd(ACTOR, tm, tv, x, rows, out, saved=sv, ws=ws)
        got = out.view(P, M, -1)[p].double().cpu()
        err = float(((got - h).norm(dim=1) / h.norm(dim=1)).nan_to_num(float("inf")).max())
        print(f"[gpu-split] {cfg.name} saving={sv is not None}: largest error of a row {err:.2e}", flush=True)
        assert bool(torch.isfinite(out).all())
        assert err < 1e-4   # (the relative bound of the parity tests)
