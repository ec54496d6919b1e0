"""What the one-launch forward promises beyond the oracle's tolerances: fp32 hidden layers take the library's tanh, weights
of one row never reach the feature of another, and in bf16 a result does not depend on how many rows are asked for.
Inputs are made on the device."""
import pytest

from paper_2603_09237_amd.configs import CONFIGS, scaled
from test_gpu_parity import _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

ACTOR, CRITIC = 0, 1
BASE = scaled(CONFIGS[1], name="bits", K=3, act_dim=5, n_hidden=3, wdtype=1)


def out_dim(cfg, net):
    return cfg.K if net == CRITIC else (2 * cfg.act_dim if cfg.sigma_state else cfg.act_dim)


def layers(cfg, net):
    """(rows, columns, offset) of every matrix inside a preference's theta_mat."""
    off, out = 0, []
    for l in range(cfg.n_hidden + 1):
        d_in = cfg.obs_dim if l == 0 else cfg.width
        d_out = out_dim(cfg, net) if l == cfg.n_hidden else cfg.width
        out.append((d_out, d_in, off))
        off += d_out * d_in
    return out


def make_theta(cfg, ctx, net, torch, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    tm = torch.empty(cfg.P, ctx.theta_mat_len(net), device="cuda")
    for do, di, off in layers(cfg, net):
        tm[:, off:off + do * di] = torch.randn(cfg.P, do * di, device="cuda", generator=g) * di ** -0.5
    tv = torch.randn(cfg.P, ctx.theta_vec_len(net), device="cuda", generator=g) * 0.1
    return tm.to(torch.bfloat16 if cfg.wdtype == 1 else torch.float32), tv


def forward(cfg, ctx, net, tm, tv, x, rows, eps, torch, saving):
    """Outputs of the selection in its own shape (time, preference, environment, value); when saving, also h and the code
    of act'(z) of every hidden layer."""
    t0, tc, j0, jc = rows
    od = out_dim(cfg, net)
    out = torch.full((cfg.T, cfg.N, od), -7.5, device="cuda")
    ws = torch.empty(ctx.workspace_bytes(rows), dtype=torch.uint8, device="cuda")
    kw, got = {}, [out]
    if net == ACTOR:
        kw = dict(eps=eps, act=torch.full_like(eps, -7.5), logp=torch.full((cfg.T, cfg.N), -7.5, device="cuda"))
        got += [kw["act"], kw["logp"]]
    saved = torch.zeros(ctx.saved_bytes(net, rows), dtype=torch.uint8, device="cuda") if saving else None
    ctx.policy_fwd(net, tm, tv, x, rows, out, saved=saved, ws=ws, **kw)
    torch.cuda.synchronize()
    res = [t.view(cfg.T, cfg.P, cfg.n_g, -1)[t0:t0 + tc, :, j0:j0 + jc] for t in got]
    if saving:
        M, W, P = tc * jc, cfg.width, cfg.P
        Mp = (M + 31) // 32 * 32
        n = (P * Mp * W + 63) // 64 * 64
        buf = saved[:2 * cfg.n_hidden * n * 2].view(torch.int16).view(2 * cfg.n_hidden, n)
        rows_of = buf[:, :P * Mp * W].view(2 * cfg.n_hidden, P, Mp, W)[:, :, :M]
        res.append(rows_of.reshape(2 * cfg.n_hidden, P, tc, jc, W).permute(2, 1, 3, 0, 4))
    return res


@pytest.mark.parametrize("W", (64, 160, 512, 528))
def test_fp32_hidden_layers_take_the_librarys_tanh(W, torch, binding):  # noqa: F811
    """One hidden layer of unit weights and a critic whose output k is hidden feature k: the output is tanh(x)."""
    n_g = 2048
    cfg = scaled(BASE, name=f"tanh-W{W}", wdtype=0, width=W, obs_dim=1, act=0, n_hidden=1, P=2, N=2 * n_g, T=1)
    ctx = binding.Context.from_config(cfg)
    tm = torch.zeros(2, ctx.theta_mat_len(CRITIC), device="cuda")
    tv = torch.zeros(2, ctx.theta_vec_len(CRITIC), device="cuda")
    tm[:, :W] = 1.0
    for k in range(cfg.K):
        tm[:, W + k * W + k] = 1.0
    x = torch.cat([torch.logspace(-30, 1.2, n_g // 2), torch.linspace(0.3, 1.5, n_g // 2 - 2), torch.tensor([0.0, 200.0])])
    x = torch.stack([x, -x]).cuda().reshape(1, 2 * n_g, 1)
    got = forward(cfg, ctx, CRITIC, tm, tv, x, (0, 1, 0, n_g), None, torch, False)[0]
    ref = torch.tanh(x).view(1, 2, n_g, 1).expand_as(got)
    exact = torch.tanh(x.double()).view(1, 2, n_g, 1)
    ulp = lambda t: float(((t.double() - exact).abs() / exact.abs().clamp_min(1e-37) * 2 ** 23).max())
    print(f"[gpu-bits] tanh W={W}: largest relative error here {ulp(got):.3f} * 2^-23, of the library {ulp(ref):.3f} * 2^-23",
          flush=True)
    n_diff = int((got != ref).sum())
    assert n_diff == 0, n_diff


def plain_forward(cfg, net, tm, tv, x, torch):
    """The network in float64 with the matrices as they stand, [T, N, outputs]."""
    h = x.double().view(cfg.T, cfg.P, cfg.n_g, -1).permute(1, 0, 2, 3).reshape(cfg.P, cfg.T * cfg.n_g, -1).cpu()
    tm, tv, voff = tm.double().cpu(), tv.double().cpu(), 0
    for l, (do, di, off) in enumerate(layers(cfg, net)):
        z = torch.stack([h[p] @ tm[p, off:off + do * di].view(do, di).t() for p in range(cfg.P)]) + tv[:, None, voff:voff + do]
        voff += do
        last = l == cfg.n_hidden
        h = torch.tanh(z) if not last or (net == ACTOR and cfg.mean_tanh) else z
    return h.view(cfg.P, cfg.T, cfg.n_g, -1).permute(1, 0, 2, 3).reshape(cfg.T, cfg.N, -1)


@pytest.mark.parametrize("wd,W,O,L", [(0, 80, 11, 3), (0, 64, 45, 2), (0, 160, 33, 1), (1, 80, 45, 3), (1, 256, 45, 2),
                                      (1, 160, 40, 1), (1, 384, 72, 2)])
def test_infinite_and_undefined_weights_stay_in_their_row(wd, W, O, L, torch, binding):  # noqa: F811
    """An infinite weight saturates its own tanh feature, a NaN row of the output layer spoils its own output: the
    neighbouring rows, which a request for whole pieces of a row also reads, must not show it."""
    cfg = scaled(BASE, name=f"inf-{wd}-W{W}-O{O}-L{L}", wdtype=wd, width=W, obs_dim=O, act=0, n_hidden=L, P=2, N=2 * 21, T=1)
    ctx = binding.Context.from_config(cfg)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(1, cfg.N, O, device="cuda", generator=g)
    for net in (ACTOR, CRITIC):
        tm, tv = make_theta(cfg, ctx, net, torch, 5 + net)
        for l, (do, di, off) in enumerate(layers(cfg, net)[:-1]):
            tm[1, off + 7 * di + 1] = float("inf")
            tm[1, off + (do - 1) * di] = float("-inf")
        off = layers(cfg, net)[-1][2]
        tm[:, off:off + W] = float("nan")
        tm[:, off + 2 * W + 3] = float("inf")
        ref = plain_forward(cfg, net, tm, tv, x, torch)
        assert ref[..., 0].isnan().all() and not ref[..., 1:].isnan().any() and ref[..., 1].isfinite().all()
        for saving in (False, True):
            got = forward(cfg, ctx, net, tm, tv, x, (0, 1, 0, cfg.n_g), torch.zeros(1, cfg.N, 5, device="cuda"), torch, saving)[0]
            got = got.double().cpu().view(ref.shape)
            say = f" {cfg.name} net={net} saving={saving}: NaN {int(got.isnan().sum())} of {int(ref.isnan().sum())}"
            print("[gpu-bits] " + say, flush=True)
            same = bool((got.isnan() == ref.isnan()).all()) and bool((got.isinf() == ref.isinf()).all())
            assert same, say
            ok = ref.isfinite()
            # (the bounds of the parity tests: fp32 1e-5 + 1e-4 |ref|; bf16 relative RMS error 1e-2)
            if wd == 0:
                assert bool(((got - ref).abs() <= 1e-5 + 1e-4 * ref.abs())[ok].all())
            else:
                assert float((got - ref)[ok].square().mean().sqrt()) < 1e-2 * float(ref[ok].square().mean().sqrt())


# (width, observation widths, time steps of 131 rows that go to the kernel for tall selections): width 512 and 256 to the
# one that reads the matrices in fragment order, 384 and 448 to the tiled GEMMs behind the three first-layer forms (O <= 32
# by multiply-adds, O a multiple of 32 and of 8 and odd O on tiles), 160 and 208 to the same kernel with taller tiles
BIT_CASES = [(512, (11, 45, 64, 100), 4), (256, (11, 45, 64, 256), 6), (384, (11, 31, 32, 40, 45, 96), 4),
             (448, (19, 45, 64), 4), (160, (11, 45), 4), (208, (31, 64), 4)]


@pytest.mark.parametrize("act", (0, 1))
@pytest.mark.parametrize("W,O,T", [(W, O, T) for W, Os, T in BIT_CASES for O in Os])
def test_bf16_results_do_not_depend_on_the_rows_asked_for(W, O, T, act, torch, binding):  # noqa: F811
    """One time step of 40 rows (32-row tiles), two of 128 (64-row tiles) and the whole selection: outputs, samples,
    log-densities, saved activations and derivative codes of the rows they share."""
    cfg = scaled(BASE, name=f"bits-W{W}-O{O}-a{act}", width=W, obs_dim=O, act=act, P=64, N=64 * 131, T=T)
    ctx = binding.Context.from_config(cfg)
    g = torch.Generator(device="cuda").manual_seed(W + O)
    x = torch.randn(cfg.T, cfg.N, O, device="cuda", generator=g)
    eps = torch.randn(cfg.T, cfg.N, cfg.act_dim, device="cuda", generator=g)
    for net in (ACTOR, CRITIC):
        tm, tv = make_theta(cfg, ctx, net, torch, 5 + net)
        for saving in (False, True):
            tall = forward(cfg, ctx, net, tm, tv, x, (0, T, 0, 131), eps, torch, saving)
            assert all(bool(t.float().isfinite().all()) for t in tall)
            for t0, tc, j0, jc in ((1, 1, 3, 40), (0, 2, 3, 128)):
                part = forward(cfg, ctx, net, tm, tv, x, (t0, tc, j0, jc), eps, torch, saving)
                diff = [int((a != b[t0:t0 + tc, :, j0:j0 + jc]).sum()) for a, b in zip(part, tall)]
                assert not any(diff), (net, saving, tc, diff, [a.numel() for a in part])
