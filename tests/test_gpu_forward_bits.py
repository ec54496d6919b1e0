"""What the one-launch forward promises beyond the oracle's tolerances: fp32 hidden layers take the library's tanh.
Inputs are made on the device and everything here is compared bit for bit."""
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
