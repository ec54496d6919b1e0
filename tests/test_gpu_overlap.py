"""The two networks' chains on streams of their own give the bits that one stream gives: gradients, updated parameters, roll-out
and loss, step after step, from a caller's stream that is not the default one, with inputs that change in between."""
import pytest

from paper_2603_09237_amd import inputs
from paper_2603_09237_amd.configs import CONFIGS, scaled
from test_gpu_parity import RAGGED, _float32_default, binding, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

ADAM = dict(lr_actor=3e-3, lr_critic=1e-2, beta1=0.9, beta2=0.999, eps=1e-8)
CASES = [(scaled(CONFIGS[1], name="overlap-adam", minibatches=2, epochs=2), dict(optimizer=ADAM)),
         (scaled(RAGGED, name="overlap-per-objective"), dict(adv_norm="per_objective", optimizer=ADAM)),
         (scaled(CONFIGS[3], name="overlap-sigma-bf16", sigma_state=1, P=8, N=8 * 60, T=9, minibatches=3), dict(keep_adv_vec=True))]


@pytest.mark.parametrize("cfg,kw", CASES, ids=lambda x: getattr(x, "name", ""))
@pytest.mark.parametrize("callback", (False, True))
def test_streams_of_their_own_give_the_same_bits(cfg, kw, callback, torch, binding):  # noqa: F811
    from paper_2603_09237_amd.step import UpdateStep
    d = inputs.make_all(cfg)
    got = {}
    for overlap in (False, True):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            st = UpdateStep(cfg, **kw)
            st.overlap = overlap
            st.load_inputs(d)
            out = []

            def keep(*_):   # behind what the caller's stream holds, before anything it is given next
                out.extend(t.clone() for n in (0, 1) for t in (st.dhp[n], st.hp[n], st.theta_vec[n]))
                out.extend(t.clone() for t in (st.mu_old, st.act, st.logp_old, st.v_roll, st.vtarg, st.adv_s, st.mu, st.v, st.stats))

            for i in range(3):
                st.run(on_minibatch=keep if callback else None)
                keep()
                st.obs.mul_(0.9)
                st.rewards.add_(0.125)
                for n in (0, 1):
                    st.hp_old[n].copy_(st.hp[n])
        torch.cuda.synchronize()
        got[overlap] = out
    assert len(got[False]) == len(got[True])
    wrong = [i for i, (a, b) in enumerate(zip(got[False], got[True])) if not torch.equal(a, b)]
    print(f"[gpu-overlap] {cfg.name} callback={callback}: {len(got[True])} tensors, different {wrong[:5]}", flush=True)
    assert not wrong


# steps that take two streams by themselves: the split forward of fp32 networks of width 256, the persistent kernels of bf16 ones of
# width 512
OWN = [scaled(CONFIGS[2], name="overlap-own-fp32-W256", P=8, N=8 * 109, T=5), scaled(CONFIGS[4], name="overlap-own-bf16-W512", P=32, N=32 * 64, T=16, rank=4, n_hidden=3)]


@pytest.mark.parametrize("cfg", OWN, ids=lambda c: c.name)
def test_streams_that_a_step_takes_by_itself_give_the_same_bits(cfg, torch, binding):  # noqa: F811
    from paper_2603_09237_amd.step import UpdateStep
    d, got = inputs.make_all(cfg), []
    for one in (False, True):
        st = UpdateStep(cfg, optimizer=ADAM)
        assert st.overlap
        if one:
            st.overlap = False
        st.load_inputs(d)
        for _ in range(3):
            st.run()
        torch.cuda.synchronize()
        got.append([t.clone() for n in (0, 1) for t in (st.dhp[n], st.hp[n], st.theta_vec[n])] +
                   [t.clone() for t in (st.act, st.logp_old, st.v_roll, st.adv_s, st.mu, st.v, st.stats)])
    wrong = [i for i, (a, b) in enumerate(zip(*got)) if not torch.equal(a, b)]
    print(f"[gpu-overlap] {cfg.name}: {len(got[0])} tensors, different {wrong[:5]}", flush=True)
    assert not wrong


# either side of the two lines of the rule, and what is far beyond them
@pytest.mark.parametrize("P,rows,L,W,two", [(4, 640, 2, 256, False), (16, 3200, 2, 128, True), (4, 96, 4, 256, False), (4, 192, 4, 256, True)])
def test_which_steps_take_two_streams(P, rows, L, W, two, torch, binding):  # noqa: F811
    from paper_2603_09237_amd.step import UpdateStep
    assert UpdateStep(scaled(CONFIGS[3], name="overlap-rule", P=P, N=P * rows // 16, T=16, n_hidden=L, width=W)).overlap is two
    assert UpdateStep(CONFIGS[3]).overlap is True


def test_rule_and_capture_stay_on_the_callers_stream(torch, binding):  # noqa: F811
    """A step bound by its submission stays on one stream; a caller's own graph records the one-stream schedule whatever
    `overlap` says, and its replays equal the eager steps."""
    from paper_2603_09237_amd.step import UpdateStep
    assert not UpdateStep(CONFIGS[1]).overlap
    cfg = scaled(CONFIGS[1], name="overlap-capture", minibatches=2)
    st = UpdateStep(cfg)
    st.load_inputs(inputs.make_all(cfg))
    st.overlap = True
    st.run()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (st.dhp[0], st.dhp[1], st.stats)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        st.run()
    for _ in range(3):
        for n in (0, 1):
            st.dhp[n].zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(ref, (st.dhp[0], st.dhp[1], st.stats)))
        st.run()


def test_profile_of_launches_on_two_streams(torch, binding):  # noqa: F811
    """The profile waits for every stream that was launched on, not for the last launch alone; a step that is profiled stays on the
    caller's stream."""
    from paper_2603_09237_amd.step import UpdateStep
    cfg = scaled(CONFIGS[3], name="overlap-profile", P=16, N=16 * 256, T=16)
    st = UpdateStep(cfg)
    st.load_inputs(inputs.make_all(cfg))
    ctx, fwd = st.ctx, lambda net, rows, stream: st.ctx.policy_fwd(
        net, st.theta_mat[net], st.theta_vec[net], st.obs, rows, st.mu_old if net == 0 else st.v_roll, ws=st.wsn[net], stream=stream)
    st.run()
    torch.cuda.synchronize()
    long, *others = [torch.cuda.Stream() for _ in range(6)]   # (some of them share the first one's hardware queue)
    for short in others:
        ctx.profile_begin()
        for _ in range(200):
            fwd(1, st.full_T1, long.cuda_stream)
        fwd(0, (0, 1, 0, 1), short.cuda_stream)
        assert sum(v[1] for v in ctx.profile_end().values()) >= 201
        assert long.query() and short.query()
    st.overlap = True
    st._run_beside = None
    ctx.profile_begin()
    st.run()
    assert ctx.profile_end()["fwd_fused"][1] > 0
