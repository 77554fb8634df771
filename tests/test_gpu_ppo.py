"""GPU parity of the PPO head update (through the C ABI) against the fp64 oracle.

Tolerances: the GPU keeps parameters and Adam state in fp32 (rounded after every step) and sums in fp64;
the oracle is fp64 throughout.  One step therefore agrees to about 1e-7 of a parameter's size; the bound
used on the parameter change after a whole update is 2e-4 of the largest change of that tensor."""
import numpy as np
import pytest

from oracle import ppo_oracle as P
from paper_2604_24273_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _mods():
    from paper_2604_24273_amd import binding as B
    from paper_2604_24273_amd import runtime as R
    B.lib()
    return B, R


def test_gae_matches_oracle():
    B, R = _mods()
    c = synth.ppo_rollout_case(3, 300, 8, 4, 0, n_envs=5)
    c["dones"][2, 299] = 1.0                      # an episode that ends with the rollout: no bootstrap
    adv, ret = R.gae(R.dev(c["rewards"]), R.dev(c["values"]), R.dev(c["dones"]), R.dev(c["last_value"]), 0.99, 0.95)
    for e in range(5):
        a_ref, r_ref = P.gae(c["rewards"][e], c["values"][e], c["dones"][e], c["last_value"][e], 0.99, 0.95)
        scale = np.abs(a_ref).max()
        assert np.abs(adv[e].cpu().numpy() - a_ref).max() <= 2e-7 * scale + 1e-7
        assert np.abs(ret[e].cpu().numpy() - r_ref).max() <= 2e-7 * np.abs(r_ref).max() + 1e-7


def _run_case(B, R, dims_p, dims_v, act, T, batch, epochs, seed, **hyper):
    d, A = dims_p[0], dims_p[-1]
    c = synth.ppo_rollout_case(seed, T, d, A, epochs)
    pw, pb = synth.mlp_params(seed, 60, dims_p)
    vw, vb = synth.mlp_params(seed, 80, dims_v)
    adv_ref, ret_ref = P.gae(c["rewards"][0], c["values"][0], c["dones"][0], c["last_value"][0], 0.99, 0.95)
    adv32, ret32 = adv_ref.astype(np.float32), ret_ref.astype(np.float32)
    tr = R.PPOTrainer((pw, pb), (vw, vb), act=B.BRL_ACT_TANH if act == "tanh" else B.BRL_ACT_RELU, **hyper)
    stats = tr.update(R.dev(c["h"]), R.dev(c["actions"]), R.dev(c["logp_old"]), R.dev(adv32), R.dev(ret32),
                      R.dev(c["perm"]), batch)
    hp = P.PPOHyper(**hyper)
    pol = P.MLPParams([w.astype(np.float64) for w in pw], [b.astype(np.float64) for b in pb], act)
    val = P.MLPParams([w.astype(np.float64) for w in vw], [b.astype(np.float64) for b in vb], act)
    out = P.ppo_update(c["h"].astype(np.float64), c["actions"], c["logp_old"].astype(np.float64), adv32.astype(np.float64),
                       ret32.astype(np.float64), pol, val, c["perm"], batch, hp)
    return tr, stats, pol, val, out, (pw, pb, vw, vb), c


@pytest.mark.parametrize("dims_p,dims_v,act,T,batch,epochs", [
    ([2560, 256, 18], [2560, 256, 1], "tanh", 256, 64, 2),       # the measured head shape
    ([96, 32, 16, 5], [96, 32, 16, 1], "relu", 200, 48, 3),      # two hidden layers, ragged rollout (8 steps dropped per epoch)
    ([64, 7], [64, 1], "tanh", 40, 40, 1),                        # single layer, one step
    ([96, 32, 16, 5], [96, 24, 1], "tanh", 128, 32, 2),           # heads of unequal depth: the deeper one's extra level runs alone
    ([64, 7], [64, 16, 8, 1], "relu", 96, 32, 2),
])
def test_head_update_matches_oracle(dims_p, dims_v, act, T, batch, epochs):
    B, R = _mods()
    tr, stats, pol, val, out, init, c = _run_case(B, R, dims_p, dims_v, act, T, batch, epochs, seed=11)
    n_steps = epochs * (T // batch)
    assert tr.step == n_steps == len(out["stats"])
    st = stats.cpu().numpy()
    ref = np.array([[s["policy_loss"], s["value_loss"], s["entropy"], s["clip_fraction"], s["grad_norm"]] for s in out["stats"]])
    # the first step starts from identical parameters: tight; later steps inherit the fp32 parameter rounding
    assert np.allclose(st[0], ref[0], rtol=2e-6, atol=1e-7), (st[0], ref[0])
    assert np.allclose(st[:, [0, 1, 2, 4]], ref[:, [0, 1, 2, 4]], rtol=2e-4, atol=1e-6)
    assert np.abs(st[:, 3] - ref[:, 3]).max() <= 1.0 / batch + 1e-6          # at most one sample on the clip boundary
    pw, pb, vw, vb = tr.tensors()
    got = list(pw) + list(pb) + list(vw) + list(vb)
    want = list(pol.weights) + list(pol.biases) + list(val.weights) + list(val.biases)
    start = list(init[0]) + list(init[1]) + list(init[2]) + list(init[3])
    for g, w, s0 in zip(got, want, start):
        change = np.abs(w - s0.astype(np.float64)).max()
        assert change > 0
        assert np.abs(g.astype(np.float64) - w).max() <= 2e-4 * change + 1e-7, (g.shape, np.abs(g - w).max(), change)
    # the forward entry point reads the same flat buffer: its outputs match the oracle's updated heads
    h_eval = R.dev(c["h"][:16])
    logits = torch.empty((16, dims_p[-1]), dtype=torch.float32, device="cuda")
    value = torch.empty((16,), dtype=torch.float32, device="cuda")
    ws = R.Workspace(B.brl_head_workspace_bytes(tr.head, 16))
    B.policy_value_head(tr.head, h_eval, 16, logits, value, ws.buf)
    l_ref = P.mlp_forward_cache(c["h"][:16], pol)[-1]
    v_ref = P.mlp_forward_cache(c["h"][:16], val)[-1][:, 0]
    assert np.abs(logits.cpu().numpy() - l_ref).max() <= 1e-4 * np.abs(l_ref).max()
    assert np.abs(value.cpu().numpy() - v_ref).max() <= 1e-4 * max(np.abs(v_ref).max(), 1.0)


def test_head_update_is_deterministic_and_resumable():
    B, R = _mods()
    dims_p, dims_v = [128, 32, 6], [128, 32, 1]
    c = synth.ppo_rollout_case(5, 128, 128, 6, 2)
    pw, pb = synth.mlp_params(5, 60, dims_p)
    vw, vb = synth.mlp_params(5, 80, dims_v)
    adv = R.dev(synth.normal(5, 90, (128,)))
    ret = R.dev(synth.normal(5, 91, (128,)))
    args = (R.dev(c["h"]), R.dev(c["actions"]), R.dev(c["logp_old"]), adv, ret)
    a = R.PPOTrainer((pw, pb), (vw, vb))
    a.update(*args, R.dev(c["perm"]), 32)
    b = R.PPOTrainer((pw, pb), (vw, vb))
    b.update(*args, R.dev(c["perm"][:1]), 32)           # the same update as two calls: the step counter carries over
    b.update(*args, R.dev(c["perm"][1:]), 32)
    assert a.step == b.step == 8
    assert torch.equal(a.params, b.params) and torch.equal(a.adam_m, b.adam_m) and torch.equal(a.adam_v, b.adam_v)
    before = a.params.clone()
    step = B.ppo_head_update(a.cfg, a.params, a.adam_m, a.adam_v, a.step, *args, 128, R.dev(c["perm"]), 0, 32, None,
                             a.ws.buf)                  # no epochs: nothing changes
    assert torch.equal(before, a.params) and step == 8


def test_no_normalisation_and_paper_hyperparameters_defaults():
    B, R = _mods()
    tr, stats, pol, val, out, init, c = _run_case(B, R, [64, 16, 3], [64, 16, 1], "tanh", 64, 16, 1, seed=13,
                                                  normalize_adv=False, clip_eps=0.2, ent_coef=0.0)
    ref = np.array([[s["policy_loss"], s["value_loss"], s["entropy"], s["clip_fraction"], s["grad_norm"]] for s in out["stats"]])
    assert np.allclose(stats.cpu().numpy()[:, [0, 1, 2, 4]], ref[:, [0, 1, 2, 4]], rtol=2e-4, atol=1e-6)
    cfg, _ = B.make_ppo_config([8, 4, 2], [8, 4, 1], B.BRL_ACT_TANH)
    assert abs(cfg.clip_eps - 0.1) < 1e-7 and abs(cfg.ent_coef - 0.05) < 1e-7 and abs(cfg.max_grad_norm - 0.5) < 1e-7
    assert abs(cfg.lr_policy - 3e-4) < 1e-7 and abs(cfg.lr_value - 1e-3) < 1e-7


@pytest.mark.parametrize("dims_p,dims_v,act,T,batch", [
    ([2567, 250, 3], [2567, 17, 1], "tanh", 70, 67),      # inputs, units and samples off every tile; rows at odd addresses
    ([9, 5], [9, 3, 1], "relu", 6, 3),                    # less than one tile in every direction, heads of unequal depth
    ([1024, 40, 24, 70], [1024, 16, 1], "tanh", 260, 130),   # more actions than a wavefront, three sample blocks
    ([1030, 256, 5], [1030, 250, 1], "tanh", 2100, 2090),    # more than 1024 tiles: a workgroup takes all inputs of its tile
    ([48, 1040, 30], [48, 1030, 1], "tanh", 48, 16),      # too many units for one workgroup per sample: a launch per level
    ([40, 640, 500, 4], [40, 8, 1], "relu", 24, 12),      # 320 k weights above the first layer, units that still fit
])
def test_head_update_at_tile_edges(dims_p, dims_v, act, T, batch):
    """Bounds as above: first-step statistics from identical parameters, parameter change relative to its largest."""
    B, R = _mods()
    tr, stats, pol, val, out, init, c = _run_case(B, R, dims_p, dims_v, act, T, batch, 2, seed=17)
    st = stats.cpu().numpy()
    ref = np.array([[s["policy_loss"], s["value_loss"], s["entropy"], s["clip_fraction"], s["grad_norm"]] for s in out["stats"]])
    assert np.allclose(st[0], ref[0], rtol=2e-6, atol=1e-7), (st[0], ref[0])
    pw, pb, vw, vb = tr.tensors()
    for g, w, s0 in zip(list(pw) + list(pb) + list(vw) + list(vb),
                        list(pol.weights) + list(pol.biases) + list(val.weights) + list(val.biases),
                        list(init[0]) + list(init[1]) + list(init[2]) + list(init[3])):
        change = np.abs(w - s0.astype(np.float64)).max()
        assert np.abs(g.astype(np.float64) - w).max() <= 2e-4 * change + 1e-7, (g.shape, np.abs(g - w).max(), change)


@pytest.mark.parametrize("T", [1, 2, 255, 257, 2048])
def test_gae_stretches(T):
    """One thread composes a stretch of steps: shorter than the workgroup, one over, and the rollout's usual length."""
    B, R = _mods()
    c = synth.ppo_rollout_case(19, T, 4, 4, 0, n_envs=3)
    adv, ret = R.gae(R.dev(c["rewards"]), R.dev(c["values"]), R.dev(c["dones"]), R.dev(c["last_value"]), 0.99, 0.95)
    for e in range(3):
        a_ref, r_ref = P.gae(c["rewards"][e], c["values"][e], c["dones"][e], c["last_value"][e], 0.99, 0.95)
        scale = max(np.abs(a_ref).max(), np.abs(r_ref).max())
        assert np.abs(adv[e].cpu().numpy() - a_ref).max() <= 2e-7 * scale + 1e-7
        assert np.abs(ret[e].cpu().numpy() - r_ref).max() <= 2e-7 * scale + 1e-7


@pytest.mark.parametrize("dims_p,dims_v,offsets", [([130, 36, 5], [130, 30, 1], (1, 2, 3)), ([96, 2100, 3], [96, 8, 1], (3, 1, 0))])
def test_head_update_on_buffers_that_start_anywhere(dims_p, dims_v, offsets):
    """params, adam_m and adam_v as views at odd elements of larger buffers: the bits of the aligned buffers, and nothing
    beside the views is touched."""
    B, R = _mods()
    T, batch = 64, 32
    c = synth.ppo_rollout_case(23, T, dims_p[0], dims_p[-1], 2)
    pwb, vwb = synth.mlp_params(23, 60, dims_p), synth.mlp_params(23, 80, dims_v)
    args = (R.dev(c["h"]), R.dev(c["actions"]), R.dev(c["logp_old"]), R.dev(synth.normal(23, 90, (T,))),
            R.dev(synth.normal(23, 91, (T,))))
    a = R.PPOTrainer(pwb, vwb)
    n = a.params.numel()
    bufs = [torch.full((n + 8,), 7.0, dtype=torch.float32, device="cuda") for _ in range(3)]
    views = [b[o:o + n] for b, o in zip(bufs, offsets)]
    for v, src in zip(views, (a.params, a.adam_m, a.adam_v)):
        v.copy_(src)
    print("ppo_head_update on views at", offsets, flush=True)
    sa = a.update(*args, R.dev(c["perm"]), batch)
    sb = torch.zeros_like(sa)
    B.ppo_head_update(a.cfg, *views, 0, *args, T, R.dev(c["perm"]), 2, batch, sb, a.ws.buf)
    assert torch.equal(sa, sb)
    for b, v, o, want in zip(bufs, views, offsets, (a.params, a.adam_m, a.adam_v)):
        assert torch.equal(v, want)
        assert bool((b[:o] == 7.0).all()) and bool((b[o + n:] == 7.0).all())


@pytest.mark.parametrize("value_hidden", [1000, 1100])
def test_head_update_norm_on_both_sides_of_its_launch(value_hidden):
    """3039 partial sums of squares (added by Adam's workgroups) and 3089 (a launch of their own): the gradient norm of the
    first step from identical parameters, and the parameters after it, bounds as above."""
    B, R = _mods()
    print("gradient norm, value head of", value_hidden, flush=True)
    tr, stats, pol, val, out, init, c = _run_case(B, R, [512, 2100, 700, 3], [512, value_hidden, 1], "tanh", 16, 8, 1, seed=29)
    st, ref = stats.cpu().numpy(), [s["grad_norm"] for s in out["stats"]]
    assert np.isclose(st[0, 4], ref[0], rtol=2e-6) and np.allclose(st[:, 4], ref, rtol=2e-4)
    assert min(ref) > 0.5                            # clipped, so the norm reaches every parameter
    pw, pb, vw, vb = tr.tensors()
    for g, w, s0 in zip(list(pw) + list(pb) + list(vw) + list(vb),
                        list(pol.weights) + list(pol.biases) + list(val.weights) + list(val.biases),
                        list(init[0]) + list(init[1]) + list(init[2]) + list(init[3])):
        change = np.abs(w - s0.astype(np.float64)).max()
        assert np.abs(g.astype(np.float64) - w).max() <= 2e-4 * change + 1e-7, (g.shape, np.abs(g - w).max(), change)


@pytest.mark.parametrize("n_envs,T", [(1, 8), (257, 8), (300, 9), (129, 16), (131, 17), (40, 63), (9, 130), (2, 2049)])
def test_gae_rollouts_share_workgroups(n_envs, T):
    """A power of two of threads per rollout, one per eight steps: both sides of its steps, and a last workgroup not full."""
    B, R = _mods()
    print("gae", n_envs, T, flush=True)
    c = synth.ppo_rollout_case(37, T, 4, 4, 0, n_envs=n_envs)
    adv, ret = R.gae(R.dev(c["rewards"]), R.dev(c["values"]), R.dev(c["dones"]), R.dev(c["last_value"]), 0.99, 0.95)
    adv, ret = adv.cpu().numpy(), ret.cpu().numpy()
    for e in range(n_envs):
        a_ref, r_ref = P.gae(c["rewards"][e], c["values"][e], c["dones"][e], c["last_value"][e], 0.99, 0.95)
        scale = max(np.abs(a_ref).max(), np.abs(r_ref).max())
        assert np.abs(adv[e] - a_ref).max() <= 2e-7 * scale + 1e-7
        assert np.abs(ret[e] - r_ref).max() <= 2e-7 * scale + 1e-7


@pytest.mark.parametrize("dims_p,dims_v,batch", [
    ([1024, 64, 5], [1024, 64, 1], 64), ([1040, 40, 5], [1040, 24, 1], 33),       # one block of samples; ranges that end early
    ([2048, 250, 3], [2048, 17, 1], 16), ([3072, 33, 4], [3072, 16, 1], 48),      # two and three rounds of parameters per thread
    ([2560, 256, 18], [2560, 256, 1], 65), ([2560, 256, 18], [2560, 256, 1], 64),  # 256 tiles: up to four blocks of samples
    ([2560, 256, 18], [2560, 256, 1], 256), ([2560, 256, 18], [2560, 256, 1], 257),
    ([1024, 64, 5], [1024, 64, 1], 65), ([3088, 33, 4], [3088, 16, 1], 48),       # either limit passed
    ([48, 7], [48, 1], 16), ([64, 16, 8, 4], [64, 16, 1], 12),
])
def test_update_and_next_first_layer_share_a_launch(dims_p, dims_v, batch):
    """A call per mini-batch never has a next first layer to take along, a call for all of them does: the same bits in
    parameters, both moments and statistics.  (Against the oracle: test_head_update_matches_oracle.)"""
    B, R = _mods()
    T = 4 * batch
    print("ppo", dims_p, dims_v, batch, flush=True)
    c = synth.ppo_rollout_case(41, T, dims_p[0], dims_p[-1], 1)
    pwb, vwb = synth.mlp_params(41, 60, dims_p), synth.mlp_params(41, 80, dims_v)
    args = (R.dev(c["h"]), R.dev(c["actions"]), R.dev(c["logp_old"]), R.dev(synth.normal(41, 90, (T,))),
            R.dev(synth.normal(41, 91, (T,))))
    whole, single = R.PPOTrainer(pwb, vwb), R.PPOTrainer(pwb, vwb)
    stats = whole.update(*args, R.dev(c["perm"]), batch)
    ident = torch.arange(batch, dtype=torch.int32, device="cuda").view(1, batch)
    parts = [single.update(*[x[rows].contiguous() for x in args], ident, batch)
             for rows in R.dev(c["perm"])[0].long().view(4, batch)]
    assert torch.equal(stats, torch.cat(parts))
    for name in ("params", "adam_m", "adam_v"):
        assert torch.equal(getattr(whole, name), getattr(single, name)), name
