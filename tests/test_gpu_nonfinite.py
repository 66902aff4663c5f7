"""Weights, observations and states that are infinite, or finite but beyond the largest bf16 value: the products on split bf16
operands have to give what a product of fp32 values gives -- a saturated tanh, an infinity, a NaN only where infinity meets
zero or its opposite.  The oracle, in fp64, is the reference for which values are NaN and for the others.
"""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import REL_TOL, dev, err, load_traj

pytestmark = pytest.mark.gpu

INF, BIG = np.float32(np.inf), np.float32(3.4e38)  # BIG: finite, rounds to infinity in bf16


@pytest.fixture(scope="module")
def M():
    import paper_2107_01460_amd as m
    return m


def with_weights(cfg, params, changes):
    p, off = params.copy(), 0
    for name, shape in W.param_layout(cfg):
        n = int(np.prod(shape))
        for block, index, v in changes:
            if block == name:
                p[off:off + n].reshape(shape)[index] = v
        off += n
    return p


def check(got, ref, cfg, name):
    """NaN in the same places, the finite values of the others within the tolerance of every parity test."""
    got, ref = np.asarray(got, np.float64).ravel(), np.asarray(ref, np.float64).ravel()
    assert np.array_equal(np.isnan(got), np.isnan(ref)), (name, np.isnan(got).mean(), np.isnan(ref).mean())
    ok = ~np.isnan(ref)
    assert np.array_equal(np.isinf(got[ok]), np.isinf(ref[ok])), name
    ok &= np.isfinite(ref)
    assert not ok.any() or err(got[ok], ref[ok], cfg) < REL_TOL[0], name


def finite_losses(tr):
    """Advantages, returns and old log-probabilities that do not depend on the (possibly NaN) forward pass."""
    rng = np.random.default_rng(5)
    tr.value[:] = rng.normal(size=tr.value.shape)
    tr.ret[:] = tr.value + 0.3 * rng.normal(size=tr.value.shape)
    tr.adv[:] = rng.normal(size=tr.adv.shape)
    tr.logp[:] = -1.8


FEED_FORWARD = {
    "w2_inf": [("actor.W2", (5, 7), INF), ("actor.W2", (9, 3), -INF), ("critic.W2", (5, 7), INF)],
    "w2_big": [("actor.W2", (5, 7), BIG), ("critic.W2", (11, 2), -BIG)],
    "w1_big": [("actor.W1", (4, 7), BIG), ("critic.W1", (7, 9), -BIG)],
    "w1_last_row_inf": [("actor.W1", (-1, 7), INF), ("critic.W1", (-1, 9), -INF)],
}


# the kernels of 64 and 128 units, the whole-network kernels of other widths up to 320, and the layer-by-layer products above
@pytest.mark.parametrize("key", sorted(FEED_FORWARD))
@pytest.mark.parametrize("ha,hc,central", [(128, 64, 0), (64, 256, 1), (192, 128, 0), (352, 512, 0)])
def test_feed_forward(M, orc, ha, hc, central, key):
    cfg = dict(W.CONFIGS[1], n_envs=30, rollout_len=5, n_minibatches=1, n_epochs=1, actor_hidden=ha, critic_hidden=hc,
               central_critic=central, max_grad_norm=0.0)
    print("case", ha, hc, central, key, flush=True)
    params = with_weights(cfg, W.init_params(cfg, bias_scale=0.1), FEED_FORWARD[key])
    sizes = M.query_sizes(cfg)
    forced = W.random_actions(cfg, cfg["rollout_len"], 3)
    s = orc.EnvState(cfg)
    orc.env_reset(cfg, s)
    otr = orc.Traj(cfg)
    with np.errstate(all="ignore"):
        orc.rollout(cfg, s, params, otr, step_offset=0, forced_actions=forced)
    gs, gtr = M.EnvState(cfg), M.Traj(cfg, debug=True)
    M.env_reset(cfg, gs)
    M.rollout(cfg, gs, dev(params), gtr, 0, M.alloc_workspace(sizes.rollout_workspace_bytes), forced_actions=dev(forced))
    assert key != "w2_inf" or np.isfinite(otr.logits).all()   # infinite, yet every unit behind it saturates
    for name in ("logits", "value", "last_value"):
        check(getattr(gtr, name).cpu().numpy(), getattr(otr, name), cfg, name)
    finite_losses(otr)
    po, mo, vo = params.copy(), np.zeros_like(params), np.zeros_like(params)
    _, ograd = orc.ppo_update(cfg, otr, po, mo, vo, adam_step0=0, perm=None)
    gtr = load_traj(M, cfg, otr)
    gp, gm, gv = dev(params), torch.zeros(params.size, device="cuda"), torch.zeros(params.size, device="cuda")
    stats, g = torch.zeros((1, 8), device="cuda"), torch.zeros(params.size, device="cuda")
    M.ppo_update(cfg, gtr, gp, gm, gv, 0, None, stats, g, M.alloc_workspace(sizes.update_workspace_bytes))
    off = 0
    for name, shape in W.param_layout(cfg):
        n = int(np.prod(shape))
        check(g[off:off + n].cpu().numpy(), ograd[off:off + n], cfg, name)
        off += n


# rows of the caller's own: small and large calls (they may take different kernels), the padding of the last input column
@pytest.mark.parametrize("ha,hc,rows", [(128, 64, 40), (128, 256, 900), (96, 64, 40), (384, 352, 40)])
def test_observations(M, orc, ha, hc, rows):
    cfg = dict(W.CONFIGS[1], n_envs=rows, rollout_len=1, n_minibatches=1, n_epochs=1, actor_hidden=ha, critic_hidden=hc)
    print("case", ha, hc, rows, flush=True)
    params = W.init_params(cfg, bias_scale=0.1)
    A, D = cfg["n_agents"], W.obs_dim(cfg)
    obs = (0.5 + np.random.default_rng(1).integers(0, 4, size=(rows, A, D))).astype(np.float32)
    obs[3, 0, 4], obs[5, 1, -1], obs[7, 2, 0], obs[rows - 1, 2, -1] = INF, -INF, BIG, -BIG
    ws = M.alloc_workspace(M.query_sizes(cfg).rollout_workspace_bytes)
    logits, value = torch.empty((rows, A, 6), device="cuda"), torch.empty((rows, A), device="cuda")
    M.policy_forward(cfg, dev(params), dev(obs), rows, logits, value, ws)
    ol, ov = orc.policy_forward(cfg, params, obs)
    assert np.isfinite(ol).all() and np.isfinite(ov).all()
    check(logits.cpu().numpy(), ol, cfg, "logits")
    check(value.cpu().numpy(), ov, cfg, "value")


RECURRENT = {
    "wh_inf": [("actor.Wh", (5, 7), INF), ("critic.Wh", (5, 7), -INF)],
    "wi_inf": [("actor.Wi", (5, 7), INF), ("critic.Wi", (6, 30), -INF)],
    "wh_big": [("actor.Wh", (5, 7), BIG), ("critic.Wh", (5, 30), -BIG)],
    "h0": [],
}


# weights of the cell in registers, streamed, and one step at a time; states that start out of range
@pytest.mark.parametrize("key", sorted(RECURRENT))
@pytest.mark.parametrize("ha,hc", [(128, 192), (320, 64)])
def test_recurrent(M, orc, ha, hc, key):
    cfg = dict(W.CONFIGS[1], n_envs=21, rollout_len=5, n_minibatches=1, n_epochs=1, actor_hidden=ha, critic_hidden=hc, recurrent=1,
               max_grad_norm=0.0)
    print("case", ha, hc, key, flush=True)
    params = with_weights(cfg, W.init_params(cfg, bias_scale=0.1), RECURRENT[key])
    sizes = M.query_sizes(cfg)
    forced = W.random_actions(cfg, cfg["rollout_len"], 3)
    s = orc.EnvState(cfg)
    orc.env_reset(cfg, s)
    otr, orec = orc.Traj(cfg), orc.RecState(cfg)
    rng = np.random.default_rng(2)
    orec.ha0[:] = 0.3 * rng.normal(size=orec.ha0.shape)
    orec.hc0[:] = 0.3 * rng.normal(size=orec.hc0.shape)
    if key == "h0":
        orec.ha0[2, 1, 3], orec.ha0[4, 0, 5], orec.hc0[3, 2, 1] = INF, BIG, -BIG
    orc.rec_rollout(cfg, s, params, otr, orec, step_offset=0, forced_actions=forced)
    gs, gtr, grec = M.EnvState(cfg), M.Traj(cfg, debug=True), M.RecState(cfg)
    M.env_reset(cfg, gs)
    grec.ha0.copy_(dev(orec.ha0))
    grec.hc0.copy_(dev(orec.hc0))
    M.rollout_recurrent(cfg, gs, dev(params), gtr, grec, 0, M.alloc_workspace(sizes.rollout_workspace_bytes), forced_actions=dev(forced))
    for name in ("logits", "value", "last_value"):
        check(getattr(gtr, name).cpu().numpy(), getattr(otr, name), cfg, name)
