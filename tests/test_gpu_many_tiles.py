"""Whole-network kernels with more row tiles than workgroups, so that a workgroup goes through several: the weights that run on from the
last layer of a tile to the first of the next, the next tile's input requested ahead, per-tile notes and output gradients used again,
sums carried over tiles, a ragged last tile.  Every hidden width (each has its own arrangement of wavefronts).  The gradient cases are
also those whose sample counts make the weight-gradient products take every output tile.
"""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import REL_TOL, TIGHT_TOL_GRAD, dev, err, err_tight, rel_err, tight_cfg
from test_gpu_fullsize import tiled_perm
from test_gpu_parity import oracle_traj
from test_gpu_split_net import reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2107_01460_amd as m
    return m


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


def check_tiled_gradient(M, orc, cs, copies):
    """One minibatch over `copies` copies of a small trajectory in a shuffled order: means over equal copies are the means over one, so
    the loss terms and the gradient are the oracle's on the small one."""
    cf = W.scaled(cs, n_envs=cs["n_envs"] * copies)
    S = cf["n_envs"] * cs["rollout_len"] * cs["n_agents"]
    print("case", cs["actor_hidden"], cs["critic_hidden"], cs["view"], cs["central_critic"], "samples", S, flush=True)
    params0, otr = oracle_traj(orc, cs)
    rng = np.random.default_rng(300)
    params = (params0 + 0.1 * np.abs(params0).mean() * rng.normal(size=params0.size)).astype(np.float32)
    otr.value[:] += (0.2 * rng.normal(size=otr.value.shape)).astype(np.float32)
    otr.logp[:] += rng.choice([-0.4, 0.0, 0.0, 0.4], size=otr.logp.shape).astype(np.float32)
    perm_s = W.make_perm(cs, seed=11)
    # bf16: the oracle mode that rounds the inputs of every product (a ratio on the clip edge may take the other branch in the mode that
    # rounds the weights only)
    po, mo, vo = params.copy(), np.zeros_like(params), np.zeros_like(params)
    ostats, ograd = orc.ppo_update(tight_cfg(cs) or cs, otr, po, mo, vo, adam_step0=0, perm=perm_s)
    gtr = M.Traj(cf)
    for f in ("obs", "action", "logp", "value", "reward", "adv", "ret", "done"):
        src = getattr(otr, f)
        getattr(gtr, f).copy_(torch.from_numpy(np.tile(src, (1, copies) + (1,) * (src.ndim - 2))))
    perm = dev(tiled_perm(cf, cs, perm_s, seed=12))
    gp, gm, gv = dev(params), torch.zeros(params.size, device="cuda"), torch.zeros(params.size, device="cuda")
    stats, gdump = torch.zeros((1, 8), device="cuda"), torch.zeros(params.size, device="cuda")
    M.ppo_update(cf, gtr, gp, gm, gv, 0, perm, stats, gdump, M.alloc_workspace(M.query_sizes(cf).update_workspace_bytes))
    g, st, Pa, tol = gdump.cpu().numpy(), stats.cpu().numpy()[0], orc.actor_param_count(cs), REL_TOL[cs["precision"]]
    if cs["precision"]:
        print("tight gradient", err_tight(g[:Pa], ograd[:Pa], True), err_tight(g[Pa:], ograd[Pa:], True), flush=True)
        assert err_tight(g[:Pa], ograd[:Pa], True) < TIGHT_TOL_GRAD and err_tight(g[Pa:], ograd[Pa:], True) < TIGHT_TOL_GRAD
    else:
        assert err(g[:Pa], ograd[:Pa], cs) < tol and err(g[Pa:], ograd[Pa:], cs) < tol
    for i in (0, 1, 2, 3, 5, 6):
        assert abs(st[i] - ostats[0, i]) < tol * max(abs(ostats[0, i]), 1e-2), (i, st[i], ostats[0, i])
    assert st[7] == 0


# 3 agents x 7 environments x 5 steps, 643 times: 67 515 samples = 2109 tiles of 32 rows and 27 (up to 2048 workgroups), 1054 of 64 and 59
# (up to 1024).  64 and 128 units: with inputs wider than the whole-minibatch kernel takes.
SMALL = dict(n_agents=3, n_envs=7, rollout_len=5, n_epochs=1, n_minibatches=1, max_grad_norm=0.0, episode_cap=4)


@pytest.mark.parametrize("ha,hc", [(32, 64), (64, 96), (96, 32), (128, 160), (160, 128), (192, 224), (224, 256), (256, 192), (288, 320), (320, 288)])
def test_fp32_gradient(M, orc, ha, hc):
    check_tiled_gradient(M, orc, W.scaled(W.CONFIGS[1], actor_hidden=ha, critic_hidden=hc, view=7, **SMALL), 643)


# weight gradients whose rows are read 16 bytes at a time (300 inputs: of a central critic of four agents), and one-row gathers
@pytest.mark.parametrize("ha,hc,agents,view", [(192, 96, 4, 5), (96, 256, 4, 5), (64, 320, 2, 7)])
def test_fp32_gradient_central(M, orc, ha, hc, agents, view):
    cs = W.scaled(W.CONFIGS[1], actor_hidden=ha, critic_hidden=hc, view=view, central_critic=1, **dict(SMALL, n_agents=agents))
    check_tiled_gradient(M, orc, cs, 1929)


# 4275 samples 16 times: 1068 tiles of 64 rows and 48.  (A power of two of copies: the gradients that are rounded to bf16 are the small
# minibatch's times one, and round alike.  The comparison's bound holds from about a thousand samples on.)
@pytest.mark.parametrize("ha,hc", [(64, 128), (128, 64), (192, 256), (256, 192), (320, 384), (384, 448), (448, 512), (512, 320)])
def test_bf16_gradient(M, orc, ha, hc):
    cs = W.scaled(W.CONFIGS[3], actor_hidden=ha, critic_hidden=hc, view=7, **dict(SMALL, n_envs=95, rollout_len=15))
    check_tiled_gradient(M, orc, cs, 16)


def forward(M, cfg, params, obs, ws):
    n = obs.shape[0]
    logits, value = torch.empty((n, 4, 6), device="cuda"), torch.empty((n, 4), device="cuda")
    M.policy_forward(cfg, params, obs.contiguous(), n, logits, value, ws)
    return logits, value


# 4 x 35 003 samples: 2187 tiles of 64 rows and 44; beside them, calls of few enough rows that every tile has a workgroup of its own
@pytest.mark.parametrize("precision,ha,hc,view", [
    (0, 32, 64, 5), (0, 96, 128, 7), (0, 160, 192, 5), (0, 224, 256, 7), (0, 288, 320, 3), (0, 256, 160, 5),
    (1, 64, 128, 7), (1, 192, 256, 5), (1, 320, 384, 7), (1, 448, 512, 5)])
def test_forward(M, precision, ha, hc, view):
    rows = 35003
    cfg = W.scaled(W.CONFIGS[3], precision=precision, actor_hidden=ha, critic_hidden=hc, view=view, n_agents=4, n_envs=rows, rollout_len=1,
                   n_minibatches=1)
    print("case", precision, ha, hc, view, flush=True)
    D = W.obs_dim(cfg)
    gen = torch.Generator(device="cuda").manual_seed(6)
    obs = torch.randint(-2, 8, (rows, 4, D), device="cuda", generator=gen) * 0.5
    # a stretch of tiles with values that are not exact in bf16, between others: what a tile notes does not reach the next one
    obs[3000:3100:7] = torch.randn((15, 4, D), device="cuda", generator=gen)
    obs[20000::5] = torch.randn((rows - 20000 + 4) // 5, 4, D, device="cuda", generator=gen)
    params = dev(W.init_params(cfg, bias_scale=0.2))
    ws = M.alloc_workspace(M.query_sizes(cfg).rollout_workspace_bytes)
    logits, value = forward(M, cfg, params, obs, ws)
    for first in range(0, rows, 5000):
        l, v = forward(M, cfg, params, obs[first:first + 5000], ws)
        assert torch.equal(l, logits[first:first + 5000]) and torch.equal(v, value[first:first + 5000]), first
    if precision == 0:
        n_actor = D * ha + ha + ha * ha + ha + 6 * ha + 6
        some = slice(1, rows, 41)
        assert rel_err(logits[some].cpu(), reference(obs[some].reshape(-1, D), params[:n_actor], D, ha, 6)) < REL_TOL[0]
        assert rel_err(value[some].cpu(), reference(obs[some].reshape(-1, D), params[n_actor:], D, hc, 1)) < REL_TOL[0]
