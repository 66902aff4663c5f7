"""Parity of the recurrent (GRU) IPPO / MAPPO path against the oracle: teacher-forced rollout with hidden states
carried over episode boundaries, sequence-minibatch gradient (back-propagation through time), optimiser loop."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import REL_TOL, dev, err, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2107_01460_amd as m
    return m


def rec_cfg(kind, **kw):
    if kind == "ippo":
        base = dict(W.CONFIGS[0], n_envs=42, rollout_len=11, actor_hidden=64, critic_hidden=64, episode_cap=5,
                    n_minibatches=1, n_epochs=1, recurrent=1)
    else:
        base = dict(W.CONFIGS[2], n_envs=36, rollout_len=9, actor_hidden=128, critic_hidden=128, episode_cap=4,
                    n_minibatches=1, n_epochs=1, recurrent=1)
    base.update(kw)
    return base


def oracle_rollout(orc, cfg, seed=1):
    params = W.init_params(cfg, bias_scale=0.2)
    s = orc.EnvState(cfg)
    orc.env_reset(cfg, s)
    tr, rec = orc.Traj(cfg), orc.RecState(cfg)
    rng = np.random.default_rng(seed)
    rec.ha0[:] = 0.3 * rng.normal(size=rec.ha0.shape)
    rec.hc0[:] = 0.3 * rng.normal(size=rec.hc0.shape)
    orc.rec_rollout(cfg, s, params, tr, rec, step_offset=300)
    orc.compute_gae(cfg, tr)
    return params, s, tr, rec


def load_rec(M, cfg, orec):
    g = M.RecState(cfg)
    g.ha0.copy_(dev(orec.ha0))
    g.hc0.copy_(dev(orec.hc0))
    return g


@pytest.mark.parametrize("kind", ["ippo", "mappo"])
def test_recurrent_rollout_teacher_forced(M, orc, kind):
    cfg = rec_cfg(kind)
    print("case", kind, cfg["n_envs"], cfg["rollout_len"], flush=True)
    params, os_, otr, orec = oracle_rollout(orc, cfg)
    gs = M.EnvState(cfg)
    M.env_reset(cfg, gs)
    gtr = M.Traj(cfg, debug=True)
    grec = load_rec(M, cfg, orec)
    ws = M.alloc_workspace(M.query_sizes(cfg).rollout_workspace_bytes)
    M.rollout_recurrent(cfg, gs, dev(params), gtr, grec, 300, ws, forced_actions=dev(otr.action))
    torch.cuda.synchronize()
    tol = REL_TOL[0]
    assert np.array_equal(gtr.obs.cpu().numpy(), otr.obs)
    assert np.array_equal(gtr.reward.cpu().numpy().view(np.uint32), otr.reward.view(np.uint32))
    assert np.array_equal(gtr.done.cpu().numpy(), otr.done)
    assert otr.done[:-1].sum() > 0
    host = gs.to_host()
    for f in M.EnvState.FIELDS:
        assert np.array_equal(host[f], getattr(os_, f)), f
    assert err(gtr.logits.cpu().numpy(), otr.logits, cfg) < tol
    assert err(gtr.value.cpu().numpy(), otr.value, cfg) < tol
    assert err(gtr.last_value.cpu().numpy(), otr.last_value, cfg) < tol
    assert err(gtr.logp.cpu().numpy(), otr.logp, cfg) < tol
    assert err(grec.ha1.cpu().numpy(), orec.ha1, cfg) < tol
    assert err(grec.hc1.cpu().numpy(), orec.hc1, cfg) < tol
    ended_last = otr.done[-1].astype(bool)
    assert np.all(grec.ha1.cpu().numpy()[ended_last] == 0)
    mism = gtr.sampled.cpu().numpy() != otr.sampled
    lim = 1e-5 + 2e-4 * np.abs(otr.logits).max()
    assert np.all(otr.gap[mism] < lim) and mism.mean() < 5e-3


@pytest.mark.parametrize("kind,clipv", [("ippo", 0), ("mappo", 0), ("mappo", 1)])
def test_recurrent_sequence_gradient(M, orc, kind, clipv):
    cfg = rec_cfg(kind, clip_value=clipv, max_grad_norm=0.0)
    print("case", kind, clipv, flush=True)
    params0, _, otr, orec = oracle_rollout(orc, cfg)
    rng = np.random.default_rng(21)
    params = (params0 + 0.05 * np.abs(params0).mean() * rng.normal(size=params0.size)).astype(np.float32)
    otr.value[:] += (0.2 * rng.normal(size=otr.value.shape)).astype(np.float32)
    otr.logp[:] += rng.choice([-0.4, 0.0, 0.0, 0.4], size=otr.logp.shape).astype(np.float32)
    perm = W.make_env_perm(cfg, seed=3)
    po, mo, vo = params.copy(), np.zeros_like(params), np.zeros_like(params)
    ostats, ograd = orc.rec_ppo_update(cfg, otr, orec, po, mo, vo, adam_step0=0, perm=perm)
    from gpu_util import load_traj
    gtr = load_traj(M, cfg, otr)
    grec = load_rec(M, cfg, orec)
    ws = M.alloc_workspace(M.query_sizes(cfg).update_workspace_bytes)
    gp, gm, gv = dev(params), torch.zeros(params.size, device="cuda"), torch.zeros(params.size, device="cuda")
    stats = torch.zeros((1, 8), device="cuda")
    gdump = torch.zeros(params.size, device="cuda")
    M.ppo_update_recurrent(cfg, gtr, grec, gp, gm, gv, 0, dev(perm), stats, gdump, ws)
    torch.cuda.synchronize()
    tol = REL_TOL[0]
    g = gdump.cpu().numpy()
    off = 0
    for name, shape in W.param_layout(cfg):          # block by block, so that a wrong block names itself
        n = int(np.prod(shape))
        assert err(g[off:off + n], ograd[off:off + n], cfg) < tol, name
        off += n
    st = stats.cpu().numpy()[0]
    assert 0.0 < ostats[0, 4] < 1.0
    for i in (0, 1, 2, 3, 5, 6):
        assert abs(st[i] - ostats[0, i]) < tol * max(abs(ostats[0, i]), 1e-2), (i, st[i], ostats[0, i])
    assert st[7] == 0
    pa, ma, va = params.copy(), np.zeros_like(params), np.zeros_like(params)
    orc.adam_step(cfg, pa, ma, va, g.astype(np.float64), 1)
    assert rel_err(gm.cpu().numpy(), ma) < 1e-5 and rel_err(gv.cpu().numpy(), va) < 1e-5
    assert rel_err(gp.cpu().numpy() - params, pa - params) < 1e-3


@pytest.mark.parametrize("kind", ["ippo", "mappo"])
def test_recurrent_update_epochs_and_minibatches(M, orc, kind):
    cfg = rec_cfg(kind, n_epochs=2, n_minibatches=3)
    params, _, otr, orec = oracle_rollout(orc, cfg)
    perm = W.make_env_perm(cfg, seed=9)
    po, mo, vo = params.copy(), np.zeros_like(params), np.zeros_like(params)
    ostats, ograd = orc.rec_ppo_update(cfg, otr, orec, po, mo, vo, adam_step0=2, perm=perm)
    from gpu_util import load_traj
    gtr = load_traj(M, cfg, otr)
    grec = load_rec(M, cfg, orec)
    ws = M.alloc_workspace(M.query_sizes(cfg).update_workspace_bytes)
    gp, gm, gv = dev(params), torch.zeros(params.size, device="cuda"), torch.zeros(params.size, device="cuda")
    stats = torch.zeros((6, 8), device="cuda")
    gdump = torch.zeros(params.size, device="cuda")
    M.ppo_update_recurrent(cfg, gtr, grec, gp, gm, gv, 2, dev(perm), stats, gdump, ws)
    torch.cuda.synchronize()
    tol = REL_TOL[0]
    st = stats.cpu().numpy()
    for i in (0, 1, 2, 5, 6):
        assert np.all(np.abs(st[:, i] - ostats[:, i]) < 20 * tol * np.maximum(np.abs(ostats[:, i]), 1e-2)), (i, st[:, i], ostats[:, i])
    assert np.all(st[:, 7] == 0)
    assert rel_err(gp.cpu().numpy() - params, po - params, floor=1.0) < 0.05
    assert err(gdump.cpu().numpy(), ograd, cfg) < 100 * tol
    # identity order when perm is NULL
    gp2, gm2, gv2 = dev(params), torch.zeros_like(gm), torch.zeros_like(gm)
    M.ppo_update_recurrent(cfg, gtr, grec, gp2, gm2, gv2, 2, None, stats, None, ws)
    po2, mo2, vo2 = params.copy(), np.zeros_like(params), np.zeros_like(params)
    orc.rec_ppo_update(cfg, otr, orec, po2, mo2, vo2, adam_step0=2, perm=None)
    assert rel_err(gp2.cpu().numpy() - params, po2 - params, floor=1.0) < 0.05


def test_recurrent_full_size(M, orc):
    """The recurrent path at the size and launch configuration the benchmark times (workload 3 with GRU networks):
    the rollout is checked on its first environments, re-simulated by the oracle with the GPU's actions and hidden
    start states; the update through the tiling property (K copies of a small oracle trajectory along the
    environment axis, environment order such that every minibatch holds K copies of the small one's sequences)."""
    from gpu_util import load_traj
    cfg = W.scaled(W.CONFIGS[2], recurrent=1, n_epochs=2)
    N, A, T, Mb, E = cfg["n_envs"], cfg["n_agents"], cfg["rollout_len"], cfg["n_minibatches"], cfg["n_epochs"]
    n_s = 8
    K = N // n_s
    cs = W.scaled(cfg, n_envs=n_s)
    tol = REL_TOL[0]
    params = W.init_params(cs, bias_scale=0.1)
    rng = np.random.default_rng(77)

    # ---- rollout at full size, first n_s environments against the oracle
    orec = orc.RecState(cs)
    orec.ha0[:] = 0.3 * rng.normal(size=orec.ha0.shape)
    orec.hc0[:] = 0.3 * rng.normal(size=orec.hc0.shape)
    gs = M.EnvState(cfg)
    M.env_reset(cfg, gs)
    gtr = M.Traj(cfg)
    grec = M.RecState(cfg)
    grec.ha0.copy_(dev(np.tile(orec.ha0, (K, 1, 1))))
    grec.hc0.copy_(dev(np.tile(orec.hc0, (K, 1))))
    sizes = M.query_sizes(cfg)
    ws = M.alloc_workspace(sizes.rollout_workspace_bytes)
    M.rollout_recurrent(cfg, gs, dev(params), gtr, grec, 900, ws)
    torch.cuda.synchronize()
    os_ = orc.EnvState(cs)
    orc.env_reset(cs, os_)
    otr = orc.Traj(cs)
    orc.rec_rollout(cs, os_, params, otr, orec, step_offset=900, forced_actions=gtr.action[:, :n_s].cpu().numpy())
    assert np.array_equal(gtr.obs[:, :n_s].cpu().numpy(), otr.obs)
    assert np.array_equal(gtr.done[:, :n_s].cpu().numpy(), otr.done)
    assert np.array_equal(gtr.reward[:, :n_s].cpu().numpy().view(np.uint32), otr.reward.view(np.uint32))
    assert err(gtr.logp[:, :n_s].cpu().numpy(), otr.logp, cfg) < tol
    assert err(gtr.value[:, :n_s].cpu().numpy(), otr.value, cfg) < tol
    assert err(gtr.last_value[:n_s].cpu().numpy(), otr.last_value, cfg) < tol
    assert err(grec.ha1[:n_s].cpu().numpy(), orec.ha1, cfg) < tol
    assert err(grec.hc1[:n_s].cpu().numpy(), orec.hc1, cfg) < tol
    del gtr, ws

    # ---- update: the oracle's small trajectory tiled K times
    orc.compute_gae(cs, otr)
    p2 = (params + 0.05 * np.abs(params).mean() * rng.normal(size=params.size)).astype(np.float32)
    otr.value[:] += (0.2 * rng.normal(size=otr.value.shape)).astype(np.float32)
    otr.logp[:] += rng.choice([-0.4, 0.0, 0.0, 0.4], size=otr.logp.shape).astype(np.float32)
    perm_s = W.make_env_perm(cs, seed=4)
    per_mb = n_s // Mb
    perm_f = np.empty((E, N), np.int32)
    for e in range(E):
        parts = []
        for m in range(Mb):
            envs = perm_s[e, m * per_mb:(m + 1) * per_mb].astype(np.int64)
            full = (envs[None, :] + (np.arange(K, dtype=np.int64) * n_s)[:, None]).reshape(-1)
            rng.shuffle(full)
            parts.append(full)
        perm_f[e] = np.concatenate(parts)
    assert np.array_equal(np.sort(perm_f[0]), np.arange(N))
    gtr = M.Traj(cfg)
    for f in ("obs", "action", "logp", "value", "reward", "adv", "ret"):
        src = getattr(otr, f)
        getattr(gtr, f).copy_(torch.from_numpy(np.tile(src, (1, K) + (1,) * (src.ndim - 2))))
    gtr.done.copy_(torch.from_numpy(np.tile(otr.done, (1, K))))
    gtr.last_value.copy_(torch.from_numpy(np.tile(otr.last_value, (K, 1))))
    wsu = M.alloc_workspace(sizes.update_workspace_bytes)
    # (A) a step size too small to move any parameter: every minibatch at the same parameters, tight bounds
    tiny = dict(n_epochs=1, lr=1e-30, max_grad_norm=0.0)
    po, mo, vo = p2.copy(), np.zeros_like(p2), np.zeros_like(p2)
    ostats, ograd = orc.rec_ppo_update(dict(cs, **tiny), otr, orec, po, mo, vo, adam_step0=0, perm=perm_s[:1])
    gp, gm, gv = dev(p2), torch.zeros(p2.size, device="cuda"), torch.zeros(p2.size, device="cuda")
    stats = torch.zeros((Mb, 8), device="cuda")
    gdump = torch.zeros(p2.size, device="cuda")
    M.ppo_update_recurrent(dict(cfg, **tiny), gtr, grec, gp, gm, gv, 0, dev(perm_f[:1]), stats, gdump, wsu)
    torch.cuda.synchronize()
    assert np.array_equal(gp.cpu().numpy(), p2)
    g = gdump.cpu().numpy()
    # Block by block.  The tiled minibatch is the hardest case fp32 summation can be given: the 2048 copies of one
    # (step, environment) sample sit next to each other, so every partial sum of a weight gradient is 2048 equal
    # terms, the partial sums of different time steps cancel to a result a thousand times smaller, and the rounding
    # of the running sums (about 2^-24 of THEIR size, in whatever order the atomics land) no longer vanishes against
    # it.  Measured: the error grows with the number of copies, not with T, and stays below 1.5e-5 of a block's
    # largest element; at up to 128 copies the same comparison holds the 1e-4 bound of the small cases.  So the
    # full-size bound is on the scale of each block: 5e-5 of its largest element.
    off = 0
    worst = 0.0
    for name, shape in W.param_layout(cs):
        n = int(np.prod(shape))
        e_blk = rel_err(g[off:off + n], ograd[off:off + n], floor=1.0)
        worst = max(worst, e_blk)
        assert e_blk < 5e-5, (name, e_blk)
        off += n
    print("worst gradient block error relative to the block's scale", worst, flush=True)
    st = stats.cpu().numpy()
    for i in (0, 1, 2, 3, 5, 6):
        assert np.all(np.abs(st[:, i] - ostats[:, i]) < tol * np.maximum(np.abs(ostats[:, i]), 1e-2)), (i, st[:, i], ostats[:, i])
    assert np.all(st[:, 7] == 0)
    # (B) E epochs x M minibatches with the configuration's step size and clipping
    po, mo, vo = p2.copy(), np.zeros_like(p2), np.zeros_like(p2)
    ostats, ograd = orc.rec_ppo_update(cs, otr, orec, po, mo, vo, adam_step0=0, perm=perm_s)
    gp, gm, gv = dev(p2), torch.zeros(p2.size, device="cuda"), torch.zeros(p2.size, device="cuda")
    stats = torch.zeros((E * Mb, 8), device="cuda")
    M.ppo_update_recurrent(cfg, gtr, grec, gp, gm, gv, 0, dev(perm_f), stats, gdump, wsu)
    torch.cuda.synchronize()
    st = stats.cpu().numpy()
    for i in (0, 1, 2, 5, 6):
        assert np.all(np.abs(st[:, i] - ostats[:, i]) < 20 * tol * np.maximum(np.abs(ostats[:, i]), 1e-2)), (i, st[:, i], ostats[:, i])
    assert np.all(st[:, 7] == 0)
    assert rel_err(gp.cpu().numpy() - p2, po - p2, floor=1.0) < 0.05


# Widths on both sides of every change of kernel (weights in registers up to 128, streamed up to 256, one step at a time
# above), with sample counts that leave ragged tiles, and both tile heights (32 sequences above 4096 per step).
@pytest.mark.parametrize("ha,hc,n_envs,T", [(32, 160, 11, 7), (96, 192, 23, 5), (224, 128, 9, 6), (256, 288, 7, 5),
                                            (320, 64, 10, 4), (64, 96, 1367, 3), (128, 32, 1371, 3), (32, 256, 1366, 3)])
def test_recurrent_other_widths(M, orc, ha, hc, n_envs, T):
    from gpu_util import load_traj
    cfg = dict(W.CONFIGS[1], n_envs=n_envs, rollout_len=T, actor_hidden=ha, critic_hidden=hc, episode_cap=2, n_minibatches=1,
               n_epochs=1, recurrent=1, max_grad_norm=0.0)
    print("case", ha, hc, n_envs, T, flush=True)
    params, _, otr, orec = oracle_rollout(orc, cfg)
    sizes = M.query_sizes(cfg)
    gs = M.EnvState(cfg)
    M.env_reset(cfg, gs)
    gtr = M.Traj(cfg, debug=True)
    grec = load_rec(M, cfg, orec)
    M.rollout_recurrent(cfg, gs, dev(params), gtr, grec, 300, M.alloc_workspace(sizes.rollout_workspace_bytes),
                        forced_actions=dev(otr.action))
    tol = REL_TOL[0]
    assert otr.done[:-1].sum() > 0
    for name in ("logits", "value", "last_value"):
        assert err(getattr(gtr, name).cpu().numpy(), getattr(otr, name), cfg) < tol, name
    assert err(grec.ha1.cpu().numpy(), orec.ha1, cfg) < tol and err(grec.hc1.cpu().numpy(), orec.hc1, cfg) < tol
    perm = W.make_env_perm(cfg, seed=3)
    po, mo, vo = params.copy(), np.zeros_like(params), np.zeros_like(params)
    ostats, ograd = orc.rec_ppo_update(cfg, otr, orec, po, mo, vo, adam_step0=0, perm=perm)
    gtr = load_traj(M, cfg, otr)
    gp, gm, gv = dev(params), torch.zeros(params.size, device="cuda"), torch.zeros(params.size, device="cuda")
    stats, gdump = torch.zeros((1, 8), device="cuda"), torch.zeros(params.size, device="cuda")
    M.ppo_update_recurrent(cfg, gtr, grec, gp, gm, gv, 0, dev(perm), stats, gdump, M.alloc_workspace(sizes.update_workspace_bytes))
    torch.cuda.synchronize()
    g = gdump.cpu().numpy()
    off = 0
    for name, shape in W.param_layout(cfg):
        n = int(np.prod(shape))
        assert err(g[off:off + n], ograd[off:off + n], cfg) < tol, name
        off += n
    st = stats.cpu().numpy()[0]
    for i in (0, 1, 2, 5, 6):
        assert abs(st[i] - ostats[0, i]) < tol * max(abs(ostats[0, i]), 1e-2), (i, st[i], ostats[0, i])


# The runs between episodes' beginnings that the update goes through: one-step runs, none but whole sequences, runs of many lengths, more
# sequences than a workgroup of the plan has threads, runs beyond the lengths that are told apart, and rollouts of one step.
@pytest.mark.parametrize("n_envs,T,density,central,mb,width", [
    (42, 11, 1.0, 0, 1, 64), (42, 11, 0.0, 1, 1, 64), (36, 33, 0.1, 0, 2, 128), (600, 5, 0.3, 1, 2, 64), (600, 1, 0.5, 0, 1, 64),
    (2, 1100, 0.002, 1, 1, 64), (34, 40, 0.15, 0, 2, 160)])
def test_recurrent_runs(M, orc, n_envs, T, density, central, mb, width):
    from gpu_util import load_traj
    cfg = dict(W.CONFIGS[0], n_envs=n_envs, rollout_len=T, actor_hidden=width, critic_hidden=width, episode_cap=50, n_minibatches=mb,
               n_epochs=1, recurrent=1, max_grad_norm=0.0, lr=1e-30, central_critic=central)
    print("case", n_envs, T, density, central, mb, width, flush=True)
    params, _, otr, orec = oracle_rollout(orc, cfg)
    rng = np.random.default_rng(5)
    otr.done[:] = rng.random(otr.done.shape) < density  # any flags: the update takes the trajectory as it is
    perm = W.make_env_perm(cfg, seed=3)
    po, mo, vo = params.copy(), np.zeros_like(params), np.zeros_like(params)
    ostats, ograd = orc.rec_ppo_update(cfg, otr, orec, po, mo, vo, adam_step0=0, perm=perm)
    gtr, grec = load_traj(M, cfg, otr), load_rec(M, cfg, orec)
    ws = M.alloc_workspace(M.query_sizes(cfg).update_workspace_bytes)
    gp, gm, gv = dev(params), torch.zeros(params.size, device="cuda"), torch.zeros(params.size, device="cuda")
    stats, gdump = torch.zeros((mb, 8), device="cuda"), torch.zeros(params.size, device="cuda")
    M.ppo_update_recurrent(cfg, gtr, grec, gp, gm, gv, 0, dev(perm), stats, gdump, ws)
    torch.cuda.synchronize()
    g = gdump.cpu().numpy()
    off = 0
    for name, shape in W.param_layout(cfg):
        n = int(np.prod(shape))
        assert err(g[off:off + n], ograd[off:off + n], cfg) < REL_TOL[0], name
        off += n
