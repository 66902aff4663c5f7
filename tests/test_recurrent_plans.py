"""The recurrent update's plans of its minibatches (row order, state rows, resets, runs): as many as are planned at once, however many there are."""
import numpy as np
import pytest
import torch

import workloads as W


def sizes(**kw):
    import paper_2107_01460_amd as M
    return M.query_sizes(W.scaled(W.CONFIGS[1], recurrent=1, n_envs=1280, rollout_len=128, **kw)).update_workspace_bytes


def test_workspace_does_not_grow_with_the_epochs():
    assert sizes(n_minibatches=4, n_epochs=1) == sizes(n_minibatches=4, n_epochs=2) == sizes(n_minibatches=4, n_epochs=100)


def test_workspace_shrinks_with_the_minibatches():
    """Smaller minibatches, smaller buffers, up to one environment each."""
    by_count = [sizes(n_minibatches=m, n_epochs=2) for m in (1, 2, 4, 32, 64, 320, 1280)]
    assert by_count == sorted(by_count, reverse=True), by_count


def against_the_oracle(orc, cfg, done, order):
    """Statistics and the last minibatch's gradient of an update whose parameters stay, so that every minibatch is by itself."""
    import paper_2107_01460_amd as M
    from gpu_util import REL_TOL, dev, err, load_traj
    from test_gpu_recurrent import load_rec, oracle_rollout
    mb = cfg["n_minibatches"] * cfg["n_epochs"]
    params, _, otr, orec = oracle_rollout(orc, cfg)
    otr.done[:] = done(np.random.default_rng(5), otr.done.shape)
    perm = W.make_env_perm(cfg, seed=3) if order else None
    ostats, ograd = orc.rec_ppo_update(cfg, otr, orec, params.copy(), np.zeros_like(params), np.zeros_like(params), adam_step0=0, perm=perm)
    gtr, grec = load_traj(M, cfg, otr), load_rec(M, cfg, orec)
    ws = M.alloc_workspace(M.query_sizes(cfg).update_workspace_bytes)
    stats, g = torch.zeros((mb, 8), device="cuda"), torch.zeros(params.size, device="cuda")
    M.ppo_update_recurrent(cfg, gtr, grec, dev(params), torch.zeros_like(g), torch.zeros_like(g), 0, dev(perm) if order else None, stats, g, ws)
    torch.cuda.synchronize()
    got = stats.cpu().numpy()
    for i in (0, 1, 2, 5, 6):  # (a minibatch may have twelve samples per step and network: sums small enough to hold to the fp32 bound)
        assert np.all(np.abs(got[:, i] - ostats[:, i]) < REL_TOL[0] * np.maximum(np.abs(ostats[:, i]), 1e-2)), i
    off = 0
    for name, shape in W.param_layout(cfg):
        n = int(np.prod(shape))
        assert err(g.cpu().numpy()[off:off + n], ograd[off:off + n], cfg) < REL_TOL[0], name
        off += n


@pytest.mark.gpu
@pytest.mark.parametrize("order", [True, False])
def test_more_minibatches_than_are_planned_at_once(orc, order):
    cfg = dict(W.CONFIGS[0], n_envs=140, rollout_len=6, actor_hidden=64, critic_hidden=96, episode_cap=4, n_minibatches=70, n_epochs=2,
               recurrent=1, max_grad_norm=0.0, lr=1e-30, central_critic=1)  # two plans of 32 minibatches and one of 6
    against_the_oracle(orc, cfg, lambda rng, shape: rng.random(shape) < 0.3, order)


# Run by run: from 24 steps on (16 above 128 units, whose groups come from a counter), pieces of 64 steps and four of them at a time, episodes
# that end at every step, at a few and at none, at the last step of a piece and at its first; every width's kernels and, in the last case, two networks of which one goes in whole sequences.
@pytest.mark.gpu
@pytest.mark.parametrize("T,n_envs,ha,hc,central,ends", [
    (24, 10, 32, 64, 0, 0.3), (16, 9, 160, 256, 1, 0.4), (33, 10, 32, 64, 0, 0.3), (64, 6, 96, 128, 0, 0.05), (65, 6, 160, 192, 1, 1.0), (129, 5, 224, 256, 0, 0.0), (300, 3, 64, 32, 0, "pieces"),
    (48, 9, 128, 352, 1, 0.1)])
def test_runs(orc, T, n_envs, ha, hc, central, ends):
    cfg = dict(W.CONFIGS[0], n_envs=n_envs, rollout_len=T, actor_hidden=ha, critic_hidden=hc, episode_cap=20, n_minibatches=1, n_epochs=2,
               recurrent=1, max_grad_norm=0.0, lr=1e-30, central_critic=central)
    print("case", T, n_envs, ha, hc, ends, flush=True)

    def done(rng, shape):
        if ends != "pieces":
            return rng.random(shape) < ends
        d = np.zeros(shape, bool)
        d[62::64, 0] = d[63::64, 1] = d[64::64, 2] = True
        return d
    against_the_oracle(orc, cfg, done, True)
