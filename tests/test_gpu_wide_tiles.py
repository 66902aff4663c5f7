"""Products in tiles of 192 columns (forward ones that come out in fewer rounds, weight gradients of many samples): the gradient of one
large minibatch, which takes them, against the average of the same samples' smaller minibatches, which do not.

Bound: a weight's gradient is a sum over samples of random sign, of standard deviation s; either side adds it in ranges of a few hundred samples
(at most 32 matrix instructions in a row), so its roundings come to about 2^-24 sqrt(32) of s sqrt(samples), the block's scale: 1e-5 of
its largest element leaves a factor of 30 for blocks whose sums cancel to less."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import dev, rel_err

pytestmark = pytest.mark.gpu


# 43 695 x 384 outputs and a 384 x 384 gradient in ranges of 544 samples, the last ragged (layer by layer); 131 076 x 384 gates, their 128 x 384
# gradients, at their line; 49 140 x 768 gates, 256 x 768 gradients
@pytest.mark.parametrize("recurrent,units,n_envs,T,parts", [(0, 384, 2913, 5, 3), (1, 128, 3972, 11, 12), (1, 256, 3276, 5, 6)])
def test_one_minibatch_against_its_parts(recurrent, units, n_envs, T, parts):
    import paper_2107_01460_amd as M
    cfg = W.scaled(W.CONFIGS[1], view=3, n_envs=n_envs, rollout_len=T, actor_hidden=units, critic_hidden=units, episode_cap=4, n_epochs=1,
                   n_minibatches=1, recurrent=recurrent, max_grad_norm=0.0, normalize_adv=0, lr=1e-30)
    print("case", recurrent, units, n_envs, T, flush=True)
    sizes = M.query_sizes(cfg)
    params = dev(W.init_params(cfg, bias_scale=0.2))
    st, tr = M.EnvState(cfg), M.Traj(cfg)
    M.env_reset(cfg, st)
    ws = M.alloc_workspace(sizes.rollout_workspace_bytes)
    rec = M.RecState(cfg) if recurrent else None
    if recurrent:
        M.rollout_recurrent(cfg, st, params, tr, rec, 7, ws)
    else:
        M.rollout(cfg, st, params, tr, 7, ws)
    M.compute_gae(cfg, tr)
    perm = (W.make_env_perm if recurrent else W.make_perm)(cfg, seed=3)

    def last_gradient(n_minibatches, order):
        c = dict(cfg, n_minibatches=n_minibatches)
        p, g, stats = params.clone(), torch.zeros_like(params), torch.zeros((n_minibatches, 8), device="cuda")
        m, v, u = torch.zeros_like(p), torch.zeros_like(p), M.alloc_workspace(M.query_sizes(c).update_workspace_bytes)
        if recurrent:
            M.ppo_update_recurrent(c, tr, rec, p, m, v, 0, dev(order), stats, g, u)
        else:
            M.ppo_update(c, tr, p, m, v, 0, dev(order), stats, g, u)
        torch.cuda.synchronize()
        return g.cpu().numpy().astype(np.float64)

    whole = last_gradient(1, perm)
    share = perm.shape[1] // parts
    mean = sum(last_gradient(parts, np.ascontiguousarray(np.roll(perm, k * share, axis=1))) for k in range(parts)) / parts
    off = 0
    for name, shape in W.param_layout(cfg):
        n = int(np.prod(shape))
        e = rel_err(whole[off:off + n], mean[off:off + n], floor=1.0)
        assert e < 1e-5, (name, e)
        off += n
    assert off == whole.size
