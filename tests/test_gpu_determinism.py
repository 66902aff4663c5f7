"""Run-to-run determinism on the GPU: the same rollout + GAE + update from the same buffers, twice.

The environment, the sampler and GAE have no reductions, so state and trajectory must be equal bit for bit.  The
gradient of the networks that take the whole-network training kernel is reduced in a fixed order (the shares inside a
workgroup added in turn through LDS, the per-workgroup copies added in a fixed grouping, the gradient norm as per-block
shares added by a fixed tree),
so their parameters must be equal bit for bit as well, and so are those of the 256-wide fp32 critic, of networks that go layer by
layer and of the bf16 networks (k splits and per-workgroup copies added in a fixed order).  The reported loss statistics of
fused_train_kernel and of the layer-by-layer loss kernel are summed with atomics."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import dev, small

pytestmark = pytest.mark.gpu

TRAJ = ("obs", "action", "logp", "value", "reward", "done", "last_value", "adv", "ret")


def one_run(M, cfg, params0, perm):
    st = M.EnvState(cfg)
    M.env_reset(cfg, st)
    tr = M.Traj(cfg)
    sizes = M.query_sizes(cfg)
    ws_r, ws_u = M.alloc_workspace(sizes.rollout_workspace_bytes), M.alloc_workspace(sizes.update_workspace_bytes)
    p = dev(params0)
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    stats = torch.zeros((cfg["n_epochs"] * cfg["n_minibatches"], 8), device="cuda")
    snaps = []
    for it in range(2):
        M.rollout(cfg, st, p, tr, it * cfg["rollout_len"], ws_r)
        M.compute_gae(cfg, tr)
        torch.cuda.synchronize()
        out = {f: getattr(tr, f).cpu().numpy() for f in TRAJ}
        out.update({"state." + f: x for f, x in st.to_host().items()})
        snaps.append(out)
        M.ppo_update(cfg, tr, p, m, v, it * cfg["n_epochs"] * cfg["n_minibatches"], dev(perm), stats, None, ws_u)
        torch.cuda.synchronize()
        snaps[-1]["stats"] = stats.cpu().numpy().copy()
    return snaps, p.cpu().numpy(), m.cpu().numpy(), v.cpu().numpy(), stats.cpu().numpy()


# (3, 8192): 65 536 critic rows per minibatch, more tiles than the critic's training kernel has workgroups
# (4, 1024): 65 536 rows, 1024 tiles on 512 workgroups
@pytest.mark.parametrize("k,n_envs,kw", [(2, 1024, {}), (3, 512, {}), (3, 8192, {}), (4, 96, {}), (4, 1024, {}), (1, 700, {}), (5, 3000, {}),
                                         (2, 700, dict(actor_hidden=352, critic_hidden=192))])
def test_two_runs_agree(k, n_envs, kw):
    import paper_2107_01460_amd as M
    cfg = small(k, n_envs=n_envs, rollout_len=16, n_minibatches=2, n_epochs=2, **kw)
    print("case", cfg["name"], flush=True)
    params0 = W.init_params(cfg, bias_scale=0.1)
    perm = W.make_perm(cfg)
    a = one_run(M, cfg, params0, perm)
    b = one_run(M, cfg, params0, perm)
    for f in a[0][0]:
        if f != "stats":
            assert np.array_equal(a[0][0][f], b[0][0][f]), f
    for f in a[0][1]:                                  # the second rollout ran under the updated parameters
        if f != "stats":
            assert np.array_equal(a[0][1][f], b[0][1][f]), f
    for x, y, name in zip(a[1:4], b[1:4], ("params", "adam_m", "adam_v")):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32)), name
    assert np.allclose(a[4], b[4], rtol=1e-5, atol=1e-6)
