"""The whole-minibatch training kernel of 64 and 128 units on observations that are not all exact in bf16: every tile in its second
form, workgroups that change to it after exact tiles, both networks in one launch; every input width it pads differently (27 of 32
columns; 54, 75 and 81 of 96, the first in two k blocks), a ragged last tile.
"""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import REL_TOL, dev, err
from test_gpu_many_tiles import SMALL
from test_gpu_parity import oracle_traj

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2107_01460_amd as m
    return m


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


# Tiles: three agents 1500 times 4922; central critics of two agents (3001 times) 3283 and of three (1800 times) 1969, their actors twice and
# three times as many.  Workgroups: 512 of 128 units, 1024 of 64 with 27 inputs, 768 with more; each goes through at least three tiles.
# "last": the last fifth of them in the second form; "early": all but the first fifth, so that most workgroups change after their first tile
# and take several in the second form; "all".  Once: four tiles.
@pytest.mark.parametrize("ha,hc,view,agents,central", [(128, 64, 3, 3, 0), (64, 128, 5, 3, 0), (128, 64, 3, 2, 1), (64, 128, 3, 3, 1)])
@pytest.mark.parametrize("which,often", [("last", True), ("early", True), ("all", True), ("all", False)])
def test_inexact_observations(M, orc, ha, hc, view, agents, central, which, often):
    copies = (3001 if agents == 2 else 1800) if often and central else 1500 if often else 1
    if copies == 1:
        hc = ha
    cs = W.scaled(W.CONFIGS[1], **dict(SMALL, actor_hidden=ha, critic_hidden=hc, view=view, n_agents=agents, central_critic=central))
    cf = W.scaled(cs, n_envs=cs["n_envs"] * copies)
    print("case", ha, hc, view, agents, central, which, copies, flush=True)
    params, otr = oracle_traj(orc, cs)
    rng = np.random.default_rng(7)
    steps = slice({"last": cs["rollout_len"] - 1, "early": 1, "all": 0}[which], None)
    otr.obs[steps] += (0.1 * rng.normal(size=otr.obs[steps].shape)).astype(np.float32)
    otr.value[:] += (0.2 * rng.normal(size=otr.value.shape)).astype(np.float32)
    otr.logp[:] += rng.choice([-0.4, 0.0, 0.0, 0.4], size=otr.logp.shape).astype(np.float32)
    po, mo, vo = params.copy(), np.zeros_like(params), np.zeros_like(params)
    ostats, ograd = orc.ppo_update(cs, otr, po, mo, vo, adam_step0=0, perm=None)
    gtr = M.Traj(cf)
    for f in ("obs", "action", "logp", "value", "reward", "adv", "ret", "done"):
        src = getattr(otr, f)
        getattr(gtr, f).copy_(torch.from_numpy(np.tile(src, (1, copies) + (1,) * (src.ndim - 2))))
    gp, gm, gv = dev(params), torch.zeros(params.size, device="cuda"), torch.zeros(params.size, device="cuda")
    stats, g = torch.zeros((1, 8), device="cuda"), torch.zeros(params.size, device="cuda")
    M.ppo_update(cf, gtr, gp, gm, gv, 0, None, stats, g, M.alloc_workspace(M.query_sizes(cf).update_workspace_bytes))
    off, g, st = 0, g.cpu().numpy(), stats.cpu().numpy()[0]
    for name, shape in W.param_layout(cs):  # block by block
        n = int(np.prod(shape))
        assert err(g[off:off + n], ograd[off:off + n], cs) < REL_TOL[0], (name, err(g[off:off + n], ograd[off:off + n], cs))
        off += n
    for i in (0, 1, 2, 3, 5, 6):
        assert abs(st[i] - ostats[0, i]) < REL_TOL[0] * max(abs(ostats[0, i]), 1e-2), (i, st[i], ostats[0, i])
