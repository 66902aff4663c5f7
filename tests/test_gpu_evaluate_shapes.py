"""Greedy evaluation blocks of shapes that none of the workloads has, against the oracle: both worlds, every view, both widths of
the one-launch kernel, entity counts on both sides of its unrolled capacities, ragged last workgroups; and actors whose steps are
launches of their own, in one kernel (192 units) and layer by layer (448)."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2107_01460_amd as m
    return m


@pytest.mark.parametrize("kind,grid,agents,food,level,view,hidden,n_envs", [
    (0, 9, 6, 3, 2, 7, 128, 23), (0, 8, 3, 4, 2, 3, 64, 70), (0, 10, 5, 5, 3, 5, 64, 61), (0, 8, 2, 2, 2, 7, 64, 67),
    (1, 8, 3, 5, 2, 3, 64, 45), (1, 10, 4, 4, 2, 7, 128, 33), (2, 9, 5, 6, 2, 5, 128, 41), (2, 8, 2, 8, 3, 7, 64, 97),
    (0, 8, 3, 4, 2, 5, 192, 37), (0, 8, 2, 2, 2, 3, 448, 29)])
def test_evaluation_block(M, orc, kind, grid, agents, food, level, view, hidden, n_envs):
    cfg = W.scaled(W.CONFIGS[0], env_kind=kind, grid=grid, n_agents=agents, n_food=food, max_level=level, view=view, n_envs=n_envs,
                   actor_hidden=hidden, critic_hidden=hidden, episode_cap=9, n_minibatches=1, rollout_len=1)
    E = 3
    print("case", kind, grid, agents, food, view, hidden, n_envs, flush=True)
    params = W.init_params(cfg, bias_scale=0.3)
    os_ = orc.EnvState(cfg)
    orc.env_reset(cfg, os_)
    oret, olen, oeps, gap = orc.evaluate(cfg, os_, params, E)
    gs, out = M.EnvState(cfg), M.EvalStats(cfg)
    M.env_reset(cfg, gs)
    M.evaluate(cfg, gs, dev(params), E, out, M.alloc_workspace(M.query_sizes(cfg).eval_workspace_bytes))
    torch.cuda.synchronize()
    # the environments whose two largest logits were never closer than an fp32 evaluation can tell apart: with logits spread
    # over about 1, one decision in a thousand is that close, and a run of six agents makes 27 x 6 = 162 of them
    clear = gap > 8e-4 * max(1.0, float(np.abs(params).max()))
    assert clear.mean() > 0.6, clear.mean()
    assert np.all(out.episodes.cpu().numpy() == E) and np.all(oeps == E)
    assert np.array_equal(out.ret_sum.cpu().numpy()[clear].view(np.uint32), oret[clear].view(np.uint32))
    assert np.array_equal(out.len_sum.cpu().numpy()[clear], olen[clear])
    host = gs.to_host()
    for f in M.EnvState.FIELDS:
        assert np.array_equal(host[f][..., clear], getattr(os_, f)[..., clear]), f


# Episodes played beside one another: from states in the middle of an episode; more episodes than rows of an environment are resident
# (700 environments with 8 to a workgroup and one of those per CU); more than there is room to record (5600 environments, two of three);
# environments whose step count is past the cap already, which play their first episode for as long as it lasts.
@pytest.mark.parametrize("agents,view,hidden,n_envs,cap,E,past", [(2, 3, 64, 45, 7, 4, 0), (4, 7, 128, 700, 3, 5, 0), (2, 3, 64, 5600, 2, 3, 0),
                                                                 (3, 5, 128, 40, 6, 3, 1)])
def test_evaluation_from_the_middle(M, orc, agents, view, hidden, n_envs, cap, E, past):
    cfg = W.scaled(W.CONFIGS[0], grid=8, n_agents=agents, n_food=2, max_level=2, view=view, n_envs=n_envs, actor_hidden=hidden,
                   critic_hidden=hidden, episode_cap=cap, n_minibatches=1, rollout_len=1)
    print("case", agents, view, hidden, n_envs, cap, E, past, flush=True)
    params = W.init_params(cfg, bias_scale=0.3)
    os_ = orc.EnvState(cfg)
    orc.env_reset(cfg, os_)
    rng = np.random.default_rng(3)
    os_.t_in_ep[:] = rng.integers(0, cap, n_envs)
    if past:
        os_.t_in_ep[::3] = cap + rng.integers(0, 4, len(os_.t_in_ep[::3]))
    gs, out = M.EnvState(cfg), M.EvalStats(cfg)
    for f in M.EnvState.FIELDS:
        getattr(gs, f).copy_(torch.from_numpy(np.ascontiguousarray(getattr(os_, f))).view(getattr(gs, f).dtype))
    oret, olen, oeps, gap = orc.evaluate(cfg, os_, params, E)
    M.evaluate(cfg, gs, dev(params), E, out, M.alloc_workspace(M.query_sizes(cfg).eval_workspace_bytes))
    torch.cuda.synchronize()
    clear = gap > 8e-4 * max(1.0, float(np.abs(params).max()))
    assert clear.mean() > 0.6, clear.mean()
    for got, want in ((out.ret_sum, oret), (out.len_sum, olen), (out.episodes, oeps)):
        assert np.array_equal(got.cpu().numpy()[clear], want[clear])
    host = gs.to_host()
    for f in M.EnvState.FIELDS:
        assert np.array_equal(host[f][..., clear], getattr(os_, f)[..., clear]), f


# Blocks whose episodes end early, in both worlds, from states with carried shelves and, in some environments, a step count past the cap: rows that play
# several episodes and the block's last one in part, from its beginning and from either third of it (caps that are no multiple of three among
# them); 2049 environments, whose rows take all the episodes there is room for; and more counted episodes than half of that room.
@pytest.mark.parametrize("kind,agents,food,view,hidden,n_envs,cap,E,past", [
    (2, 5, 4, 5, 64, 45, 31, 4, 1), (2, 8, 3, 7, 128, 33, 24, 7, 0), (1, 4, 5, 3, 128, 38, 11, 3, 1), (0, 3, 1, 5, 128, 40, 40, 2, 1),
    (2, 3, 3, 3, 64, 2049, 20, 5, 0), (2, 3, 4, 3, 64, 2049, 6, 9, 0)])
def test_evaluation_of_episodes_that_end_early(M, orc, kind, agents, food, view, hidden, n_envs, cap, E, past):
    cfg = W.scaled(W.CONFIGS[0], env_kind=kind, grid=8, n_agents=agents, n_food=food, max_level=1 if kind == 0 else 2, view=view, n_envs=n_envs,
                   actor_hidden=hidden, critic_hidden=hidden, episode_cap=cap, n_minibatches=1, rollout_len=1)
    print("case", kind, agents, food, view, hidden, n_envs, cap, E, past, flush=True)
    params = W.init_params(cfg, bias_scale=1.0 if kind else 0.3)
    os_ = orc.EnvState(cfg)
    orc.env_reset(cfg, os_)
    rng = np.random.default_rng(11)
    for _ in range(cap // 2):
        orc.env_step(cfg, os_, rng.integers(0, 6, (n_envs, agents)).astype(np.int32))
    if past:
        os_.t_in_ep[::4] = cap + rng.integers(0, 3, len(os_.t_in_ep[::4]))
    gs, out = M.EnvState(cfg), M.EvalStats(cfg)
    for f in M.EnvState.FIELDS:
        getattr(gs, f).copy_(torch.from_numpy(np.ascontiguousarray(getattr(os_, f))).view(getattr(gs, f).dtype))
    oret, olen, oeps, gap = orc.evaluate(cfg, os_, params, E)
    M.evaluate(cfg, gs, dev(params), E, out, M.alloc_workspace(M.query_sizes(cfg).eval_workspace_bytes))
    torch.cuda.synchronize()
    clear = gap > 8e-4 * max(1.0, float(np.abs(params).max()))
    print("clear", clear.mean(), "steps of an episode", olen.mean() / E, flush=True)
    assert clear.mean() > 0.3, clear.mean()
    for got, want in ((out.ret_sum, oret), (out.len_sum, olen), (out.episodes, oeps)):
        assert np.array_equal(got.cpu().numpy()[clear], want[clear])
    host = gs.to_host()
    for f in M.EnvState.FIELDS:
        assert np.array_equal(host[f][..., clear], getattr(os_, f)[..., clear]), f
