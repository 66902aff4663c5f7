"""marl_rollout_static on both sides of its limit: it takes the configurations whose rollout_workspace_bytes fit
MARL_STATIC_SCRATCH_BYTES (the caller can ask beforehand), and those that only the split copies of their weights push over it, with the
results of marl_rollout."""
import os
import re

import pytest
import torch

import workloads as W
from gpu_util import dev

pytestmark = pytest.mark.gpu


def limit():
    header = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "marl.h")
    return eval(re.search(r"#define MARL_STATIC_SCRATCH_BYTES \((.*)\)", open(header).read()).group(1))


# networks that run on chip; the size reported grows with the environments all the same, by both hidden layers of a step of the 192 and
# 96 units
@pytest.mark.parametrize("ha,hc,central", [(192, 256, 1), (128, 96, 0)])
def test_rollout_static_limit(ha, hc, central):
    import paper_2107_01460_amd as M
    base = W.scaled(W.CONFIGS[1], actor_hidden=ha, critic_hidden=hc, central_critic=central, rollout_len=2, n_minibatches=1)
    need = lambda n: M.query_sizes(W.scaled(base, n_envs=n)).rollout_workspace_bytes
    n = max(k for k in range(1, 20000) if need(k) <= limit())
    assert need(n + 1) > limit()
    params = dev(W.init_params(base, bias_scale=0.1))
    for envs in (n, n + 1):
        cfg = W.scaled(base, n_envs=envs)
        print("case", ha, hc, envs, need(envs), flush=True)
        st, tr = M.EnvState(cfg), M.Traj(cfg, debug=True)
        M.env_reset(cfg, st)
        if envs > n:
            with pytest.raises(M.MarlError, match="-5"):
                M.rollout_static(cfg, st, params, tr, 3)
            continue
        check_against_rollout(M, cfg, params, st, tr)


def check_against_rollout(M, cfg, params, st, tr):
    M.rollout_static(cfg, st, params, tr, 3)
    s2, t2 = M.EnvState(cfg), M.Traj(cfg, debug=True)
    M.env_reset(cfg, s2)
    M.rollout(cfg, s2, params, t2, 3, M.alloc_workspace(M.query_sizes(cfg).rollout_workspace_bytes))
    for f in ("obs", "action", "logits", "value", "last_value", "reward", "done"):
        assert torch.equal(getattr(tr, f), getattr(t2, f)), f


# layer-by-layer actors beside critics on chip, at the most environments that are taken: over the limit by the critic's split weights
@pytest.mark.parametrize("ha,hc,agents,view,central,envs", [(512, 320, 8, 7, 1, 144), (352, 64, 3, 5, 0, 913)])
def test_rollout_static_over_the_limit_by_split_weights(ha, hc, agents, view, central, envs):
    import paper_2107_01460_amd as M
    cfg = W.scaled(W.CONFIGS[1], actor_hidden=ha, critic_hidden=hc, n_agents=agents, view=view, central_critic=central, n_envs=envs,
                   rollout_len=2, n_minibatches=1)
    assert M.query_sizes(cfg).rollout_workspace_bytes > limit()
    print("case", ha, hc, envs, flush=True)
    st, tr = M.EnvState(cfg), M.Traj(cfg, debug=True)
    M.env_reset(cfg, st)
    check_against_rollout(M, cfg, dev(W.init_params(cfg, bias_scale=0.1)), st, tr)
