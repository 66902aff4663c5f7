"""An environment's run does not depend on how many others share the launch: its random streams are keyed by its own index,
and every size of call computes with the same arithmetic, so the same environments come out bit for bit.  (A sampled
action is a discrete choice: logits that differ in the last bit are, somewhere among millions of them, another run.)
"""
import pytest
import torch

import workloads as W
from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2107_01460_amd as m
    return m


def run(M, cfg, params):
    st, tr = M.EnvState(cfg), M.Traj(cfg, debug=True)
    M.env_reset(cfg, st)
    ws = M.alloc_workspace(M.query_sizes(cfg).rollout_workspace_bytes)
    if not cfg["recurrent"]:
        M.rollout(cfg, st, params, tr, 7, ws)
        return tr, ()
    rec = M.RecState(cfg)
    M.rollout_recurrent(cfg, st, params, tr, rec, 7, ws)
    return tr, (rec.ha1, rec.hc1)


# environments per launch around 512 workgroups of the rollout kernels (32 environments each at 64 units and two agents, 10 at
# 128 units and three), and a handful; networks whose steps are launches of their own, in one kernel each (192 units; 64-row tiles from
# 16 384 samples on) and layer by layer (352); the recurrent ones around 4096 samples per step, where
# the cell's kernels change their tile, with weights in registers and streamed
@pytest.mark.parametrize("k,sizes,kw", [
    (5, (37, 512 * 32, 512 * 32 + 1), {}),
    (2, (37, 512 * 10, 512 * 10 + 1), {}),
    (2, (37, 600), dict(actor_hidden=192, critic_hidden=256)),
    (2, (37, 5461, 5462), dict(actor_hidden=192, critic_hidden=320)),
    (2, (37, 600, 3000), dict(actor_hidden=352, critic_hidden=480)),
    (2, (37, 1365, 1366), dict(recurrent=1, actor_hidden=128, critic_hidden=192)),
    (2, (37, 1365, 1366), dict(recurrent=1, actor_hidden=256, critic_hidden=64)),
])
def test_rollout_does_not_depend_on_the_batch(M, k, sizes, kw):
    base = W.scaled(W.CONFIGS[k - 1], rollout_len=4, n_minibatches=1, n_epochs=1, episode_cap=3, **kw)
    params = dev(W.init_params(base, bias_scale=0.1))
    ref = None
    for n in sorted(sizes, reverse=True):
        print("case", k, kw, n, flush=True)
        tr, state = run(M, W.scaled(base, n_envs=n), params)
        if ref is None:
            ref, ref_state = tr, state
            continue
        for f in ("obs", "action", "sampled", "logits", "logp", "reward", "done", "value"):
            assert torch.equal(getattr(tr, f), getattr(ref, f)[:, :n]), (n, f)
        assert torch.equal(tr.last_value, ref.last_value[:n]), n
        for a, b in zip(state, ref_state):
            assert torch.equal(a, b[:n]), n


@pytest.mark.parametrize("hidden", [64, 128, 192, 256, 384])
def test_evaluation_does_not_depend_on_the_batch(M, hidden):
    base = W.scaled(W.CONFIGS[1], rollout_len=1, n_minibatches=1, episode_cap=6, actor_hidden=hidden)
    params = dev(W.init_params(base, bias_scale=0.1))
    ref = None
    for n in (1100, 37):
        cfg = W.scaled(base, n_envs=n)
        print("case", hidden, n, flush=True)
        st, out = M.EnvState(cfg), M.EvalStats(cfg)
        M.env_reset(cfg, st)
        M.evaluate(cfg, st, params, 2, out, M.alloc_workspace(M.query_sizes(cfg).eval_workspace_bytes))
        got = [out.ret_sum, out.len_sum] + [getattr(st, f) for f in M.EnvState.FIELDS]
        if ref is None:
            ref = got
            continue
        for a, b in zip(got, ref):
            assert torch.equal(a, b[..., :n])
