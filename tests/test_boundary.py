"""The C-ABI library loads without a GPU, exports every symbol the header declares, and rejects bad
arguments on the host before anything is launched."""
import ctypes as C
import os
import re

import pytest
import torch

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def M():
    import paper_2107_01460_amd as m
    if not os.path.exists(m.binding._LIB_PATH):
        from paper_2107_01460_amd import build
        build.build(verbose=False)
    m.lib()
    return m


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "marl.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(marl_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(M):
    names = declared_symbols()
    assert len(names) >= 12
    for n in names:
        assert hasattr(M.lib(), n), n
    assert set(M.binding.EXPORTS) == set(names)


def test_query_sizes_and_parameter_counts(M):
    for cfg in W.CONFIGS:
        s = M.query_sizes(cfg)
        assert s.n_params == W.param_count(cfg)
        assert s.obs_dim == W.obs_dim(cfg) and s.critic_in_dim == W.critic_in_dim(cfg)
        T, N, A = cfg["rollout_len"], cfg["n_envs"], cfg["n_agents"]
        assert s.obs_bytes == 4 * (T + 1) * N * A * s.obs_dim
        assert s.step_scalar_bytes == 4 * T * N * A and s.done_bytes == T * N
        assert s.rollout_workspace_bytes > 0 and s.update_workspace_bytes > s.n_params * 8


@pytest.mark.parametrize("field,value", [
    ("grid", 1), ("grid", 65), ("n_agents", 9), ("n_food", 0), ("view", 4), ("actor_hidden", 100),
    ("critic_hidden", 1024), ("n_minibatches", 7), ("precision", 2), ("clip_eps", 0.0), ("gamma", 1.5),
    ("max_level", 0), ("max_level", 16), ("central_critic", 2), ("lr", 0.0), ("n_minibatches", 0), ("n_epochs", 0)])
def test_bad_config_rejected(M, field, value):
    cfg = W.scaled(W.CONFIGS[1], **{field: value})
    s = M.binding.Sizes()
    rc = M.lib().marl_query_sizes(C.byref(M.make_config(cfg)), C.byref(s))
    assert rc == -3, (field, rc)
    st = M.binding.EnvStateC(*([0x1000] * 8))
    assert M.lib().marl_env_reset(C.byref(M.make_config(cfg)), st, None) == -3


def test_zero_minibatches_rejected_for_recurrent_networks(M):
    """n_minibatches is a divisor in the checks of the recurrent configuration: zero must be an error, not a trap."""
    s = M.binding.Sizes()
    for nm in (0, -1):
        cfg = W.scaled(W.CONFIGS[0], recurrent=1, n_minibatches=nm)
        assert M.lib().marl_query_sizes(C.byref(M.make_config(cfg)), C.byref(s)) == -3


def test_recurrent_sizes(M):
    cfg = W.scaled(W.CONFIGS[2], recurrent=1)
    sz = M.query_sizes(cfg)
    assert sz.n_params == W.param_count(cfg)
    assert sz.hidden_actor_bytes == 4 * cfg["n_envs"] * cfg["n_agents"] * cfg["actor_hidden"]
    assert sz.hidden_critic_bytes == 4 * cfg["n_envs"] * cfg["critic_hidden"]
    assert sz.rollout_workspace_bytes > 0 and sz.update_workspace_bytes > 0
    assert M.query_sizes(W.CONFIGS[2]).hidden_actor_bytes == 0


def test_warehouse_config_checks(M):
    L = M.lib()
    sz = M.binding.Sizes()
    ok = M.make_config(W.scaled(W.CONFIGS[1], env_kind=2, max_level=3))
    assert L.marl_query_sizes(C.byref(ok), C.byref(sz)) == 0
    assert L.marl_query_sizes(C.byref(M.make_config(W.scaled(W.CONFIGS[1], env_kind=3))), C.byref(sz)) == -3
    # more requested shelves than shelves
    assert L.marl_query_sizes(C.byref(M.make_config(W.scaled(W.CONFIGS[0], env_kind=1, max_level=2))), C.byref(sz)) == -3


def test_too_many_entities_rejected(M):
    cfg = W.scaled(W.CONFIGS[0], grid=2, n_agents=3, n_food=2)
    s = M.binding.Sizes()
    assert M.lib().marl_query_sizes(C.byref(M.make_config(cfg)), C.byref(s)) == -3


def test_null_and_misaligned_pointers_rejected_before_launch(M):
    cfg = M.make_config(W.CONFIGS[0])
    L = M.lib()
    good = 0x10000
    null_state = M.binding.EnvStateC(*([good] * 7 + [None]))
    assert L.marl_env_reset(C.byref(cfg), null_state, None) == -1
    odd_state = M.binding.EnvStateC(*([good] * 7 + [good + 4]))
    assert L.marl_env_reset(C.byref(cfg), odd_state, None) == -2
    ok_state = M.binding.EnvStateC(*([good] * 8))
    assert L.marl_observe(C.byref(cfg), ok_state, None, None) == -1
    assert L.marl_env_step(C.byref(cfg), ok_state, good, good + 8, good, good, None) == -2
    traj = M.binding.TrajC(*([good] * 9 + [None, None]))
    assert L.marl_rollout(C.byref(cfg), ok_state, None, traj, 0, None, None, good, None) == -1
    assert L.marl_compute_gae(C.byref(cfg), M.binding.TrajC(*([good] * 7 + [None, good, None, None])), None) == -1
    assert L.marl_ppo_update(C.byref(cfg), traj, good, good, good, -1, None, good, None, good, None) == -5
    assert L.marl_ppo_update(C.byref(cfg), traj, good, good, good, 0, good + 2, good, None, good, None) == -2
    assert L.marl_policy_forward(C.byref(cfg), good, good, -1, good, good, good, None) == -5
    assert L.marl_sample_actions(C.byref(cfg), good, None, None, 1 << 31, 0, good, None, good, None) == -5
    ev = M.binding.EvalStatsC(good, good, good)
    assert L.marl_evaluate(C.byref(cfg), ok_state, good, 0, ev, good, None) == -5
    assert L.marl_evaluate(C.byref(cfg), ok_state, good, 1 << 20, ev, good, None) == -5
    assert L.marl_evaluate(C.byref(cfg), ok_state, None, 1, ev, good, None) == -1
    assert L.marl_evaluate(C.byref(cfg), ok_state, good, 1, M.binding.EvalStatsC(good, None, good), good, None) == -1
    rs = M.binding.RecStateC(good, good, good, good)
    # the recurrent entry points take recurrent configurations only, and the feed-forward ones refuse them
    assert L.marl_rollout_recurrent(C.byref(cfg), ok_state, good, traj, rs, 0, None, None, good, None) == -3
    rcfg = M.make_config(W.scaled(W.CONFIGS[0], recurrent=1))
    assert L.marl_rollout(C.byref(rcfg), ok_state, good, traj, 0, None, None, good, None) == -3
    assert L.marl_ppo_update(C.byref(rcfg), traj, good, good, good, 0, None, good, None, good, None) == -3
    assert L.marl_rollout_recurrent(C.byref(rcfg), ok_state, good, traj, M.binding.RecStateC(good, None, good, good), 0,
                                    None, None, good, None) == -1
    assert L.marl_ppo_update_recurrent(C.byref(rcfg), traj, rs, good, good, good, -1, None, good, None, good, None) == -5
    assert L.marl_ppo_update_recurrent(C.byref(rcfg), traj, rs, good, good + 4, good, 0, None, good, None, good, None) == -2
    bad = M.make_config(W.scaled(W.CONFIGS[0], recurrent=1, n_minibatches=3))     # 64 environments do not split in 3
    assert L.marl_ppo_update_recurrent(C.byref(bad), traj, rs, good, good, good, 0, None, good, None, good, None) == -3
    # the single-call training step: counters and both workspaces are required, feed-forward networks only
    assert L.marl_train_step(C.byref(cfg), ok_state, good, traj, good, good, None, None, good, good, good, None) == -1
    assert L.marl_train_step(C.byref(cfg), ok_state, good, traj, good, good, good, None, good, good, None, None) == -1
    assert L.marl_train_step(C.byref(cfg), ok_state, good, traj, good, good, good + 8, None, good, good, good, None) == -2
    assert L.marl_train_step(C.byref(rcfg), ok_state, good, traj, good, good, good, None, good, good, good, None) == -3
    assert L.marl_query_sizes(None, None) == -1
    assert M.status_string(0) == "ok" and "null" in M.status_string(-1)
    d, n, w = C.c_double(), C.c_int64(), C.c_double()
    assert L.marl_timing_read(99, C.byref(d), C.byref(n), C.byref(w)) == -5
    assert L.marl_timing_read(0, None, None, None) == -1


def test_missing_library_fails_loudly(M, monkeypatch):
    monkeypatch.setattr(M.binding, "_lib", None)
    monkeypatch.setattr(M.binding, "_LIB_PATH", "/nonexistent/libmarl_gfx950.so")
    with pytest.raises(M.MarlError):
        M.binding.lib()


@pytest.mark.parametrize("view", [3, 5])
def test_update_workspace_of_networks_in_one_training_kernel(M, view):
    """512 copies of the larger network's gradient and little else: the output-layer copies of the other routes are not counted."""
    s = M.query_sizes(W.scaled(W.CONFIGS[0], n_envs=2, rollout_len=1, n_minibatches=1, view=view))
    assert s.update_workspace_bytes < 4 * (512 * s.n_actor_params + 16 * s.n_params)


@pytest.mark.skipif(torch.cuda.device_count() > 0, reason="the calls that are accepted would run, on addresses that are none")
@pytest.mark.parametrize("ha,hc,agents,view,central,most", [
    (512, 320, 8, 7, 1, 144), (480, 320, 8, 7, 1, 157), (352, 64, 3, 5, 0, 913), (448, 64, 3, 5, 0, 686), (64, 448, 4, 5, 0, 515)])
def test_rollout_static_takes_what_only_split_weights_push_over_its_limit(ha, hc, agents, view, central, most):
    """One network layer by layer, the other on chip: the split copies of the second one's weights are larger than plain ones, and the
    environments that fitted beside plain ones still fit (MARL_E_LAUNCH: accepted, no GPU here)."""
    import paper_2107_01460_amd as M
    for envs, code in ((most, -4), (most + 1, -5)):
        cfg = W.scaled(W.CONFIGS[1], actor_hidden=ha, critic_hidden=hc, n_agents=agents, view=view, central_critic=central, n_envs=envs,
                       rollout_len=1, n_minibatches=1)
        assert M.query_sizes(cfg).rollout_workspace_bytes > 8 * 1024 * 1024
        good = 0x10000
        st, traj = M.binding.EnvStateC(*([good] * 8)), M.binding.TrajC(*([good] * 9 + [None, None]))
        assert M.lib().marl_rollout_static(C.byref(M.make_config(cfg)), st, good, traj, 0, None, None, None) == code, envs


def test_current_stream_without_the_private_name(M, monkeypatch):
    """A torch that lacks the short way to the current stream's handle takes the long one."""
    class Current:
        cuda_stream = 0x1234
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Current)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(M.binding, "_raw_stream", None)
    assert M.binding._stream(None) == 0x1234
    monkeypatch.setattr(M.binding, "_raw_stream", lambda device: 0x5678 + device)
    assert M.binding._stream(None) == 0x5678
    assert M.binding._stream(Current) == 0x1234


@pytest.mark.gpu
def test_current_stream_both_ways(M, monkeypatch):
    for s in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(s):
            short = M.binding._stream(None)
            monkeypatch.setattr(M.binding, "_raw_stream", None)
            assert M.binding._stream(None) == short == s.cuda_stream
            monkeypatch.undo()
