"""Training rollouts on both sides of the line where the tile grows from 16 samples to 32 or 64 (256 groups of 16 samples at 128
units, 512 at 64): the same environments bit for bit, since a sample's sums run in the same order in tiles of either height."""
import pytest
import torch

import workloads as W
from gpu_util import dev
from test_gpu_batch_size import M, run  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,units,agents,food,level,view", [
    (0, 64, 2, 1, 2, 3), (0, 64, 1, 2, 2, 5), (0, 64, 7, 3, 2, 7), (1, 64, 3, 5, 2, 3), (2, 64, 5, 6, 2, 5),
    (0, 128, 3, 3, 3, 5), (0, 128, 1, 1, 1, 3), (0, 128, 8, 6, 3, 7), (1, 128, 4, 4, 2, 7), (2, 128, 5, 6, 2, 3)])
def test_tiles_of_either_height_give_the_same_run(M, kind, units, agents, food, level, view):  # noqa: F811
    line = (512 if units == 64 else 256) * (16 // agents)  # environments in the largest launch of small tiles
    base = W.scaled(W.CONFIGS[0], env_kind=kind, grid=10, n_agents=agents, n_food=food, max_level=level, view=view, actor_hidden=units,
                    critic_hidden=64, rollout_len=5, n_minibatches=1, n_epochs=1, episode_cap=4)
    params = dev(W.init_params(base, bias_scale=0.2))
    ref, _ = run(M, W.scaled(base, n_envs=line + 1), params)
    for n in (line, line - 1, 16 // agents + 1, 1):
        print("case", kind, units, agents, view, n, flush=True)
        tr, _ = run(M, W.scaled(base, n_envs=n), params)
        for f in ("obs", "action", "sampled", "logits", "logp", "reward", "done"):
            assert torch.equal(getattr(tr, f), getattr(ref, f)[:, :n]), (n, f)
