"""The bf16 networks at the edges of their tiles: every hidden width, inputs of one and of several 192-column pieces, sample
counts around the 32- and 64-row tiles and around the size from which the taller tiles are used."""
import pytest
import torch

import workloads as W
from gpu_util import dev, small
from test_gpu_parity import check_policy_forward, check_single_minibatch_gradient

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2107_01460_amd as M
    return M


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


@pytest.mark.parametrize("ha,hc,view,central,n_envs", [
    (64, 320, 3, 0, 1), (192, 448, 5, 0, 5), (384, 128, 7, 1, 11), (448, 192, 7, 0, 16), (320, 512, 5, 1, 33), (512, 64, 3, 1, 43)])
def test_widths(M, orc, ha, hc, view, central, n_envs):
    kw = dict(actor_hidden=ha, critic_hidden=hc, view=view, central_critic=central)
    check_policy_forward(M, orc, small(4, **kw), 70 + ha // 64)
    check_single_minibatch_gradient(M, orc, small(4, n_envs=n_envs, n_epochs=1, n_minibatches=1, max_grad_norm=0.0, **kw), 4)


@pytest.mark.parametrize("ha,hc", [(512, 256), (64, 128), (192, 448)])
def test_forward_does_not_depend_on_the_number_of_rows(M, ha, hc):
    """Both tile heights (the line is at 16 384 samples) take a sample's sums in the same order."""
    cfg = W.scaled(W.CONFIGS[3], actor_hidden=ha, critic_hidden=hc, n_agents=4, n_envs=4200, rollout_len=1, n_minibatches=1)
    D = W.obs_dim(cfg)
    g = torch.Generator(device="cuda").manual_seed(5)
    obs = torch.randint(0, 4, (4200, 4, D), device="cuda", generator=g).float()
    params = dev(W.init_params(cfg, bias_scale=0.2))
    ws = M.alloc_workspace(M.query_sizes(cfg).rollout_workspace_bytes)

    def forward(first, n):
        logits, value = torch.empty((n, 4, 6), device="cuda"), torch.empty((n, 4), device="cuda")
        M.policy_forward(cfg, params, obs[first:first + n].contiguous(), n, logits, value, ws)
        return logits, value

    all_l, all_v = forward(0, 4200)
    for first, n in ((0, 1), (7, 8), (8, 9), (100, 16), (100, 17), (3, 4095), (3, 4096), (3, 4097)):
        print("case", ha, hc, n, flush=True)
        l, v = forward(first, n)
        assert torch.equal(l, all_l[first:first + n]) and torch.equal(v, all_v[first:first + n]), n
