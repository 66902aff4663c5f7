"""The fp32 networks whose row tile goes through the whole network in one kernel, at the edges of its tiles: every hidden width
up to 320, inputs of one and of several staged pieces, sample counts around the 32- and 64-row tiles and around the size
from which forward passes take the taller one; inputs that are exact in bf16 (fewer products) beside inputs that are not."""
import pytest
import torch

import workloads as W
from gpu_util import REL_TOL, dev, rel_err, small
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


# (64 and 128 units: inputs wider than the whole-minibatch kernel takes)
@pytest.mark.parametrize("ha,hc,view,central,n_envs", [
    (32, 64, 7, 1, 1), (64, 128, 7, 0, 5), (96, 288, 3, 0, 11), (128, 224, 7, 1, 16), (160, 192, 5, 1, 33),
    (256, 320, 7, 0, 43), (320, 96, 5, 1, 22), (288, 256, 3, 0, 3)])
def test_widths(M, orc, ha, hc, view, central, n_envs):
    kw = dict(actor_hidden=ha, critic_hidden=hc, view=view, central_critic=central)
    check_policy_forward(M, orc, small(2, **kw), 80 + ha // 32)
    check_single_minibatch_gradient(M, orc, small(2, n_envs=n_envs, n_epochs=1, n_minibatches=1, max_grad_norm=0.0, **kw), 2)


def reference(x, p, din, h, nout):
    """Two tanh layers and a linear one in 64 bits; x [rows][din], p the network's parameters."""
    sizes = (din * h, h, h * h, h, h * nout, nout)
    w1, b1, w2, b2, w3, b3 = torch.split(p.double().cpu(), sizes)
    y = torch.tanh(x.double().cpu() @ w1.reshape(din, h) + b1)
    return torch.tanh(y @ w2.reshape(h, h) + b2) @ w3.reshape(h, nout) + b3


@pytest.mark.parametrize("ha,hc,view", [(256, 192, 7), (64, 128, 5), (32, 320, 3), (224, 96, 7), (160, 288, 5)])
def test_forward_does_not_depend_on_the_batch(M, ha, hc, view):
    """Both tile heights (the line is at 16 384 samples) take a sample's sums in the same order, beside any neighbours."""
    cfg = W.scaled(W.CONFIGS[1], actor_hidden=ha, critic_hidden=hc, view=view, n_agents=4, n_envs=4200, rollout_len=1, n_minibatches=1)
    D = W.obs_dim(cfg)
    g = torch.Generator(device="cuda").manual_seed(5)
    obs = torch.randint(-2, 8, (4200, 4, D), device="cuda", generator=g) * 0.5
    params = dev(W.init_params(cfg, bias_scale=0.2))
    ws = M.alloc_workspace(M.query_sizes(cfg).rollout_workspace_bytes)

    def forward(x):
        n = x.shape[0]
        logits, value = torch.empty((n, 4, 6), device="cuda"), torch.empty((n, 4), device="cuda")
        M.policy_forward(cfg, params, x.contiguous(), n, logits, value, ws)
        return logits, value

    mixed = obs.clone()
    mixed[::5] = torch.randn((840, 4, D), device="cuda", generator=g)  # no tile is without such rows
    exact_l, exact_v = forward(obs)
    all_l, all_v = forward(mixed)
    same = torch.arange(4200, device="cuda") % 5 != 0
    assert torch.equal(all_l[same], exact_l[same]) and torch.equal(all_v[same], exact_v[same])
    n_actor = D * ha + ha + ha * ha + ha + 6 * ha + 6
    some = slice(0, 4200, 7)
    assert rel_err(all_l[some].cpu(), reference(mixed[some].reshape(-1, D), params[:n_actor], D, ha, 6)) < REL_TOL[0]
    assert rel_err(all_v[some].cpu(), reference(mixed[some].reshape(-1, D), params[n_actor:], D, hc, 1)) < REL_TOL[0]
    # more than 2048 samples: below, networks of 64, 128 and 256 units take the small calls' kernel
    for first, n in ((0, 513), (7, 520), (8, 521), (100, 4095), (100, 4096), (100, 4097)):
        print("case", ha, hc, n, flush=True)
        l, v = forward(mixed[first:first + n])
        assert torch.equal(l, all_l[first:first + n]) and torch.equal(v, all_v[first:first + n]), n
