"""Products in tiles of 192 columns (forward ones that come out in fewer rounds, weight gradients of many samples): the gradient of one
large minibatch, which takes them, against the average of the same samples' smaller minibatches, which do not, and against torch in
64 bits.

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
SHAPES = [(0, 384, 2913, 5, 3), (1, 128, 3972, 11, 12), (1, 256, 3276, 5, 6)]


def rollout_of(M, recurrent, units, n_envs, T):
    cfg = W.scaled(W.CONFIGS[1], view=3, n_envs=n_envs, rollout_len=T, actor_hidden=units, critic_hidden=units, episode_cap=4, n_epochs=1,
                   n_minibatches=1, recurrent=recurrent, max_grad_norm=0.0, normalize_adv=0, lr=1e-30)
    params = dev(W.init_params(cfg, bias_scale=0.2))
    st, tr = M.EnvState(cfg), M.Traj(cfg)
    M.env_reset(cfg, st)
    ws = M.alloc_workspace(M.query_sizes(cfg).rollout_workspace_bytes)
    rec = M.RecState(cfg) if recurrent else None
    if recurrent:
        M.rollout_recurrent(cfg, st, params, tr, rec, 7, ws)
    else:
        M.rollout(cfg, st, params, tr, 7, ws)
    M.compute_gae(cfg, tr)
    return cfg, params, tr, rec


def last_gradient(M, cfg, params, tr, rec, n_minibatches, order):
    c = dict(cfg, n_minibatches=n_minibatches)
    p, g, stats = params.clone(), torch.zeros_like(params), torch.zeros((n_minibatches, 8), device="cuda")
    m, v, u = torch.zeros_like(p), torch.zeros_like(p), M.alloc_workspace(M.query_sizes(c).update_workspace_bytes)
    if rec is not None:
        M.ppo_update_recurrent(c, tr, rec, p, m, v, 0, dev(order), stats, g, u)
    else:
        M.ppo_update(c, tr, p, m, v, 0, dev(order), stats, g, u)
    torch.cuda.synchronize()
    return g.cpu().numpy().astype(np.float64)


def assert_close(cfg, got, want):
    off = 0
    for name, shape in W.param_layout(cfg):
        n = int(np.prod(shape))
        e = rel_err(got[off:off + n], want[off:off + n], floor=1.0)
        assert e < 1e-5, (name, e)
        off += n
    assert off == got.size


@pytest.mark.parametrize("recurrent,units,n_envs,T,parts", SHAPES)
def test_one_minibatch_against_its_parts(recurrent, units, n_envs, T, parts):
    import paper_2107_01460_amd as M
    print("case", recurrent, units, n_envs, T, flush=True)
    cfg, params, tr, rec = rollout_of(M, recurrent, units, n_envs, T)
    perm = (W.make_env_perm if recurrent else W.make_perm)(cfg, seed=3)
    whole = last_gradient(M, cfg, params, tr, rec, 1, perm)
    share = perm.shape[1] // parts
    mean = sum(last_gradient(M, cfg, params, tr, rec, parts, np.ascontiguousarray(np.roll(perm, k * share, axis=1))) for k in range(parts)) / parts
    assert_close(cfg, whole, mean)


def exact_gradient(cfg, params, tr):
    """The same minibatch's gradient by torch in 64 bits (all rows, no normalisation, initial hidden states of zero)."""
    T, A = cfg["rollout_len"], cfg["n_agents"]
    p = params.double().requires_grad_()
    b, off = {}, 0
    for name, shape in W.param_layout(cfg):
        n = int(np.prod(shape))
        b[name] = p[off:off + n].view(shape)
        off += n
    x = tr.obs[:T].double().view(T, -1, W.obs_dim(cfg))

    def outputs(net):
        w = lambda k: b[net + "." + k]
        if not cfg["recurrent"]:
            return torch.tanh(torch.tanh(x.reshape(-1, x.shape[-1]) @ w("W1") + w("b1")) @ w("W2") + w("b2")) @ w("W3") + w("b3")
        H = w("be").numel()
        h, out = torch.zeros((x.shape[1], H), dtype=torch.float64, device="cuda"), []
        for t in range(T):
            if t > 0:
                h = h * (1 - tr.done[t - 1].double()).repeat_interleave(A)[:, None]
            gi = torch.tanh(x[t] @ w("We") + w("be")) @ w("Wi") + w("bi")
            gh = h @ w("Wh") + w("bh")
            r, z = torch.sigmoid(gi[:, :H] + gh[:, :H]), torch.sigmoid(gi[:, H:2 * H] + gh[:, H:2 * H])
            n = torch.tanh(gi[:, 2 * H:] + r * gh[:, 2 * H:])
            h = (1 - z) * n + z * h
            out.append(h @ w("W3") + w("b3"))
        return torch.cat(out)

    logp = torch.log_softmax(outputs("actor"), dim=1)
    ratio = torch.exp(logp.gather(1, tr.action.long().view(-1, 1))[:, 0] - tr.logp.double().view(-1))
    adv = tr.adv.double().view(-1)
    eps = cfg["clip_eps"]
    loss = -torch.minimum(ratio * adv, ratio.clamp(1 - eps, 1 + eps) * adv).mean() + cfg["ent_coef"] * (logp.exp() * logp).sum(1).mean()
    loss = loss + cfg["vf_coef"] * 0.5 * (outputs("critic")[:, 0] - tr.ret.double().view(-1)).square().mean()
    return torch.autograd.grad(loss, p)[0].cpu().numpy()


# Bound as above; what the forward pass rounds, about 2^-24 of a sample's own share, is of random sign as well.
@pytest.mark.parametrize("recurrent,units,n_envs,T,parts", SHAPES)
def test_one_minibatch_against_64_bits(recurrent, units, n_envs, T, parts):
    import paper_2107_01460_amd as M
    print("case", recurrent, units, n_envs, T, flush=True)
    cfg, params, tr, rec = rollout_of(M, recurrent, units, n_envs, T)
    perm = (W.make_env_perm if recurrent else W.make_perm)(cfg, seed=3)
    assert_close(cfg, last_gradient(M, cfg, params, tr, rec, 1, perm), exact_gradient(cfg, params, tr))
