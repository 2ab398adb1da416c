"""Grouped bf16 scans round the decays no earlier than their products: the queries
meet the state unscaled and e^{g_r} multiplies the fp32 sum, and the decays of the
masked scores come from an fp64 difference.  Inputs whose other steps are exact
leave one rounding to bf16 in the output: half a unit in the last place of the exact
value, and SLACK of it for the fp32 arithmetic before (the logarithms' last places
and the rounding of their sum, at most 64 in size, 2^-17 and 2^-18; the exponential).
Queries scaled and rounded to bf16 first are off by up to two such units, and
logarithms rounded to fp32 move a decay by up to 2^-11."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SLACK = 2.0 ** -16
H = 16                                              # independent streams


def one_hot(T, Dk):
    x = torch.zeros(T, Dk)
    x[torch.arange(T), torch.arange(T) % Dk] = 1.0
    return x[:, None].expand(T, H, Dk)


def run(gdn, q, k, v, alpha, beta, state):
    """H streams in groups of one chunk; the output [T, H, Dv] as fp64 on the host."""
    q, k, v = (x[None].to("cuda", torch.bfloat16).contiguous() for x in (q, k, v))
    alpha, beta = (x[None].cuda().contiguous() for x in (alpha, beta))
    out, _ = gdn.forward(q, k, v, alpha, beta, None if state is None else state[None].cuda(), scan_group=1)
    return out[0].double().cpu()


def check(out, ref):
    half_ulp = torch.exp2(torch.floor(torch.log2(ref.abs())) - 8)
    over = ((out - ref).abs() - half_ulp) / ref.abs()
    assert over.max() <= SLACK, over.max()


@pytest.mark.parametrize("Dk,Dv", [(64, 64), (128, 128), (64, 128), (128, 64)])
@pytest.mark.parametrize("rate", [0.05, 1.0])
def test_decayed_state(gdn, Dk, Dv, rate):
    """Nothing is written: o_t = e^{g_t} H_0[t % Dk] in the first chunk, H_0 in bf16."""
    g = torch.Generator().manual_seed(71 + Dk + Dv)
    T = 192
    alpha = torch.exp(-rate * torch.rand(T, H, generator=g))
    state = torch.randn(H, Dk, Dv, generator=g).bfloat16().float()
    out = run(gdn, one_hot(T, Dk), one_hot(T, Dk), torch.zeros(T, H, Dv), alpha, torch.zeros(T, H), state)[:64]
    dec = torch.exp(torch.cumsum(torch.log(alpha.double()), 0))[:64, :, None]
    check(out, dec * state.double().transpose(0, 1)[torch.arange(64) % Dk])


@pytest.mark.parametrize("D", [64, 128])
def test_scores_after_strong_forgetting(gdn, D):
    """A chunk whose first 40 gates are zero (log decay -87.3 each) and whose later ones
    forget slowly: one token writes a row of ones at t = 41, and the later tokens read
    e^{g_t - g_41}."""
    g = torch.Generator().manual_seed(73 + D)
    T = 192
    alpha = torch.exp(-0.2 * torch.rand(T, H, generator=g))
    alpha[:40] = 0.0
    beta = torch.zeros(T, H)
    beta[41] = 1.0
    qk = torch.zeros(T, H, D)
    qk[..., 3] = 1.0
    out = run(gdn, qk, qk, torch.ones(T, H, D), alpha, beta, None)[42:64]
    dec = torch.exp(torch.cumsum(torch.log(alpha.double())[42:64], 0))
    check(out, dec[..., None].expand(-1, -1, D))
