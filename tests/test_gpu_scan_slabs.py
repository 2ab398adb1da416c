"""Calls whose chunk records outgrow the memory-side cache run in slabs of chunks
with the state carried between them; the profiled call runs in one pass.  Same
kernels and sums: the outputs and states are the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,T,Dk,Dv,state", [
    (1, 32, 5312, 128, 128, True),     # 83 chunks, 145 MB: two slabs of 42 and 41
    (2, 24, 3300, 128, 128, True),     # 52 chunks, 137 MB: just over the size from which there are two
    (1, 32, 5249, 128, 128, False),    # a last chunk of one token, no state in
    (4, 20, 8000, 64, 64, True),       # 125 chunks of 80 narrow heads: three slabs
    (2, 24, 6401, 64, 128, True),
])
def test_slabs_bitwise(gdn, B, H, T, Dk, Dv, state):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + H)

    def randn(*s):
        return torch.randn(s, generator=g, device="cuda")

    q, k = (torch.nn.functional.normalize(randn(B, T, H, Dk), dim=-1).bfloat16() for _ in range(2))
    v = randn(B, T, H, Dv).bfloat16()
    alpha = torch.sigmoid(randn(B, T, H) + 4.0)      # slow decay: the carried state matters
    beta = torch.sigmoid(randn(B, T, H))
    s0 = 0.1 * randn(B, H, Dk, Dv) if state else None
    ws = gdn.workspace(q, v)
    out1, st1 = torch.empty_like(v), torch.empty(B, H, Dk, Dv, device="cuda")
    gdn.gdn_profile_stages(q, k, v, alpha, beta, s0, out1, st1, ws, reps=1)
    out, st = gdn.forward(q, k, v, alpha, beta, s0, ws=ws)
    assert torch.equal(out, out1) and torch.equal(st, st1)
    if state:                                        # in place
        gdn.forward(q, k, v, alpha, beta, s0, out=out, state_out=s0, ws=ws)
        assert torch.equal(out, out1) and torch.equal(s0, st1)
