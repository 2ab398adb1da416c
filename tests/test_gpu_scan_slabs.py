"""Calls whose chunk records outgrow the memory-side cache run in slabs of chunks
with the state carried between them; fewer heads of the same call, with less than
132 MB of records, in one pass.  Same kernels and sums: the outputs and states are
the same bits, also where the stages are timed over several launches."""
import statistics

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
    out, st = gdn.forward(q, k, v, alpha, beta, s0, ws=ws)
    n = 16 if H == 32 else H                         # heads of a part: at most 102 MB of records
    for b in range(B):
        for h in range(0, H, n):
            cut = [x[b:b + 1, :, h:h + n].contiguous() for x in (q, k, v, alpha, beta)]
            out1, st1 = gdn.forward(*cut, s0[b:b + 1, h:h + n].contiguous() if state else None)
            assert torch.equal(out[b:b + 1, :, h:h + n], out1) and torch.equal(st[b:b + 1, h:h + n], st1)
    out1, st1 = torch.empty_like(v), torch.empty(B, H, Dk, Dv, device="cuda")
    gdn.gdn_profile_stages(q, k, v, alpha, beta, s0, out1, st1, ws, reps=3)
    assert torch.equal(out, out1) and torch.equal(st, st1)
    if state:                                        # in place
        gdn.forward(q, k, v, alpha, beta, s0, out=out, state_out=s0, ws=ws)
        assert torch.equal(out, out1) and torch.equal(s0, st1)


def test_profile_times_the_call_that_runs(gdn):
    """T = 16384, H = 16 takes 270 us in slabs and 385 in one pass; the stages of the
    call add up to no more than it takes (10 % for the timing itself)."""
    B, T, H, D = 1, 16384, 16, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, k, v = (torch.randn(B, T, H, D, generator=g, device="cuda").bfloat16() for _ in range(3))
    q, k = (torch.nn.functional.normalize(x, dim=-1) for x in (q, k))
    alpha, beta = (torch.sigmoid(torch.randn(B, T, H, generator=g, device="cuda")) for _ in range(2))
    ws = gdn.workspace(q, v)
    out, st = torch.empty_like(v), torch.empty(B, H, D, D, device="cuda")
    times = []
    for _ in range(8):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(10):
            gdn.forward(q, k, v, alpha, beta, None, out=out, state_out=st, ws=ws)
        e1.record()
        torch.cuda.synchronize()
        times.append(e0.elapsed_time(e1) / 10)
    stages = min(sum(gdn.gdn_profile_stages(q, k, v, alpha, beta, None, out, st, ws, reps=10)) for _ in range(3))
    assert stages <= 1.1 * statistics.median(times), (stages, times)
