"""The fp32 fused operator's rotation table and unrotated Gram pass at the edges of
their ranges: one-token frames of one head (the table fills its region), grids
narrower and wider than a frame, one and several splits for both head sizes (with
several, only tiles on and above the diagonal are formed).  Against the fp64
oracle at the fp32 path's bound (1e-4)."""
import pytest

from test_gpu_frame_fused_f32 import check, fused_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("F,N,lat_w", [(1, 1, 1), (1, 1, 2**31 - 1), (5, 1, 3), (1, 70, 1), (2, 67, 2**31 - 1), (1, 129, 128)])
def test_table_rows(gdn, D, F, N, lat_w):
    inp = fused_inputs(1, F, frame_tokens=N, B=1, H=1, Dk=D, Dv=D, lat_w=lat_w, t0=9, seed=49600 + 7 * F + N + D)
    check(gdn, inp, f"F{F} N{N} D{D} lat_w={lat_w}", bidirectional=F > 1)


@pytest.mark.parametrize("Dk,Dv", [(64, 128), (128, 64)])
@pytest.mark.parametrize("splits", [1, 2, 5])
def test_unrotated_gram_splits(gdn, Dk, Dv, splits):
    inp = fused_inputs(1, 2, frame_tokens=300, B=1, H=2, Dk=Dk, Dv=Dv, lat_w=20, seed=49700 + splits + Dk)
    check(gdn, inp, f"Dk{Dk} Dv{Dv} splits={splits}", token_splits=splits)
