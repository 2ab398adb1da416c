"""The fused operator's latent coordinates where their steps can go wrong: widths
below, at and beside the steps of the key features (4 or 8 tokens a pass, 52 or 56
to the next block) and of the output (192 to a wave's next tile), a width no token
reaches, and splits that end inside a block.  Enough frames and heads that an output
wave takes several tiles.  Against the fp64 oracle at the bf16 path's bound."""
import pytest

import gdn_inputs
from test_gpu_frame_fused import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,lat_w", [(64, 64, w) for w in (1, 3, 8, 55, 56, 57, 191, 192, 193, 2**31 - 1)] +
                         [(128, 64, 3), (128, 64, 52), (128, 64, 193)])
def test_widths(gdn, D, H, lat_w):
    inp = gdn_inputs.make_fused_inputs(1, 4, frame_tokens=413, H=H, Dk=D, Dv=D, lat_w=lat_w, t0=2,
                                       seed=39000 + D + lat_w % 997)
    check(gdn, inp, f"D{D} lat_w={lat_w}")


@pytest.mark.parametrize("splits", [1, 2, 3])
def test_ragged_splits(gdn, splits):
    inp = gdn_inputs.make_fused_inputs(1, 2, frame_tokens=331, H=2, Dk=128, Dv=64, lat_w=37, seed=39070 + splits)
    check(gdn, inp, f"splits={splits}", token_splits=splits)
