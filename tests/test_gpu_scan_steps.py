"""The scan over chunks where its loops and its choice of workgroup can go wrong:
every remainder of the unrolled loops (four compute steps, three output steps),
a partial last chunk in each of them, one and two column tiles per workgroup,
and group counts around the group scan's four register sets.  Against the fp64
oracle; bounds as in test_gpu_parity (1e-4 in fp32, 2e-2 in bf16)."""
import pytest

import gdn_inputs
from test_gpu_parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [127, 129, 192, 256, 320, 385, 448, 511])
def test_step_remainders(gdn, dtype, T):
    inp = gdn_inputs.make_inputs(1, B=1, T=T, H=2, Dk=128, Dv=64, dtype=dtype, seed=9100 + T)
    check(gdn, inp, f"T{T} H2 {dtype}")


@pytest.mark.parametrize("B,H,Dk,Dv", [(1, 33, 128, 128), (3, 22, 64, 64), (1, 32, 128, 128)])
@pytest.mark.parametrize("T", [1, 190, 257])
def test_two_column_tiles(gdn, B, H, Dk, Dv, T):
    """264 tiles (more than CUs: pairs), 264 of D = 64, and 256 (one tile each)."""
    inp = gdn_inputs.make_inputs(1, B=B, T=T, H=H, Dk=Dk, Dv=Dv, dtype="bf16", seed=9300 + H + T)
    check(gdn, inp, f"B{B} T{T} H{H} D{Dk}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,G", [(192, 1), (256, 1), (320, 1), (450, 1), (640, 2)])
def test_group_counts(gdn, dtype, T, G):
    inp = gdn_inputs.make_inputs(1, B=1, T=T, H=2, Dk=64, Dv=128, dtype=dtype, seed=9500 + T)
    check(gdn, inp, f"T{T} groups of {G} {dtype}", scan_group=G)
