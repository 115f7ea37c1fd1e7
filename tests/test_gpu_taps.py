"""Mixed-nest plans whose nwg_conv2d runs on the level-1 taps (U in four values
per channel pair instead of nine points), against the fp64 direct oracle, at the
edges of the contraction's blocks: both depths, channel counts that are whole
chunks of 8 and (on the quad layout) are not, output channels and tiles that are
not multiples of 4, 32, 64 or 128, more items than work-groups, several images.
"""
import numpy as np
import pytest
import torch

from oracle.direct import direct_conv2d
from paper_2102_13272_amd import nwg
from paper_2102_13272_amd.workloads import make_case
from tests.gpu_util import assert_close, dev

pytestmark = pytest.mark.gpu

MIX = nwg.NWG_TILE_MIX_F23_F33


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nwg.load_library()


# (B, M, N, H, W, r, pad)
CASES = [
    (1, 8, 1, 12, 12, 13, 6),         # one tile, one output channel, one chunk
    (1, 16, 5, 20, 31, 8, 3),         # even kernel, the smallest of depth 3
    (2, 24, 33, 26, 25, 11, 5),       # N one past a block, T = 18
    (3, 40, 64, 45, 61, 14, 6),       # the last r with level-1 digit 3 dead at depth 3
    (1, 32, 66, 100, 60, 13, 0),      # T = 32
    (2, 8, 130, 56, 56, 9, 4),        # N two past 128, T = 50
    (1, 136, 32, 24, 24, 12, 5),      # M over 128
    (1, 8, 3, 40, 40, 16, 8),         # depth 4, T = 4
    (1, 16, 36, 75, 40, 25, 12),      # T = 6
    (2, 8, 70, 60, 60, 31, 15),       # T = 8
    (1, 24, 17, 37, 37, 38, 20),      # the last r of depth 4 with digit 3 dead
    (4, 8, 32, 144, 144, 17, 8),      # T = 64: 64-tile input transform
    (3, 8, 129, 108, 72, 19, 9),      # T = 18
    (1, 12, 20, 30, 30, 13, 6),       # M = 12: the quad layout
    (1, 16, 20, 30, 30, 15, 7),       # r = 15: level-1 digit 3 live, the quad layout
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%d_M%d_N%d_%dx%d_r%d_p%d" % c)
def test_mixed_layers_on_taps_match_oracle(case):
    B, M, N, H, W, r, pad = case
    print(f"taps case {case}", flush=True)
    _, x, w = make_case(B, M, N, H, W, r, pad, seed=sum(case), x_dist="normal",
                        w_dist="fanin_normal")
    xd, wd = dev(x), dev(w)
    ref = direct_conv2d(x, w, pad)
    with nwg.Plan(B, M, N, H, W, r, pad, tile=MIX) as plan:
        y = torch.full(plan.y_shape, float("nan"), device="cuda")
        for _ in range(2):                    # the second call on the first's buffers
            plan.conv2d(xd, wd, y)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        # F(3,3) at one outer level: 3e-6 of the output, at two: 1.1e-5
        assert_close(got, ref, rel_tol=1e-5 if r <= 15 else 4e-5, what=str(case))
        # the stage calls (the public layouts) give the same convolution
        U = torch.empty(plan.u_shape, device="cuda")
        V = torch.empty(plan.v_shape, device="cuda")
        Z = torch.empty(plan.z_shape, device="cuda")
        z = torch.full(plan.y_shape, float("nan"), device="cuda")
        plan.kernel_transform(wd, U)
        plan.input_transform(xd, V)
        plan.contract(U, V, Z)
        plan.output_transform(Z, z)
        torch.cuda.synchronize()
        assert_close(got, z.cpu().numpy().astype(np.float64),
                     rel_tol=1e-5 if r <= 15 else 4e-5, what=f"{case} against the stage calls")
