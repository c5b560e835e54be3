"""Projection at the sizes where each tile shape is chosen (one and several rounds of workgroups, ragged last tiles, equal
shares of tiles per XCD along either axis): the sums run in the same order in all of them, so the results agree bit for bit
with those of the 256-row tiles; and every shape at the edges of what the kernel takes, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2408_01890_amd import lisa, synth
from tests.test_gpu_parity import PROJ_MFMA, check_projection, log
from tests.test_gpu_project_small import EDGES

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("shape,H,Hkv,r,dk,L,B", [
    (6, 32, 8, 22, 128, 129, 1),       # 128 x 64
    (5, 32, 8, 22, 128, 1000, 1),      # 128 x 128, one round
    (5, 8, 4, 8, 64, 10900, 1),        # 128 x 128, two rounds
    (3, 32, 8, 22, 128, 2300, 1),      # 128 x 192, one round; shares along the rows
    (3, 64, 64, 32, 128, 300, 1),      # the same; shares along the columns
    (4, 32, 8, 22, 128, 8100, 1),      # 128 x 192, several rounds
    (2, 32, 32, 22, 128, 1101, 1),     # 128 x 256, one round
    (2, 32, 8, 22, 128, 1501, 2),      # the same; sequences end inside a tile
    (1, 32, 8, 22, 128, 4300, 1),      # 256 x 192, in equal shares
    (1, 40, 40, 20, 128, 1301, 1),     # the same, one round
    (0, 32, 32, 22, 128, 2204, 1),     # 256 x 256
    (0, 8, 4, 8, 64, 20000, 1),        # many row tiles of few columns
])
def test_projection_tile_shapes_agree(shape, H, Hkv, r, dk, L, B):
    cfg = synth.LayerShape("proj_shapes", "bf16", B, H, Hkv, L, 192, dk, r, 64, 10000.0)
    pin = synth.make_projection_inputs(cfg, device=DEV)
    assert lisa.project_choice(torch.bfloat16, B, L, 192, H, Hkv, r, dk) == shape

    def project():
        return lisa.lisa_project_qkv(pin["x"], pin["w"], H, Hkv, r, dk, rope_theta=10000.0)

    got = project()
    for tn in (192, 256):
        with lisa.tune(project_tn=tn):
            want = project()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("shape", range(7))
@pytest.mark.parametrize("case", PROJ_MFMA + EDGES, ids=lambda c: f"B{c[0]}H{c[1]}-{c[2]}L{c[3]}d{c[4]}r{c[6]}")
def test_projection_every_shape_at_the_edges(case, shape):
    B, H, Hkv, L, D, dk, r, theta, pos0, dim_major, extra = case
    log(f"[case] projection shape {shape} {case}")
    cfg = synth.LayerShape("proj_edges", "bf16", B, H, Hkv, L, D, dk, r, 64, theta)
    pin = synth.make_projection_inputs(cfg, device=DEV)
    with lisa.tune(project_tn=shape):
        assert lisa.project_choice(torch.bfloat16, B, L, D, H, Hkv, r, dk) == shape
        path = check_projection(cfg, pin, {b: np.arange(L) for b in range(B)}, theta, pos0, dim_major, pos0 + L + extra)
    assert path == "project_mfma"
