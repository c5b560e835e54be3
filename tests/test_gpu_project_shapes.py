"""Projection at the sizes where each tile shape is chosen (one and several rounds of workgroups, ragged last tiles, equal
shares of tiles per XCD along either axis): the sums run in the same order in all of them, so the results agree bit for bit
with the 256 x 192 tiles; those are checked against a plain product elsewhere."""
import pytest
import torch

from paper_2408_01890_amd import lisa, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("H,Hkv,r,dk,L,B", [
    (32, 8, 22, 128, 129, 1),        # 128 x 64
    (32, 8, 22, 128, 1000, 1),       # 128 x 128, one round
    (32, 8, 22, 128, 2300, 1),       # 128 x 192, one round
    (32, 8, 22, 128, 1501, 2),       # 128 x 256, one round; sequences end inside a tile
    (32, 8, 22, 128, 4300, 1),       # 128 x 192, two rounds
    (32, 32, 22, 128, 1101, 1),      # 128 x 128, two rounds
    (32, 32, 22, 128, 2204, 1),      # 256 x 256
    (40, 40, 20, 128, 1301, 1),
    (8, 4, 8, 64, 20000, 1),         # many row tiles of few columns: shares along the rows
])
def test_projection_tile_shapes_agree(H, Hkv, r, dk, L, B):
    cfg = synth.LayerShape("proj_shapes", "bf16", B, H, Hkv, L, 192, dk, r, 64, 10000.0)
    pin = synth.make_projection_inputs(cfg, device=DEV)

    def project():
        return lisa.lisa_project_qkv(pin["x"], pin["w"], H, Hkv, r, dk, rope_theta=10000.0)

    got = project()
    for tn in (192, 256):
        with lisa.tune(project_tn=tn):
            want = project()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
