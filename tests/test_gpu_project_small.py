"""Projection with 128 x 64 tiles (few token rows): the sizes of the other geometries, whose sums run in the same
order, so the results agree bit for bit; and one past the edges of its own tiles."""
import numpy as np
import pytest
import torch

from paper_2408_01890_amd import lisa, synth
from tests.test_gpu_parity import PROJ_MFMA, check_projection, log

pytestmark = pytest.mark.gpu
DEV = "cuda"
EDGES = [  # B, H, Hkv, L, d_model, d_k, r, theta, pos0, dim_major, extra
    (1, 8, 2, 129, 128, 128, 22, 10000.0, 0, True, 7), (1, 3, 3, 257, 64, 32, 7, None, 5, False, 0),
    (3, 33, 11, 85, 192, 64, 32, 500000.0, 0, True, 1),
    (1, 64, 64, 300, 192, 128, 32, None, 0, False, 0)]      # more small tiles than compute units: 128 x 192 instead


@pytest.mark.parametrize("case", PROJ_MFMA + EDGES, ids=lambda c: f"B{c[0]}H{c[1]}-{c[2]}L{c[3]}d{c[4]}r{c[6]}")
def test_projection_small_tiles(case):
    B, H, Hkv, L, D, dk, r, theta, pos0, dim_major, extra = case
    log(f"[case] projection small tiles {case}")
    cfg = synth.LayerShape("proj_small", "bf16", B, H, Hkv, L, D, dk, r, 64, theta)
    pin = synth.make_projection_inputs(cfg, device=DEV)
    path = check_projection(cfg, pin, {b: np.arange(L) for b in range(B)}, theta, pos0, dim_major, pos0 + L + extra)
    assert path == "project_mfma"
    small = lisa.lisa_project_qkv(pin["x"], pin["w"], H, Hkv, r, dk, rope_theta=theta or 0.0, dim_major=dim_major)
    with lisa.tune(project_tn=192):
        wide = lisa.lisa_project_qkv(pin["x"], pin["w"], H, Hkv, r, dk, rope_theta=theta or 0.0, dim_major=dim_major)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(small, wide))
