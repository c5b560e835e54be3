"""Projection of one to four token rows, a wave per pair of weight rows: odd ranks (a row without a partner), several
sequences and tokens, cached positions, both cache layouts, widths of whole and part batches of loads."""
import numpy as np
import pytest

from paper_2408_01890_amd import synth
from tests.test_gpu_parity import DEV, check_projection, log
from tests.test_gpu_split import stages


pytestmark = pytest.mark.gpu
CASES = [  # B, H, Hkv, L, d_model, d_k, r, theta, pos0, dim_major, extra
    (1, 32, 8, 1, 4096, 128, 22, 500000.0, 300, True, 7), (2, 8, 4, 1, 512, 64, 11, None, 5, True, 0),
    (1, 5, 1, 3, 2560, 32, 1, None, 0, False, 3), (4, 3, 3, 1, 5120, 96, 32, 10000.0, 17, False, 0), (1, 40, 8, 2, 1536, 128, 20, 10000.0, 9, True, 1)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"B{c[0]}H{c[1]}-{c[2]}L{c[3]}d{c[4]}r{c[6]}")
def test_projection_of_few_rows(case):
    B, H, Hkv, L, D, dk, r, theta, pos0, dim_major, extra = case
    log(f"[case] projection rows {case}")
    cfg = synth.LayerShape("proj_rows", "bf16", B, H, Hkv, L, D, dk, r, 64, theta)
    pin = synth.make_projection_inputs(cfg, device=DEV)
    path, ran = stages(lambda: check_projection(cfg, pin, {b: np.arange(L) for b in range(B)}, theta, pos0, dim_major, pos0 + L + extra))
    assert path == "project_skinny" and "k_project_rows" in ran
