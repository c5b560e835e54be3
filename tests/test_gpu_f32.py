"""float32 prefill layers at the edges of their tiles (16 query rows, 16 keys, four waves of key tiles; 64
keys per lane group in the scores kernel): every row against the float64 oracle at 1e-5."""
import numpy as np
import pytest
import torch

from oracle import cref
from paper_2408_01890_amd import lisa, synth
from tests import helpers as hp
from tests.test_gpu_parity import SENTINEL, log

pytestmark = pytest.mark.gpu
DEV = "cuda"
TOL = hp.TOL[torch.float32]

CASES = [  # B, H, Hkv, Lq, Lk, d_k, r, F
    (1, 8, 8, 2, 2, 64, 11, 32),
    (2, 8, 8, 33, 33, 64, 11, 32),
    (1, 8, 2, 17, 129, 128, 5, 33),       # a chunk of rows; d_k = 128; four heads per kv head
    (1, 3, 3, 64, 64, 64, 1, 8),         # fewer heads than the padded form
    (2, 13, 13, 65, 80, 64, 7, 40),
    (1, 32, 8, 47, 47, 128, 22, 64),      # widest form
    (1, 8, 8, 260, 260, 64, 11, 32),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"h{c[1]}_{c[3]}x{c[4]}_dk{c[5]}")
def test_f32_layers(case):
    B, H, Hkv, Lq, Lk, dk, r, F = case
    log(f"[case] f32 {case}")
    cfg = synth.LayerShape(f"f32_h{H}_{Lq}x{Lk}", "f32", B, H, Hkv, Lk, 128, dk, r, F)
    inp = synth.make_prefill_inputs(cfg, 400 + Lk, DEV, ffn="fan_in")
    for k in ("q", "q_lr"):
        inp[k] = inp[k][:, :, Lk - Lq:].contiguous()
    a0 = torch.full((B, H, Lq, Lk), SENTINEL, dtype=torch.float32, device=DEV)
    a1 = torch.full_like(a0, SENTINEL)
    _, o0 = lisa.std_attn_scores(inp["q"], inp["k"], inp["v"], scores_out=a0)
    o1, _ = lisa.lisa_attn_prefill(inp["q_lr"], inp["k_lr"], inp["v"], a0, inp["w1"], inp["w2"], scores_out=a1)
    o2, _ = lisa.lisa_attn_prefill(inp["q_lr"], inp["k_lr"], inp["v"], a0, inp["w1"], inp["w2"], write_scores=False)
    torch.cuda.synchronize()
    above = torch.ones(Lq, Lk, dtype=torch.bool, device=DEV).triu(Lk - Lq + 1)
    assert bool((a0[..., above] == SENTINEL).all()) and bool((a1[..., above] == SENTINEL).all())
    assert torch.equal(o1, o2)
    rows = np.arange(Lq)
    for b in range(B):
        ref = hp.oracle_std_rows(inp["q"], inp["k"], b, rows)
        assert hp.scores_row_rel_err(hp.gather_score_rows(a0, b, rows), ref, rows, Lq, Lk) <= TOL
        o_ref = cref.softmax_v_rows(hp.f64(inp["v"][b]), rows, ref, Lq)
        assert hp.row_rel_err(hp.gather_out_rows(o0, b, rows), o_ref) <= TOL
        a_ref, o_ref = cref.lisa_rows(hp.f64(inp["q_lr"][b]), hp.f64(inp["k_lr"][b]), hp.f64(inp["v"][b]), hp.f64(inp["w1"]),
                                      hp.f64(inp["w2"]), rows, hp.gather_score_rows(a0, b, rows))
        assert hp.scores_row_rel_err(hp.gather_score_rows(a1, b, rows), a_ref, rows, Lq, Lk) <= TOL
        assert hp.row_rel_err(hp.gather_out_rows(o1, b, rows), o_ref) <= TOL
