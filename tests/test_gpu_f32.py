"""float32 prefill layers at the edges of their tiles (attention: 16 query rows, the 16-key tiles dealt to four waves;
scores: tiles of 16 rows x 16 keys, runs of them in a workgroup where there are many), against the float64
oracle at 1e-5."""
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


@pytest.mark.parametrize("dtype,dk", [("f32", 64), ("f32", 128), ("bf16", 128)])
@pytest.mark.parametrize("B,H,Hkv,Lq,Lk", [
    (1, 8, 8, 16, 128), (1, 8, 8, 17, 129),    # a workgroup's tiles, and a second workgroup with one
    (1, 4, 2, 2, 3001), (2, 3, 3, 47, 1031),   # few rows, many keys; row blocks that see fewer tiles than there are workgroups
])
def test_f32_scores_alone_are_those_of_the_layer(B, H, Hkv, Lq, Lk, dtype, dk):
    """Without V the tiles of a row block are dealt to several workgroups: the same scores bit for bit, and no others."""
    if dtype == "bf16":
        Lk += (Lk % 8 == 0)                                   # (row-major rows of ragged length run in float32)
    log(f"[case] f32 scores alone {dtype} {B} {H} {Lq}x{Lk} dk{dk}")
    g = torch.Generator(device=DEV).manual_seed(6)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.randn((B, H, Lq, dk), generator=g, device=DEV).to(dt)
    k, v = (torch.randn((B, Hkv, Lk, dk), generator=g, device=DEV).to(dt) for _ in range(2))
    a, b = (torch.full((B, H, Lq, Lk), SENTINEL, dtype=lisa.score_dtype(dt), device=DEV) for _ in range(2))
    lisa.std_attn_scores(q, k, v, scores_out=a)
    lisa.std_attn_scores(q, k, scores_out=b)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    for n in range(B):
        rows = np.arange(Lq)
        ref = hp.oracle_std_rows(q, k, n, rows)
        tol = TOL if dtype == "f32" else 2.0 ** -8           # half scores: see test_gpu_ragged_rows.py
        assert hp.scores_row_rel_err(hp.gather_score_rows(b, n, rows), ref, rows, Lq, Lk) <= tol


@pytest.mark.parametrize("B,H,L,F,silu", [
    (1, 4, 897, 16, False),      # 57 x 57 tiles: runs of two, the last one clipped
    (3, 4, 900, 16, True),       # runs of six that share the staged weights
    (1, 8, 50, 33, True),
    (1, 32, 40, 128, True),      # weights that do not fit the LDS beside A_delta: the generic scores kernel
])
def test_f32_scores_in_runs_of_tiles(B, H, L, F, silu):
    log(f"[case] f32 scores B{B} H{H} {L} F{F} silu={silu}")
    cfg = synth.LayerShape(f"f32_runs_{L}", "f32", B, H, H, L, 128, 64, 11, F)
    inp = synth.make_prefill_inputs(cfg, 500 + L, DEV, ffn="fan_in", std_layer=False)
    g = torch.Generator(device=DEV).manual_seed(23)
    prev = torch.randn((B, H, L, L), generator=g, device=DEV)
    out, scores = lisa.lisa_attn_prefill(inp["q_lr"], inp["k_lr"], inp["v"], prev, inp["w1"], inp["w2"],
                                         act=lisa.ACT_SILU if silu else lisa.ACT_RELU)
    torch.cuda.synchronize()
    rows = np.unique(np.clip([0, 15, 16, 31, 47, 95, 447, 448, L - 17, L - 2, L - 1], 0, L - 1))
    for b in range(B):
        a_ref, o_ref = cref.lisa_rows(*(hp.f64(inp[n][b]) for n in ("q_lr", "k_lr", "v")), hp.f64(inp["w1"]), hp.f64(inp["w2"]),
                                      rows, hp.gather_score_rows(prev, b, rows), act=cref.ACT_SILU if silu else cref.ACT_RELU)
        assert hp.scores_row_rel_err(hp.gather_score_rows(scores, b, rows), a_ref, rows, L, L) <= TOL
        assert hp.row_rel_err(hp.gather_out_rows(out, b, rows), o_ref) <= TOL


def _rows_err(out, scores, v, Lq):
    """Worst row of `out` against the float64 softmax of the float32 scores that the layer took or emitted."""
    worst, rows = 0.0, np.arange(Lq)
    for b in range(out.shape[0]):
        ref = cref.softmax_v_rows(hp.f64(v[b]), rows, hp.gather_score_rows(scores, b, rows), Lq)
        worst = max(worst, hp.row_rel_err(hp.gather_out_rows(out, b, rows), ref))
    return worst


@pytest.mark.parametrize("dk", [64, 128])
@pytest.mark.parametrize("shift", [0.0, 50.0, -200.0, 200.0, 1000.0])
def test_f32_softmax_far_from_zero(shift, dk):
    """The softmax depends on the differences of the scores alone, so the distance of all of them from zero costs
    nothing: s - m is exact to its own float32 rounding (2^-24 of a difference of 8 or less)."""
    log(f"[case] f32 softmax around {shift} dk{dk}")
    B, H, Hkv, Lq, Lk = 1, 8, 4, 70, 301
    g = torch.Generator(device=DEV).manual_seed(17)
    prev = torch.randn((B, H, Lq, Lk), generator=g, device=DEV) + shift
    q = torch.randn((B, H, Lq, dk), generator=g, device=DEV)
    k, v = (torch.randn((B, Hkv, Lk, dk), generator=g, device=DEV) for _ in range(2))
    q[..., 0], k[..., 0] = abs(shift) ** 0.5, shift / max(abs(shift), 1.0) ** 0.5 * dk ** 0.5
    out, _ = lisa.lisa_attn_prefill(None, None, v, prev, None, None, mix=lisa.MIX_SHARE)
    scores, o_std = lisa.std_attn_scores(q, k, v, scores_out=torch.zeros_like(prev))
    torch.cuda.synchronize()
    assert _rows_err(out, prev, v, Lq) <= TOL
    assert _rows_err(o_std, scores, v, Lq) <= TOL
