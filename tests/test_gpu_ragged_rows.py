"""Row-major scores whose row length is no multiple of 8: rows start at any 2-byte boundary, the last
chunk of a row straddles the next row and the very last one the end of the tensor.  The matrix-core
prefill kernels against the float64 oracle, every row; nothing beyond a row's last visible key, and
nothing outside the tensor, is written."""
import numpy as np
import pytest
import torch

from oracle import cref
from paper_2408_01890_amd import lisa, synth
from tests import helpers as hp
from tests.test_gpu_parity import SENTINEL, check_prefill, log, tuned  # noqa: F401

pytestmark = pytest.mark.gpu
DEV = "cuda"
GUARD = 64


def guarded(shape):
    """A score tensor in the middle of a larger buffer of sentinels, and the two guards."""
    n = int(np.prod(shape))
    buf = torch.full((n + 2 * GUARD,), SENTINEL, dtype=torch.float16, device=DEV)
    return buf[GUARD:GUARD + n].view(shape), buf[:GUARD], buf[GUARD + n:]


def untouched(scores, guards, Lq, Lk):
    above = torch.ones(Lq, Lk, dtype=torch.bool, device=DEV).triu(Lk - Lq + 1)
    return bool(torch.all(scores[..., above] == SENTINEL)) and all(bool(torch.all(g == SENTINEL)) for g in guards)


STD = [  # B, H, Hkv, Lq, Lk: one key past a chunk, one short of one, odd, a chunk of rows, below one tile
    (2, 4, 2, 33, 33), (1, 8, 8, 95, 95), (1, 3, 3, 130, 257), (2, 2, 1, 2, 9), (1, 4, 4, 129, 129)]


@pytest.mark.parametrize("B,H,Hkv,Lq,Lk", STD)
def test_std_layer_ragged_rows(B, H, Hkv, Lq, Lk):
    log(f"[case] ragged std B{B} H{H}/{Hkv} {Lq}x{Lk}")
    g = torch.Generator(device=DEV).manual_seed(5)
    q = torch.randn((B, H, Lq, 128), generator=g, device=DEV).to(torch.bfloat16)
    k, v = (torch.randn((B, Hkv, Lk, 128), generator=g, device=DEV).to(torch.bfloat16) for _ in range(2))
    scores, *guards = guarded((B, H, Lq, Lk))
    _, out = lisa.std_attn_scores(q, k, v, scores_out=scores)
    torch.cuda.synchronize()
    assert lisa.last_path() == "mfma_std"
    assert untouched(scores, guards, Lq, Lk)
    rows, tol = np.arange(Lq), hp.TOL[torch.bfloat16]
    for b in range(B):
        ref = hp.oracle_std_rows(q, k, b, rows)
        assert hp.scores_row_rel_err(hp.gather_score_rows(scores, b, rows), ref, rows, Lq, Lk) <= tol
        o_ref = cref.softmax_v_rows(hp.f64(v[b]), rows, ref, Lq)
        assert hp.row_rel_err(hp.gather_out_rows(out, b, rows), o_ref) <= tol


LISA = [  # H, Hkv, Lq, Lk, F, mix, knobs, path
    (8, 4, 97, 97, 32, "add", {}, "mfma_fused"),
    (8, 8, 1, 9, 32, "add", {}, "mfma_fused"),
    (16, 16, 47, 351, 64, "add", dict(prefill_split=4, prefill_groups=1), "mfma_fused"),
    (32, 8, 161, 161, 64, "add", dict(prefill_groups=2, prefill_pair=1, prefill_split=2), "mfma_fused"),
    (32, 8, 68, 131, 64, "add", dict(prefill_groups=1), "mfma_fused"),
    (32, 32, 63, 190, 64, "add", dict(prefill_slices=2, prefill_pair=1), "mfma_fused"),
    (40, 40, 65, 65, 80, "add", dict(prefill_slices=2), "mfma_fused"),
    (24, 24, 79, 79, 64, "add", {}, "mfma_fused"),
    (16, 8, 79, 79, 64, "concat", {}, "mfma_scores"),
    (32, 8, 50, 243, 256, "concat", {}, "mfma_scores"),
    (40, 40, 33, 33, 256, "concat", {}, "mfma_scores"),
    (8, 8, 45, 77, 160, "add", {}, "generic"),               # float32 scores through the matrix-core softmax
]


@pytest.mark.parametrize("emit", [True, False])
@pytest.mark.parametrize("case", LISA, ids=lambda c: f"h{c[0]}_{c[2]}x{c[3]}_f{c[4]}_{c[5]}")
def test_lisa_layer_ragged_rows(case, emit, tuned):
    H, Hkv, Lq, Lk, F, mix, knobs, path = case
    B = 2
    log(f"[case] ragged lisa {case} emit={emit}")
    tuned(**knobs)
    cfg = synth.LayerShape(f"ragged_h{H}_{Lq}x{Lk}", "bf16", B, H, Hkv, Lk, 256, 128, 20, F)
    inp = synth.make_prefill_inputs(cfg, 300 + Lk, DEV, mix=mix, ffn="fan_in", std_layer=False)
    inp["q_lr"] = inp["q_lr"][:, :, Lk - Lq:].contiguous()
    g = torch.Generator(device=DEV).manual_seed(9)
    prev = torch.randn((B, H, Lq, Lk), generator=g, device=DEV).to(torch.float16)
    m = lisa.MIX_CONCAT if mix == "concat" else lisa.MIX_ADD
    scores, *guards = guarded((B, H, Lq, Lk))
    out, _ = lisa.lisa_attn_prefill(inp["q_lr"], inp["k_lr"], inp["v"], prev, inp["w1"], inp["w2"], mix=m,
                                    write_scores=emit, scores_out=scores if emit else None)
    torch.cuda.synchronize()
    assert lisa.last_path() == path
    assert untouched(scores, guards, Lq, Lk)
    check_prefill(cfg, inp, prev, out, scores if emit else None, {b: np.arange(Lq) for b in range(B)},
                  mix=int(mix == "concat"))
