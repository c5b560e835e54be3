"""Row-major scores whose row length is no multiple of 8: rows start at any 2-byte boundary.  Such layers run in float32
arithmetic whatever their element type, and are held to its tolerance: against the float64 oracle, every row;
nothing beyond a row's last visible key, and nothing outside the tensor, is written."""
import numpy as np
import pytest
import torch

from oracle import cref
from paper_2408_01890_amd import lisa, synth
from tests import helpers as hp
from tests.test_gpu_parity import SENTINEL, log

pytestmark = pytest.mark.gpu
DEV = "cuda"
GUARD = 64
TOL_O = hp.TOL[torch.float32]       # O leaves as float32
# A_n leaves as half, rounded once: half a spacing, 2^-9 below 8, of rows whose RMS is 1 or more and whose largest
# element is below 8 RMS (or scaled alike); as much again for the sums
TOL_A = 2.0 ** -8


def guarded(shape):
    """A score tensor in the middle of a larger buffer of sentinels, and the two guards."""
    n = int(np.prod(shape))
    buf = torch.full((n + 2 * GUARD,), SENTINEL, dtype=torch.float16, device=DEV)
    return buf[GUARD:GUARD + n].view(shape), buf[:GUARD], buf[GUARD + n:]


def untouched(scores, guards, Lq, Lk):
    above = torch.ones(Lq, Lk, dtype=torch.bool, device=DEV).triu(Lk - Lq + 1)
    return bool(torch.all(scores[..., above] == SENTINEL)) and all(bool(torch.all(g == SENTINEL)) for g in guards)


STD = [  # B, H, Hkv, Lq, Lk: one key past a tile, one short of one, odd, a chunk of rows, below one tile
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
    assert lisa.last_path() == "generic"
    assert untouched(scores, guards, Lq, Lk)
    out16, _ = lisa.std_attn_scores(q, k, v, want_scores=False, out_dtype=torch.bfloat16)[::-1]
    assert torch.equal(out16, out.to(torch.bfloat16))
    rows = np.arange(Lq)
    for b in range(B):
        ref = hp.oracle_std_rows(q, k, b, rows)
        assert hp.scores_row_rel_err(hp.gather_score_rows(scores, b, rows), ref, rows, Lq, Lk) <= TOL_A
        o_ref = cref.softmax_v_rows(hp.f64(v[b]), rows, ref, Lq)
        assert hp.row_rel_err(hp.gather_out_rows(out, b, rows), o_ref) <= TOL_O


def check_rows(inp, prev, out, scores, rows, mix=0):
    Lq, Lk = inp["q_lr"].shape[2], inp["k_lr"].shape[2]
    for b in range(inp["v"].shape[0]):
        a_ref, o_ref = hp.oracle_lisa_rows(inp, b, rows, hp.gather_score_rows(prev, b, rows), mix=mix)
        err_o = hp.row_rel_err(hp.gather_out_rows(out, b, rows), o_ref)
        err_a = 0.0 if scores is None else hp.scores_row_rel_err(hp.gather_score_rows(scores, b, rows), a_ref, rows, Lq, Lk)
        log(f"[parity] ragged {Lq}x{Lk}: err_out={err_o:.3e} err_scores={err_a:.3e}")
        assert err_o <= TOL_O and err_a <= TOL_A


LISA = [  # H, Hkv, Lq, Lk, F, mix, act
    (8, 4, 97, 97, 32, "add", "relu"),
    (8, 8, 1, 9, 32, "add", "relu"),                          # a single row
    (16, 16, 47, 351, 64, "add", "relu"),
    (32, 8, 161, 161, 64, "add", "silu"),
    (12, 4, 68, 131, 40, "add", "relu"),                      # heads and hidden units that fill no block
    (40, 40, 65, 65, 80, "add", "relu"),
    (24, 24, 79, 79, 64, "add", "relu"),
    (16, 8, 79, 79, 64, "concat", "silu"),
    (32, 8, 50, 243, 256, "concat", "relu"),
    (6, 3, 33, 50, 24, "concat", "relu"),
    (40, 40, 33, 33, 128, "concat", "relu"),
    (40, 40, 33, 33, 256, "concat", "relu"),                  # weights that do not fit the LDS beside A_delta
    (8, 8, 45, 77, 160, "add", "relu"),
    (16, 16, 1100, 1100 + 1, 64, "add", "relu"),              # runs of key tiles that share the staged weights
]


@pytest.mark.parametrize("emit", [True, False])
@pytest.mark.parametrize("case", LISA, ids=lambda c: f"h{c[0]}_{c[2]}x{c[3]}_f{c[4]}_{c[5]}_{c[6]}")
def test_lisa_layer_ragged_rows(case, emit):
    H, Hkv, Lq, Lk, F, mix, act = case
    B = 2
    log(f"[case] ragged lisa {case} emit={emit}")
    cfg = synth.LayerShape(f"ragged_h{H}_{Lq}x{Lk}", "bf16", B, H, Hkv, Lk, 256, 128, 20, F)
    inp = synth.make_prefill_inputs(cfg, 300 + Lk, DEV, mix=mix, ffn="fan_in", std_layer=False)
    inp["q_lr"] = inp["q_lr"][:, :, Lk - Lq:].contiguous()
    g = torch.Generator(device=DEV).manual_seed(9)
    prev = torch.randn((B, H, Lq, Lk), generator=g, device=DEV).to(torch.float16)
    scores, *guards = guarded((B, H, Lq, Lk))
    out, _ = lisa.lisa_attn_prefill(inp["q_lr"], inp["k_lr"], inp["v"], prev, inp["w1"], inp["w2"], write_scores=emit,
                                    mix=lisa.MIX_CONCAT if mix == "concat" else lisa.MIX_ADD,
                                    act=lisa.ACT_SILU if act == "silu" else lisa.ACT_RELU,
                                    scores_out=scores if emit else None)
    torch.cuda.synchronize()
    assert lisa.last_path() == "generic"
    assert untouched(scores, guards, Lq, Lk)
    rows = np.arange(Lq) if Lq < 500 else np.array([0, 15, 16, 500, Lq - 2, Lq - 1])
    if act == "relu":
        return check_rows(inp, prev, out, scores if emit else None, rows, int(mix == "concat"))
    for b in range(B):
        a_ref, o_ref = cref.lisa_rows(*(hp.f64(inp[n][b]) for n in ("q_lr", "k_lr", "v")), hp.f64(inp["w1"]), hp.f64(inp["w2"]),
                                      rows, hp.gather_score_rows(prev, b, rows), mix=int(mix == "concat"), act=cref.ACT_SILU)
        assert hp.row_rel_err(hp.gather_out_rows(out, b, rows), o_ref) <= TOL_O
        if emit:
            assert hp.scores_row_rel_err(hp.gather_score_rows(scores, b, rows), a_ref, rows, Lq, Lk) <= TOL_A


def test_lisa_layer_ragged_rows_in_chunks():
    """More float32 scores and padded operands than the workspace holds at a time (256 MB): the rows on both sides of the border."""
    B, H, L = 2, 32, 1031
    log(f"[case] ragged lisa in chunks {L}")
    cfg = synth.LayerShape("ragged_chunks", "bf16", B, H, 8, L, 256, 128, 22, 64)
    inp = synth.make_prefill_inputs(cfg, 77, DEV, ffn="fan_in", std_layer=False)
    g = torch.Generator(device=DEV).manual_seed(9)
    prev = torch.randn((B, H, L, L), generator=g, device=DEV).to(torch.float16)
    scores, *guards = guarded((B, H, L, L))
    lisa.profile_enable(True)
    try:
        out, _ = lisa.lisa_attn_prefill(inp["q_lr"], inp["k_lr"], inp["v"], prev, inp["w1"], inp["w2"], scores_out=scores)
        torch.cuda.synchronize()
        assert lisa.profile_collect()["k_split_scores"][0] == 2        # (launches)
    finally:
        lisa.profile_enable(False)
    assert untouched(scores, guards, L, L)
    operands = B * H * 1040 * 64 + B * 8 * 1088 * 64                   # rows of 64 bytes, L rounded up to 16 and to 64
    edge = ((256 << 20) - operands) // (B * H * 1056 * 4) // 16 * 16   # float32 scores in tiles of 32 keys
    assert edge == 960
    check_rows(inp, prev, out, scores, np.array([0, 17, edge - 17, edge - 16, edge - 1, edge, edge + 1, edge + 15, edge + 16, L - 1]))


@pytest.mark.parametrize("mix", [lisa.MIX_PLUS, lisa.MIX_SHARE])
def test_layers_without_a_module_ragged_rows(mix):
    B, H, L = 2, 32, 1031
    log(f"[case] ragged without a module mix={mix}")
    g = torch.Generator(device=DEV).manual_seed(3)
    q, k = (torch.randn((B, n, L, 22), generator=g, device=DEV).to(torch.bfloat16) for n in (H, 8))
    v = torch.randn((B, 8, L, 128), generator=g, device=DEV).to(torch.bfloat16)
    prev = torch.randn((B, H, L, L), generator=g, device=DEV).to(torch.float16)
    share = mix == lisa.MIX_SHARE
    out, _ = lisa.lisa_attn_prefill(None if share else q, None if share else k, v, prev, None, None, mix=mix)
    torch.cuda.synchronize()
    rows = np.array([0, 700, 1007, 1008, L - 1])
    for b in range(B):
        _, o_ref = cref.lisa_rows(None if share else hp.f64(q[b]), None if share else hp.f64(k[b]), hp.f64(v[b]), None, None,
                                  rows, hp.gather_score_rows(prev, b, rows), mix=mix, Lq=L)
        assert hp.row_rel_err(hp.gather_out_rows(out, b, rows), o_ref) <= TOL_O
