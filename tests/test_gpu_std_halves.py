"""Standard prefill layers with two waves per row block (few workgroups, more than 256 keys): lengths at which one key half
has a tile more than the other, starts beyond a row's diagonal or ends in part of a tile, in both score layouts; and
the softmax from given scores behind the CONCAT module.  Against float64, every row."""
import pytest
import torch

from paper_2408_01890_amd import lisa
from tests.test_gpu_parity import log
from tests.test_gpu_split import err, reference, softmax_v, stages

pytestmark = pytest.mark.gpu
DEV = "cuda"
# probabilities as bf16: 2^-9 of each, of rows of O whose largest element is below 8 RMS (test_gpu_tiled_scores: 2e-2)
TOL_O, TOL_A = 2e-2, 2.0 ** -9

CASES = [  # Lq, Lk, causal: a tile, two, three in the last pair (row 0 sees one key); chunks behind cached keys
    (264, 264, True), (288, 288, True), (320, 320, True), (130, 1032, True), (2, 264, True), (33, 296, False), (128, 4096, True)]


@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("Lq,Lk,causal", CASES)
def test_std_layer_key_halves(Lq, Lk, causal, tiled):
    B, H, Hkv = 2, 4, 2
    log(f"[case] std halves {Lq}x{Lk} tiled={tiled}")
    g = torch.Generator(device=DEV).manual_seed(Lk)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV).to(torch.bfloat16)
    q, k, v = rn(B, H, Lq, 128), rn(B, Hkv, Lk, 128), rn(B, Hkv, Lk, 128)
    a0, o0 = lisa.std_attn_scores(q, k, v, causal=causal, tiled=tiled)
    a1, _ = lisa.std_attn_scores(q, k, causal=causal, tiled=tiled)
    torch.cuda.synchronize()
    assert lisa.last_path() == "mfma_std"
    rep = lambda t: t.cpu().double().repeat_interleave(H // Hkv, 1)
    A = q.cpu().double() @ rep(k).transpose(-1, -2).contiguous() / 128 ** 0.5
    vis = torch.ones(Lq, Lk, dtype=torch.bool).tril(Lk - Lq) if causal else torch.ones(Lq, Lk, dtype=torch.bool)
    for a in (a0, a1):
        got = (lisa.untile_scores(a, Lq, Lk) if tiled else a).cpu().double()
        assert float((got - A).abs()[..., vis].max()) <= TOL_A * float(A.abs().max())
    assert err(o0.flatten(2), softmax_v(A, rep(v), causal).flatten(2)) <= TOL_O


@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("Lq,Lk", [(264, 264), (40, 1032)])
def test_softmax_from_given_scores_key_halves(Lq, Lk, tiled):
    B, H, F, r = 1, 8, 64, 20
    log(f"[case] given halves {Lq}x{Lk} tiled={tiled}")
    g = torch.Generator(device=DEV).manual_seed(Lk)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)
    q, k, v = rn(B, H, Lq, r).to(torch.bfloat16), rn(B, H, Lk, r).to(torch.bfloat16), rn(B, H, Lk, 128).to(torch.bfloat16)
    w1, w2 = (rn(2 * H, F) / 4).to(torch.bfloat16), (rn(F, H) / 8).to(torch.bfloat16)
    prev = rn(B, H, Lq, Lk).to(torch.float16)
    out, a1 = lisa.lisa_attn_prefill(q, k, v, lisa.tile_scores(prev) if tiled else prev, w1, w2, mix=lisa.MIX_CONCAT, tiled=tiled, Lq=Lq)
    torch.cuda.synchronize()
    assert lisa.last_path() == "mfma_scores"
    A = (lisa.untile_scores(a1, Lq, Lk) if tiled else a1).cpu().double()   # what the softmax is given
    assert err(out.flatten(2), softmax_v(A.nan_to_num(0.0), v.cpu().double(), True).flatten(2)) <= TOL_O


@pytest.mark.parametrize("Lq,Lk", [(264, 264), (40, 1032), (2, 264)])
@pytest.mark.parametrize("masked", [0, 70])
def test_softmax_from_float32_scores_key_halves(Lq, Lk, masked):
    """A layer whose scores come from the float32 or generic kernels (12 heads); `masked` keys of -inf, which leave the first key
    half of the early rows without any."""
    B, H, F, r = 2, 12, 160, 20
    log(f"[case] given float32 halves {Lq}x{Lk} masked={masked}")
    g = torch.Generator(device=DEV).manual_seed(Lk)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)
    q, k, v = rn(B, H, Lq, r).to(torch.bfloat16), rn(B, H, Lk, r).to(torch.bfloat16), rn(B, H, Lk, 128).to(torch.bfloat16)
    prev = rn(B, H, Lq, Lk).to(torch.float16)
    prev[..., :masked] = float("-inf")
    if masked:                                               # A_n = A_{n-1} + A_delta: -inf passes through
        w1 = w2 = None
        mix = lisa.MIX_PLUS
        kd = k.cpu().double().transpose(-1, -2).contiguous()
        A = prev.cpu().double() + q.cpu().double() @ kd / r ** 0.5
    else:
        w1, w2, mix = (rn(H, F) / 4).to(torch.bfloat16), (rn(F, H) / 8).to(torch.bfloat16), lisa.MIX_ADD
        A = reference(q, k, v, prev, w1, w2, "add", True)[0]
    (out, _), ran = stages(lambda: lisa.lisa_attn_prefill(q, k, v, prev, w1, w2, mix=mix))
    assert "k_softmax_v_mfma" in ran
    rows = slice(max(0, masked + Lq - Lk), None)             # (rows that see more than masked keys)
    assert torch.isfinite(out).all()
    assert err(out[:, rows].flatten(2), softmax_v(A, v.cpu().double(), True)[:, rows].flatten(2)) <= TOL_O
