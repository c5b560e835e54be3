"""Prefill layers that pass on scores masked with -inf (padding in front of a prompt): a masked key weighs nothing, and a
row that sees nothing but masked keys is not NaN."""
import pytest
import torch

from paper_2408_01890_amd import lisa
from tests import helpers as hp
from tests.test_gpu_parity import log

pytestmark = pytest.mark.gpu
DEV = "cuda"

CASES = [  # dtype, H, Hkv, L, d_k, pad
    ("f32", 8, 8, 130, 64, 70),          # a whole tile of every wave, and the first row blocks
    ("f32", 4, 2, 33, 128, 17),
    ("bf16", 8, 8, 130, 128, 70),        # rows of ragged length: float32 arithmetic
    ("bf16", 12, 4, 77, 128, 32),
    ("bf16", 8, 8, 136, 128, 70),        # the fused kernel
    ("bf16", 32, 8, 160, 128, 64),
    ("bf16", 12, 4, 128, 128, 64),       # generic scores, softmax on the matrix cores
]


def masked_layer(dtype, H, Hkv, L, dk, pad, mix, tiled=False):
    """(out, emitted scores, scores as given, v, what the layer adds to them) of a layer without an alignment module."""
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(31)
    prev = torch.randn((2, H, L, L), generator=g, device=DEV).to(lisa.score_dtype(dt))
    prev[..., :pad] = float("-inf")
    v = torch.randn((2, Hkv, L, dk), generator=g, device=DEV).to(dt)
    q_lr = k_lr = None
    delta = torch.zeros((2, H, L, L), dtype=torch.float64)
    if mix == lisa.MIX_PLUS:
        q_lr = torch.randn((2, H, L, 20), generator=g, device=DEV).to(dt)
        k_lr = torch.randn((2, Hkv, L, 20), generator=g, device=DEV).to(dt)
        kx = k_lr.double().cpu().repeat_interleave(H // Hkv, dim=1)
        delta = (q_lr.double().cpu() @ kx.transpose(-1, -2).contiguous()) / 20 ** 0.5
    given = lisa.tile_scores(prev) if tiled else prev
    out, scores = lisa.lisa_attn_prefill(q_lr, k_lr, v, given, None, None, mix=mix, tiled=tiled, Lq=L)
    torch.cuda.synchronize()
    return out, lisa.untile_scores(scores, L, L) if tiled else scores, prev, v, delta


def check_masked(out, scores, prev, v, delta, tol, zeros):
    B, H, L, _ = prev.shape
    pad = int(torch.isinf(prev[0, 0, 0]).sum())
    seen = torch.ones(L, L, dtype=torch.bool).tril()
    a = prev.double().cpu() + delta
    vx = v.double().cpu().repeat_interleave(H // v.shape[1], dim=1)
    ref = torch.softmax(a.masked_fill(~seen, float("-inf")), -1)[:, :, pad:] @ vx
    got = out.double().cpu().permute(0, 2, 1, 3)
    assert torch.isfinite(got).all()
    assert hp.row_rel_err(got[:, :, pad:].permute(2, 0, 1, 3).numpy(), ref.permute(2, 0, 1, 3).numpy()) <= tol
    if zeros:
        assert bool((got[:, :, :pad] == 0).all())
    s = scores.double().cpu()
    masked = seen & (torch.arange(L) < pad)
    assert bool((s[..., masked] <= -60000).all())             # -inf, or the lowest finite half


@pytest.mark.parametrize("mix", [lisa.MIX_SHARE, lisa.MIX_PLUS], ids=["share", "plus"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}_h{c[1]}_{c[3]}_dk{c[4]}_pad{c[5]}")
def test_masked_keys_weigh_nothing(case, mix):
    dtype, H, Hkv, L, dk, pad = case
    log(f"[case] masked prefill {case} mix={mix}")
    check_masked(*masked_layer(dtype, H, Hkv, L, dk, pad, mix), tol=1e-5 if dtype == "f32" else 2e-2, zeros=dtype == "f32" or L % 8 != 0 or H == 12)


@pytest.mark.parametrize("mix", [lisa.MIX_SHARE, lisa.MIX_PLUS], ids=["share", "plus"])
def test_masked_keys_weigh_nothing_on_tiled_scores(mix):
    log(f"[case] masked prefill, tiled, mix={mix}")
    check_masked(*masked_layer("bf16", 16, 4, 200, 128, 70, mix, tiled=True), tol=2e-2, zeros=False)


@pytest.mark.parametrize("H,B,Lk", [(8, 2, 300), (16, 1, 1100), (32, 40, 2300)])   # (the last: beyond 16 MB of scratch)
def test_masked_keys_weigh_nothing_in_a_decode_step(H, B, Lk):
    """LiSA_plus: the row of the layer before plus the low-rank correction."""
    log(f"[case] masked decode, LiSA_plus, {H} {B} {Lk}")
    g = torch.Generator(device=DEV).manual_seed(32)
    dt, r, dk, Lmax = torch.bfloat16, 20, 128, (Lk + 7) // 8 * 8
    prev = torch.randn((B, H, Lk), generator=g, device=DEV).half()
    prev[..., 30:290] = float("-inf")
    v = torch.randn((B, 1, Lmax, dk), generator=g, device=DEV).to(dt)
    q_lr = torch.randn((B, H, r), generator=g, device=DEV).to(dt)
    k_lr = torch.randn((B, 1, r, Lmax), generator=g, device=DEV).to(dt)
    out, _ = lisa.lisa_attn_decode(q_lr, k_lr, v, Lk, prev, None, None, mix=lisa.MIX_PLUS)
    a = prev.double().cpu() + (q_lr.double().cpu() @ k_lr[:, 0].double().cpu())[..., :Lk] / r ** 0.5
    ref = torch.softmax(a, -1) @ v[:, 0, :Lk].double().cpu()
    err = (out.double().cpu() - ref).norm(dim=-1) / ref.norm(dim=-1)
    assert torch.isfinite(out).all() and float(err.max()) <= 2e-2
