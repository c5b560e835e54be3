"""Scores of ragged layers in tiles of 16 and of 32 keys: a sequence of a large batch (many tiles: 32 keys) comes out as it does
alone (few: 16 keys).  The sums of a position run in the same order in both, but A_delta * scale + y may be one rounding or two,
so a float32 score moves by 2^-24 of itself: 1e-6 of a probability at |A| <= 16, and a half score by its last place where it
lies next to a rounding boundary (2e-6: the same of terms up to 16 that cancel)."""
import pytest
import torch

from paper_2408_01890_amd import lisa, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("H,Hkv,F,r,mix,B,Lq,past", [
    (32, 8, 64, 22, "add", 9, 125, 0), (32, 32, 64, 22, "add", 5, 137, 66), (40, 40, 80, 20, "add", 6, 151, 0),
    (33, 11, 66, 32, "add", 4, 203, 0), (32, 32, 256, 20, "concat", 6, 141, 0), (20, 4, 96, 9, "concat", 5, 97, 130)])
def test_small_tiles_equal_large_ones(H, Hkv, F, r, mix, B, Lq, past):
    Lk = Lq + past
    cfg = synth.LayerShape("tiles", "bf16", B, H, Hkv, Lk, 512, 128, r, F, None)
    t = synth.make_prefill_inputs(cfg, Lq, DEV, mix=mix, ffn="fan_in")
    q_lr = t["q_lr"][:, :, past:].contiguous()
    g = torch.Generator(device=DEV).manual_seed(Lk)
    prev = torch.randn((B, H, Lq, Lk), generator=g, device=DEV, dtype=torch.float16)
    m = lisa.MIX_CONCAT if mix == "concat" else lisa.MIX_ADD

    def layer(s):
        scores = torch.zeros_like(prev[s])
        out, _ = lisa.lisa_attn_prefill(*(x[s].clone() for x in (q_lr, t["k_lr"], t["v"], prev)), t["w1"], t["w2"], mix=m, scores_out=scores)
        torch.cuda.synchronize()
        return out, scores

    out, scores = layer(slice(0, B))
    for b in (0, B - 1):
        o1, s1 = layer(slice(b, b + 1))
        assert (out[b] - o1[0]).norm() <= 2e-6 * o1[0].norm()
        diff = (scores[b].float() - s1[0].float()).abs()
        assert (diff <= 2.0 ** -10 * s1[0].float().abs() + 2e-6).all() and (diff > 0).float().mean() <= 2e-3
