"""The geometry that a fused prefill call chooses (head groups, row slices, key shares, pairs of units, chunks of slots per XCD)
against plain units of 16 rows: A_n does not depend on it and is the same bit for bit, O differs by what bf16 probabilities against
another running maximum and key shares summed apart give (each rounds to 2^-9; 2e-3 of the 2-norm is four times what is seen)."""
import pytest
import torch

from paper_2408_01890_amd import lisa, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("H,Hkv,F,r,B,Lq,past,tiled,geometry", [   # geometry: slices, head groups, key shares, pairs
    (32, 8, 64, 22, 1, 97, 0, True, (1, 4, 1, 0)), (32, 8, 64, 22, 1, 704, 0, True, (1, 4, 2, 0)),
    (32, 8, 64, 22, 1, 1250, 0, True, (1, 2, 2, 0)), (32, 32, 64, 22, 1, 416, 0, True, (1, 4, 2, 0)),
    (32, 32, 64, 22, 3, 656, 0, True, (1, 4, 1, 1)), (32, 16, 128, 16, 2, 333, 0, True, (1, 4, 2, 0)),
    (32, 8, 64, 22, 2, 2000, 0, True, (1, 2, 1, 1)),
    (40, 40, 80, 20, 1, 512, 0, True, (1, 5, 2, 0)), (40, 40, 80, 20, 3, 272, 0, True, (1, 5, 1, 0)),
    (40, 8, 40, 32, 2, 1111, 0, True, (1, 5, 1, 0)), (40, 40, 80, 22, 2, 1216, 0, True, (2, 5, 1, 1)),
    (40, 40, 80, 22, 8, 352, 0, True, (2, 5, 1, 1)), (40, 40, 80, 22, 7, 576, 0, True, (2, 5, 1, 0)),
    (16, 4, 32, 8, 2, 500, 0, True, (1, 2, 2, 0)), (24, 24, 48, 12, 1, 300, 0, True, (1, 1, 2, 0)),
    (24, 24, 48, 12, 1, 704, 0, True, (1, 1, 4, 0)), (8, 8, 16, 4, 5, 190, 0, True, (1, 1, 1, 0)),
    (32, 8, 64, 22, 1, 16, 2000, True, (1, 4, 4, 0)), (24, 8, 48, 16, 1, 40, 1000, True, (1, 1, 4, 0)),
    (16, 16, 32, 8, 2, 33, 700, True, (1, 2, 4, 0)),
    (32, 8, 64, 22, 2, 200, 312, False, (1, 2, 4, 0)), (40, 40, 80, 20, 1, 776, 0, False, (1, 5, 2, 0)),
    (24, 8, 96, 32, 3, 136, 40, False, (1, 1, 1, 0))])
def test_chosen_geometry_agrees_with_plain_units(H, Hkv, F, r, B, Lq, past, tiled, geometry):
    Lk = Lq + past
    cfg = synth.LayerShape("geometry", "bf16", B, H, Hkv, Lk, 512, 128, r, F, None)
    t = synth.make_prefill_inputs(cfg, Lq + H, DEV, ffn="identity_noise" if F >= 2 * H else "fan_in")
    desc = lisa.make_desc(lisa.BF16, B, H, Hkv, Lq, Lk, 128, r=r, F=F, write_scores=1, score_tiled=int(tiled))
    assert lisa.launch_choice(desc, lisa.CHOICE_PREFILL)[:4] == geometry
    q_lr = t["q_lr"][:, :, past:].contiguous()
    g = torch.Generator(device=DEV).manual_seed(Lk)
    prev = torch.randn(lisa.scores_shape(B, H, Lq, Lk, tiled), generator=g, device=DEV, dtype=torch.float16)

    def layer():
        scores = torch.zeros_like(prev)
        out, _ = lisa.lisa_attn_prefill(q_lr, t["k_lr"], t["v"], prev, t["w1"], t["w2"], scores_out=scores, tiled=tiled)
        torch.cuda.synchronize()
        assert lisa.last_path() == "mfma_fused"
        return out, scores

    out, scores = layer()
    with lisa.tune(prefill_slices=1, prefill_split=1, prefill_pair=0, prefill_groups=H // 8):
        want, want_scores = layer()
    assert (out - want).norm() <= 2e-3 * want.norm()
    if tiled:                                                # (rows past the end and entries above the diagonal are unspecified)
        vis = lisa.tile_scores(torch.ones(1, 1, Lq, Lk, dtype=torch.float16, device=DEV).tril(past)) > 0
        scores, want_scores = scores.where(vis, 0), want_scores.where(vis, 0)
    assert torch.equal(scores, want_scores)
