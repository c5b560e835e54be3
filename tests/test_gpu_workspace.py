"""What a prefill call finds in its workspace must not matter: with every byte 0xff (NaN in half, bfloat16 and float32) it gives
what it gives on zeros, bit for bit.  The forms that leave part of their scratch unwritten: float32 tiles of 32 keys of which
tiles of 16 write one half at the diagonal, rows and keys padded to whole tiles, key shares without keys, FFN images."""
import pytest
import torch

from paper_2408_01890_amd import lisa, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("H,Hkv,F,r,mix,act,dtype,B,Lq,past,tiled", [
    # ragged layers: tiles of 16 keys (few tiles), of 32 (many), rows behind cached keys
    (32, 8, 64, 22, "add", 0, "bf16", 1, 125, 0, False), (40, 40, 80, 20, "add", 0, "bf16", 1, 201, 0, False),
    (32, 32, 256, 20, "concat", 0, "bf16", 1, 150, 0, False), (33, 11, 66, 32, "add", 1, "bf16", 1, 67, 38, False),
    (32, 8, 64, 22, "add", 0, "bf16", 9, 125, 0, False), (20, 4, 96, 9, "concat", 0, "bf16", 5, 97, 130, False),
    (8, 8, 32, 11, "add", 0, "bf16", 3, 33, 0, False),
    # fused kernel: one, two and four key shares, row slices
    (32, 8, 64, 22, "add", 0, "bf16", 1, 97, 0, True), (32, 8, 64, 22, "add", 0, "bf16", 1, 1250, 0, True),
    (24, 8, 48, 16, "add", 1, "bf16", 1, 40, 1000, True), (32, 8, 64, 22, "add", 0, "bf16", 1, 3, 2000, True),
    (40, 40, 80, 22, "add", 0, "bf16", 2, 1216, 0, True),
    # CONCAT in tiles and in whole rows, float32
    (32, 32, 256, 20, "concat", 0, "bf16", 1, 160, 0, True), (40, 40, 256, 20, "concat", 0, "bf16", 2, 136, 0, False),
    (8, 8, 32, 11, "add", 0, "f32", 2, 70, 9, False)])
@pytest.mark.parametrize("write_scores", [True, False])
def test_workspace_contents_do_not_matter(H, Hkv, F, r, mix, act, dtype, B, Lq, past, tiled, write_scores):
    Lk = Lq + past
    cfg = synth.LayerShape("poison", dtype, B, H, Hkv, Lk, 256, 64 if dtype == "f32" else 128, r, F, None)
    t = synth.make_prefill_inputs(cfg, Lq, DEV, mix=mix, ffn="fan_in")
    q_lr = t["q_lr"][:, :, past:].contiguous()
    g = torch.Generator(device=DEV).manual_seed(Lk)
    prev = torch.randn(lisa.scores_shape(B, H, Lq, Lk, tiled), generator=g, device=DEV).to(cfg.score_dtype)
    m = lisa.MIX_CONCAT if mix == "concat" else lisa.MIX_ADD
    desc = lisa.make_desc(cfg.torch_dtype, B, H, Hkv, Lq, Lk, cfg.d_k, r=r, F=F, mix=m, act=act, write_scores=int(write_scores),
                          out_f32=int(dtype != "f32"), score_tiled=int(tiled))
    need = lisa.workspace_bytes(desc, lisa.WS_PREFILL)

    def layer(fill):
        ws = torch.full((max(need, 16),), fill, dtype=torch.uint8, device=DEV)
        scores = torch.zeros_like(prev) if write_scores else None
        out, _ = lisa.lisa_attn_prefill(q_lr, t["k_lr"], t["v"], prev, t["w1"], t["w2"], mix=m, act=act, scores_out=scores,
                                        write_scores=write_scores, workspace=ws, tiled=tiled)
        torch.cuda.synchronize()
        return out, scores

    out, scores = layer(0xff)
    want, want_scores = layer(0)
    assert bool(out.isfinite().all()) and torch.equal(out, want)
    if write_scores:
        vis = torch.ones(1, 1, Lq, Lk, dtype=torch.float16, device=DEV).tril(past)
        vis = (lisa.tile_scores(vis) if tiled else vis) > 0
        assert torch.equal(scores.where(vis, 0), want_scores.where(vis, 0))
