"""What the dispatch chooses on both sides of its lines (host only): each line was drawn where the two sides' times cross, and
the sizes here are ones at which the other side was measured slower."""
import ctypes as C

import pytest
import torch

from paper_2408_01890_amd import lisa


def std(B, H, Hkv, Lq, past=0, **kw):
    return lisa.make_desc(lisa.BF16, B, H, Hkv, Lq, Lq + past, 128, **kw)


@pytest.mark.parametrize("B,H,Lq,past,order", [
    (2, 32, 201, 0, 1), (4, 8, 333, 0, 1), (2, 32, 509, 1022, 0),                           # all at once; rows behind more keys
    (2, 32, 265, 0, 0), (2, 32, 301, 0, 0), (3, 32, 199, 0, 0), (8, 32, 65, 0, 1), (4, 40, 99, 0, 1),
    (4, 8, 777, 0, 1), (5, 24, 227, 0, 1), (2, 32, 395, 0, 0), (3, 40, 301, 0, 0),
    (16, 32, 129, 100, 0), (8, 32, 501, 0, 0), (8, 40, 777, 0, 0), (32, 40, 777, 0, 0)])
def test_order_of_ragged_standard_layers(B, H, Lq, past, order):
    assert lisa.launch_choice(std(B, H, H, Lq, past), lisa.CHOICE_STD_ORDER) == (order,)


@pytest.mark.parametrize("B,H,Lq,dk,order", [
    (1, 8, 128, 64, 1), (2, 8, 504, 64, 2), (8, 16, 512, 64, 2), (3, 32, 1000, 128, 2), (8, 32, 128, 128, 2),
    (8, 16, 1500, 64, 0), (13, 12, 410, 64, 0), (16, 32, 600, 64, 0), (8, 32, 700, 128, 0), (8, 32, 1000, 128, 0), (1000, 32, 9, 128, 0), (8, 32, 17, 128, 0), (8, 32, 33, 128, 2)])
def test_order_of_float32_standard_layers(B, H, Lq, dk, order):
    d = lisa.make_desc(lisa.F32, B, H, H, Lq, Lq, dk)
    assert lisa.launch_choice(d, lisa.CHOICE_STD_ORDER) == (order,)


def test_order_of_more_row_blocks_than_one_grid_axis_holds():
    """65535 heads of 257 row blocks: in a single axis of 256 threads each these pass the 2^32 threads an axis may have."""
    d = lisa.make_desc(lisa.F32, 1, 65535, 1, 4112, 1, 64, causal=0)
    assert lisa.launch_choice(d, lisa.CHOICE_STD_ORDER) == (0,)


@pytest.mark.parametrize("H,Hkv,d_model,L,shape", [
    (32, 32, 4096, 2048, 1), (32, 32, 4096, 4096, 1), (32, 32, 4096, 6144, 1), (32, 8, 4096, 4096, 1), (40, 40, 5120, 2560, 1),
    (32, 32, 4096, 777, 3), (32, 8, 4096, 2204, 3), (32, 8, 4096, 900, 5), (32, 8, 4096, 777, 6), (40, 40, 5120, 2304, 4),
    (40, 40, 5120, 900, 2), (32, 32, 4096, 8192, 0), (32, 32, 4096, 128, None)])
def test_projection_tile_shape(H, Hkv, d_model, L, shape):
    assert lisa.project_choice(torch.bfloat16, 1, L, d_model, H, Hkv, 22, 128) == shape


def prefill(H, Hkv, F, B, Lq, past=0, **kw):
    return lisa.make_desc(lisa.BF16, B, H, Hkv, Lq, Lq + past, 128, r=22, F=F, write_scores=1, score_tiled=1, **kw)


@pytest.mark.parametrize("H,Hkv,F,B,Lq,past,geometry", [
    # slices, head groups, key shares, pairs
    (32, 8, 64, 1, 16, 8192, (1, 4, 4, 0)), (32, 32, 64, 4, 32, 8192, (1, 4, 4, 0)), (40, 40, 80, 1, 136, 960, (1, 5, 4, 0)),
    (8, 8, 16, 1, 128, 8192, (1, 1, 4, 0)), (24, 8, 48, 1, 512, 8192, (1, 1, 4, 0)), (16, 4, 32, 4, 16, 8192, (1, 2, 4, 0)),
    (24, 24, 48, 1, 704, 0, (1, 1, 4, 0)), (8, 2, 64, 1, 704, 0, (1, 1, 4, 0)),
    (32, 32, 128, 1, 352, 0, (1, 4, 2, 0)), (32, 8, 64, 1, 1248, 0, (1, 2, 2, 0)),
    (32, 8, 64, 4, 8192, 0, (1, 2, 1, 1)), (32, 32, 64, 3, 1312, 0, (1, 2, 1, 1)),
    (40, 40, 80, 8, 4096, 0, (2, 5, 1, 1)), (40, 40, 80, 3, 704, 0, (2, 5, 1, 1)), (8, 2, 64, 1, 2816, 0, (1, 1, 2, 1))])
def test_geometry_of_the_fused_prefill(H, Hkv, F, B, Lq, past, geometry):
    """Few rows behind many keys take four key shares, whatever the layer: with two they ran up to twice as long."""
    assert lisa.launch_choice(prefill(H, Hkv, F, B, Lq, past), lisa.CHOICE_PREFILL)[:4] == geometry


@pytest.mark.parametrize("act", [lisa.ACT_RELU, lisa.ACT_SILU])
@pytest.mark.parametrize("H,Hkv,F", [(8, 8, 16), (16, 4, 64), (24, 8, 48), (32, 32, 64), (32, 8, 64), (40, 40, 80)])
def test_prefill_workspace_with_key_shares_is_bounded(H, Hkv, F, act):
    """Partial results of fewer than 1024 units (16 rows of the heads of the smallest head group, 520 bytes each), whatever the
    length; none beyond the lengths that had them when counts of units alone decided."""
    group = 24 if H == 24 else 16 if act == lisa.ACT_SILU and H in (16, 32) else 8
    for B in (1, 3, 8):
        for past in (0, 2048):
            for Lq in [*range(16, 2400, 37), *range(2400, 9000, 331)]:
                d = prefill(H, Hkv, F, B, Lq, past, act=act)
                need = lisa.workspace_bytes(d, lisa.WS_PREFILL)
                with lisa.tune(prefill_split=1):
                    plain = lisa.workspace_bytes(d, lisa.WS_PREFILL)
                assert plain - 2 ** 17 <= need <= plain + 1024 * 16 * group * 520 + 2 ** 17     # (the FFN image: 1 - 2 head groups)
                units = -(-Lq // 16) * B * (H // group)
                if units >= 512 or Lq + past <= 7 * 32:
                    assert need <= plain + 2 ** 17


def test_forced_key_shares_are_taken_where_row_slices_exist():
    for split in (2, 4):
        with lisa.tune(prefill_split=split):
            assert lisa.launch_choice(prefill(40, 40, 80, 8, 4096), lisa.CHOICE_PREFILL)[:3] == (1, 5, split)
    with lisa.tune(prefill_slices=2, prefill_split=2):       # (slices have one share)
        assert lisa.launch_choice(prefill(40, 40, 80, 8, 4096), lisa.CHOICE_PREFILL)[:3] == (2, 5, 1)


@pytest.mark.parametrize("kw", [
    dict(), dict(act=lisa.ACT_SILU), dict(mix=lisa.MIX_PLUS), dict(act=lisa.ACT_SINGLE, F=32), dict(mix=lisa.MIX_SHARE, r=0),
    dict(mix=lisa.MIX_CONCAT, F=256), dict(score_tiled=0, Lq=97, Lk=97)])
def test_prefill_refuses_one_byte_less_than_the_workspace_needs(kw):
    args = dict(dtype=lisa.BF16, B=1, H=32, Hkv=8, Lq=96, Lk=1024, d_k=128, r=22, F=64, write_scores=1, score_tiled=1)
    args.update(kw)
    d = lisa.make_desc(**args)
    need = lisa.workspace_bytes(d, lisa.WS_PREFILL)
    fake = C.c_void_p(0x10000)                               # never dereferenced on the host
    call = [fake] * 9
    call[7] = C.c_void_p(0x20000)                            # (scores_out is not scores_prev)
    assert need > 0 and lisa.library().lisa_attn_prefill(C.byref(d), *call, need - 1, None) == -5
