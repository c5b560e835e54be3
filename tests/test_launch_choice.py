"""What the dispatch chooses on both sides of its lines (host only): each line was drawn where the two sides' times cross, and
the sizes here are ones at which the other side was measured slower."""
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
    (8, 16, 1500, 64, 0), (13, 12, 410, 64, 0), (16, 32, 600, 64, 0), (8, 32, 700, 128, 0), (8, 32, 1000, 128, 0), (1000, 32, 9, 128, 0)])
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
