"""The order in which the attention kernels' workgroups take row groups and sequences, at sizes on both sides of the lines where
it changes: every sequence of a batch must come out as it does alone (bit for bit where the same kernel runs, else within what
float32 sums in another order give) and float32 rows as in float64."""
import pytest
import torch

from paper_2408_01890_amd import lisa

pytestmark = pytest.mark.gpu
DEV = "cuda"


def qkv(B, H, Hkv, L, dk, dtype, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    shapes = ((B, H, L, dk), (B, Hkv, L, dk), (B, Hkv, L, dk))
    return [torch.randn(s, generator=g, device=DEV).to(dtype) for s in shapes]


@pytest.mark.parametrize("B,H,Hkv,L,tiled", [
    (2, 8, 2, 520, True), (3, 8, 8, 264, False),          # by length
    (5, 40, 40, 520, True), (9, 32, 8, 392, False),       # sequence by sequence: more than 640 row groups
    (3, 8, 2, 333, False), (2, 16, 16, 97, False),        # rows of odd length: 32 rows a workgroup, by length
    (2, 32, 8, 265, False), (5, 8, 8, 777, False), (3, 40, 8, 301, False)])   # sequence by sequence, by length, and again not
def test_batch_equals_its_sequences(B, H, Hkv, L, tiled):
    q, k, v = qkv(B, H, Hkv, L, 128, torch.bfloat16, L)
    vis = torch.ones(L, L, dtype=torch.bool, device=DEV).tril()
    a, o = lisa.std_attn_scores(q, k, v, tiled=tiled)
    for b in range(B):
        a1, o1 = lisa.std_attn_scores(q[b:b + 1], k[b:b + 1], v[b:b + 1], tiled=tiled)
        torch.cuda.synchronize()
        if tiled:
            a_b, a_1 = (lisa.untile_scores(t, L, L)[0] for t in (a[b:b + 1], a1))
        else:
            a_b, a_1 = a[b], a1[0]
        assert torch.equal(a_b[:, vis], a_1[:, vis])
        # (a sequence alone may take two waves per row block: bf16 probabilities against another maximum)
        assert (o[b] - o1[0]).norm() <= 4e-3 * o1[0].norm()


@pytest.mark.parametrize("B,H,Hkv,L,dk", [(1, 4, 2, 255, 64), (1, 4, 2, 273, 64), (2, 8, 8, 257, 64), (3, 8, 4, 401, 64),
                                          (2, 4, 4, 300, 128), (7, 8, 8, 305, 64), (9, 32, 8, 129, 64)])
def test_float32_rows_in_every_order(B, H, Hkv, L, dk):
    q, k, v = qkv(B, H, Hkv, L, dk, torch.float32, L + B)
    vis = torch.ones(L, L, dtype=torch.bool, device=DEV).tril()
    kk, vv = (t.double().repeat_interleave(H // Hkv, 1) for t in (k, v))
    s = q.double() @ kk.transpose(2, 3).contiguous() / dk ** 0.5
    want = (s.masked_fill(~vis, float("-inf")).softmax(-1) @ vv).transpose(1, 2)
    a, o = lisa.std_attn_scores(q, k, v)
    # a layer whose module passes A_{n-1} through, plus zero A_delta: softmax from given scores
    eye = torch.eye(H, device=DEV)
    w1, w2 = torch.cat([eye, -eye], 1).contiguous(), torch.cat([eye, -eye], 0).contiguous()
    zq, zk = torch.zeros((B, H, L, 4), device=DEV), torch.zeros((B, Hkv, L, 4), device=DEV)
    o2, a2 = lisa.lisa_attn_prefill(zq, zk, v, a, w1, w2)
    torch.cuda.synchronize()
    for got in (o, o2):
        assert (got.double() - want).norm() <= 2e-6 * want.norm()      # (L rounded products and probabilities of 6e-8 each)
    assert (a.double() - s)[:, :, vis].norm() <= 1e-6 * s[:, :, vis].norm()
    assert torch.equal(a2[:, :, vis], a[:, :, vis])
