"""bf16 layers in float32 arithmetic on the bf16 matrix instructions (row-major score rows of any length): the sizes where
tiles, operand rows and tensors end, against float64."""
import pytest
import torch

from paper_2408_01890_amd import lisa
from tests.test_gpu_parity import log
from tests.test_gpu_ragged_rows import SENTINEL, guarded

pytestmark = pytest.mark.gpu
DEV = "cuda"
# float32 sums of up to 2000 terms and three-part products: a few 2^-24 of the row's RMS; the benchmark's float32 tolerance
TOL_O = 1e-5
TOL_A = 2.0 ** -8                  # one rounding to half, of scores below 8 RMS (see test_gpu_ragged_rows)

CASES = [  # B, H, Hkv, Lq, Lk, r, F, mix, causal: three-part products
    (1, 32, 32, 2, 9, 1, 64, "add", True),      # operand rows shorter than what a lane reads, at the tensor's end
    (2, 24, 3, 31, 31, 7, 33, "add", True),
    (1, 32, 16, 32, 33, 8, 31, "add", True),
    (1, 32, 4, 33, 63, 9, 64, "add", True),
    (30, 8, 1, 31, 67, 7, 33, "add", True),
    (3, 16, 16, 161, 171, 8, 31, "add", True),
    (1, 33, 11, 17, 65, 31, 96, "add", True),   # heads that fill no block of 8 waves
    (1, 40, 8, 65, 97, 32, 97, "add", True),
    (1, 40, 40, 16, 1003, 22, 128, "add", True),   # weights for which the tiles have 16 keys
    (2, 8, 8, 40, 1111, 32, 64, "add", False),  # every key visible to every row
    (1, 32, 32, 18, 41, 20, 256, "concat", True),
    (1, 37, 37, 5, 23, 11, 40, "concat", True),    # an odd number of heads, two per load
    (2, 24, 3, 47, 49, 20, 256, "concat", False),
    (2, 8, 2, 201, 211, 20, 40, "concat", False),
    (2, 16, 2, 201, 211, 20, 256, "concat", True),
]
CASES_F32 = [  # the float32 kernel
    (1, 8, 8, 2, 9, 1, 32, "add", True),
    (2, 8, 1, 31, 31, 7, 33, "add", True),
    (1, 16, 16, 32, 33, 8, 31, "add", True),
    (2, 16, 2, 47, 49, 20, 256, "concat", False),
    (1, 32, 32, 20, 37, 33, 64, "add", True),   # more ranks than one product takes
    (1, 8, 4, 3, 5, 4, 32, "add", True),        # fewer keys than a lane reads
]


def reference(q, k, v, prev, w1, w2, mix, causal, act="relu"):
    d = torch.float64
    q, k, v, prev, w1, w2 = (t.cpu().to(d) for t in (q, k, v, prev, w1, w2))
    rep = lambda t: t.repeat_interleave(q.shape[1] // t.shape[1], 1)
    delta = q @ rep(k).transpose(-1, -2).contiguous() / q.shape[-1] ** 0.5
    x = torch.cat([prev, delta], 1) if mix == "concat" else prev
    A = ((torch.relu if act == "relu" else torch.nn.functional.silu)(x.permute(0, 2, 3, 1) @ w1) @ w2).permute(0, 3, 1, 2)
    if mix == "add":
        A = A + delta
    return A, softmax_v(A, rep(v), causal)


def softmax_v(A, v, causal):
    Lq, Lk = A.shape[-2:]
    if causal:
        A = A.masked_fill(torch.ones(Lq, Lk, dtype=torch.bool).triu(Lk - Lq + 1), float("-inf"))
    return (torch.softmax(A, -1) @ v).permute(0, 2, 1, 3)


def err(got, ref):                 # largest difference over the RMS of its row
    got, ref = got.cpu().double(), ref
    return float(((got - ref).abs().amax(-1) / ref.pow(2).mean(-1).sqrt()).max())


def stages(call):
    """What `call()` returns, and the kernels that it launched: {name: (launches, ms)}."""
    lisa.profile_enable(True)
    try:
        res = call()
        torch.cuda.synchronize()
        return res, lisa.profile_collect()
    finally:
        lisa.profile_enable(False)


def check_layer(B, H, Hkv, Lq, Lk, r, F, mix, causal):
    """Scores and output of one layer against float64; the names of the kernels it launched."""
    log(f"[case] split lisa {B, H, Hkv, Lq, Lk, r, F, mix, causal}")
    g = torch.Generator(device=DEV).manual_seed(Lk)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)
    q, k, v = rn(B, H, Lq, r).to(torch.bfloat16), rn(B, Hkv, Lk, r).to(torch.bfloat16), rn(B, Hkv, Lk, 128).to(torch.bfloat16)
    din = 2 * H if mix == "concat" else H
    w1, w2 = (rn(din, F) / din ** 0.5).to(torch.bfloat16), (rn(F, H) / F ** 0.5).to(torch.bfloat16)
    prev = rn(B, H, Lq, Lk).to(torch.float16)
    scores, *guards = guarded((B, H, Lq, Lk))
    (out, _), ran = stages(lambda: lisa.lisa_attn_prefill(q, k, v, prev, w1, w2, causal=causal, scores_out=scores,
                                                          mix=lisa.MIX_CONCAT if mix == "concat" else lisa.MIX_ADD))
    A, O = reference(q, k, v, prev, w1, w2, mix, causal)
    vis = torch.ones(Lq, Lk, dtype=torch.bool).tril(Lk - Lq) if causal else torch.ones(Lq, Lk, dtype=torch.bool)
    assert all(bool(torch.all(t == SENTINEL)) for t in guards) and bool(torch.all(scores.cpu()[..., ~vis] == SENTINEL))
    rms = (A * vis).pow(2).sum((1, 3)).div(vis.sum(-1) * H).sqrt()[:, None, :, None]
    assert float((((scores.cpu().double() - A) / rms).abs() * vis).max()) <= TOL_A
    assert err(out.flatten(2), O.flatten(2)) <= TOL_O
    return ran


@pytest.mark.parametrize("case", CASES + CASES_F32, ids=lambda c: "_".join(map(str, c)))
def test_lisa_layer(case):
    assert ("k_f32_lisa_scores" if case in CASES_F32 else "k_split_scores") in check_layer(*case)


@pytest.mark.parametrize("kernel,B,H,Lq,Lk,F,mix", [         # both sides of each line, causal
    ("f32", 1, 8, 201, 201, 256, "concat"), ("split", 2, 8, 201, 201, 64, "add"),     # 169 and 338 tiles of 16 x 16
    ("f32", 1, 16, 255, 255, 33, "add"), ("split", 1, 16, 257, 257, 33, "add"),       # 256 and 289
    ("f32", 1, 16, 255, 255, 256, "add"), ("split", 1, 16, 255, 255, 257, "add"),
    ("f32", 1, 17, 65, 65, 16, "add"), ("split", 1, 17, 65, 65, 17, "add"),
    ("f32", 2, 32, 9, 9, 32, "add"), ("split", 2, 32, 9, 9, 33, "add"),               # one key tile, more heads x units
    ("f32", 16, 40, 9, 15, 64, "add"), ("split", 16, 40, 9, 15, 65, "add"), ("split", 16, 20, 9, 9, 129, "concat"),
    ("split", 260, 12, 17, 17, 20, "add"), ("f32", 130, 12, 17, 17, 20, "add"),       # 520 and 260 tiles of 32 keys
    ("f32", 152, 16, 17, 31, 64, "concat"), ("split", 153, 16, 17, 31, 64, "concat"),
    ("f32", 140, 8, 60, 62, 64, "add"), ("split", 140, 8, 60, 66, 64, "add"),         # 8 heads, rows of up to 64 keys
    ("f32", 140, 7, 9, 127, 64, "concat"), ("split", 140, 7, 9, 129, 64, "concat"),
    ("f32", 90, 8, 33, 33, 128, "add"), ("split", 260, 8, 33, 33, 128, "add"),        # 360 and 1040 tiles
    ("f32", 300, 32, 2, 33, 64, "add"), ("split", 120, 32, 2, 33, 64, "add"),
])
def test_scores_of_few_or_short_rows(kernel, B, H, Lq, Lk, F, mix):
    """float32 matrix instructions where they are sooner, three-part products elsewhere."""
    ran = check_layer(B, H, H, Lq, Lk, 20, F, mix, True)
    assert {"f32": "k_f32_lisa_scores", "split": "k_split_scores"}[kernel] in ran


@pytest.mark.parametrize("Lq,Lk,causal", [(2, 4097, True), (31, 1155, False), (32, 33, True), (33, 129, True), (64, 65, True), (3, 5, True)])
def test_std_layer(Lq, Lk, causal):
    B, H, Hkv = 2, 4, 2
    log(f"[case] split std {Lq}x{Lk}")
    g = torch.Generator(device=DEV).manual_seed(Lk)
    q = torch.randn((B, H, Lq, 128), generator=g, device=DEV).to(torch.bfloat16)
    k, v = (torch.randn((B, Hkv, Lk, 128), generator=g, device=DEV).to(torch.bfloat16) for _ in range(2))
    only, *guards = guarded((B, H, Lq, Lk))
    lisa.std_attn_scores(q, k, causal=causal, scores_out=only)       # scores alone: tiles dealt to several workgroups
    scores, out = lisa.std_attn_scores(q, k, v, causal=causal)
    torch.cuda.synchronize()
    assert all(bool(torch.all(t == SENTINEL)) for t in guards)
    rep = lambda t: t.cpu().double().repeat_interleave(H // Hkv, 1)
    A = q.cpu().double() @ rep(k).transpose(-1, -2).contiguous() / 128 ** 0.5
    vis = torch.ones(Lq, Lk, dtype=torch.bool).tril(Lk - Lq) if causal else torch.ones(Lq, Lk, dtype=torch.bool)
    assert torch.equal(only.cpu()[..., vis], scores.cpu()[..., vis])
    assert float((scores.cpu().double() - A).abs()[..., vis].max()) <= 2.0 ** -9 * float(A.abs().max())
    assert err(out.flatten(2), softmax_v(A, rep(v), causal).flatten(2)) <= TOL_O


def chunk_rows(B, H, Hkv, L):
    """Query rows per chunk: 256 MB less the padded operands, of float32 scores in tiles of 32 keys, in blocks of 16 rows."""
    up = lambda n, m: (n + m - 1) // m * m
    operands = up(B * H * up(L, 16) * 64, 256) + up(B * Hkv * up(L, 64) * 64, 256)
    return ((256 << 20) - operands) // (B * H * up(L, 32) * 4) // 16 * 16


def test_chunk_border():
    """The last two blocks of rows of a chunk of float32 scores and the first two of the next."""
    B, H, L = 2, 40, 1001
    log("[case] split chunk border")
    edge = chunk_rows(B, H, H, L)
    assert edge == 784
    g = torch.Generator(device=DEV).manual_seed(1)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)
    q, k, v = rn(B, H, L, 22).to(torch.bfloat16), rn(B, H, L, 22).to(torch.bfloat16), rn(B, H, L, 128).to(torch.bfloat16)
    w1, w2 = (rn(H, 80) / 6).to(torch.bfloat16), (rn(80, H) / 9).to(torch.bfloat16)
    prev = rn(B, H, L, L).to(torch.float16)
    (out, scores), ran = stages(lambda: lisa.lisa_attn_prefill(q, k, v, prev, w1, w2))
    assert ran["k_split_scores"][0] == 2                             # (launches)
    for i in (0, edge - 17, edge - 16, edge - 1, edge, edge + 15, edge + 16, L - 1):   # row i alone: one row of i + 1 keys
        A, O = reference(q[:, :, i:i + 1], k[:, :, :i + 1], v[:, :, :i + 1], prev[:, :, i:i + 1, :i + 1], w1, w2, "add", True)
        assert err(out[:, i:i + 1].flatten(2), O.flatten(2)) <= TOL_O
        assert err(scores[:, :, i, :i + 1].flatten(1), A[:, :, 0].flatten(1)) <= TOL_A


@pytest.mark.parametrize("causal", [True, False])
def test_batch_past_the_workspace_budget(causal):
    """16 rows of float32 scores beside the padded operands pass 256 MB: the kernels without copies take the call, half of
    the batch fits.  Both are float32 sums of the same terms."""
    B, H, Lq, Lk, r, F = 16, 40, 2, 6561, 22, 64
    log(f"[case] split budget causal={causal}")
    g = torch.Generator(device=DEV).manual_seed(1)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)
    q, k, v = rn(B, H, Lq, r).to(torch.bfloat16), rn(B, 1, Lk, r).to(torch.bfloat16), rn(B, 1, Lk, 128).to(torch.bfloat16)
    w1, w2 = (rn(H, F) / H ** 0.5).to(torch.bfloat16), (rn(F, H) / F ** 0.5).to(torch.bfloat16)
    prev = rn(B, H, Lq, Lk).to(torch.float16)
    run = lambda s: lisa.lisa_attn_prefill(q[s], k[s], v[s], prev[s], w1, w2, causal=causal)
    (whole, a), ran = stages(lambda: run(slice(None)))
    assert "k_f32_lisa_scores" in ran
    for s in (slice(0, B // 2), slice(B // 2, B)):
        (out, b), ran = stages(lambda: run(s))
        assert "k_split_scores" in ran
        vis = slice(None, Lk - 1) if causal else slice(None)          # (the last key: row 1 alone)
        assert err(whole[s], out.cpu().double()) <= TOL_O
        x, y = a[s][..., vis].cpu().double(), b[..., vis].cpu().double()
        assert float((x - y).abs().max()) <= TOL_A * float(y.pow(2).mean().sqrt())


@pytest.mark.parametrize("B,Lq,Lk,std,given", [  # the side of the line that a standard layer and given scores fall on
    (2, 2, 2, "f32", "f32"), (2, 9, 9, "f32", "f32"), (2, 15, 15, "f32", "f32"), (2, 16, 17, "split", "f32"), (1, 3, 47, "split", "f32"),
    (1, 16, 49, "split", "split"), (2, 17, 17, "split", "split"), (4100, 5, 31, "f32", "f32"), (4100, 2, 33, "split", "f32")])
def test_attention_of_few_keys(B, Lq, Lk, std, given):
    """One block of 16 rows that sees few keys: float32 matrix instructions or three-part products, both in float32 arithmetic."""
    H, Hkv = 4, 2
    log(f"[case] split few keys {B}x{Lq}x{Lk}")
    g = torch.Generator(device=DEV).manual_seed(Lk)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV).to(torch.bfloat16)
    q, k, v = rn(B, H, Lq, 128), rn(B, Hkv, Lk, 128), rn(B, Hkv, Lk, 128)
    prev = rn(B, H, Lq, Lk).half()
    (scores, out), ran = stages(lambda: lisa.std_attn_scores(q, k, v))
    assert set(ran) == {f"k_{std}_attn"}
    (shared, _), ran = stages(lambda: lisa.lisa_attn_prefill(None, None, v, prev, None, None, mix=lisa.MIX_SHARE))
    assert f"k_{given}_softmax_v" in ran
    rep = lambda t: t.cpu().double().repeat_interleave(H // Hkv, 1)
    A = q.cpu().double() @ rep(k).transpose(-1, -2).contiguous() / 128 ** 0.5
    vis = torch.ones(Lq, Lk, dtype=torch.bool).tril(Lk - Lq)
    assert float((scores.cpu().double() - A).abs()[..., vis].max()) <= 2.0 ** -9 * float(A.abs().max())
    assert err(out.flatten(2), softmax_v(A, rep(v), True).flatten(2)) <= TOL_O
    assert err(shared.flatten(2), softmax_v(prev.cpu().double(), rep(v), True).flatten(2)) <= TOL_O
