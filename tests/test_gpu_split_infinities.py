"""Infinities in layers whose operands go through the bf16 matrix instructions in parts (row-major score rows of any length):
the parts of an infinite number give what the number itself gives, against float64."""
import pytest
import torch

from paper_2408_01890_amd import lisa
from tests.test_gpu_parity import log
from tests.test_gpu_split import TOL_O, err, reference, softmax_v, stages

pytestmark = pytest.mark.gpu
DEV = "cuda"

CASES = [  # H, Hkv, Lq, Lk, F, mix, act, what is infinite at the masked keys
    (8, 8, 301, 301, 32, "add", "relu", "-prev"),       # hidden units +inf behind the negative columns of W1
    (8, 2, 301, 301, 32, "add", "relu", "+prev"),       # A_{n-1} = +inf
    (32, 8, 77, 301, 64, "add", "relu", "one +prev"),   # in one head: one infinite term per sum
    (40, 8, 77, 301, 128, "add", "relu", "+prev"),      # tiles of 16 keys
    (8, 8, 301, 301, 32, "add", "silu", "+prev"),
    (32, 32, 77, 301, 64, "concat", "relu", "-prev"),
    (16, 4, 141, 301, 64, "concat", "relu", "delta"),    # A_delta = +inf
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "_".join(map(str, c)))
def test_infinite_scores_at_masked_keys(case):
    """The module turns what is infinite at the first `pad` keys into scores of -inf: they weigh nothing.  Weights of magnitude
    1 to 2, so that a term of 3e38 in the place of an infinite one would pass the float32 range."""
    H, Hkv, Lq, Lk, F, mix, act, what = case
    log(f"[case] split infinities {case}")
    B, r, pad = 2, 20, 37
    g = torch.Generator(device=DEV).manual_seed(7)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)
    q, k, v = rn(B, H, Lq, r), rn(B, Hkv, Lk, r), rn(B, Hkv, Lk, 128).to(torch.bfloat16)
    prev = rn(B, H, Lq, Lk) / 128                            # (finite scores of a few units)
    din = 2 * H if mix == "concat" else H
    w1 = 1 + torch.rand((din, F), generator=g, device=DEV)
    w2 = -1 - torch.rand((F, H), generator=g, device=DEV)
    if mix == "concat":
        q, k = q / 16, k / 16
    if what == "-prev":
        prev[..., :pad] = float("-inf")
        w1[:H, ::2] *= -1                                    # (every other hidden unit +inf, its neighbour 0)
    elif what == "+prev":
        prev[..., :pad] = float("inf")
    elif what == "one +prev":
        prev[:, 3, :, :pad] = float("inf")
    else:
        q, k = q.abs() + 0.1, k / 16
        k[:, :, :pad] = 3e38
        q[..., 0] = 2.0                                      # (2 * 3e38: past the float32 range)
    q, k, w1, w2, prev = q.to(torch.bfloat16), k.to(torch.bfloat16), w1.to(torch.bfloat16), w2.to(torch.bfloat16), prev.half()
    (out, scores), ran = stages(lambda: lisa.lisa_attn_prefill(
        q, k, v, prev, w1, w2, mix=lisa.MIX_CONCAT if mix == "concat" else lisa.MIX_ADD,
        act=lisa.ACT_SILU if act == "silu" else lisa.ACT_RELU))
    assert "k_split_scores" in ran
    seen = torch.ones(Lq, Lk, dtype=torch.bool).tril(Lk - Lq)
    rows = slice(max(0, pad + Lq - Lk), None)                # (rows that see more than masked keys)
    kd = k.clone()
    if what == "delta":
        kd[:, :, :pad] = float("inf")                        # (6e38 is finite in float64)
    A, O = reference(q, kd, v, prev, w1, w2, mix, True, act)
    masked = seen & (torch.arange(Lk) < pad)
    assert bool((A[..., masked] == float("-inf")).all())
    assert bool((scores.cpu()[..., masked] <= -60000).all())
    assert torch.isfinite(out).all()
    assert err(out[:, rows].flatten(2), O[:, rows].flatten(2)) <= TOL_O


@pytest.mark.parametrize("Lq,Lk,causal", [(301, 301, True), (40, 301, True), (33, 129, False), (2, 65, True), (19, 19, True)])
@pytest.mark.parametrize("kind", ["std", "share", "add"])
def test_infinite_v(kind, Lq, Lk, causal):
    """An infinite element of V makes its feature infinite in the rows that see its key, whatever bits the probability has (all
    of them 1 in half of the heads: equal scores), NaN makes it NaN, and the other rows and features stay what they are."""
    B, H, Hkv, r, F = 2, 8, 4, 20, 32
    log(f"[case] split infinite V {kind} {Lq}x{Lk}")
    g = torch.Generator(device=DEV).manual_seed(Lk)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)
    v = rn(B, Hkv, Lk, 128).to(torch.bfloat16)
    at = {(Lk // 2, 5): float("inf"), (Lk - 2, 70): float("-inf"), (0, 127): float("inf"), (Lk // 3, 33): float("nan")}
    rep = lambda t: t.cpu().double().repeat_interleave(H // Hkv, 1)
    if kind == "std":
        q, k = rn(B, H, Lq, 128).to(torch.bfloat16), rn(B, Hkv, Lk, 128).to(torch.bfloat16)
        q[:, ::2] = 0
        A = q.cpu().double() @ rep(k).transpose(-1, -2).contiguous() / 128 ** 0.5
    else:
        q, k, prev = rn(B, H, Lq, r).to(torch.bfloat16), rn(B, Hkv, Lk, r).to(torch.bfloat16), rn(B, H, Lq, Lk).half()
        w1, w2 = (rn(H, F) / H ** 0.5).to(torch.bfloat16), (rn(F, H) / F ** 0.5).to(torch.bfloat16)
        prev[:, ::2] = 1.0
        if kind == "add":
            q[:, ::2] = 0
            prev[:] = prev[:, :1]
            w2[:, ::2] = 0                                   # (A_n = 0 in every other head)
            A = reference(q, k, v, prev, w1, w2, "add", causal)[0]
        else:
            A = prev.cpu().double()
    O = softmax_v(A, rep(v), causal)                         # [B,Lq,H,128], of the finite V
    last = torch.arange(Lq) + Lk - Lq if causal else torch.full((Lq,), Lk - 1)
    for (key, d), x in at.items():
        v[:, :, key, d] = x
        O[:, last >= key, :, d] = x
    if kind == "std":
        out = lisa.std_attn_scores(q, k, v, causal=causal)[1]
    elif kind == "add":
        out = lisa.lisa_attn_prefill(q, k, v, prev, w1, w2, causal=causal)[0]
    else:
        out = lisa.lisa_attn_prefill(None, None, v, prev, None, None, mix=lisa.MIX_SHARE, causal=causal)[0]
    torch.cuda.synchronize()
    got, fin = out.cpu().double(), torch.isfinite(O)
    assert torch.equal(got[~fin].nan_to_num(nan=7.0), O[~fin].nan_to_num(nan=7.0))
    rms = O.masked_fill(~fin, 0).pow(2).mean(-1, keepdim=True).sqrt()
    assert float(((got - O).masked_fill(~fin, 0).abs() / rms).max()) <= TOL_O
