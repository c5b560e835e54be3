"""Decode steps by data flow, stacks and single layers: the sizes where the split can go wrong.  Every layer of every sequence
against the oracle, and kept score rows against rows that stay inside the workspace, bit for bit."""
import pytest
import torch

from oracle import cref
from paper_2408_01890_amd import lisa, synth
from paper_2408_01890_amd import patterns as pt
from tests import helpers as hp
from tests.test_gpu_parity import log, oracle_decode_lisa, run_pattern_stack

pytestmark = pytest.mark.gpu
DEV = "cuda"

MIXED = (pt.STD, pt.LISA, pt.SHARE, pt.LISA, pt.STD, pt.SHARE, pt.SHARE, pt.LISA, pt.LISA, pt.LISA, pt.LISA, pt.STD)
# more layers than one group takes (48): the row passes from group to group, to a LiSA layer and, through
# layers that share directly, from one group to the one after the next
LONG = (pt.STD,) + (pt.LISA,) * 49 + (pt.STD,)
LONG_SHARE = (pt.STD, pt.LISA) + (pt.SHARE,) * 96 + (pt.LISA, pt.SHARE, pt.STD)

CASES = [  # H, Hkv, ctx, d_k, r, F, B, Lmax, dim_major, kinds
    (8, 8, 15, 128, 22, 16, 1, 16, True, MIXED),       # one block of 16 positions
    (8, 4, 127, 128, 7, 32, 2, 128, True, MIXED),      # exactly one block of 128 keys; odd rank; two heads per kv head
    (40, 40, 128, 128, 22, 80, 1, 131, True, MIXED),   # one key in the second block; rows that are not 16-byte aligned
    # few workgroups, so that the last one of an output merges its spans (512 keys of d_k = 128, 1024 of 64)
    (8, 8, 511, 128, 22, 16, 1, 512, True, MIXED),     # exactly one span
    (8, 8, 512, 128, 22, 16, 1, 520, True, MIXED),     # one key in the second
    (8, 2, 1500, 128, 11, 32, 2, 1504, True, MIXED),   # three spans, four heads per kv head
    (8, 8, 1023, 64, 20, 16, 1, 1024, True, MIXED),
    (8, 4, 1024, 64, 20, 16, 1, 1025, False, MIXED),
    (16, 4, 300, 64, 20, 33, 2, 320, False, MIXED),    # row-major K_LR, d_k = 64, four heads per kv head
    (40, 8, 257, 128, 22, 80, 1, 264, True, MIXED),    # five heads per kv head
    (64, 2, 64, 64, 16, 128, 1, 72, True, MIXED),      # widest chain; 32 heads per kv head
    (33, 33, 40, 64, 3, 100, 1, 48, True, MIXED),      # heads in a block of their own
    (8, 8, 20, 64, 12, 16, 1, 24, True, LONG),
    (8, 8, 140, 64, 12, 16, 1, 144, True, LONG_SHARE),
    (8, 2, 700, 128, 12, 16, 1, 704, True, LONG_SHARE),   # two spans: counters, then a group of sharing layers alone, which has none
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"h{c[0]}_{c[1]}_ctx{c[2]}_dk{c[3]}_f{c[5]}_n{len(c[9])}")
def test_decode_stack_sizes(case):
    H, Hkv, ctx, dk, r, F, B, Lmax, dim_major, kinds = case
    log(f"[case] stack {case[:9]} {len(kinds)} layers")
    # (the identity-like FFN of the shared inputs needs F >= 2H)
    stk = synth.DecodeStack(f"stack_h{H}_ctx{ctx}", "bf16", B, H, Hkv, ctx, 256, dk, r, max(F, 2 * H), len(kinds), 1)
    run_pattern_stack(stk, kinds, list(range(B)), dim_major=dim_major, Lmax=Lmax)


@pytest.mark.parametrize("ctx", [200, 700])
def test_stack_whose_layers_share_result_buffers(ctx):
    """Two score rows used in turn and one output for all layers: what the single calls leave in this order."""
    H, Hkv, dk, r, F, B, Lk = 8, 4, 128, 22, 32, 2, ctx + 1
    log(f"[case] stack with shared result buffers, ctx {ctx}")
    stk = synth.DecodeStack("shared", "bf16", B, H, Hkv, ctx, 256, dk, r, F, len(MIXED), 1)
    code = {pt.STD: lisa.LAYER_STD, pt.LISA: lisa.LAYER_LISA, pt.SHARE: lisa.LAYER_SHARE}
    rows = [torch.empty((B, H, Lk), dtype=torch.float16, device=DEV) for _ in range(4)]
    outs = [torch.empty((B, H, dk), dtype=torch.float32, device=DEV) for _ in range(2)]
    layers = []
    for n, kind in enumerate(MIXED):
        ly = synth.make_decode_layer(stk, n, device=DEV, kind=kind)
        rec = dict(kind=code[kind], v_cache=ly["v_cache"], out=outs[0], score_row=rows[n % 2])
        if kind == pt.STD:
            rec.update(q=ly["q"], k_cache=ly["k_cache"])
            lisa.std_attn_decode(ly["q"], ly["k_cache"], ly["v_cache"], Lk, out=outs[1], score_row_out=rows[2 + n % 2])
        elif kind == pt.LISA:
            rec.update(q=ly["q_lr"], k_cache=ly["k_lr_cache"], w1=ly["w1"], w2=ly["w2"])
            lisa.lisa_attn_decode(ly["q_lr"], ly["k_lr_cache"], ly["v_cache"], Lk, rows[2 + (n + 1) % 2], ly["w1"], ly["w2"],
                                  out=outs[1], score_row_out=rows[2 + n % 2], write_scores=True)
        else:
            lisa.lisa_attn_decode(None, None, ly["v_cache"], Lk, rows[2 + (n + 1) % 2], None, None, mix=lisa.MIX_SHARE,
                                  out=outs[1], score_row_out=rows[2 + n % 2], write_scores=True)
        layers.append(rec)
    stack = lisa.DecodeStack(layers, Lk, r=r, F=F)
    for _ in range(2):
        stack.step()
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1])
        assert torch.equal(rows[0], rows[2]) and torch.equal(rows[1], rows[3])


SINGLE = [  # H, Hkv, ctx, d_k, r, F, B, concat: one workgroup's keys and one more; many spans; both forms of the V stream
    (8, 8, 511, 128, 22, 16, 1, False), (8, 2, 512, 128, 22, 16, 2, False), (16, 4, 1030, 64, 20, 64, 1, True),
    (8, 4, 5000, 128, 11, 40, 1, False), (32, 32, 600, 128, 20, 256, 8, True), (40, 40, 513, 128, 22, 80, 7, False)]


@pytest.mark.parametrize("case", SINGLE, ids=lambda c: f"h{c[0]}_{c[1]}_ctx{c[2]}_dk{c[3]}_b{c[6]}")
def test_single_layer_decode_spans(case):
    H, Hkv, ctx, dk, r, F, B, concat = case
    log(f"[case] single decode {case}")
    Lk, tol = ctx + 1, hp.TOL[torch.bfloat16]
    stk = synth.DecodeStack("single", "bf16", B, H, Hkv, ctx, 256, dk, r, F, 2, 1)
    std = synth.make_decode_layer(stk, 0, device=DEV)
    row, out = lisa.std_attn_decode(std["q"], std["k_cache"], std["v_cache"], Lk)
    ly = synth.make_decode_layer(stk, 1, device=DEV, mix="concat" if concat else "add", ffn="fan_in")
    o2, row2 = lisa.lisa_attn_decode(ly["q_lr"], ly["k_lr_cache"], ly["v_cache"], Lk, row, ly["w1"], ly["w2"],
                                     mix=lisa.MIX_CONCAT if concat else lisa.MIX_ADD)
    o3, row3 = lisa.lisa_attn_decode(None, None, ly["v_cache"], Lk, row, None, None, mix=lisa.MIX_SHARE)
    torch.cuda.synchronize()
    assert torch.equal(row3, row)
    for b in range(0, B, 3):
        ref = hp.oracle_std_rows(std["q"][:, :, None, :], std["k_cache"][:, :, :Lk], b, [0])
        assert hp.row_rel_err(hp.f64(row[b])[None], ref) <= tol
        o_ref = cref.softmax_v_rows(hp.f64(std["v_cache"][b])[:, :Lk], [0], ref, 1)
        assert hp.row_rel_err(hp.f64(out[b])[None], o_ref) <= tol
        a_ref, o_ref = oracle_decode_lisa(ly, b, Lk, hp.f64(row[b]), True, mix=int(concat))
        assert hp.row_rel_err(hp.f64(row2[b])[None], a_ref) <= tol and hp.row_rel_err(hp.f64(o2[b])[None], o_ref) <= tol
        o_ref = cref.softmax_v_rows(hp.f64(ly["v_cache"][b])[:, :Lk], [0], hp.f64(row[b])[None], 1)
        assert hp.row_rel_err(hp.f64(o3[b])[None], o_ref) <= tol


@pytest.mark.parametrize("H,Hkv,B,std_spread,add_spread", [
    (8, 8, 47, True, True), (8, 8, 48, False, False),         # 376 and 384 units of 128 keys: the line of narrow layers
    (24, 24, 48, False, True), (24, 24, 80, False, False),    # 640 units: the line of wide ADD modules
    (8, 4, 80, True, True),                                   # two query heads per kv head: below 16 MB of scratch always
])
def test_single_layers_on_both_sides_of_the_line(H, Hkv, B, std_spread, add_spread):
    """Which kernels a single layer takes, and that both give the oracle's results there."""
    Lk, dk, r, F, tol = 1024, 128, 22, 64, hp.TOL[torch.bfloat16]
    log(f"[case] single decode, {H}/{Hkv} heads, {B} sequences")
    stk = synth.DecodeStack("line", "bf16", B, H, Hkv, Lk - 1, 256, dk, r, F, 2, 1)
    std, ly = synth.make_decode_layer(stk, 0, device=DEV), synth.make_decode_layer(stk, 1, device=DEV, ffn="fan_in")

    def stages(call):
        lisa.profile_enable(True)
        try:
            return call(), set(lisa.profile_collect())
        finally:
            lisa.profile_enable(False)

    (row, out), names = stages(lambda: lisa.std_attn_decode(std["q"], std["k_cache"], std["v_cache"], Lk))
    assert ("k_stack_pv" in names) == std_spread and ("k_decode_part_std" in names) != std_spread
    (o2, row2), names = stages(lambda: lisa.lisa_attn_decode(ly["q_lr"], ly["k_lr_cache"], ly["v_cache"], Lk, row, ly["w1"], ly["w2"]))
    assert ("k_stack_pv" in names) == add_spread and ("k_decode_part_lisa" in names) != add_spread
    torch.cuda.synchronize()
    for b in (0, B // 2, B - 1):
        ref = hp.oracle_std_rows(std["q"][:, :, None, :], std["k_cache"][:, :, :Lk], b, [0])
        assert hp.row_rel_err(hp.f64(row[b])[None], ref) <= tol
        o_ref = cref.softmax_v_rows(hp.f64(std["v_cache"][b])[:, :Lk], [0], ref, 1)
        assert hp.row_rel_err(hp.f64(out[b])[None], o_ref) <= tol
        a_ref, o_ref = oracle_decode_lisa(ly, b, Lk, hp.f64(row[b]), True)
        assert hp.row_rel_err(hp.f64(row2[b])[None], a_ref) <= tol and hp.row_rel_err(hp.f64(o2[b])[None], o_ref) <= tol


@pytest.mark.parametrize("H,Hkv,dk,Lk,B,masked", [
    (8, 8, 128, 128, 1, (0, 40)),       # all of a wave's first 32 keys
    (8, 2, 64, 1500, 2, (0, 1100)),     # a whole workgroup's keys, merged with the next one's
    (8, 8, 128, 700, 1, (512, 700)),    # the last workgroup's
    (32, 32, 128, 2100, 4, (100, 400)),  # the long stream: 128 keys per wave
    (32, 1, 128, 16500, 8, (300, 1000)),  # scratch beyond 16 MB: k_decode_part, chunks of 128 keys
])
def test_masked_keys_weigh_nothing(H, Hkv, dk, Lk, B, masked):
    """Keys whose shared score is -inf (padding in front of a prompt) over whole pieces of the split."""
    log(f"[case] masked keys {H} {Hkv} {dk} {Lk} {B} {masked}")
    g = torch.Generator().manual_seed(5)
    row = torch.randn((B, H, Lk), generator=g).half()
    row[..., masked[0]:masked[1]] = float("-inf")
    v = torch.randn((B, Hkv, Lk, dk), generator=g).to(torch.bfloat16)
    out, _ = lisa.lisa_attn_decode(None, None, v.to(DEV), Lk, row.to(DEV), None, None, mix=lisa.MIX_SHARE)
    ref = (torch.softmax(row.double(), -1).reshape(B, Hkv, H // Hkv, Lk) @ v.double()).reshape(B, H, dk)
    # float32 sums of exact products; the result leaves as the output type of the call
    tol = 1e-5 if out.dtype == torch.float32 else hp.TOL[torch.bfloat16]
    err = (out.double().cpu() - ref).norm(dim=-1) / ref.norm(dim=-1)
    assert torch.isfinite(out).all() and float(err.max()) <= tol
