"""lisa_kd_huber on row-major scores at the sizes where its numbering of the pieces can go wrong, against the float64 oracle:
rows that start anywhere in a line, a last piece that is not whole, fewer elements than a piece, a middle row without a partner,
more pieces than the grid takes in one share."""
import pytest
import torch

from oracle import npref
from paper_2408_01890_amd import lisa
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda"
RTOL = 2e-6      # float32 per element and per piece of 16 bytes, float64 from there on


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dtype,B,H,Lq,Lk", [
    (torch.float16, 1, 1, 1, 1), (torch.float16, 1, 1, 2, 3), (torch.float16, 1, 3, 1, 7), (torch.float32, 1, 1, 1, 3),
    (torch.float16, 2, 3, 5, 63), (torch.float16, 1, 2, 7, 64), (torch.float16, 1, 2, 8, 65), (torch.float32, 1, 3, 33, 33),
    (torch.float16, 1, 5, 129, 511), (torch.float16, 2, 8, 203, 203), (torch.float16, 1, 1, 3, 20011),
    (torch.float16, 1, 8, 1501, 1501), (torch.float32, 1, 8, 1031, 1200)])
def test_kd_huber_rows_of_any_length(dtype, B, H, Lq, Lk, causal):
    g = torch.Generator(device=DEV).manual_seed(Lq * Lk)
    t = (torch.randn((B, H, Lq, Lk), generator=g, device=DEV) * 3).to(dtype)
    s = (t.float() + torch.randn((B, H, Lq, Lk), generator=g, device=DEV) * 2).to(dtype)
    want = npref.kd_loss(hp.f64(s), hp.f64(t), 1.0, causal)
    if causal:                                               # what lies above the diagonal must not count
        hidden = torch.ones(Lq, Lk, dtype=torch.bool, device=DEV).triu(Lk - Lq + 1)
        s, t = s.masked_fill(hidden, float("nan")), t.masked_fill(hidden, float("nan"))
    got = lisa.lisa_kd_huber(s, t, causal=causal).cpu().numpy()
    assert abs(got[1] - want) <= RTOL * want and got[0] == got[1]
