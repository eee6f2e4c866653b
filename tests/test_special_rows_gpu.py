"""Rows with special values in the streaming forms, each against the FP64 result or
the one-row kernels' of the same row: row scales of 0.  A cap on the row groups
makes a few rows enough for a plan to stream."""
import pytest
import torch

from paper_2609_01864_amd import credit as C

from test_stream_gpu import capped  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


# 16-byte vectors that end in a part, in one wave, several, and the most of a form
@pytest.mark.parametrize("N", [17, 4111, 20001, 65000])
def test_fp8_softmax_of_a_row_scaled_by_zero(capped, N):
    # a row of zeros quantised with amax / 448 has the scale 0, and any code
    # then stands for 0: the uniform row, whose codes are all 448 = 0x7E
    print(f"[special] fp8 softmax scale 0 9 x {N}", flush=True)
    q = (torch.randn((9, N), device="cuda") * 50).clamp(-448, 448).to(torch.float8_e4m3fn)
    s = torch.rand(9, device="cuda") * 1e-2 + 1e-3
    want = C.softmax_fwd(q, s, p=C.plan("resident"), h=capped)
    z = s.clone()
    z[3] = z[8] = 0.0
    q.view(torch.uint8)[8] = 0
    y, ys = C.softmax_fwd(q, z, p=C.plan("resident"), h=capped)
    for r in (3, 8):
        assert bool((y.view(torch.uint8)[r] == 0x7E).all())
        # a sum of N ones, one division by it and one by 448
        assert abs(ys[r].item() * 448 * N - 1) <= 4 * 2.0 ** -24
    keep = [r for r in range(9) if r not in (3, 8)]
    assert torch.equal(y.view(torch.uint8)[keep], want[0].view(torch.uint8)[keep]) and torch.equal(ys[keep], want[1][keep])
    assert capped.check_errors() == C.OK
