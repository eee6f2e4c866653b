"""Rows with special values in the streaming forms, each against the FP64 result or
the one-row kernels' of the same row: row scales of 0, and rows whose first byte
is the last of a line.  A cap on the row groups
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


# the widest rows of one and two waves' 256 vectors each that begin at any byte of a line
@pytest.mark.parametrize("waves", [1, 2, 5])
def test_fp8_softmax_of_rows_at_the_end_of_a_line(capped, waves):
    # 127 bytes before the row and the row itself are one byte more than the waves'
    # vectors hold with a phase of 126: the row's last element is a vector of its own
    N = 4096 * waves - 126
    M, ld = 9, 4096 * waves
    print(f"[special] fp8 softmax phase 127 {M} x {N}", flush=True)
    flat = (torch.randn(M * ld + 128, device="cuda") * 50).clamp(-448, 448).to(torch.float8_e4m3fn)
    x = flat[127:127 + M * ld].view(M, ld)[:, :N]
    x[2, N - 1] = 448.0
    s = torch.rand(M, device="cuda") * 1e-2 + 1e-3
    out = torch.full_like(flat, 1.0)[127:127 + M * ld].view(M, ld)[:, :N]
    assert x.data_ptr() % 128 == 127 and out.data_ptr() % 128 == 127
    y, ys = C.softmax_fwd(x, s, out=out, p=C.plan("resident"), h=capped)
    ref = torch.softmax(x.double() * s.double()[:, None], 1)
    assert bool((ys.double() * 448 / ref.amax(1) - 1).abs().max() <= 1e-5)
    v = ref / ys.double()[:, None]
    step = torch.clamp(2.0 ** torch.floor(torch.log2(v.clamp_min(2.0 ** -6))) / 8, min=2.0 ** -9)
    assert bool(((y.double() - v).abs() <= step + 1e-5 * v).all())
    assert capped.check_errors() == C.OK
