"""Rows with special values in the streaming forms, each against the FP64 result or
the one-row kernels' of the same row: row scales of 0, rows whose first byte
is the last of a line, NaN, infinities and lone large elements under LayerNorm,
constant FP8 rows, FP8 rows of tiny outputs, huge gradients, logits of any size (in
every kernel), and FP8 rows beside rows of another kind.  A cap on the row groups
makes a few rows enough for a plan to stream."""
import pytest
import torch

from paper_2609_01864_amd import credit as C

from _cases import ALL_PLANS
from test_stream_gpu import DTN, capped  # noqa: F401  (fixture)
from test_stream_rows_gpu import ULP, _bound, _logits_ref

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


TD = {"f32": torch.float32, "bf16": torch.bfloat16}


# rows held by one wave, by several, and by the members of a split row
@pytest.mark.parametrize("N,k", [(8, 1), (130, 1), (512, 1), (1000, 1), (1024, 1), (5003, 1), (512, 4), (5003, 4)])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
def test_layernorm_of_rows_with_nan_or_infinity(capped, dtype, N, k):
    M = 33
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    if dtype == "fp8" and N < 16:
        N = 16
    print(f"[special] layernorm nan / inf {dtype} {M} x {N} {p}", flush=True)
    x = torch.randn((M, N), device="cuda") + 10
    bad = {1: (N // 2 + 3, float("nan")), 6: (0, float("nan")), 11: (N - 1, float("nan"))}
    if dtype != "fp8":  # e4m3 has no infinity
        bad |= {14: (N // 2 + 3, float("inf")), 17: (0, float("inf")), 20: (N - 1, -float("inf"))}
    g, b = torch.rand(N, device="cuda") + 0.5, torch.randn(N, device="cuda")
    if dtype == "fp8":
        q = x.to(torch.float8_e4m3fn)
        w = q.clone()
        for r, (c, _) in bad.items():
            w.view(torch.uint8)[r, c] = 0x7F
        s = torch.rand(M, device="cuda") + 0.5
    else:
        q, s = x.to(TD[dtype]), None
        w = q.clone()
        for r, (c, v) in bad.items():
            w[r, c] = v
        w[23] = float("inf")
        bad[23] = (0, float("inf"))
    good = C.layernorm_fwd(q, g, b, x_scale=s, p=p, h=capped)
    y, ys, mean, rstd = C.layernorm_fwd(w, g, b, x_scale=s, p=p, h=capped)
    rows = sorted(bad)
    # the variance of a row with a NaN or an infinity is NaN, in FP64 too
    assert bool(torch.isnan(rstd[rows]).all()) and not bool(torch.isfinite(mean[rows]).any())
    if dtype != "fp8":
        assert bool(torch.isnan(y[rows].float()).all())
    keep = [r for r in range(M) if r not in bad]
    for a, e in zip((y, ys, mean, rstd), good):
        if a is not None:
            assert torch.equal(a[keep].view(torch.uint8), e[keep].view(torch.uint8))
    assert capped.check_errors() == C.OK


# slices of one wave whose lanes are mostly idle, and of a second wave with few
@pytest.mark.parametrize("dtype,N", [("f32", 67), ("f32", 132), ("bf16", 132), ("bf16", 260), ("f32", 530), ("bf16", 1050)])
def test_layernorm_of_rows_with_one_large_element(capped, dtype, N):
    M, epv = 66, 4 if dtype == "f32" else 8
    print(f"[special] layernorm spike {dtype} {M} x {N}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randn((M, N), device="cuda", generator=gen)
    x[:, N - epv] = 40 + 60 * torch.rand(M, device="cuda", generator=gen)
    x = x.to(TD[dtype])
    g, b = torch.ones(N, device="cuda"), torch.zeros(N, device="cuda")
    _, _, mean, rstd = C.layernorm_fwd(x, g, b, p=C.plan("resident"), h=capped)
    xd = x.double()
    rs = 1 / torch.sqrt(xd.var(1, correction=0) + 1e-5)
    # M2 = sum d^2 - (sum d)^2 / n about a shift of at most a twelfth of the
    # element: the sum of squares is at most 1.4 M2, of 16 terms a lane and 8
    # more roundings; half of their relative error in rstd, and 4 of its own
    assert bool(((rstd.double() / rs - 1).abs() <= (0.5 * 1.4 * 24 + 4) * 2.0 ** -24).all())
    assert bool(((mean.double() - xd.mean(1)).abs() <= 8 * 2.0 ** -24 * xd.abs().amax(1)).all())
    assert capped.check_errors() == C.OK


@pytest.mark.parametrize("N,k", [(16, 1), (1000, 1), (1024, 1), (5001, 1), (16384, 1), (4096, 4), (20001, 8)])
def test_fp8_layernorm_of_constant_rows(capped, N, k):
    # x - mean is 0 in every element, so y is beta, whatever 1 / sqrt(eps) times the value
    M = 29  # over three rounds of two groups of four rows
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    print(f"[special] fp8 layernorm constant {M} x {N} {p}", flush=True)
    q = (torch.randn((M, N), device="cuda") * 50).clamp(-448, 448).to(torch.float8_e4m3fn)
    for r, v in ((2, 448.0), (5, -416.0), (6, 1.125), (11, 0.0), (16, 104.0)):
        q[r] = v
    rows = [2, 5, 6, 11, 16]
    s = torch.rand(M, device="cuda") + 0.5
    g, b = torch.rand(N, device="cuda") + 0.5, torch.randn(N, device="cuda")
    one = C.Handle(0)
    try:
        for beta in (torch.zeros(N, device="cuda"), b):
            y, ys, mean, rstd = C.layernorm_fwd(q, g, beta, x_scale=s, p=p, h=capped)
            w, ws, _, _ = C.layernorm_fwd(q, g, beta, x_scale=s, p=p, h=one)
            amax = beta.abs().max()
            want = (amax / 448 if amax > 0 else torch.ones_like(amax)).expand(len(rows))
            assert torch.allclose(ys[rows], want, rtol=2.0 ** -23, atol=0)
            assert torch.equal(ys[rows], ws[rows]) and torch.equal(y.view(torch.uint8)[rows], w.view(torch.uint8)[rows])
            assert torch.equal(mean[rows], (q[rows, 0].float() * s[rows]))
    finally:
        one.close()
    assert capped.check_errors() == C.OK


@pytest.mark.parametrize("N,k", [(512, 1), (5001, 1), (4096, 4)])
def test_fp8_layernorm_of_tiny_outputs(capped, N, k):
    # 448 / amax is infinite below 1.3e-36: the codes saturate
    M = 29  # over three rounds of two groups of four rows
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    print(f"[special] fp8 layernorm tiny outputs {M} x {N} {p}", flush=True)
    q = (torch.randn((M, N), device="cuda") * 50).clamp(-448, 448).to(torch.float8_e4m3fn)
    s = torch.rand(M, device="cuda") + 0.5
    b = torch.zeros(N, device="cuda")
    one = C.Handle(0)
    try:
        for scale in (1e-30, 1e-36, 1e-37):
            g = (torch.rand(N, device="cuda") + 0.5) * scale
            y, ys, _, _ = C.layernorm_fwd(q, g, b, x_scale=s, p=p, h=capped)
            w, _, _, _ = C.layernorm_fwd(q, g, b, x_scale=s, p=p, h=one)
            assert not bool(torch.isnan(y.float()).any())
            if scale == 1e-37:  # every code is +-448
                assert torch.equal(y.view(torch.uint8), w.view(torch.uint8))
    finally:
        one.close()
    assert capped.check_errors() == C.OK


# slices held one, two and four vectors a lane
@pytest.mark.parametrize("N,k", [(200, 1), (2000, 1), (4111, 1), (9001, 1), (30001, 4)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_logits_backward_of_huge_gradients(capped, dtype, N, k):
    # the gradient is linear, and a power of two is exact at every step of it
    M = 17
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    print(f"[special] logits backward, huge gradients {dtype} {M} x {N} {p}", flush=True)
    x = (3 * torch.randn((M, N), device="cuda")).to(TD[dtype])
    dy = torch.randn((M, N), device="cuda").to(TD[dtype])
    dx, _ = C.softmax_logits_bwd(x, dy, p=p, h=capped)
    for e in (40, 100, 112):
        got, _ = C.softmax_logits_bwd(x, dy * 2.0 ** e, p=p, h=capped)
        assert bool(torch.isfinite(got.float()).all())
        big = dx.float().abs() > 2.0 ** -100
        assert torch.equal(got.double()[big], dx.double()[big] * 2.0 ** e)
    assert capped.check_errors() == C.OK


def far_rows(N, td):
    """Rows masked in part or throughout with values of any size, and others of huge logits."""
    low = torch.finfo(td).min
    x = torch.randn((21, N), device="cuda", generator=torch.Generator(device="cuda").manual_seed(N))
    for r, v in enumerate((-1e4, -3e8, -5e8, -1e9, -3e9, -1e10, -1e30, low, 6e8, 1e10, 3e38)):
        x[r] = v                                 # constant: uniform
    x[11, N // 3:] = -1e9                        # masked in part
    x[12, : (6 * N) // 10] = -1e10
    x[13, N // 5:] = low
    x[14] = -1e9                                 # two masks, the larger one's elements share 1
    x[14, N // 2:] = low
    x[15] = -1e30
    x[15, ::3] = -1e10
    x[16, N // 4] = 1e10                         # one element is all there is
    x[17] *= 1e9
    x[18] *= 1e30
    x[19] = low
    x[19, N - 1] = -1e30
    return x.to(td)                              # row 20: ordinary


@pytest.mark.parametrize("form", ["one_row", "streaming"])
@pytest.mark.parametrize("N", [17, 1000, 5001, 40000, 70001])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_softmax_of_logits_of_any_size(capped, gpu_handle, dtype, N, form):
    h = capped if form == "streaming" else gpu_handle
    x = far_rows(N, TD[dtype])
    dy = torch.randn(x.shape, device="cuda").to(x.dtype)
    want = torch.softmax(x.double(), 1)
    ref, yy, g = _logits_ref(x, dy)
    assert bool(torch.isfinite(want).all())
    for v, k in ALL_PLANS:
        p = C.plan(v, k)
        if h.plan_legal(C.SOFTMAX, C.FWD, DTN[dtype], 21, N, p):
            print(f"[special] softmax of any logits {form} {dtype} {N} {p}", flush=True)
            y, _ = C.softmax_fwd(x, p=p, h=h)
            tol = 2e-6 if dtype == "f32" else ULP["bf16"] * want + 2.0 ** -132
            assert bool(((y.double() - want).abs() <= tol).all()), p
        if h.plan_legal(C.SOFTMAX_LOGITS, C.BWD, DTN[dtype], 21, N, p):
            dx = C.softmax_logits_bwd(x, dy, p=p, h=h)[0].double()
            assert bool(((dx - ref).abs() <= _bound(dtype, yy, g) + 2.0 ** -132).all()), p
    assert h.check_errors() == C.OK


@pytest.mark.parametrize("N,k", [(1000, 1), (5001, 1), (16384, 1), (20001, 8)])
def test_fp8_layernorm_rows_do_not_depend_on_each_other(capped, N, k):
    # four rows share a round; one whose spread is small beside its mean takes
    # its moments in a second pass
    M = 32
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    print(f"[special] fp8 layernorm neighbours {M} x {N} {p}", flush=True)
    q = (torch.randn((M, N), device="cuda") * 40 + 15).clamp(-448, 448).to(torch.float8_e4m3fn)
    s = torch.rand(M, device="cuda") + 0.5
    g, b = torch.rand(N, device="cuda") + 0.5, torch.randn(N, device="cuda")
    want = C.layernorm_fwd(q, g, b, x_scale=s, p=p, h=capped)
    q[1::4] = 416.0
    q[1::4, ::7] = 448.0
    got = C.layernorm_fwd(q, g, b, x_scale=s, p=p, h=capped)
    keep = [r for r in range(M) if r % 4 != 1]
    for a, e in zip(got, want):
        assert torch.equal(a[keep].view(torch.uint8), e[keep].view(torch.uint8))
    assert capped.check_errors() == C.OK
