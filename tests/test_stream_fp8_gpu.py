"""The streaming forms of the FP8 LayerNorm and softmax forward at the sizes where
their slices end -- one vector, whole waves, one vector more, the largest,
partial vectors, short and empty members, a last round with fewer rows --
against the oracle, the LayerNorm's plan when none is given, and rows whose
spread is far below their mean, that are constant or hold a NaN code."""
import numpy as np
import pytest
import torch

from paper_2609_01864_amd import credit as C

from _cases import EPS, Case, OPNUM, check_case
from test_stream_gpu import capped  # noqa: F401  (fixture)

VECS = {1: (1, 2, 63, 64, 65, 512, 1000, 1024), 2: (1, 64, 129, 1024), 8: (1, 130, 300, 1024), 32: (1, 33, 64)}


@pytest.mark.gpu
@pytest.mark.parametrize("k", sorted(VECS))
def test_slice_edges(capped, k):
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    seen = 0
    for n, vec in enumerate(VECS[k]):
        full = vec * k * 16
        for N in {full, full - 1, full - 15, full - max(1, k - 1) * 16 - 2}:
            if N < 16:
                continue
            M = (25, 29, 34)[n % 3]  # over three rounds of two groups of four rows
            if not capped.plan_legal(*OPNUM["layernorm_fwd"], C.FP8, M, N, p):
                continue
            g = capped.geometry(*OPNUM["layernorm_fwd"], C.FP8, M, N, p)
            seen += g["rows"] == 4 and g["block"] == 64 * -(-(-(-N // 16 // k)) // 64)
            print(f"[stream] fp8 {M} x {N} {p} {g}", flush=True)
            case = Case("layernorm_fwd", "fp8", M, N, seed=n + N)
            ref = case.reference()
            out = case.run(capped, p, ref=ref)
            check_case(case, out, ref)
            for pad, off in ((5, 0), (16, 3)):
                check_case(case, case.run(capped, p, ld_pad=pad, offset=off, ref=ref), ref)
            if k > 1:
                capped.set_option(C.OPT_TEST_SKEW, 1)
                try:
                    skewed = case.run(capped, p, ref=ref)
                finally:
                    capped.set_option(C.OPT_TEST_SKEW, 0)
                for key in out:
                    if isinstance(out[key], np.ndarray):
                        assert np.array_equal(out[key], skewed[key]), key
    assert seen >= 4
    assert capped.check_errors() == C.OK


@pytest.mark.gpu
@pytest.mark.parametrize("k", [1, 4])
def test_offset_constant_and_nan_rows(capped, k):
    M, N = 30, 4096 * k
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    gen = torch.Generator(device="cuda").manual_seed(k)
    x = torch.randn((M, N), device="cuda", generator=gen) * 60
    x[3] = 416 + 20 * torch.sign(x[3])      # two neighbouring codes
    x[4] = 448
    x[4, 7::512] = 416
    x[5] = 104                              # constant
    x[6] = 0
    q = x.clamp(-448, 448).to(torch.float8_e4m3fn)
    s = torch.rand(M, device="cuda", generator=gen) * 1e-2 + 1e-3
    g = torch.rand(N, device="cuda", generator=gen) + 0.5
    b = torch.randn(N, device="cuda", generator=gen) * 0.1
    print(f"[stream] fp8 special {p}", flush=True)
    y, ys, mean, rstd = C.layernorm_fwd(q, g, b, x_scale=s, p=p, h=capped)
    xd = q.double() * s.double()[:, None]
    mu, var = xd.mean(1), xd.var(1, correction=0)
    rs = 1 / torch.sqrt(var + EPS)
    # the mean to a few roundings of it; 1 / sqrt(var + eps) to those of the
    # variance, whose moments are taken about the mean
    assert bool(((mean.double() - mu).abs() <= 8 * 2.0 ** -24 * xd.abs().amax(1)).all())
    assert bool(((rstd.double() - rs).abs() <= 64 * 2.0 ** -24 * rs + rs ** 3 * (8 * 2.0 ** -24 * mu) ** 2).all())
    ref = (xd - mu[:, None]) * rs[:, None] * g.double() + b.double()
    amax = ref.abs().amax(1)
    # a rounding of the mean, scaled by 1 / spread, before the e4m3 step
    tol = rs * 8 * 2.0 ** -24 * mu.abs() * 1.5 + 1e-5
    assert bool(((ys.double() * 448 - amax).abs() <= 1e-5 * amax + tol).all())
    step = torch.clamp(2.0 ** torch.floor(torch.log2((ref / ys.double()[:, None]).abs().clamp_min(2.0 ** -6))) / 8, 2.0 ** -9)
    err = (y.double() * ys.double()[:, None] - ref).abs()
    assert bool((err <= ys.double()[:, None] * step + tol[:, None] + 1e-5 * ref.abs()).all())
    # a row with a NaN code: the same bytes as the one-row kernel, other rows untouched
    bad = q.clone()
    bad.view(torch.uint8)[9, N // 3] = 0x7F
    z, zs, zm, zr = C.layernorm_fwd(bad, g, b, x_scale=s, p=p, h=capped)
    one = C.Handle(0)
    try:
        w, ws, wm, wr = C.layernorm_fwd(bad[9:10], g, b, x_scale=s[9:10], p=C.plan("resident"), h=one)
    finally:
        one.close()
    assert torch.equal(z[9].view(torch.uint8), w[0].view(torch.uint8)) and torch.equal(zs[9], ws[0])
    assert bool(torch.isnan(zm[9])) and bool(torch.isnan(zr[9]))
    keep = [i for i in range(M) if i != 9]
    assert torch.equal(z.view(torch.uint8)[keep], y.view(torch.uint8)[keep]) and torch.equal(zs[keep], ys[keep])
    # a parameter that is not finite takes the clamp
    g2 = g.clone()
    g2[5] = float("inf")
    v, vs, _, _ = C.layernorm_fwd(q, g2, b, x_scale=s, p=p, h=capped)
    one = C.Handle(0)
    try:
        w, ws, _, _ = C.layernorm_fwd(q[0:1], g2, b, x_scale=s[0:1], p=C.plan("resident"), h=one)
    finally:
        one.close()
    assert torch.equal(v[0].view(torch.uint8), w[0].view(torch.uint8)) and torch.equal(vs[0], ws[0])
    assert capped.check_errors() == C.OK


@pytest.mark.gpu
def test_plan_of_a_call_without_one(capped):
    h = C.Handle(0)
    try:
        M, N = 4100, 20000  # slices of up to 16384 elements: two members
        q = (torch.randn((M, N), device="cuda") * 50).to(torch.float8_e4m3fn)
        s = torch.rand(M, device="cuda") * 1e-2 + 1e-3
        g, b = torch.rand(N, device="cuda"), torch.rand(N, device="cuda")
        got = C.layernorm_fwd(q, g, b, x_scale=s, h=h)
        want = C.layernorm_fwd(q, g, b, x_scale=s, p=C.plan("split", 2), h=h)
        assert all(torch.equal(a.view(torch.uint8), w.view(torch.uint8)) for a, w in zip(got, want))
        assert h.check_errors() == C.OK
    finally:
        h.close()


@pytest.mark.gpu
@pytest.mark.parametrize("k", [1, 2, 8])
def test_softmax_slice_edges_and_phases(capped, k):
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    vecs = (1, 2, 64, 65, 255, 256, 257, 1000, 4087, 4096) if k == 1 else (256, 512, 4096) if k == 2 else (256, 1024)
    seen = 0
    for n, vec in enumerate(vecs):
        full = vec * k * 16
        for N in {full, full - 1, full - 15} if k == 1 else {full}:
            if not capped.plan_legal(*OPNUM["softmax_fwd"], C.FP8, 7, N, p):
                continue
            g = capped.geometry(*OPNUM["softmax_fwd"], C.FP8, 7, N, p)
            one = C.plan_geometry(None, *OPNUM["softmax_fwd"], C.FP8, 7, N, p)
            seen += g["block"] != one["block"] or g["vpt"] != one["vpt"]
            print(f"[stream] fp8 softmax 7 x {N} {p} {g}", flush=True)
            case = Case("softmax_fwd", "fp8", 7, N, seed=n + N)
            ref = case.reference()
            check_case(case, case.run(capped, p, ref=ref), ref)
            for pad, off in ((0, 1), (5, 0), (77, 13), (128, 128)):
                check_case(case, case.run(capped, p, ld_pad=pad, offset=off, ref=ref), ref)
    assert seen >= 1  # (slices of 1024 vectors have the one-row kernels' geometry)
    assert capped.check_errors() == C.OK


@pytest.mark.gpu
def test_softmax_nan_row(capped):
    q = (torch.randn((9, 20001), device="cuda") * 50).to(torch.float8_e4m3fn)
    s = torch.rand(9, device="cuda") * 1e-2 + 1e-3
    y, ys = C.softmax_fwd(q, s, p=C.plan("resident"), h=capped)
    bad = q.clone()
    bad.view(torch.uint8)[4, 777] = 0x7F
    print("[stream] fp8 softmax nan", flush=True)
    z, zs = C.softmax_fwd(bad, s, p=C.plan("resident"), h=capped)
    keep = [i for i in range(9) if i != 4]
    assert bool(torch.isnan(zs[4])) and torch.equal(zs[keep], ys[keep])
    assert torch.equal(z.view(torch.uint8)[keep], y.view(torch.uint8)[keep])
    assert capped.check_errors() == C.OK
