"""The streaming form of the int8 row quantisation: codes and scales bit-exact
against the oracle at the sizes where its slices end, on rows of every BF16
significand of the largest element with ties, multiples and neighbours of the
decision boundaries, on rows whose factor is not an ordinary one, and -- beside
the one-row kernel -- on rows with infinities and NaN."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_01864_amd import credit as C

from test_stream_gpu import DTN, EPV, capped  # noqa: F401  (fixture)

TD = {"f32": torch.float32, "bf16": torch.bfloat16}
VECS = {1: (1, 2, 64, 65, 127, 256, 257, 1025, 2048, 2049, 4096, 4097), 2: (1, 65, 256, 641, 1025), 8: (1, 130, 640), 32: (1, 33)}


def _exact(x):
    codes, scale = oracle.quantize_rows(x.float().cpu().numpy(), "int8")
    return np.asarray(codes).view(np.int8), np.asarray(scale, dtype=np.float32)


@pytest.mark.gpu
@pytest.mark.parametrize("k", sorted(VECS))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_slice_edges(capped, dtype, k):
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    for n, vec in enumerate(VECS[k]):
        full = vec * k * EPV[dtype]
        for N in sorted({full, full - 1, full - max(1, k - 1) * EPV[dtype] - 2}):
            if N < EPV[dtype] or not capped.plan_legal(C.QUANT_INT8, C.FWD, DTN[dtype], 11, N, p):
                continue
            print(f"[quant] {dtype} 11 x {N} {p}", flush=True)
            gen = torch.Generator(device="cuda").manual_seed(n)
            ld = N + (0, 3, 8)[n % 3]
            flat = torch.randn(11 * ld + 8, device="cuda", generator=gen).to(TD[dtype])
            x = flat[n % 5:n % 5 + 11 * ld].view(11, ld)[:, :N]
            codes, scale = C.quantize_rows(x, "int8", p=p, h=capped)
            want, ws = _exact(x)
            assert np.array_equal(codes.cpu().numpy(), want)
            assert np.array_equal(scale.cpu().numpy(), ws)
    assert capped.check_errors() == C.OK


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_every_significand_of_the_largest(capped, dtype):
    # row m: the largest element is m / 128; then every BF16 value below it in
    # eleven binades, and the FP32 neighbours of its decision boundaries
    rows = []
    for m in range(128, 256):
        am = m / 128
        v = [s * q / 128 * 2.0 ** -u for u in range(11) for q in range(128, 256) for s in (1, -1) if q * 2.0 ** -u <= m]
        if dtype == "f32":
            for c in range(127):
                b = np.float32((c + 0.5) * am / 127)
                v += [float(b), float(np.nextafter(b, np.float32(0))), float(np.nextafter(b, np.float32(9)))]
        rows.append([am, am / 2, -am / 2] + v)
    N = max(map(len, rows))
    x = torch.tensor([r + [0.0] * (N - len(r)) for r in rows], dtype=torch.float32).to(TD[dtype]).cuda()
    scales = torch.tensor([1.0, 2.0 ** -20, 2.0 ** 90, 2.0 ** -99]).repeat(32)[:, None].cuda()
    x = (x.float() * scales).to(TD[dtype])
    print(f"[quant] {dtype} significands {tuple(x.shape)}", flush=True)
    codes, scale = C.quantize_rows(x, "int8", p=C.plan("resident"), h=capped)
    want, ws = _exact(x)
    assert np.array_equal(codes.cpu().numpy(), want)
    assert np.array_equal(scale.cpu().numpy(), ws)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_special_rows(capped, dtype):
    x = torch.randn((13, 6001), device="cuda").to(TD[dtype])
    x[1] = 0
    x[2] *= 2.0 ** -120
    x[3, 17] = float("inf")
    x[4, 5000] = float("nan")
    x[5] = float("nan")
    x[6, 6000] = -float("inf")
    x[7] = 0
    x[7, 3] = float("nan")
    x[8] = -x[8].abs()
    print(f"[quant] {dtype} special", flush=True)
    codes, scale = C.quantize_rows(x, "int8", p=C.plan("resident"), h=capped)
    one = C.Handle(0)
    try:
        for i in range(13):
            c1, s1 = C.quantize_rows(x[i:i + 1], "int8", p=C.plan("resident"), h=one)
            assert torch.equal(codes[i], c1[0]), i
            assert torch.equal(scale[i], s1[0]) or bool(torch.isnan(scale[i]) & torch.isnan(s1[0])), i
    finally:
        one.close()
