"""The streaming form of the forward operators and of the softmax backward from
the logits at the sizes where its slices and vectors end, as
test_stream_gpu.py does for the normalisation backward -- and for softmax,
whose long rows begin on their first 128-byte line, over every phase of a row
in its line, over tensors that do and do not agree on it, in place, and with
masked, infinite and NaN elements."""
import numpy as np
import pytest
import torch

from paper_2609_01864_amd import credit as C

from _cases import Case, OPNUM, check_case
from test_stream_gpu import DTN, EPV, _streams, capped  # noqa: F401  (fixture)

VECS = {1: (1, 2, 64, 65, 127, 256, 257, 513, 1025, 2049, 4087, 4096), 2: (1, 64, 129, 256, 513, 640, 1024, 1030),
        8: (1, 130, 300, 700), 32: (1, 33, 64)}
OPS = ["layernorm_fwd", "rmsnorm_fwd", "softmax_fwd"]
ULP = {"f32": 2.0 ** -23, "bf16": 2.0 ** -8}


@pytest.mark.gpu
@pytest.mark.parametrize("k", sorted(VECS))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("op", OPS)
def test_slice_edges(capped, op, dtype, k):
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    seen = 0
    for n, vec in enumerate(VECS[k]):
        full = vec * k * EPV[dtype]
        for N in {full, full - 1, full - (EPV[dtype] - 1), full - max(1, k - 1) * EPV[dtype] - 2}:
            if N < EPV[dtype]:
                continue
            M = (17, 19, 22)[n % 3]  # over two rounds of two groups of up to four rows
            if not capped.plan_legal(*OPNUM[op], DTN[dtype], M, N, p):
                continue
            g, st = _streams(capped, op, dtype, M, N, p)
            seen += st
            print(f"[stream] {op} {dtype} {M} x {N} {p} {g} stream={st}", flush=True)
            case = Case(op, dtype, M, N, seed=n + N)
            ref = case.reference()
            check_case(case, case.run(capped, p, ref=ref), ref)
    assert seen >= 4
    assert capped.check_errors() == C.OK


def _logits_ref(x, dy):
    y = torch.softmax(x.double(), 1)
    g = dy.double()
    return y * (g - (g * y).sum(1, keepdim=True)), y, g


def _bound(dtype, y, g):
    """One rounding of the result, and 64 of the FP32 terms it cancels from."""
    terms = y * (g.abs() + (g * y).abs().sum(1, keepdim=True))
    return terms * (64 * 2.0 ** -24 + (ULP["bf16"] if dtype == "bf16" else 0)) + 1e-30


@pytest.mark.gpu
@pytest.mark.parametrize("k", sorted(VECS))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_logits_backward_slice_edges(capped, dtype, k):
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    for n, vec in enumerate(VECS[k]):
        for N in {vec * k * EPV[dtype], vec * k * EPV[dtype] - 1, vec * k * EPV[dtype] - 2 * k - 1}:
            if N < EPV[dtype] or not capped.plan_legal(C.SOFTMAX_LOGITS, C.BWD, DTN[dtype], 17, N, p):
                continue
            print(f"[stream] logits {dtype} {N} {p}", flush=True)
            gen = torch.Generator(device="cuda").manual_seed(n)
            x = (3 * torch.randn((17, N), device="cuda", generator=gen)).to(td)
            dy = torch.randn((17, N), device="cuda", generator=gen).to(td)
            dx = C.softmax_logits_bwd(x, dy, p=p, h=capped)[0].double()
            ref, y, g = _logits_ref(x, dy)
            assert bool(((dx - ref).abs() <= _bound(dtype, y, g)).all())
    assert capped.check_errors() == C.OK


@pytest.mark.gpu
@pytest.mark.parametrize("k", [1, 4])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_phase_of_rows(capped, dtype, k):
    # row lengths of every residue modulo a line, tensors that begin at
    # different elements, results in place
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    line = 128 // (4 if dtype == "f32" else 2)
    M, base = 17, 640 * EPV[dtype] * k
    for extra in range(line):
        N = base + extra
        ld = N + (0, 0, 3)[extra % 3]
        flat = torch.randn(M * ld + line, device="cuda").to(td)
        x = flat[extra % 5:extra % 5 + M * ld].view(M, ld)[:, :N]
        keep = flat.clone()
        want = torch.softmax(x.double(), 1)
        y, _ = C.softmax_fwd(x, p=p, h=capped)
        print(f"[phase] {dtype} {N} ld {ld} {p}", flush=True)
        tol = 2e-6 if dtype == "f32" else ULP["bf16"] * want + 1e-30
        assert bool(((y.double() - want).abs() <= tol).all())
        assert torch.equal(flat, keep)
        # the same layout for the result: rows agree on their phase
        y = torch.empty_like(flat)[extra % 5:extra % 5 + M * ld].view(M, ld)[:, :N]
        C.softmax_fwd(x, out=y, p=p, h=capped)
        assert bool(((y.double() - want).abs() <= tol).all())
        C.softmax_fwd(x, out=x, p=p, h=capped)
        assert torch.equal(x, y)
        x.copy_(keep[extra % 5:extra % 5 + M * ld].view(M, ld)[:, :N])
        assert torch.equal(flat, keep)  # nothing outside the rows was written
    assert capped.check_errors() == C.OK


@pytest.mark.gpu
@pytest.mark.parametrize("k", [1, 4])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_masked_and_special_rows(capped, dtype, k):
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    for N in (1000 * k, 5001 * k, 40000):
        if not capped.plan_legal(C.SOFTMAX, C.FWD, DTN[dtype], 17, N, p):
            continue
        print(f"[special] {dtype} {N} {p}", flush=True)
        x = torch.randn((17, N), device="cuda")
        x[0, N // 3:] = -float("inf")
        x[1, N // 3:] = torch.finfo(td).min
        x[2, :-1] = torch.finfo(td).min
        x[3, 5] = 300.0
        x[4, : N // 2] = -200.0  # outputs far below the row's largest
        x[5] = 90.0 + 0 * x[5]
        x = x.to(td)
        dy = torch.randn((17, N), device="cuda").to(td)
        y, _ = C.softmax_fwd(x, p=p, h=capped)
        want = torch.softmax(x.double(), 1)
        tol = 2e-6 if dtype == "f32" else ULP["bf16"] * want + 2.0 ** -132
        assert bool(((y.double() - want).abs() <= tol).all())
        if capped.plan_legal(C.SOFTMAX_LOGITS, C.BWD, DTN[dtype], 17, N, p):
            dx = C.softmax_logits_bwd(x, dy, p=p, h=capped)[0].double()
            ref, yy, g = _logits_ref(x, dy)
            assert bool(((dx - ref).abs() <= _bound(dtype, yy, g) + 2.0 ** -132).all())
        bad = x.clone()
        bad[7, 11] = float("nan")
        bad[8, N - 1] = float("inf")
        bad[9] = -float("inf")
        z, _ = C.softmax_fwd(bad, p=p, h=capped)
        assert bool(torch.isnan(z[7:10].float()).all())
        assert torch.equal(z[:7], y[:7]) and torch.equal(z[10:], y[10:])
    assert capped.check_errors() == C.OK
