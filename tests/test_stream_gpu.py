"""The streaming form of the row-resident / split-row kernels at the sizes where
its slices end: one vector, whole waves, one vector more, each change of
vectors per lane and rows per round, partial vectors at the end of the row,
members of a split row with a short slice or none, and a last round with
fewer rows than the others -- against the oracle.  A cap on the row groups
makes a few rows enough for several rounds; the geometry shows which form a
plan runs in."""
import numpy as np
import pytest

from paper_2609_01864_amd import build as B
from paper_2609_01864_amd import credit as C

from _cases import Case, OPNUM, check_case

EPV = {"f32": 4, "bf16": 8}
DTN = {"f32": C.F32, "bf16": C.BF16}
# vectors of a slice at which a form begins or ends, by split factor
VECS = {1: (1, 2, 63, 64, 65, 129, 256, 257, 512, 1024, 1025, 2048), 2: (1, 64, 128, 129, 256, 257, 512, 513, 1024),
        8: (1, 130, 300, 1000), 32: (1, 33, 64)}
OPS = ["layernorm_bwd", "rmsnorm_bwd"]


def test_no_stream_instance_uses_private_memory(lib_built):
    # their split plans take the occupancy query at its word (no probe)
    import json

    with open(B.RESOURCES) as f:
        rep = {k: v for k, v in json.load(f).items() if "k_stream" in k}
    assert len(rep) >= 8 and all(r["scratch_bytes"] == 0 for r in rep.values())


@pytest.fixture(scope="module")
def capped(lib_built):
    h = C.Handle(0)
    h.set_option(C.OPT_MAX_GROUPS, 2)
    yield h
    h.close()


def _streams(h, op, dtype, M, N, p):
    """Whether the plan's launch differs from the one-row kernels' geometry."""
    o, d = OPNUM[op]
    g = h.geometry(o, d, DTN[dtype], M, N, p)
    one = C.plan_geometry(None, o, d, DTN[dtype], M, N, p)
    return g, g is not None and any(g[f] != one[f] for f in ("block", "vpt", "rows"))


@pytest.mark.gpu
@pytest.mark.parametrize("k", sorted(VECS))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("op", OPS)
def test_slice_edges(capped, op, dtype, k):
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    seen = 0
    for n, vec in enumerate(VECS[k]):
        full = vec * k * EPV[dtype]
        # the whole slice; a partial last vector; a short or empty last member
        for N in {full, full - 1, full - (EPV[dtype] - 1), full - max(1, k - 1) * EPV[dtype] - 2}:
            if N < EPV[dtype]:
                continue
            M = (7, 9, 4)[n % 3]
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


@pytest.mark.gpu
@pytest.mark.parametrize("op", OPS)
def test_strides_alignment_skew_and_determinism(capped, op):
    for dtype in ("f32", "bf16"):
        for k, N in ((1, 1003), (1, 4096), (4, 4096 * 2 + 6), (8, 20000)):
            p = C.plan("split", k) if k > 1 else C.plan("resident")
            case = Case(op, dtype, 7, N, seed=k)
            ref = case.reference()
            print(f"[stream] {op} {dtype} {N} {p}", flush=True)
            plain = case.run(capped, p, ref=ref)
            again = case.run(capped, p, ref=ref)
            for key in plain:
                if isinstance(plain[key], np.ndarray):
                    assert np.array_equal(plain[key], again[key]), key
            for pad, off in ((3, 0), (8, 5)):
                check_case(case, case.run(capped, p, ld_pad=pad, offset=off, ref=ref), ref)
            if k > 1:
                capped.set_option(C.OPT_TEST_SKEW, 1)
                try:
                    skewed = case.run(capped, p, ref=ref)
                finally:
                    capped.set_option(C.OPT_TEST_SKEW, 0)
                for key in plain:
                    if isinstance(plain[key], np.ndarray):
                        assert np.array_equal(plain[key], skewed[key]), key


@pytest.mark.gpu
def test_missing_member_times_out(capped):
    import torch

    x, dy = (torch.randn(9, 8192, device="cuda") for _ in range(2))
    g = torch.rand(8192, device="cuda") + 0.5
    mean, rstd = x.mean(1), torch.rsqrt(x.var(1, correction=0) + 1e-5)
    p = C.plan("split", 4)
    assert _streams(capped, "layernorm_bwd", "f32", 9, 8192, p)[1]
    capped.set_option(C.OPT_SPIN_LIMIT, 64)
    capped.set_option(C.OPT_TEST_DROP_PUBLISH, 1)
    try:
        print("[stream] forced timeout", flush=True)
        C.layernorm_bwd(x, dy, g, mean, rstd, p=p, h=capped)
        assert capped.check_errors() == C.ERR_TIMEOUT
    finally:
        capped.set_option(C.OPT_TEST_DROP_PUBLISH, 0)
        capped.set_option(C.OPT_SPIN_LIMIT, 1 << 22)
    out = C.layernorm_bwd(x, dy, g, mean, rstd, p=p, h=capped)
    assert capped.check_errors() == C.OK
    xd, gd = x.double().requires_grad_(True), g.double()
    (ref,) = torch.autograd.grad(torch.nn.functional.layer_norm(xd, (8192,), gd, None, 1e-5), (xd,), dy.double())
    assert torch.max(torch.abs(out[0].double() - ref)).item() <= 1e-5 * max(1.0, ref.abs().max().item())
