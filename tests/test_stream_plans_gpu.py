"""Which plans stream, where the rule draws its lines for long split slices of
the norm forward, against the oracle on both sides of each line; and the plan
of a call without one, which is the first that streams: its outputs are those
of the same call with that plan named, bit for bit."""
import pytest
import torch

from paper_2609_01864_amd import credit as C

from _cases import Case, check_case
from test_stream_gpu import EPV, _streams, capped  # noqa: F401  (fixture)

# vectors per slice: the last that keeps the one-row kernel, the first that streams
LINES = {("layernorm_fwd", "f32", 4): ((1280, 1281), (3072, 3073)), ("rmsnorm_fwd", "f32", 4): ((1536, 1537), (2816, 2817)),
         ("layernorm_fwd", "f32", 8): ((1280, 1281),), ("rmsnorm_fwd", "f32", 8): ((1792, 1793),),
         ("layernorm_fwd", "bf16", 2): ((3072, 3073),), ("rmsnorm_fwd", "bf16", 2): ((3072, 3073),)}


@pytest.mark.gpu
@pytest.mark.parametrize("op,dtype,k", sorted(LINES))
def test_lines_of_long_split_slices(capped, op, dtype, k):
    p = C.plan("split", k)
    for line in LINES[op, dtype, k]:
        forms = []
        for vec in line:
            M, N = 13, vec * k * EPV[dtype] - EPV[dtype] - 1  # not whole: a short last member
            g, st = _streams(capped, op, dtype, M, N, p)
            print(f"[plans] {op} {dtype} {M} x {N} {p} {g} stream={st}", flush=True)
            # a streaming form of 4 waves and the one-row kernel's 8 vectors differ
            # in the workgroups per CU alone
            forms.append((g["block"], g["vpt"], g["rows"], g["per_cu"]))
            assert not st or vec == line[1]
            case = Case(op, dtype, M, N, seed=vec)
            ref = case.reference()
            check_case(case, case.run(capped, p, ref=ref), ref)
        assert forms[0] != forms[1]
    assert capped.check_errors() == C.OK


@pytest.mark.gpu
@pytest.mark.parametrize("op,dtype,M,N,k", [("layernorm_bwd", "f32", 1500, 20000, 8), ("layernorm_fwd", "bf16", 1024, 65536, 4),
                                            ("rmsnorm_fwd", "bf16", 1024, 65536, 4)])
def test_call_without_a_plan(lib_built, op, dtype, M, N, k):
    h = C.Handle(0)
    try:
        T = torch.float32 if dtype == "f32" else torch.bfloat16
        gen = torch.Generator(device="cuda").manual_seed(N)
        x = torch.randn((M, N), device="cuda", generator=gen).to(T)
        dy = torch.randn((M, N), device="cuda", generator=gen).to(T)
        g, b = torch.rand(N, device="cuda"), torch.rand(N, device="cuda")
        mean, rstd = torch.zeros(M, device="cuda"), torch.ones(M, device="cuda")
        f = {"layernorm_bwd": lambda p: C.layernorm_bwd(x, dy, g, mean, rstd, p=p, h=h),
             "layernorm_fwd": lambda p: C.layernorm_fwd(x, g, b, p=p, h=h),
             "rmsnorm_fwd": lambda p: C.rmsnorm_fwd(x, g, p=p, h=h)}[op]
        got, want = f(None), f(C.plan("split", k))
        same = [torch.equal(a, w) for a, w in zip(got, want) if a is not None]
        assert same and all(same)
        assert h.check_errors() == C.OK
    finally:
        h.close()
