"""The kernel that a plan runs, which its geometry alone does not tell: a streaming
form of four waves has the one-row kernel's block, vectors and rows."""
import pytest

from paper_2609_01864_amd import credit as C


def test_without_a_handle(lib_built):
    s = (C.LAYERNORM, C.FWD, C.BF16, 4096, 5120)
    assert C.plan_kernel(None, *s, C.plan("two_pass")) == "k_twopass"
    assert C.plan_kernel(None, *s, C.plan("split", 2)) == "k_resident"
    assert C.plan_kernel(None, C.LAYERNORM, C.FWD, C.FP8, 4096, 1 << 22, C.plan("resident")) is None


@pytest.mark.gpu
@pytest.mark.parametrize("op,d,dt,M,N,k,name", [
    (C.SOFTMAX, C.FWD, C.FP8, 4096, 65536, 4, "k_stream_softmax"), (C.SOFTMAX, C.FWD, C.FP8, 16, 65536, 4, "k_resident"),
    (C.LAYERNORM, C.FWD, C.FP8, 4096, 65536, 8, "k_stream_ln_fp8"), (C.LAYERNORM, C.FWD, C.F32, 1024, 524288, 16, "k_resident"),
    (C.RMSNORM, C.FWD, C.BF16, 8192, 4096, 1, "k_stream"), (C.LAYERNORM, C.BWD, C.BF16, 2048, 131072, 16, "k_stream"),
    (C.SOFTMAX_LOGITS, C.BWD, C.F32, 4096, 3000, 1, "k_stream_softmax"), (C.SOFTMAX, C.BWD, C.F32, 4096, 3000, 1, "k_resident"),
    (C.QUANT_INT8, C.FWD, C.BF16, 4096, 11008, 1, "k_stream_quant"), (C.QUANT_FP8, C.FWD, C.BF16, 4096, 11008, 1, "k_resident"),
    (C.RMSNORM, C.FWD, C.F32, 1024, 131072, 16, "k_multirow")])
def test_of_a_handle(gpu_handle, op, d, dt, M, N, k, name):
    p = C.plan("split", k) if k > 1 else C.plan("resident")
    assert gpu_handle.kernel(op, d, dt, M, N, p) == name
    if name == "k_stream_softmax" and dt == C.FP8:  # the case that the geometry does not show
        g, one = gpu_handle.geometry(op, d, dt, M, N, p), C.plan_geometry(None, op, d, dt, M, N, p)
        assert (g["block"], g["vpt"], g["rows"]) == (one["block"], one["vpt"], one["rows"])
