"""Which kernel a plan runs on either side of the lines between the streaming and the
one-row kernels, at shapes where the wrong one is 6 to 25 percent slower (host.cpp
has the times)."""
import pytest
import torch

from paper_2609_01864_amd import credit as C

pytestmark = pytest.mark.gpu

SM, LN, RMS, BW = (C.SOFTMAX, C.FWD), (C.LAYERNORM, C.FWD), (C.RMSNORM, C.FWD), (C.SOFTMAX_LOGITS, C.BWD)
# op, dtype, M, N, members, streams?
CASES = [
    # split, aligned or even BF16 rows: 5 to 12 waves do not, 4 (even rows) and 13 do
    (SM, C.BF16, 2493, 66826, 4, False), (SM, C.BF16, 76, 262960, 16, False), (SM, C.BF16, 844, 30320, 2, False),
    (SM, C.BF16, 332, 56774, 2, True), (SM, C.BF16, 3072, 15002, 2, True), (SM, C.BF16, 768, 51304, 2, True),
    # odd rows: only 6, 9 and 10 waves do not
    (SM, C.BF16, 6144, 29895, 2, True), (SM, C.BF16, 3072, 22001, 2, False), (SM, C.BF16, 3072, 37001, 2, False),
    # split FP32: from more than 6 rounds on
    (SM, C.F32, 576, 24642, 2, False), (SM, C.F32, 3072, 26338, 2, True),
    # split backward from the logits
    (BW, C.BF16, 211, 75016, 8, False), (BW, C.BF16, 332, 51800, 2, False), (BW, C.BF16, 3072, 54320, 2, True),
    (BW, C.BF16, 768, 208199, 8, True),
    # row-resident
    (SM, C.BF16, 1100, 10624, 1, True), (SM, C.BF16, 3000, 10496, 1, False), (SM, C.BF16, 4600, 16576, 1, False),
    (SM, C.BF16, 600, 1152, 1, False), (SM, C.BF16, 2048, 1152, 1, True),
    (BW, C.BF16, 1700, 10752, 1, False), (BW, C.BF16, 3000, 11992, 1, True), (BW, C.F32, 600, 4864, 1, False),
    (BW, C.F32, 4600, 4864, 1, True), (BW, C.BF16, 4600, 4816, 1, False),
    (SM, C.FP8, 450, 1441, 1, False), (SM, C.FP8, 1800, 1441, 1, True), (SM, C.FP8, 450, 1452, 1, True),
    (LN, C.BF16, 1250, 1280, 1, False), (LN, C.BF16, 1250, 1300, 1, True), (LN, C.BF16, 1600, 1280, 1, True),
    (RMS, C.BF16, 1250, 1280, 1, False), (RMS, C.F32, 520, 4096, 1, False), (RMS, C.F32, 1100, 4096, 1, True),
]


@pytest.mark.parametrize("op,dt,M,N,k,stream", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_kernel_on_either_side(gpu_handle, op, dt, M, N, k, stream):
    p = C.plan("resident") if k == 1 else C.plan("split", k)
    assert ("stream" in gpu_handle.kernel(*op, dt, M, N, p)) == stream


def test_fp8_softmax_fills_the_simds(gpu_handle):
    # workgroups of 4 waves: as many as fit, not as few as end in the same rounds
    s = (C.SOFTMAX, C.FWD, C.FP8, 2500, 12770)
    geo = gpu_handle.geometry(*s, C.plan("resident"))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert geo["block"] == 256 and geo["grid"] == geo["per_cu"] * cus


def test_two_pass_softmax_grid_is_what_the_device_holds(gpu_handle):
    # an eighth workgroup per CU would run after the others: 45 us, not 37
    geo = gpu_handle.geometry(C.SOFTMAX, C.FWD, C.BF16, 8979, 940, C.plan("two_pass"))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert geo["grid"] <= 7 * cus
