"""The elementwise codecs over widths and alignments at the edges of their
grouped form: rows of fewer than four elements, groups of four that cross one
row boundary, rows just below and above one workgroup's 4096 elements, totals
with 0-3 elements left over, and unaligned tensors.  Every code and value is
decided by one correctly rounded FP32 operation and one conversion on both
sides, so equality is exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_01864_amd import credit as C

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (5, 1), (7, 3), (3, 4), (6, 5), (1000, 7), (65, 63), (3, 4093), (3, 4095), (5, 4096), (3, 4097),
          (2, 8191), (1, 40001), (9, 12290)]


@pytest.mark.parametrize("dt", [C.F32, C.BF16, C.FP8], ids=["f32", "bf16", "fp8"])
@pytest.mark.parametrize("skip", [0, 1], ids=["aligned", "unaligned"])
def test_codec_shapes(gpu_handle, dt, skip):
    fmt = {C.F32: "f32", C.BF16: "bf16", C.FP8: "fp8"}[dt]
    rng = np.random.default_rng(11)
    for M, N in SHAPES:
        print(f"[codec shapes] {fmt} {M} x {N} skip={skip}", flush=True)
        x = (rng.standard_normal((M, N)) * 20).astype(np.float32)
        s = rng.uniform(0.01, 3.0, M).astype(np.float32)
        buf = torch.empty(M * N + skip, device="cuda")
        t = buf[skip:].view(M, N)
        t.copy_(torch.from_numpy(x))
        for sc in (None, s):
            v = x if sc is None else (x / sc[:, None]).astype(np.float32)
            got = C.encode(t, dt, None if sc is None else torch.from_numpy(sc).cuda(), h=gpu_handle)
            raw = got.cpu() if dt != C.BF16 else got.view(torch.int16).cpu()
            ref = v if dt == C.F32 else oracle.encode_from_f32(v.reshape(-1), fmt).reshape(M, N)
            host = raw.numpy().view(np.uint16) if dt == C.BF16 else raw.numpy()
            if dt == C.FP8:  # +0 and -0 are one value
                assert np.array_equal(oracle.decode_e4m3(host.reshape(-1)), oracle.decode_e4m3(ref.reshape(-1)))
            else:
                assert np.array_equal(host, ref)
            cb = torch.empty(M * N + skip, dtype=got.dtype, device="cuda")
            c = cb[skip:].view(M, N)
            c.copy_(got)
            back = C.decode(c, None if sc is None else torch.from_numpy(sc).cuda(), h=gpu_handle).cpu().numpy()
            if dt == C.F32:
                val = v
            elif dt == C.BF16:
                val = (host.astype(np.uint32) << 16).view(np.float32)
            else:
                val = oracle.decode_e4m3(host.reshape(-1)).reshape(M, N).astype(np.float32)
            ref_back = val if sc is None else (val * sc[:, None]).astype(np.float32)
            assert np.array_equal(back, ref_back)
