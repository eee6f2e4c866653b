"""dgamma / dbeta of the normalisation backward over the shapes at which the
column reduction's tiles end: widths around its 32- and 64-column tiles and
the width where one replaces the other, and row counts that leave one partial
row, fewer than the slices, and several batches of eight per slice.  The
oracle's rule: per column 1e-5 of the summed magnitudes plus 1e-6."""
import pytest

from paper_2609_01864_amd import credit as C

from _cases import Case, check_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op", ["layernorm_bwd", "rmsnorm_bwd"])
@pytest.mark.parametrize("M,N", [(1, 31), (2, 32), (9, 33), (700, 63), (1300, 65), (300, 1000), (3, 32767),
                                 (5, 32768), (40, 65537)])
def test_column_sums(gpu_handle, op, M, N):
    case = Case(op, "f32", M, N, seed=M + N)
    ref = case.reference()
    for v in ("two_pass", "resident", "split"):
        p = C.plan(v, 16 if v == "split" else 1)
        if not gpu_handle.plan_legal(C.LAYERNORM if op[0] == "l" else C.RMSNORM, C.BWD, C.F32, M, N, p):
            continue
        print(f"[column sums] {op} {M} x {N} {p}", flush=True)
        check_case(case, case.run(gpu_handle, p, ref=ref), ref)
