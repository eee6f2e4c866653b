"""The plan of calls without one: the timed learned selector never leaves such calls
slower than it found them."""
import pytest

from paper_2609_01864_amd import credit as C

pytestmark = pytest.mark.gpu


def test_timed_selector_times_the_plan_of_a_call_without_one(lib_built):
    # FP8 LayerNorm of wide rows: the network's two best plans take 1.6 and 2
    # times as long as the plan that a call without one runs
    h = C.Handle(0)
    try:
        s = (C.LAYERNORM, C.FWD, C.FP8, 1024, 262144)
        f = h.mlp_predict(C.features(*s)[None, :])[0]
        legal = [c for c in range(C.NUM_PLANS) if h.plan_legal(*s, C.plan_of_class(c))]
        two = [C.plan_of_class(c).as_tuple() for c in sorted(legal, key=lambda c: -f[c])[:2]]
        h.set_selector(C.SEL_LEARNED_TIMED)
        p, pred = h.select(*s)
        print(f"[default plan] {two} {p} {pred}", flush=True)
        best = min(h.time_plan(*s, C.plan("split", k), 7) for k in (16, 32))
        assert pred <= 1.2 * best and p.as_tuple() not in two
    finally:
        h.close()
