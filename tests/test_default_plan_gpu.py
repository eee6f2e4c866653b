"""The plan of calls without one: the timed learned selector never leaves such calls
slower than it found them, and it does not depend on calls made under other
options."""
import json

import pytest
import torch

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


def test_default_plan_follows_the_rows_option(lib_built, monkeypatch, tmp_path):
    # with the rows per workgroup set no norm forward streams, so what a call
    # picked before is not what it would pick now
    path = tmp_path / "calls.jsonl"
    monkeypatch.setenv("CREDIT_LOG", str(path))
    M, N = 4096, 20000
    q = (torch.randn((M, N), device="cuda") * 50).to(torch.float8_e4m3fn)
    s = torch.rand(M, device="cuda") * 1e-2 + 1e-3
    g, b = torch.rand(N, device="cuda"), torch.rand(N, device="cuda")
    used, fresh = C.Handle(0), C.Handle(0)
    try:
        print("[default plan] rows option", flush=True)
        C.layernorm_fwd(q, g, b, x_scale=s, h=used)
        used.set_option(C.OPT_ROWS, 1)
        fresh.set_option(C.OPT_ROWS, 1)
        C.layernorm_fwd(q, g, b, x_scale=s, h=used)
        C.layernorm_fwd(q, g, b, x_scale=s, h=fresh)
        used.set_option(C.OPT_ROWS, 0)
        C.layernorm_fwd(q, g, b, x_scale=s, h=used)
        torch.cuda.synchronize()
    finally:
        used.close()
        fresh.close()
    plans = [json.loads(line)["plan"] for line in path.read_text().splitlines()]
    assert plans[0] != plans[1] and plans[1] == plans[2] and plans[3] == plans[0]


def test_default_plan_of_few_short_rows_is_the_networks(lib_built, monkeypatch, tmp_path):
    # too few rows to stream row-resident: not a reason to split short rows
    # (LayerNorm backward 823 x 512 BF16: 12.7 us resident, 25.5 at k = 16)
    path = tmp_path / "calls.jsonl"
    monkeypatch.setenv("CREDIT_LOG", str(path))
    x, dy = (torch.randn((823, 512), device="cuda").bfloat16() for _ in range(2))
    g = torch.rand(512, device="cuda")
    h = C.Handle(0)
    try:
        print("[default plan] few short rows", flush=True)
        C.layernorm_bwd(x, dy, g, None, None, h=h)
        torch.cuda.synchronize()
        f = h.mlp_predict(C.features(C.LAYERNORM, C.BWD, C.BF16, 823, 512)[None, :])[0]
    finally:
        h.close()
    used = json.loads(path.read_text().splitlines()[-1])["plan"]
    assert used == [1, 1] and f.argmax() == 1
