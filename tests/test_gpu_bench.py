"""The benchmark script end to end: one JSON line with the fields its readers rely on, and the stages that it adds up."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.gpu
def test_bench_prints_one_json_line_with_roofline_and_cpu_baseline():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--steps", "2", "--warmup", "1"],
                       capture_output=True, text=True, timeout=600, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [l for l in r.stdout.splitlines() if l.startswith("{")]
    assert len(lines) == 1
    d = json.loads(lines[0])
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert key in d, key
    assert d["n_gpus"] == 1 and d["steps"] == 2 and d["warmup"] == 1
    assert d["config"]["workload"] == "mistral7b_4k" and d["dtype"] == "bf16" and d["data"] == "synthetic"
    assert d["value"] > 0 and abs(d["value"] - d["config"]["context_tokens"] / (d["ms_per_step"] * 1e-3)) < 1e-6 * d["value"]
    rf = d["roofline"]
    assert rf["bound"] == "mfma" and rf["unit"] == "TFLOP/s" and rf["peak"] == 2500.0
    assert 0.0 < rf["frac"] < 1.0 and abs(rf["frac"] - rf["achieved"] / rf["peak"]) < 1e-9
    assert rf["traffic"] is None or rf["traffic"] > 0
    cb = d["cpu_baseline"]
    assert cb["kind"] == "oracle" and cb["value"] > 0 and cb["cores"] >= 1 and cb["unit"] == d["unit"] and cb["sample"]
    assert d["ceilings"]["mfma_loop_bf16_tflop_s"] > rf["achieved"]
    # the products' time has the sums over their K parts in it, also where a norm does them; no stage is priced that did not run
    stages = d["stages_ms"]
    assert stages["gemm_parts_norm"] > 0
    products = sum(ms for name, ms in stages.items() if name.startswith("gemm"))
    assert abs(products - rf["gemm_ms_per_step"]) < 1e-3
    assert abs(rf["achieved"] - rf["algorithmic_gflop_per_step"] / rf["gemm_ms_per_step"]) < 1e-6 * rf["achieved"]
    assert rf["gemm_launches_per_step"] == 4 * 32 + 2   # four products a layer, fresh values, LM head
    assert all(r["achieved"] > 0 for r in d["stage_rooflines"].values())
    assert "rmsnorm" not in d["stage_rooflines"]        # its launches are not all of the norms


@pytest.mark.gpu
def test_sums_of_parts_have_a_stage_of_their_own():
    import torch
    from types import SimpleNamespace

    from paper_2603_13289_amd import binding as rc
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    sh = SimpleNamespace(n_layers=3, d_model=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ffn=3072, vocab=256, rope_base=1e4,
                         rms_eps=1e-5, dtype="bf16")
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    ones = torch.ones(1024, dtype=torch.bfloat16, device="cuda")
    layers = [dict(wq=rnd(1024, 1024), wk=rnd(256, 1024), wv=rnd(256, 1024), wo=rnd(1024, 1024), w_gate=rnd(3072, 1024),
                   w_up=rnd(3072, 1024), w_down=rnd(1024, 3072), g_attn=ones, g_ffn=ones) for _ in range(3)]
    model = rc.Model(sh, layers, ones, rnd(256, 1024))
    table = torch.zeros((1, 1), dtype=torch.int32, device="cuda")
    k = torch.zeros((3, 1, 2, 70, 128), dtype=torch.bfloat16, device="cuda")
    cache = rc.PagedKV.from_pools(list(k.unbind(0)), list(torch.zeros_like(k).unbind(0)), table, rc.RC_BF16)
    rc.rc_profile_enable(True)
    try:
        rc.rc_prefill(model, [rnd(70, 1024)], [0], cache, torch.zeros((1, 256), dtype=torch.float32, device="cuda"),
                      rc.alloc_workspace(rc.rc_prefill_workspace_bytes(model, [70])))
        stages = rc.rc_profile_read()
    finally:
        rc.rc_profile_enable(False)
    # 70 rows: of the products that add to the residual the down projections are cut along K (the output projections are
    # not), and the norms of the second and third layer add their parts up
    assert stages["gemm_parts_norm"][1] == 2 and stages["rmsnorm"][1] == 4
