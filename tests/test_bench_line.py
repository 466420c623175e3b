"""The benchmark's printed line stays one short JSON line whatever the legs measured (a record that keeps only the end of the
output must hold it whole), with the values of the full result."""
import json

import bench

LEG = {f"leg_{i}": [0.123456789] * 50 for i in range(40)}
ROOF = dict(frac=0.9123456789, roofline_tokens_per_s=80.0, link_engine="compute_units", link_GBps_measured=56.6, t_roof_s=1.0,
            faults_per_token=68.0, fault_rate=0.2, side=LEG)
FULL = dict(metric="m", value=74.123456789, unit="tokens/s", n_gpus=1, steps=20, warmup=5, ms_per_step=13.5, higher_is_better=True,
            scaling="weak", vs_baseline=None, dtype="bf16", data="synthetic",
            config=dict(workload="x" * 150, layers=48, d_model=2048, d_ff=768, experts=128, top_k=8, batch=1,
                        expert_budget_bytes=14495514624, cap_per_layer=32, expert_blob_bytes=9437184),
            roofline=dict(bound="hbm", achieved=4000.0, peak=8000.0, unit="GB/s", frac=0.5, traffic=None, traffic_detail=LEG),
            path_roofline=ROOF, cpu_baseline=dict(value=1.04, unit="tokens/s", cores=16, kind="oracle", sample="16 layer-steps"),
            pager="device", kernel_timing="gateup",
            passes={n: dict(tokens_per_s=74.0, ms_per_step=13.5, path_roofline=ROOF, kernel_census=LEG) for n in ("host", "device")},
            prefill=dict(tokens_per_s=1900.0, pass_ms=1050.0, cap_per_layer=32, faults=6144, roofline=ROOF, mfma=LEG, hbm=LEG,
                         resident=dict(tokens_per_s=1e5, pass_ms=18.4, kernels=LEG)),
            sweep=[dict(cap=c, paged_tokens_per_s=40.0, speedup_vs_zero_copy=3.0, speedup_vs_bulk=40.0, resident=LEG)
                   for c in (8, 16, 32, 64, 128)],
            controller=LEG, configurator=LEG, prefetch=[LEG] * 3,
            pageable_legs={n: dict(tokens_per_s=38.0, path_roofline=ROOF, gateup_kernel=LEG) for n in ("a", "b")})


def test_line_is_short_and_holds_the_contract():
    line = json.dumps(bench.summary(FULL))
    assert len(line) < 2000 and "\n" not in line
    got = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data", "config"):
        assert got[k] == FULL[k]
    assert got["path_roofline"]["frac"] == 0.912346 and got["sweep"][2] == [32, 40.0, 3.0]


def test_line_without_the_side_legs():
    bare = dict(FULL, roofline=None, cpu_baseline=None, prefill=None, sweep=None, pageable_legs=None)
    got = bench.summary(bare)
    assert got["roofline"] is None and "prefill" not in got and got["value"] == FULL["value"]
