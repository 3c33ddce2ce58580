"""bench.py's serving harness on the host, with the GPU passes replaced by timed stand-ins (the
fake server of test_serve_policy): every mode runs on the same traces, the summary pools the
seeds per (mode, rate), picks the better time-sliced order, and sets Eq. 6 beside the wait."""
import json

import numpy as np

import bench
from paper_2509_21301_amd import sched, serve, synth
from tests.test_sched_host import curves
from tests.test_serve_policy import fake_server


class FakeSetup:
    """ServingSetup's serve() over the fake server."""

    def serve(self, kw, trace, keep_log=False):
        kw = dict(kw)
        srv, _ = fake_server(kw.pop("mode"), **{k: kw.pop(k) for k in ("slice_order", "decode_limit") if k in kw})
        srv.decode_cus = kw.get("decode_cus", srv.decode_cus)
        srv.alpha = kw.get("alpha", srv.alpha)
        srv.minimum = kw.get("minimum", srv.minimum)
        res = srv.run(trace)
        if keep_log:
            res["partition_timeline"] = [[round(t * 1e3, 2), st, cus] for t, st, cus in srv.partition_log]
            res["arrivals_ms"] = [r.arrival * 1e3 for r in trace]
        return res


def test_run_serving_summary(monkeypatch):
    small = serve.poisson_trace
    monkeypatch.setattr(serve, "poisson_trace", lambda rate, window, seed: small(rate, window, seed, n_text=(5, 9),
                                                                                   n_out=(6, 12)))
    monkeypatch.setattr(serve.nova, "make_cu_mask", lambda n, first=0: [0xFFFFFFFF] * 8)
    monkeypatch.setattr(serve.nova, "set_stage_partition", lambda stage, mask: None)
    out = bench.run_serving(serve, sched, FakeSetup(), curves(2), 32, [100.0], [1, 2], 0.05, timeline_at=(100.0, 1))
    modes = {r["mode"] for r in out["runs"]}
    assert modes == {"nova_rate_static", "nova_adaptive", "time_sliced_decode_first", "time_sliced_prefill_first",
                     "pf_limit", "multi_stream"}
    assert len(out["runs"]) == 12
    rows = {r["mode"]: r for r in out["summary"]}
    best = rows["time_sliced_best"]
    assert best["chosen"] in ("time_sliced_decode_first", "time_sliced_prefill_first")
    assert best["max_e2e_s"] == min(rows["time_sliced_decode_first"]["max_e2e_s"],
                                    rows["time_sliced_prefill_first"]["max_e2e_s"])
    for m in modes:
        rs = [r for r in out["runs"] if r["mode"] == m]
        assert abs(rows[m]["max_e2e_s"] - np.mean([r["max_e2e_s"] for r in rs])) < 1e-3
        assert rows[m]["seeds"] == 2 and "eq6_predicted_wait_s" in rows[m]
    assert any("partition_timeline" in r for r in out["runs"] if r["mode"] == "nova_adaptive")
    a = out["adaptive_params"]
    assert a["sm_min"] <= min(a["sm_op_v"], a["sm_op_p"])


def test_result_line_is_short():
    """A full run's results as one line that a capture of 14,000 characters holds, the headline intact."""
    head = {"metric": "m", "value": 1.5, "unit": "patches/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 87.5,
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
            "config": {"global_batch": 8}}
    row = {k: 0.123456 for k in ("max_e2e_s", "max_e2e_s_std", "avg_e2e_s", "avg_ttft_s", "avg_tbt_ms", "throughput_req_s",
                                 "avg_queue_wait_s", "eq6_predicted_wait_s", "utilization")}
    big = {"corun": [dict(share=p, decode_ms=3.333, encode_ms=77.77, prefill_ms=55.55) for p in range(32, 256, 8)],
           "serving": [dict(row, mode="time_sliced_prefill_first", rate_req_s=4.0) for _ in range(16)],
           "serving_runs": [dict(row, mode="nova_adaptive", seed=s) for s in range(12)],
           "partition_timeline": {"timeline": [[8909.41, 2, 96]] * 1300}}
    line = bench.result_line({**head, **big})
    assert len(line) < 9000 and "\n" not in line
    got = json.loads(line)
    assert {k: got[k] for k in head} == head
    assert got["corun"] == big["corun"] and got["serving"][0]["max_e2e_s"] == row["max_e2e_s"]


def test_prefill_flops_count_what_the_result_needs():
    """A one-layer prefill: K and V of every row, and one row of everything else."""
    c = synth.LlmConfig(hidden=256, n_q=4, n_kv=2, head_dim=64, inter=688, vocab=4096, layers=1)
    s, d = 96, 64
    lin, attn = bench.prefill_flops(c, s)
    assert lin == 2 * (s * 256 * 2 * 2 * d + 256 * 2 * 4 * d + 3 * 256 * 688 + 256 * 4096)
    assert attn == 2 * 2 * s * 4 * d
    c2 = synth.LlmConfig(hidden=256, n_q=4, n_kv=2, head_dim=64, inter=688, vocab=4096, layers=3)
    lin2, attn2 = bench.prefill_flops(c2, s)
    assert lin2 - lin == 2 * 2 * s * 256 * (2 * 2 * d + 2 * 4 * d + 3 * 688) and attn2 - attn == 2 * 2 * s * s * 4 * d
