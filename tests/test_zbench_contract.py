"""The benchmark's output contract, on a short run: one JSON line with the fields the driver
reads, a roofline object against the HBM peak, and a refusal of more than one GPU."""
import json
import os
import subprocess
import sys

import pytest

from card_inputs import SHAPES, ModelShape

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(*flags):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *flags], cwd=ROOT, capture_output=True,
                          text=True, timeout=600)


def test_more_than_one_gpu_is_refused_with_a_message():
    p = _run("--gpus", "2")
    assert p.returncode != 0
    assert "ONE GPU" in p.stderr and p.stdout.strip() == ""


@pytest.mark.gpu
def test_short_run_prints_one_json_line_with_the_contract_fields(monkeypatch, capsys):
    import runpy

    monkeypatch.setattr(sys, "argv", ["bench.py", "--steps", "6", "--warmup", "2", "--no-cpu-baseline", "--sweep", "quick"])
    monkeypatch.chdir(ROOT)
    runpy.run_path(os.path.join(ROOT, "bench.py"), run_name="__main__")
    lines = [ln for ln in capsys.readouterr().out.splitlines() if ln.strip()]
    assert len(lines) == 1
    d = json.loads(lines[0])
    assert d["metric"] == "verified_tokens_per_s" and d["unit"] == "tokens/s"
    assert d["n_gpus"] == 1 and d["steps"] == 6 and d["warmup"] == 2
    assert d["higher_is_better"] is True and d["vs_baseline"] is None and d["data"] == "synthetic"
    assert "workload" in d["config"] and "model" not in d["config"]
    assert abs(d["value"] - 8 / (d["ms_per_step"] * 1e-3)) <= 1e-6 * d["value"]  # r = 8 rows per step
    rf = d["roofline"]
    assert rf["bound"] == "hbm" and rf["unit"] == "GB/s" and rf["peak"] == 8000.0
    assert abs(rf["frac"] - rf["achieved"] / rf["peak"]) < 1e-9
    assert 0.2 < rf["frac"] < 1.0
    assert abs(rf["achieved"] - d["algorithmic_bytes_per_step"] / (rf["avg_launch_us"] * 1e-6) / 1e9) <= 1e-6 * rf["achieved"]
    # bytes of the weights as the kernel reads them (12 of 16 bits from the coded copy), and what the counters read for such a step
    whole = SHAPES["llama8b"].streamed_weight_bytes()
    coded = d["config"]["weights"].startswith("coded")
    assert d["algorithmic_bytes_per_step"] == rf["bytes_per_launch"] == whole * (3 if coded else 4) // 4 + SHAPES["llama8b"].kv_bytes(1024)
    assert d["bf16_equivalent"]["bytes"] == whole + SHAPES["llama8b"].kv_bytes(1024)
    assert (rf["traffic"] is None) == (rf["traffic_source"] is None)
    if coded:
        assert 0.9 * rf["bytes_per_launch"] <= rf["traffic"] <= 1.2 * rf["bytes_per_launch"]
    # the other synthetic configurations ride in the same line
    sw = d["sweep"]
    assert not [e for e in sw if "section" in e], [e for e in sw if "section" in e]  # no section failed
    pts = [e for e in sw if e.get("kind") not in ("cache_loop", "concurrent_loop", "draft_level")]
    assert pts and all(e["ms_per_step"] > 0 and 0.1 < e["hbm_frac"] < 1.0 and e["verified_tokens_per_s"] > 0 for e in pts)
    for e in pts:
        frac = e["algorithmic_bytes"] / (e["kernel_ms"] * 1e-3) / 8e12
        assert abs(e["hbm_frac"] - frac) <= 1e-9 * frac
        in_whole = e["bf16_equivalent"]["bytes"] - SHAPES[e["shape"]].kv_bytes(e["ctx"])
        assert e["algorithmic_bytes"] == e["bf16_equivalent"]["bytes"] - (in_whole // 4 if e["weights"].startswith("coded") else 0)
    conc = [e for e in sw if e.get("kind") == "concurrent_loop"]
    assert conc and all("error" in e or (e["text_equals_plain_decode"] and e["accepted_tokens_per_s"] > 0) for e in conc)
    pts = [e for e in pts if e.get("kind") != "concurrent_loop"]
    dl = [e for e in sw if e.get("kind") == "draft_level"]
    assert len(dl) == 2 and all(e["ms_per_level"] > 0 and e["K"] == 40 for e in dl)
    # the weights are streamed once per call of 32 rows, and once by the pass; the fractions of the peaks are of what was moved and issued
    assert [(e["route"], e["lanes"], e["weight_streams_per_level"]) for e in dl] == [("calls", 1, 2), ("one pass", 2, 1)]
    assert dl[1]["weights"].startswith("whole")  # the pass reads these, calls the coded copy where there is one
    draft = ModelShape("tiny-draft", 1, 128, 2, 1, 64, 344, 1024)  # what a quick run forwards
    for e in dl:
        kv = draft.kv_bytes(e["ctx"])
        assert e["bytes_per_stream"] == draft.streamed_weight_bytes() * (3 if e["weights"].startswith("coded") else 4) // 4 + kv
        frac = e["weight_streams_per_level"] * e["bytes_per_stream"] / (e["ms_per_level"] * 1e-3) / 8e12
        assert abs(e["hbm_frac"] - frac) <= 1e-9 * frac
    issued = [e["mfma_tflops_issued"] / e["model_tflops"] * e["K"] / 2 for e in dl]  # rows
    assert [round(i, 6) for i in issued] == [32 + 8, 16 + 16 + 16]  # calls of 32 and 8 rows; tiles of calls of 24 and 16 rows
    kinds = ("whole, 16 bits each", "coded, 12 bits each")
    assert all(e[key] in kinds for e in sw for key in (("target_weights", "draft_weights") if e.get("kind") == "concurrent_loop" else ("weights",)))
    loops = [e for e in sw if e.get("kind") == "cache_loop"]
    assert loops and all("error" in e or (e["accepted_tokens_per_s"] > 0 and 1.0 <= e["mean_accepted_len"] <= e["r"])
                         for e in loops)


@pytest.mark.gpu
def test_timeline_probe_reports_the_ten_phases_of_a_layer(monkeypatch, capsys):
    """bench.py --timeline: the kernel's own time stamps of one decoder layer, on the smallest shape."""
    import runpy

    monkeypatch.setattr(sys, "argv", ["bench.py", "--shape", "tiny", "--timeline", "1", "--sweep", "none", "--no-cpu-baseline"])
    monkeypatch.chdir(ROOT)
    runpy.run_path(os.path.join(ROOT, "bench.py"), run_name="__main__")
    lines = [ln for ln in capsys.readouterr().out.splitlines() if ln.strip()]
    assert len(lines) == 1
    t = json.loads(lines[0])["timeline"]
    assert t["workgroups"] == 256 and len(t["phases"]) == 10
    assert all(v >= 0 for v in t["phases"].values())  # the stamps of a workgroup are in order
    assert 0 < t["layer_total"] < 1000 and abs(sum(t["phases"].values()) - t["layer_total"]) < 0.2 * t["layer_total"] + 1
    assert t["attention_detail"]["workgroups_with_a_task"] >= 1
    # medians of the workgroups that have a tile (16 of them in the O-projection)
    assert all(0 <= v < 1000 for tag in ("qkv", "o_proj", "down") for v in t[f"{tag}_detail"].values())
