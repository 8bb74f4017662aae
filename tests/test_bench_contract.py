"""bench.py's host-side contract (no GPU): more than one GPU is refused with a
message, and the committed window-pass traffic summary is read only while
the kernel sources match the profiled ones, and the printed line is short
enough for the last 2000 characters of a captured output."""
import json
import os
import subprocess
import sys

from conftest import ROOT


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr and r.stdout == ""


def test_traffic_summary_follows_the_sources(monkeypatch, tmp_path):
    sys.path.insert(0, ROOT)
    import bench
    h = bench.window_source_hash()
    assert len(h) == 16
    f = tmp_path / "traffic.md"
    f.write_text(f"traffic_bytes_per_launch: 123456\nsource_hash: {h}\n")
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(f))
    assert bench.committed_traffic() == 123456.0
    f.write_text("traffic_bytes_per_launch: 123456\nsource_hash: 0000000000000000\n")
    assert bench.committed_traffic() is None
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(tmp_path / "missing.md"))
    assert bench.committed_traffic() is None


def test_printed_line_is_short():
    """A filled result of the full run, per-layer lists and all."""
    sys.path.insert(0, ROOT)
    import bench
    layer = {"layer": "layer3.5.c2", "call": "qconv", "M": 50176, "N": 256, "K": 1024, "ms": 0.0368, "tops": 714.9}
    agg = {"layers": 8, "ridge_ops_per_byte": 625.0, "achieved": 1035.1, "frac": 0.2071, "ms_per_forward": 0.457}
    kernel = {"kernel": "k_qconv", "achieved": 1234.5, "unit": "TOP/s", "peak": 5000.0, "frac": 0.1234,
              "ms_per_forward": 3.787, "launches": 54}
    out = {"metric": "calibration images/s (ResNet-50 b256 DFX); FL-search GB/s; int8 MFMA % peak",
           "value": 53685.12, "unit": "images/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 4.768,
           "ms_per_step_cold": 10.892, "ms_per_step_mispredicted": 15.123, "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None, "dtype": "int8", "data": "synthetic",
           "config": {"workload": "resnet50_b256_224_dfx_calibration_forward", "batch": 256, "image": 224,
                      "weight_wl": 8, "act_wl": 8, "fl_range": [-8, 15], "parallelism": "single_gpu",
                      "predicted_cblocks": 53, "timed_forwards_rerun": 0},
           "roofline": {"bound": "alu", "achieved": 13.45, "peak": 39.32, "unit": "TOP/s", "frac": 0.3421,
                        "traffic": 108123456.0, "kernel": "k_cblock_pred", "launches": 53, "avg_launch_ms": 0.07171,
                        "ops_per_launch": 980000000, "ops_per_output_value": bench.PRED_OPS_PER_VALUE,
                        "ms_per_forward": 3.801, "int8_tops": 531.2},
           "fl_search_gbs": 4780.1, "fl_search": dict(kernel), "requant": dict(kernel),
           "mfma": dict(kernel, compute_bound_layers=agg, own_roofline={"ms": 3.2, "frac": 0.2}, per_layer=[layer] * 54),
           "predicted_cblock": {"per_layer": [layer] * 53},
           "sweep": {"workload": "resnet50_b256_224_sensitivity_sweep", "layer_evaluations": 1890, "seconds": 0.8882,
                     "layer_eval_images_per_s": 544735.2, "setup_seconds_untimed": 1.03},
           "configs": dict({"fc": {"workload": "fc_256x512_b32_wl8", "us_per_call": 58.12, "calls": "x" * 80}},
                           **{n: {"workload": n, "batch": 128, "images_per_s": 123456.7, "ms_per_forward": 4.123,
                                  "ms_per_forward_cold": 4.567, "compute_bound_layers": agg}
                              for n in ("alexnet", "vgg16", "resnet18")}),
           "cpu_baseline": {"value": 1.08083, "unit": "images/s", "cores": 16, "kind": "oracle",
                            "sample": "ResNet-50 DFX calibration forward of 12 images 224x224 (exact CPU oracle, "
                                      "parameters pre-quantized; 11.1 s forward, 12.5 s set-up untimed)",
                            "cpu_model": "y" * 40, "single_core": {"values": 1 << 22}, "configs": {"fc": layer}}}
    line = json.dumps(bench.summary(out))
    assert len(line) < 1850
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config"):
        assert json.loads(line)[k] == out[k]
