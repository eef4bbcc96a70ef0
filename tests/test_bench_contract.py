"""bench.py's command-line contract on a machine without a GPU."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_exits_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    msg = json.loads(r.stdout.strip().splitlines()[-1])
    assert "one GPU" in msg["error"]


def test_cpu_oracle_leg_reports_cores_and_sample():
    env = dict(os.environ, OMP_NUM_THREADS="1")
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--cpu-oracle-only",
                        "--cpu-seconds", "0.5"], capture_output=True, text=True, timeout=300,
                       env=env)
    assert r.returncode == 0, r.stderr
    rec = json.loads(r.stdout.strip().splitlines()[-1])
    assert rec["kind"] == "oracle" and rec["cores"] == 1 and rec["unit"] == "MLUPS"
    assert rec["value"] > 0 and "1024x1024" in rec["sample"]


def test_roofline_arithmetic():
    """The roofline fields of a fused launch: minimum bytes = 72 B per FP32 site
    per launch (populations in and out, force in) whatever the steps per
    launch; frac against 8 TB/s; the one-step byte model as effective_gbs."""
    sys.path.insert(0, ROOT)
    import bench
    rf = bench.roofline("fp32", 1 << 20, 40.0, 8, "k_stepN<float, 16, 8, 512, 0> (tile)", None)
    want = 72 * (1 << 20) / 40e-6 / 1e9
    assert rf["min_bytes_per_launch"] == 72 * (1 << 20)
    assert abs(rf["achieved"] - want) < 0.1 and abs(rf["frac"] - want / 8000.0) < 1e-4
    assert abs(rf["effective_gbs"] - 8 * want) < 1.0
    assert rf["traffic"] is None and rf["valu_frac"] is None
    assert bench.PEAK_VALU_LANE_OPS == 256 * 4 * 16 * 2.4e9


def test_valu_fraction_is_of_a_rate_that_can_be_reached(monkeypatch):
    """Kernels in FP32 arithmetic issue additions in half the clocks of FP64
    instructions: 8192^2 FP16 (590.9 M wave instructions in 930 us) is 0.52 of that
    rate, not above 1; FP64 is priced at the full-width rate."""
    sys.path.insert(0, ROOT)
    import bench
    rec = {"traffic_bytes_per_launch": 3.05e9, "valu_insts_per_launch": 590910224.0}
    monkeypatch.setattr(bench, "measured_counters", lambda name, kernel=None: rec)
    want = 64 * 590910224.0 / 930e-6 / (256 * 4 * 16 * 2.4e9)
    for prec, f in (("fp16", 2), ("fp32", 2), ("fp64", 1)):
        rf = bench.roofline(prec, 8192 ** 2, 930.0, 8, "k_wave<__half, 8, 1> (wavefront)", "x")
        assert abs(rf["valu_frac"] - want / f) < 1e-3
    assert want > 1 > want / 2
