"""bench.py's command line and the one JSON line it prints (the driver's contract)."""
import json
import os
import re
import subprocess
import sys

import numpy as np
import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr and r.stdout.strip() == ""


def test_compulsory_bytes_of_the_prefetch():
    """Both sets in one launch: a row that both look up is counted once, lookups, bags and pooled rows of either add up."""
    sys.path.insert(0, ROOT)
    from bench import compulsory_gather_bytes
    from synth.generate import SetData
    from tests.helpers import small_cfg
    cfg = small_cfg(n_tasks=2, n_fields=2, emb_dim=4, rows_per_field=10, n_dense=5, layer_dims=(13, 8, 1), mlp_dtype=1)

    def one(task_offsets, lens, idx):
        n = task_offsets[-1]
        return SetData(np.array(task_offsets), torch.tensor([0] + list(np.cumsum(lens))), torch.tensor(idx, dtype=torch.int32),
                       torch.zeros(n, 5), torch.zeros(n))
    sup = one([0, 2, 3], [1, 2, 1, 0, 1, 1], [3, 5, 6, 3, 9, 9])      # task 0: rows (0,3) (1,5) (1,6)
    qry = one([0, 1, 2], [2, 1, 1, 1], [3, 4, 5, 0, 0])               # task 0: rows (0,3) (0,4) (1,5)
    rows, lookups, bags, samples = 4, 4 + 3, 4 + 2, 2 + 1
    assert compulsory_gather_bytes(cfg, sup, qry, 1) == rows * 16 + lookups * 4 + bags * 8 + samples * 32 * 6


@pytest.mark.parametrize("args,tasks", [("--config c5_large --tasks 256 --batches 1", 256), ("--config c3_medium --batches 1", None)])
def test_counter_summary_names_the_tasks_of_its_run(tmp_path, args, tasks):
    """A summary of a share of a workload's tasks says so: bench.py divides the whole run's launches by it."""
    for name in ("FETCH_SIZE", "WRITE_SIZE"):
        (tmp_path / f"{name}.csv").write_text('"Kernel_Name","Counter_Name","Counter_Value"\n'
                                              f'"stream_copy_kernel(int)","{name}",1024\n"pair_count_kernel(int)","{name}",512\n')
    out = tmp_path / "out.json"
    subprocess.run([sys.executable, os.path.join(ROOT, "bench_profiles.py"), "hbm", "--fetch", str(tmp_path / "FETCH_SIZE.csv"), "--write",
                    str(tmp_path / "WRITE_SIZE.csv"), "--copy-gib", str(1 / 1024), "--workload", "w", "--json", str(out), "--bench-args", args],
                   check=True, capture_output=True, timeout=120)
    d = json.loads(out.read_text())
    assert d["tasks_in_the_profiled_run"] == tasks and d["bytes_per_step"] == {"pair_count": 2 * 512 * 1024.0}


@pytest.mark.parametrize("workload", ["c3_medium", "c5_large"])
def test_committed_counter_summaries_name_the_tasks_of_their_run(workload):
    path = os.path.join(ROOT, "profiles", f"hbm_traffic_{workload}")
    with open(path + ".txt") as fh:
        given = re.search(r"bench\.py .*--tasks (\d+)", fh.read())
    with open(path + ".json") as fh:
        assert json.load(fh)["tasks_in_the_profiled_run"] == (int(given.group(1)) if given else None)


@pytest.mark.gpu
@pytest.mark.parametrize("bf,layers", [(0, 2), (0, 6), (1, 2)])
def test_timed_launches_of_the_weight_gradients(bf, layers):
    """The timing report's launches, bytes and operations of the weight gradients: in fp32 a pass's products share launches
    of at most four, in bf16 each has its own."""
    from paper_2401_04338_amd import GMeta
    from tests.helpers import small_cfg
    from tests.test_gpu_parity import _inputs, _params_dev, _to_dev
    cfg = small_cfg(n_tasks=3, n_support=16, n_query=8, layer_dims=(17,) + (40,) * layers + (1,), mlp_dtype=bf)
    sup, qry, params = _inputs(cfg)
    ctx = GMeta.from_config(cfg, workspace_bytes=1 << 28)
    ctx.profile(True)
    ctx.meta_step(_to_dev(sup, ctx.device), _to_dev(qry, ctx.device), _params_dev(params, ctx.device), cfg.inner_lr, 1, 2)
    r = ctx.profile_report()["gemm_wgrad"]
    ctx.close()
    assert r["launches"] == 3 * (layers if bf else -(-layers // 4))   # inner step, query set, tangent pass
    width = 32 * 64 + (layers - 1) * 64 * 64   # products' outputs, padded
    # one product per row of either set; in the tangent pass two (the first layer's second only where rows are adapted further)
    least = 2.0 * width * (3 * 16 + 3 * 8 + 3 * 16)
    assert least <= r["flops"] <= least + 2.0 * width * 3 * 16 and r["bytes"] > 0


@pytest.mark.gpu
def test_json_line_of_a_small_run():
    """The smallest config, a few steps: one JSON line on stdout with every field of the contract, the roofline of the
    dominant kernel family and the oracle timed beside it."""
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--config", "c1_tiny", "--steps", "3", "--warmup", "1",
                        "--cpu-seconds", "1"], capture_output=True, text=True, timeout=600, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [ln for ln in r.stdout.splitlines() if ln.strip()]
    assert len(lines) == 1, lines
    d = json.loads(lines[0])
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert key in d, key
    assert d["n_gpus"] == 1 and d["steps"] == 3 and d["warmup"] == 1 and d["higher_is_better"] is True
    assert d["unit"] == "samples/s" and d["data"] == "synthetic" and d["vs_baseline"] is None
    assert d["config"]["workload"] == "c1_tiny" and "model" not in d["config"]
    assert d["value"] > 0 and d["ms_per_step"] > 0
    # value is samples of one step over the time of one step
    assert abs(d["value"] - d["config"]["samples_per_step"] / (d["ms_per_step"] * 1e-3)) <= 1e-6 * d["value"]
    roof = d["roofline"]
    for key in ("bound", "achieved", "peak", "unit", "frac", "traffic"):
        assert key in roof, key
    assert roof["bound"] in ("hbm", "mfma", "alu") and roof["peak"] > 0
    assert abs(roof["frac"] - roof["achieved"] / roof["peak"]) <= 1e-9
    cpu = d["cpu_baseline"]
    for key in ("value", "unit", "cores", "kind", "sample"):
        assert key in cpu, key
    assert cpu["kind"] == "oracle" and cpu["value"] > 0 and cpu["cores"] >= 1


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,runs", [((512, 256), True), ((256, 128), True), ((96, 64), False), ((32,), False), ((), False)])
def test_query_gradient_over_runs_of_tasks(hidden, runs):
    """One second-order inner step, bf16: the query gradient summed over runs beside the chain's operand (a launch more per hidden layer) where
    the layers are wide enough to pay for it, in fp32 per task otherwise; against the oracle either way."""
    from paper_2401_04338_amd import GMeta
    from tests.helpers import small_cfg
    from tests.test_gpu_parity import TOL_BF16, _compare_step, _inputs
    cfg = small_cfg(n_tasks=96, n_support=16, n_query=40, n_fields=10, emb_dim=64, rows_per_field=200, bag_max=2, mlp_dtype=1,
                    layer_dims=(10 * 64 + 5,) + hidden + (1,))
    sup, qry, params = _inputs(cfg)
    ctx = GMeta.from_config(cfg, workspace_bytes=2 << 30)
    ctx.configure("chain_factors", 1)   # (the direction as matrices)
    ctx.profile(True)
    _compare_step(cfg, ctx, sup, qry, params, 1, 2, TOL_BF16, f"{hidden}, over runs: {runs}", operand="bf16")
    launches = ctx.profile_report().get("gemm_wgrad", {"launches": 0})["launches"]
    ctx.close()
    assert launches == (4 if runs else 3) * len(hidden)   # inner step, query set (twice), tangent pass
