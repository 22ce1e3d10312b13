"""bench.py's command-line modes: every mode function main() dispatches to exists (host only)."""
import ast
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_dispatched_mode_is_defined():
    tree = ast.parse(open(os.path.join(ROOT, "bench.py")).read())
    defined = {n.name for n in tree.body if isinstance(n, ast.FunctionDef)}
    main = next(n for n in tree.body if isinstance(n, ast.FunctionDef) and n.name == "main")
    called = {c.func.id for c in ast.walk(main) if isinstance(c, ast.Call) and isinstance(c.func, ast.Name)}
    modes = {name for name in called if name.endswith("_main")}
    assert modes, "main() dispatches to no mode function"
    assert modes <= defined, f"main() calls undefined mode functions: {sorted(modes - defined)}"


def test_a_workload_takes_little_of_the_printed_line():
    """The line is read from the last few KB of the output: a workload's entry carries no sweep, no kernel
    table and no roofline of its own."""
    import json
    import sys
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench
    roof = {"achieved": 4750.8, "peak": 8000.0, "kernel": "k" * 40}
    res = {"workload": "w" * 400, "chosen": "SPLIT(Sp=224,Sd=32,k=29)", "wall_us": 8456.1, "agg_wall_us": 9000.2,
           "speedup_vs_agg": 1.0643, "iteration_us": 8400.3, "agg_iteration_us": 8990.1, "predicted_us": 8333.3,
           "decode_step_us": 291.4, "sweep": [{"Sp": 32 * i, "measured_us": 1.5} for i in range(7)],
           "sweep_best": {"measured_us": 8411.1}, "kernels_us": {str(i): 1.0 for i in range(12)},
           "decode_roofline": {"split": roof, "standalone_256": roof},
           "prefill_roofline": {"split": None, "standalone_256": roof}}
    out = bench.summary(res)
    assert len(json.dumps(out)) < 500
    assert out["wall_us"] == 8456.1 and out["decode_gbps"] == 4750.8 and out["prefill_tflops"] is None
    assert out["sweep_best_us"] == 8411.1 and out["decode_step_us"] == 291.4
