"""Host checks of bench.py (no GPU): every module-level name its functions
call is defined, the multi-GPU request exits with a message before touching
the device."""
import ast
import builtins
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BENCH = os.path.join(ROOT, "bench.py")


def test_every_called_module_name_is_defined():
    tree = ast.parse(open(BENCH).read())
    defined = set(dir(builtins))
    for node in tree.body:
        if isinstance(node, (ast.FunctionDef, ast.ClassDef)):
            defined.add(node.name)
        elif isinstance(node, (ast.Import, ast.ImportFrom)):
            defined.update((a.asname or a.name).split(".")[0] for a in node.names)
        elif isinstance(node, ast.Assign):
            defined.update(t.id for t in node.targets if isinstance(t, ast.Name))
    missing = set()
    # each top-level function with everything nested in it is one scope
    for fn in [n for n in tree.body if isinstance(n, ast.FunctionDef)]:
        local = set()
        for n in ast.walk(fn):
            if isinstance(n, ast.Name) and isinstance(n.ctx, ast.Store):
                local.add(n.id)
            elif isinstance(n, (ast.FunctionDef, ast.Lambda)):
                a = n.args
                local.update(x.arg for x in a.args + a.kwonlyargs)
                if isinstance(n, ast.FunctionDef):
                    local.add(n.name)
            elif isinstance(n, (ast.Import, ast.ImportFrom)):
                local.update((x.asname or x.name).split(".")[0] for x in n.names)
        for n in ast.walk(fn):
            if isinstance(n, ast.Call) and isinstance(n.func, ast.Name):
                if n.func.id not in local and n.func.id not in defined:
                    missing.add(n.func.id)
    assert not missing, sorted(missing)


KERNEL_NAMES = [
    # the compiler's name, as a profiler prints it; the library's launch name
    ("void xp::(anonymous namespace)::k_conv_gemm_lds<96, 96, 1, 3, 32, 3, false, 0, false, false>(xp::ConvArgs, int)",
     "k_conv_gemm_lds<96,96,1,3,32,3,false,0,false,false>"),
    ("void xp::(anonymous namespace)::k_conv_gemm_lds<32, 32, 1, 1, 64, 4, true, 0, false, true>(xp::ConvArgs, int)",
     "k_conv_gemm_lds<32,32,1,1,64,4,true,0,false,true>"),
    ("void xp::(anonymous namespace)::k_conv_gemm_lds<64, 64, 2, 2, 64, 2, true, 2, true, false>(xp::ConvArgs, int)",
     "k_conv_gemm_lds<64,64,2,2,64,2,true,2,true,false>"),
    ("void xp::(anonymous namespace)::k_wgrad_lds<128, 64, 4, 2, 64, false>(xp::WgradArgs, int, int)",
     "k_wgrad_lds<128,64,4,2,64,false>"),
    ("void xp::(anonymous namespace)::k_wgrad_lds<64, 64, 2, 2, 64, true>(xp::WgradArgs, int, int)",
     "k_wgrad_lds<64,64,2,2,64,true>"),
    ("void xp::(anonymous namespace)::k_conv_gemm_image<7>(xp::ConvArgs, int, int, int, int)", "k_conv_gemm_image<7>"),
    ("void xp::(anonymous namespace)::k_wgrad_image<5>(xp::WgradArgs, int, int, int, int)", "k_wgrad_image<5>"),
    ("void xp::k_conv_gemm<unsigned short, 32, 64, 2, 2, false, 4, 2, 0>(xp::ConvArgs)",
     "k_conv_gemm<bf16,32,64,2,2,false,4,2>"),
    ("void xp::k_conv_gemm<float, 64, 64, 2, 2, false, 1, 1, 2>(xp::ConvArgs)",
     "k_conv_gemm<f32,64,64,2,2,false,1,1,strided_dgrad>"),
    ("void xp::k_wgrad<float, 64, 64, 2, 2, false>(xp::WgradArgs)", "k_wgrad<f32,64,64,2,2,false>"),
    ("xp::k_colfinal_v(xp::ColArgs)", "k_colfinal_v"),
]


def test_profiler_and_launch_names_of_a_kernel_share_a_key():
    """Stored HBM traffic is looked up by launch name and stored by the profiler's."""
    sys.path.insert(0, ROOT)
    import bench
    keys = [bench.kernel_key(a) for a, _ in KERNEL_NAMES]
    assert keys == [bench.kernel_key(b) for _, b in KERNEL_NAMES]
    assert all(k.startswith("k_") for k in keys) and len(set(keys)) == len(keys)


def test_result_line_is_short():
    """The line of a full run stays within the last kilobytes that a log keeps, with
    the metric's figures in it."""
    sys.path.insert(0, ROOT)
    import bench
    roof = {"bound": "mfma", "achieved": 317.349, "peak": 2500.0, "unit": "TFLOP/s", "frac": 0.12694,
            "kernel": "k_conv_gemm_lds<96,96,1,3,32,3,false,0,false,false>", "launches_per_step": 48.0,
            "avg_launch_us": 17.076, "avg_launch_us_raw_events": 19.195, "work_per_launch": 5419008000.0}
    top = [{"kernel": f"k_conv_gemm_lds<128,128,4,2,64,2,false,{i},false,false>", "ms_per_step": 0.8657,
            "launches_per_step": 208.0, "avg_us": 4.16, "achieved": 135.6, "unit": "GB/s", "frac": 0.0169} for i in range(12)]
    leg = {"workload": "resnet101_mid_stage", "dtype": "bf16", "s_fwd": 1, "ms_per_step": 6.1561, "roofline": roof,
           "roofline_conv_gemm": roof, "roofline_weight_gradient": roof, "mfma_util_all_gemm": 0.05579, "top_kernels": top[:5]}
    part = {"model": "m" * 70, "per_stage": [{"layers": [0, 7], "in_shape": [224, 224, 3], "ms_per_step": 33.8659}] * 4,
            "note": "n" * 150}
    sweep = {k: {"ms": 0.26, "GB_s": 6113.0, "frac_hbm": 0.7641} for k in
             ("predict_s0", "predict_s1", "predict_s2", "predict_s3", "predict_s7", "adam", "adam_zero_grad_2pred",
              "momentum_sgd_zero_grad_2pred", "rmsprop_zero_grad_2pred")}
    out = {"metric": "m" * 80, "value": 22660.46, "unit": "samples/s", "ms_per_step": 5.6486, "config": {"workload": "w" * 200},
           "roofline": roof, "roofline_conv_gemm": roof, "roofline_weight_gradient": None, "top_kernels": top,
           "peaks_measured": {"hbm_copy_GB_s": 6192.6, "mfma_bf16_TFLOP_s": 2204.6,
                              "graph_fork_join": [{"spin": 0, "width": 1, "branches_us": 3.24}] * 8},
           "predict_adam_sweep": {"n_params": 10 ** 8, "t": 100, **sweep, "stream_ceiling": {"read": {"GB_s": 6000.0}}},
           "interleaved_schedule": {"samples_per_s": 22459.32, "ms_per_minibatch": 5.6992, "note": "n" * 170},
           "vgg16_partitioned": part, "resnet101_partitioned": part, "inception_v3_partitioned": part,
           "vendor_reference": [{"shape": "conv 3x3 64->96, 32x35x35", "ours_us": 13.09, "ours_launches": ["k" * 50],
                                 "miopen_conv_us": 17.53, "hipblaslt_gemm_us": 19.27, "ours_TFLOP_s": 331.1}] * 4,
           "configs": [leg] * 8, "cpu_baseline": {"value": 6.068, "unit": "samples/s", "cores": 16, "kind": "oracle",
                                                  "sample": "s" * 200, "single_thread": {"note": "n" * 200}}}
    assert len(json.dumps(out)) > 12000
    line = bench.result_line(out)
    text = json.dumps(line)
    assert len(text) < 5000
    assert line["value"] == 22660.46 and line["roofline"] == roof and line["roofline_weight_gradient"] is None
    assert line["predict_adam_sweep"]["GB_s"]["predict_s1"] == 6113.0 and line["cpu_baseline"]["value"] == 6.068
    small = {k: out[k] for k in ("metric", "value", "unit", "roofline", "roofline_conv_gemm", "top_kernels")}
    assert bench.result_line(small)["value"] == 22660.46  # a run without the other measurements


def test_multi_gpu_request_exits_with_a_message():
    r = subprocess.run([sys.executable, BENCH, "--gpus", "2"], capture_output=True, text=True,
                       cwd=ROOT, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in json.loads(r.stdout.strip().splitlines()[-1])["error"]
