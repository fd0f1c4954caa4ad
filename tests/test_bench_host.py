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


def test_multi_gpu_request_exits_with_a_message():
    r = subprocess.run([sys.executable, BENCH, "--gpus", "2"], capture_output=True, text=True,
                       cwd=ROOT, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in json.loads(r.stdout.strip().splitlines()[-1])["error"]
