"""The C-ABI library loads and exports every function that include/mobile_moe.h declares; host-side
argument validation returns the documented codes without touching a GPU."""
import ctypes
import os
import re

import pytest

from paper_2510_12357_amd import binding as mm
from paper_2510_12357_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "mobile_moe.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"^\s*(?:const\s+)?[A-Za-z_][\w\s\*]*?\b(\w+)\s*\([^;{]*\)\s*;", text, flags=re.M)
    return sorted(set(names))


def test_header_functions_are_exported():
    if not os.path.exists(mm.LIB_PATH):
        pytest.skip("libmobile_moe.so not built (python -m paper_2510_12357_amd.build)")
    lib = ctypes.CDLL(mm.LIB_PATH)
    names = declared_functions()
    assert len(names) >= 15 and "moe_route" in names and "expert_cache_fetch" in names
    for n in names:
        assert hasattr(lib, n), f"{n} declared in mobile_moe.h but not exported"
    assert set(mm.EXPORTS) == set(names)


def test_config_validation_codes_without_gpu():
    if not os.path.exists(mm.LIB_PATH):
        pytest.skip("libmobile_moe.so not built")
    base = wl.CONFIGS["fine60_decode"]
    assert mm.moe_dispatch_workspace_bytes(mm.make_config(base)) >= 4 * base.E
    need = mm.moe_expert_ffn_workspace_bytes(mm.make_config(base))
    assert need >= 2 * (base.T * base.k_big * base.I + base.T * base.shared_I[0])
    lib = mm.load_library()
    for bad, code in ((base.with_(k_little=5), -2), (base.with_(H=2052), -3), (base.with_(E=300), -3),
                      (base.with_(k_big=70, k_little=1, E=80), -3), (base.with_(T=-1), -2)):
        c = mm.make_config(bad)
        assert mm.moe_dispatch_workspace_bytes(c) == 0
        rc = lib.moe_combine(ctypes.byref(c), None, None, None, None, None, None, None)
        assert rc == code, (bad, rc, mm.moe_last_error())
        assert mm.moe_last_error()


def test_bench_refuses_more_than_one_gpu():
    """Every box of this build has one GPU: the benchmark says so instead of starting ranks."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0 and "single-GPU" in (r.stderr + r.stdout)


def test_kernel_choice_is_refused_where_the_kernel_does_not_apply():
    if not os.path.exists(mm.LIB_PATH):
        pytest.skip("libmobile_moe.so not built")
    lib = mm.load_library()

    def code(cfg, kernel, variant):
        c = mm.make_config(cfg)
        return lib.moe_profile_expert_ffn(ctypes.byref(c), kernel, variant, None, None, None, None, (ctypes.c_void_p * 1)(), 1, 0,
                                          None, None, None, 0, None)
    few, many = wl.CONFIGS["fine60_decode"].with_(T=255), wl.CONFIGS["fine60_decode"].with_(T=256)
    for args in ((many, 0, 1), (few, 1, 0), (few, 2, 0), (many.with_(dtype="bf16w8"), 2, 0), (many.with_(dtype="bf16mx4"), 2, 1),
                 (few.with_(dtype="bf16w8"), 0, 2), (many.with_(dtype="fp32"), 1, 0), (few.with_(dtype="fp32"), 0, 2), (few, 0, 0),
                 (few, 0, 3), (many, 1, 4), (many, 2, 2), (many.with_(dtype="bf16w8"), 1, 2), (many, 2, -1), (many, 3, 0), (many, -1, 0)):
        assert code(*args) == -3, args
    assert code(many, 2, 0) == -1                                # the other checks are moe_expert_ffn's: x is NULL
    # gate/up of a whole step, of its routed part alone; panels count as kernel 0
    for cfg, whole, routed in ((few.with_(T=128), 0, 0), (few, 1, 0), (many, 1, 1), (few.with_(T=4096), 2, 1), (many.with_(dtype="bf16w8"), 0, 0),
                               (few.with_(T=4096, dtype="bf16w8"), 1, 1), (many.with_(dtype="fp32"), 0, 0)):
        c = mm.make_config(cfg)
        assert lib.moe_profile_expert_ffn_kernel(ctypes.byref(c), 1, 1) == whole
        assert lib.moe_profile_expert_ffn_kernel(ctypes.byref(c), 1, 0) == routed
    assert lib.moe_profile_expert_ffn_kernel(ctypes.byref(mm.make_config(few.with_(k_little=5))), 1, 1) == -2
