"""The rule that lets a step of few tokens stream its weights in panels (csrc/ffn_route.cpp) without a GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2510_12357_amd import workloads as wl
from test_ffn_route_host import CSRC, DTYPES, ROOT, STREAM


@pytest.fixture(scope="module")
def panels(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    if cxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("panels") / "ffn_panels_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "host", "ffn_panels_check.cpp"), os.path.join(CSRC, "ffn_route.cpp"), "-o", out],
                   check=True)

    def ask(cfg, routed=True, shared=True):
        v = [DTYPES[cfg.dtype], cfg.T, cfg.H, cfg.E, cfg.I, cfg.k_big, cfg.k_little, len(cfg.shared_I), *cfg.shared_I,
             int(routed), int(shared)]
        r = subprocess.run([out], input=" ".join(map(str, v)) + "\n", capture_output=True, text=True, check=True)
        kernel, yes = map(int, r.stdout.split())
        assert not yes or kernel == STREAM
        return bool(yes)
    return ask


def _layer(H, E, I, k, T, shared=(), dtype="bf16"):
    return wl.LayerConfig("r", T=T, H=H, E=E, I=I, k_big=k, k_little=max(1, k // 2), shared_I=shared, dtype=dtype)


def test_large_layers_stream_in_panels(panels):
    """Large layers (narrow formats: medium ones too); bf16 with few experts from 65 tokens on and where enough rows are
    hit, fallback passes from 8 tokens on; many experts from 8 (16) tokens on; never the shared experts alone."""
    few, many = wl.CONFIGS["coarse8"], wl.CONFIGS["fine60_decode"]
    for T in (1, 2, 64, 65, 255):
        assert panels(many.with_(T=T)) and panels(few.with_(T=T)) == (T > 64)
        assert panels(many.with_(T=T), True, False) == (T >= 8)
        assert not panels(many.with_(T=T), False, True) and not panels(many.with_(T=T, dtype="fp32"))
        for dtype in ("bf16w8", "bf16mx4"):
            assert panels(few.with_(T=T, dtype=dtype)) and panels(many.with_(T=T, dtype=dtype), True, False)
            assert panels(_layer(4096, 16, 1024, 2, T, (), dtype)) and not panels(_layer(2048, 8, 2048, 2, T, (2048,), dtype))
        assert not panels(_layer(4096, 16, 1024, 2, T))
        assert panels(_layer(2048, 256, 512, 8, T, (512,))) == (T >= 8)
    assert not panels(many.with_(T=256)) and not panels(_layer(2048, 20, 4096, 2, 1)) and panels(_layer(2048, 20, 4096, 2, 4))
