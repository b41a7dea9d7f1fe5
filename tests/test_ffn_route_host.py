"""The rules that choose the kernel of a moe_route or moe_expert_ffn call (csrc/ffn_route.cpp: plain host C++) without a GPU:
a call that runs a part of a step goes by that part."""
import os
import shutil
import subprocess

import pytest

import test_gpu_decode_step as decode
import test_gpu_kernel_edges as edges
import test_gpu_parity as parity
from paper_2510_12357_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_12357_amd", "csrc")
CUS = 256
DTYPES = {"bf16": 0, "fp32": 1, "bf16w8": 2, "bf16mx4": 3}
STREAM, TILED, WIDE, PANELS = 0, 1, 2, 3
ONE_LAUNCH, GEMV, GEMM = 0, 1, 2


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    if cxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("route") / "ffn_route_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-static-libubsan", "-Wall", "-Wextra", "-Werror", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host", "ffn_route_check.cpp"),
                    os.path.join(CSRC, "ffn_route.cpp"), "-o", out], check=True)
    env = dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0")
    env.pop("LD_PRELOAD", None)

    def run(cfg, routed, shared):
        v = [DTYPES[cfg.dtype], cfg.T, cfg.H, cfg.E, cfg.I, cfg.k_big, cfg.k_little, len(cfg.shared_I), *cfg.shared_I,
             int(routed), int(shared), CUS]
        r = subprocess.run([out], input=" ".join(map(str, v)) + "\n", capture_output=True, text=True, check=True, env=env)
        v = tuple(map(int, r.stdout.split()))
        run.even, run.lines, run.counts = v[8:10], v[10], v[11]
        return v[:8]

    def ask(cfg, routed=True, shared=True):
        """Kernel of both launches with what it is told: token tiles two (STREAM), order of tiles (TILED, WIDE), row tiles
        two (PANELS); (gate/up's, down's) where they differ."""
        gate_up, down, rows_gate_up, rows_down, two, wide, once, _ = run(cfg, routed, shared)
        assert (not two or STREAM in (gate_up, down)) and (not once or TILED in (gate_up, down)) and (not wide or PANELS in (gate_up, down))
        told = {STREAM: (two, two), PANELS: (wide, wide)}
        g, d = ((k, told.get(k, (rows_gate_up, rows_down))[i]) for i, k in enumerate((gate_up, down)))
        if gate_up == down:
            return gate_up, (g[1] if g[1] == d[1] else (g[1], d[1]))
        return g, d
    ask.raw = run
    ask.lines = lambda cfg: (run(cfg, True, True), run.lines)[1]
    ask.even = lambda cfg, shared=True: (run(cfg, True, shared), run.even)[1]
    ask.counts = lambda cfg: (run(cfg, True, True), run.counts)[1]
    ask.router = lambda cfg: run(cfg, True, True)[7]
    ask.weights_once = lambda cfg, routed=True: run(cfg, routed, True)[6]
    return ask


LAYERS = ["fine60_decode", "fine64_prefill", "shared2_offload", "coarse8"]


@pytest.mark.parametrize("layer", LAYERS)
@pytest.mark.parametrize("T", [256, 700, 2500, 4096])
def test_a_part_of_a_step_goes_by_what_it_runs(route, layer, T):
    """Fallback passes and waves (routed part alone) have rows that only the device knows: bf16 stays on
    the 128 x 256 tiles, and so do shared experts alone while there are fewer than 1.5 wide tiles per CU.
    Their tiles are alike, so the contiguous order stays, but for 8-bit experts that are all there is.  Few rows
    stream in panels."""
    cfg = wl.CONFIGS[layer].with_(T=T)
    few = T == 256 or (T == 700 and layer != "coarse8")
    assert route(cfg, True, False) == (PANELS if layer == "coarse8" and T == 256 else TILED, 0)
    assert route(cfg.with_(dtype="bf16mx4"), True, False) == (PANELS if few else TILED, 0)
    assert route(cfg.with_(dtype="bf16w8"), True, False) == ((PANELS, 0) if few else (TILED, int(layer == "fine64_prefill" and T < 2500)))
    if cfg.shared_I:
        tiles = sum(-(-i // 128) for i in cfg.shared_I) * -(-T // 256)
        assert route(cfg, False, True) == (WIDE if tiles >= 1.5 * CUS else TILED, 0)
        for narrow in ("bf16w8", "bf16mx4"):
            assert route(cfg.with_(dtype=narrow), False, True) == (TILED, 0)


def test_whole_steps(route):
    c = {k: wl.CONFIGS[k] for k in LAYERS + ["tiny_fp32"]}
    assert route(c["coarse8"].with_(T=4096)) == (WIDE, 0) and route(c["coarse8"].with_(T=1000)) == (TILED, 0)
    assert route(c["fine60_decode"].with_(T=4096)) == (WIDE, 1) and route(c["fine60_decode"].with_(T=2000)) == (TILED, 0)
    assert route(c["shared2_offload"].with_(T=2500)) == (WIDE, 1) and route(c["shared2_offload"].with_(T=3300)) == (WIDE, 0)
    assert route(c["fine64_prefill"].with_(T=4096)) == (WIDE, 1) and route(c["fine64_prefill"].with_(T=3000)) == (TILED, 0)
    assert route(c["fine64_prefill"].with_(T=777, dtype="bf16w8")) == (PANELS, 1) and route(c["fine64_prefill"].with_(T=900, dtype="bf16w8")) == (TILED, 1)
    assert route(c["fine60_decode"].with_(T=600, dtype="bf16mx4")) == (PANELS, 1) and route(c["fine60_decode"].with_(T=780, dtype="bf16mx4")) == (TILED, 1)
    assert route(c["fine60_decode"].with_(T=255)) == ((TILED, 0), (PANELS, 0)) and route(c["tiny_fp32"].with_(T=512)) == (STREAM, 0)


def _layer(H, E, I, k, T, shared=(), dtype="bf16"):
    return wl.LayerConfig("r", T=T, H=H, E=E, I=I, k_big=k, k_little=max(1, k // 2), shared_I=shared, dtype=dtype)


def test_wide_tiles_in_large_layers_only(route):
    """Below 805 MB of weights there are few wide tiles per CU or short rows; with few experts, fewer than five
    tiles per CU want 400 rows.  Shared experts alone want as many where their rows are shorter than 2048."""
    for H, E, I, k, shared in ((512, 8, 512, 2, ()), (512, 16, 256, 2, (512,)), (1024, 32, 512, 4, ()), (2048, 8, 2048, 2, (2048,)),
                               (2048, 16, 1408, 4, ()), (512, 64, 1024, 8, ()), (2048, 12, 4096, 2, ()), (2048, 24, 2048, 2, ()),
                               (520, 64, 264, 6, (1000,))):
        assert all(route(_layer(H, E, I, k, T, shared))[0] == TILED for T in (1200, 2500, 4096, 6000, 12000))
    assert [route(_layer(4096, 8, 4096, 2, T))[0] for T in (1500, 2200, 4096)] == [TILED, WIDE, WIDE]
    assert [route(_layer(2048, 8, 8192, 2, T))[0] for T in (1500, 4096)] == [TILED, WIDE]
    assert [route(_layer(6144, 8, 16384, 2, T))[0] for T in (1000, 1500)] == [TILED, WIDE]
    assert [route(_layer(4096, 64, 1536, 6, T, (3072,)))[0] for T in (2200, 3000)] == [TILED, WIDE]
    assert route(_layer(512, 16, 256, 2, 8192, (4096,)), False, True)[0] == TILED
    assert [route(_layer(1024, 16, 256, 2, T, (14336,)), False, True)[0] for T in (2048, 3000)] == [TILED, WIDE]
    assert route(_layer(4096, 16, 256, 2, 3072, (4096,)), False, True)[0] == WIDE


def test_weights_go_past_the_caches_where_the_layer_cannot_stay_in_them(route):
    for H, E, I, k, shared, once in ((2048, 64, 1024, 8, (), 1), (2048, 60, 1408, 4, (5632,), 1), (4096, 16, 1024, 2, (), 1),
                                     (4096, 15, 1024, 2, (), 0), (2048, 32, 1024, 4, (2048,), 1), (2048, 16, 1408, 4, (), 0),
                                     (2048, 8, 2048, 2, (2048,), 0), (1024, 32, 512, 4, (), 0)):
        for T in (700, 1000):
            assert route.weights_once(_layer(H, E, I, k, T, shared)) == once
            assert route.weights_once(_layer(H, E, I, k, T, shared), routed=False) == once
        for dtype in ("bf16w8", "bf16mx4"):
            assert not route.weights_once(_layer(H, E, I, k, 256, shared, dtype))
    for H, I, shared in ((2048, 1032, ()), (2080, 1024, ()), (2048, 1024, (2064,))):       # rows that are not whole lines of 128 bytes
        assert not route.weights_once(_layer(H, 64, I, 8, 256, shared))


def test_narrow_weights_by_rows_where_tiles_differ(route):
    """Beside shared experts in layers of 403 MB (of bf16) and more; alone 8-bit experts in large layers."""
    for dtype in ("bf16w8", "bf16mx4"):
        for H, E, I, k, shared, T in ((2048, 60, 1408, 4, (5632,), 780), (4096, 32, 2048, 4, (4096,), 580), (2048, 48, 1408, 4, (2816,), 840)):
            assert route(_layer(H, E, I, k, T, shared, dtype)) == (TILED, 1)
        for H, E, I, k, shared in ((512, 64, 256, 6, (1024,)), (512, 16, 256, 2, (512,)), (1024, 32, 512, 4, ()), (2048, 24, 2048, 2, ()),
                                   (4096, 16, 1024, 2, ()), (1024, 8, 1024, 2, ()), (640, 128, 512, 1, (768,)),
                                   (1408, 64, 640, 6, (2176,))):
            on = [route(_layer(H, E, I, k, T, shared, dtype)) for T in (256, 400, 800, 1500, 2000)]
            assert (TILED, 0) in on and all(r == (TILED, 0) or r[0] == PANELS or r == ((TILED, 0), (PANELS, 1)) for r in on)
        for T in (900, 2000):
            assert route(_layer(2048, 64, 1024, 8, T, (), dtype)) == (TILED, int(dtype == "bf16w8"))


def test_two_token_tiles_where_groups_are_large(route):
    """Streaming kernel, bf16, whole steps where an expert has 36 rows; in layers of 805 MB and more, which run in panels from
    20 rows on, above 64 tokens.
    Parts of a step, small layers and the narrower formats stay with one tile."""
    few, many, medium = wl.CONFIGS["coarse8"], wl.CONFIGS["fine60_decode"], _layer(2048, 16, 1408, 4, 1)
    for T in (1, 64, 65, 128, 146, 147, 255):
        assert route(few.with_(T=T), False, True) == route(many.with_(T=T), False, True) == (STREAM, 0)
        assert route(medium.with_(T=T), True, False) == route(medium.with_(T=T), False, True) == (STREAM, 0)
        assert route(few.with_(T=T)) == (((TILED, 0), (PANELS, 0)) if T > 128 else (PANELS, 0) if T > 106 else (STREAM, int(T > 64)))
        assert route(few.with_(T=T, dtype="fp32")) == (STREAM, 0)
        for dtype in ("bf16w8", "bf16mx4"):
            assert route(medium.with_(T=T, dtype=dtype)) == (STREAM, 0)
    for H, E, I, k, shared, lines in ((1024, 8, 1024, 2, (), {187: 0, 188: 1}), (2048, 8, 2048, 2, (2048,), {170: 0, 188: 1}),
                                      (2048, 16, 1408, 4, (), {128: 0, 187: 1}), (4096, 16, 1024, 2, (), {255: 0}),
                                      (512, 8, 512, 2, (), {255: 0}), (512, 16, 256, 2, (512,), {255: 0}), (520, 64, 264, 6, (1000,), {255: 0}),
                                      (1024, 128, 768, 8, (), {255: 0})):
        for T, two in lines.items():
            assert route(_layer(H, E, I, k, T, shared)) == (STREAM, two), (H, E, I, T)


def test_router_in_one_launch_while_its_reads_are_small(route):
    """Up to 64 tokens always; up to 256 with at most 64 experts while the gate matrix, read once per
    token, comes to no more than 100 MB, 60 MB in fp32."""
    def router(E, H, T, dtype="bf16"):
        return route.router(wl.LayerConfig("r", T=T, H=H, E=E, I=8, k_big=1, k_little=1, dtype=dtype))
    for E, H in ((8, 4096), (60, 2048), (256, 8192)):
        assert [router(E, H, T) for T in (1, 64, 257)] == [ONE_LAUNCH, ONE_LAUNCH, GEMM]
    for E, H, T, dtype in ((60, 2048, 200, "bf16"), (64, 2048, 256, "bf16"), (64, 4096, 200, "bf16"), (8, 4096, 256, "fp32"),
                           (60, 2048, 128, "fp32"), (33, 72, 256, "fp32")):
        assert router(E, H, T, dtype) == ONE_LAUNCH
    for E, H, T, dtype in ((65, 64, 65, "bf16"), (128, 2048, 65, "bf16"), (256, 256, 65, "bf16"), (64, 4096, 201, "bf16"),
                           (64, 2048, 128, "fp32"), (60, 2048, 200, "fp32"), (32, 8192, 65, "fp32"), (256, 1024, 256, "bf16")):
        assert router(E, H, T, dtype) == GEMV


def test_router_tests_reach_both_kernels(route):
    """The 100-token steps that the parity test compares with one launch run on the logits kernel for every
    data type, with odd expert counts too; so do tests of the logits against the oracle."""
    two = [(d, E) for d, _, E, _ in _cases(parity.test_one_launch_router_equals_the_two_kernels)
           if route.router(wl.LayerConfig("r", T=100, H=264, E=E, I=8, k_big=1, k_little=1, dtype=d)) == GEMV]
    assert {d for d, _ in two} == {"bf16", "fp32"} and any(E % 2 for _, E in two) and any(E == 256 for _, E in two)
    gemv = [c for c in _cases(parity.test_gate_logits)
            if route.router(wl.LayerConfig("r", T=c[1], H=c[2], E=c[3], I=8, k_big=1, k_little=1, dtype=c[0])) == GEMV]
    assert {c[0] for c in gemv} == {"bf16", "fp32"} and any(c[1] % 4 for c in gemv)


def test_tiles_that_fill_their_rounds(route):
    """bf16 tiles while the weights set the pace, each launch by its rows; narrow weights, wide tiles, panels and small layers never."""
    c = wl.CONFIGS
    assert [route.even(c["fine60_decode"].with_(T=T)) for T in (255, 300, 800, 1200, 2000)] == [(0, 0), (1, 1), (1, 1), (0, 1), (0, 0)]
    assert [route.even(c["coarse8"].with_(T=T)) for T in (300, 400, 700, 1000)] == [(0, 0), (1, 1), (0, 1), (0, 0)]
    assert route.even(c["fine60_decode"].with_(T=300), shared=False) == (1, 1)
    for dtype in ("bf16w8", "bf16mx4"):
        assert route.even(c["fine60_decode"].with_(T=1000, dtype=dtype)) == (0, 0)
    assert route.even(wl.LayerConfig("small", T=300, H=512, E=8, I=512, k_big=2, k_little=1)) == (0, 0)


def test_narrow_weights_in_whole_lines(route):
    """MXFP4 tiles of large layers, 8-bit ones of whole lines per row while their experts have fewer than 200 rows on average; bf16, panels and smaller layers never."""
    c = wl.CONFIGS["fine64_prefill"]
    assert [route.lines(c.with_(T=T, dtype="bf16mx4")) for T in (255, 1500, 4096)] == [0, 1, 1]
    assert [route.lines(c.with_(T=T, dtype="bf16w8")) for T in (255, 1500, 4096)] == [0, 1, 0]
    assert route.lines(c.with_(T=1500)) == 0
    for odd in (dict(I=1040), dict(H=2064), dict(shared_I=(1040,))):
        assert route.lines(c.with_(T=1500, dtype="bf16w8", **odd)) == 0
    for H, line in ((1024, 0), (4096, 1)):
        assert route.lines(wl.LayerConfig("l", T=2000, H=H, E=16, I=1024, k_big=2, k_little=1, dtype="bf16mx4")) == line


def test_narrow_tiles_are_tested_in_every_pair_of_choices(route):
    """By rows or contiguous, lines or chunks: what variants 0 and 1 do not have is tested through the public call."""
    seen = set()
    for d, T, E, I, sh in _cases(edges.test_narrow_tiles_as_the_rules_take_them):
        c = wl.LayerConfig("n", T=T, H=2048, E=E, I=I, k_big=8, k_little=4, shared_I=sh, dtype=d)
        gate_up, down, rows_gate_up, rows_down = route.raw(c, True, True)[:4]
        assert gate_up == down == TILED and rows_gate_up == rows_down
        seen.add((d, rows_down, route.lines(c)))
    assert {("bf16mx4", 0, 1), ("bf16w8", 1, 0), ("bf16w8", 1, 1), ("bf16mx4", 1, 1)} <= seen


def test_dispatch_beside_gate_up_is_tested_where_the_rules_take_it(route):
    """Its cases run in panels, as whole steps and (most of them) as fallback passes."""
    cases = _cases(edges.test_dispatch_built_by_the_gate_up_launch)
    layers = [wl.LayerConfig("f", T=T, H=H, E=E, I=I, k_big=K, k_little=kl, shared_I=sh, dtype=d) for d, T, E, K, kl, H, I, sh in cases]
    assert all(route.raw(c, True, True)[0] == PANELS for c in layers)
    assert sum(route.raw(c, True, False)[0] == PANELS for c in layers) >= 5


def test_full_size_decode_tests_reach_the_one_launch_kernel(route):
    """moe_layer_decode leaves it where gate/up runs in panels."""
    layer = lambda d, T, H, E, I, K, kl, sh: wl.LayerConfig("d", T=T, H=H, E=E, I=I, k_big=K, k_little=kl, shared_I=sh, dtype=d)  # noqa: E731
    cases = [layer(*c) for c in _cases(decode.test_one_launch_full_size)]
    assert all(route.raw(c, True, True)[0] != PANELS for c in cases) and {c.dtype for c in cases} == {"bf16", "bf16w8"}
    assert all(route.raw(wl.CONFIGS["fine60_decode"].with_(T=T), True, True)[0] == PANELS for T, in _cases_of_one(decode.test_fine60_decode_full_size))


def test_selection_counts_while_its_table_is_small(route):
    """The dispatch reads a table of a row per 16 tokens in every workgroup: with many tokens or experts a count launch is faster."""
    layer = lambda T, E, dtype="bf16": wl.LayerConfig("c", T=T, H=64, E=E, I=8, k_big=1, k_little=1, dtype=dtype)  # noqa: E731
    for E, last in ((1, 8192), (16, 8192), (60, 2184), (64, 2048), (128, 1024), (200, 655), (256, 512)):
        for dtype in ("bf16", "fp32", "bf16w8"):
            assert [route.counts(layer(T, E, dtype)) for T in (256, 257, last, last + 1, 65535, 1 << 20)] == [0, 1, 1, 0, 0, 0]
    edge = {c[:2] for c in _cases(edges.test_step_in_one_call_with_many_tokens_or_experts)}
    assert {route.counts(layer(*c)) for c in edge} == {0, 1}


def _cases_of_one(test):
    return [(a,) for m in test.pytestmark if m.name == "parametrize" for a in m.args[1]]


def _cases(test):
    return [tuple(a) for m in test.pytestmark if m.name == "parametrize" for a in m.args[1]]
