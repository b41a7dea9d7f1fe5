"""The rules that let a step of few token rows per expert stream its weights in panels (csrc/ffn_route.cpp) without a GPU."""
import pytest

from paper_2510_12357_amd import workloads as wl
from test_ffn_route_host import route  # noqa: F401


@pytest.fixture(scope="module")
def panels(route):  # noqa: F811
    """Kernels of gate/up and the down projection: S, T, W or P; with a 2 where panels hold two tiles per wave."""
    def ask(cfg, routed=True, shared=True):
        gate_up, down, _, _, _, wide, _, _ = route.raw(cfg, routed, shared)
        assert not wide or cfg.dtype in ("bf16w8", "bf16mx4")
        return "STWP"[gate_up] + "STWP"[down] + "2" * wide
    return ask


def _layer(H, E, I, k, T, shared=(), dtype="bf16"):
    return wl.LayerConfig("r", T=T, H=H, E=E, I=I, k_big=k, k_little=max(1, k // 2), shared_I=shared, dtype=dtype)


def test_large_layers_stream_in_panels(panels):
    """Large layers, narrow formats medium ones too; never the shared experts alone, nor many experts that few tokens hit."""
    few, many = wl.CONFIGS["coarse8"], wl.CONFIGS["fine60_decode"]
    for T in (1, 2, 64, 65, 128):
        assert panels(many.with_(T=T)) == "PP" and panels(few.with_(T=T)) == ("PP" if T > 106 else "SS")
        assert panels(many.with_(T=T), False, True) == panels(many.with_(T=T, dtype="fp32")) == "SS"
        for dtype in ("bf16w8", "bf16mx4"):
            assert panels(few.with_(T=T, dtype=dtype))[:2] == panels(many.with_(T=T, dtype=dtype), True, False) == "PP"
            assert panels(_layer(4096, 16, 1024, 2, T, (), dtype))[:2] == "PP" and panels(_layer(2048, 8, 2048, 2, T, (2048,), dtype)) == "SS"
        assert panels(_layer(4096, 16, 1024, 2, T)) == "SS"
    assert panels(_layer(4096, 8, 8192, 2, 65, (8192,))) == "PP"
    for dtype in ("bf16w8", "bf16mx4"):
        for E, line in ((128, 16), (256, 32)):
            layer = _layer(2048, E, 1024, 8, 1, (), dtype)
            assert [panels(layer.with_(T=T)) for T in (7, 8)] == ["SS", "PP"]
            assert [panels(layer.with_(T=T), True, False) for T in (line - 1, line)] == ["SS", "PP"]
    # 8-bit: down projections of few columns; short rows, experts of 5 .. 13 rows
    assert panels(_layer(512, 72, 2880, 2, 60, (2880,), "bf16w8")) == "PS" and panels(_layer(768, 72, 2880, 2, 60, (2880,), "bf16w8")) == "PP"
    for layer in (_layer(2048, 64, 1024, 8, 1, (), "bf16w8"), _layer(2048, 32, 1024, 4, 1, (2048,), "bf16w8")):
        per = layer.E * 2 / 3 / layer.k_little                # tokens per row of an expert
        for rows, kernels in ((4, "PP"), (4.6, "SS"), (12.9, "SS"), (14, "PP")):
            assert panels(layer.with_(T=int(rows * per))) == kernels, rows
            assert panels(layer.with_(T=int(rows * per)), True, False) == panels(layer.with_(T=int(rows * per), dtype="bf16mx4"))[:2] == "PP"


def test_bf16_launches_choose_by_themselves(panels):
    """gate/up leaves the panels where its groups are of one token tile and many of them are hit, the down projection while few are."""
    fine64, wide_rows = _layer(2048, 64, 1024, 8, 1), _layer(4096, 64, 1536, 6, 1, (3072,))
    for layer, expect in ((fine64, {1: "SS", 2: "PP", 8: "PP", 9: "SP", 117: "SP", 118: "PP", 128: "PP"}),
                          (wide_rows, {1: "SP", 2: "PP", 10: "PP", 11: "SP", 64: "SP", 65: "PP", 128: "PP"}),
                          (wl.CONFIGS["shared2_offload"], {1: "PP", 2: "PP", 128: "PP"}),
                          (_layer(2048, 48, 1408, 4, 1, (2816,)), {1: "SS", 2: "PP"}), (_layer(2048, 64, 1408, 6, 1), {1: "SS", 2: "PS", 3: "PP"}),
                          (_layer(2048, 20, 4096, 2, 1), {1: "SS", 2: "PS", 6: "PS", 7: "PP", 255: "PP"}),
                          (_layer(2048, 128, 768, 8, 1, (768,)), {7: "SS", 8: "SP", 128: "SP"}),
                          (_layer(640, 128, 4096, 4, 1, (8192,)), {7: "SS", 8: "PS", 128: "PS"}),
                          (_layer(2048, 160, 1408, 8, 1, (1408, 1408)), {8: "SP", 208: "SP", 209: "PP"}),
                          (_layer(1024, 64, 4096, 8, 1), {1: "PS", 255: "PS"}), (_layer(2048, 24, 2048, 2, 64, (2048,)), {64: "SS"})):
        for T, want in expect.items():
            assert panels(layer.with_(T=T)) == want, (layer, T)
    for layer, expect in ((wl.CONFIGS["fine60_decode"], {11: "SS", 12: "PS", 24: "PS", 25: "PP", 33: "PP", 127: "PP", 128: "SP", 255: "SP"}),
                          (wide_rows, {11: "SS", 12: "PS", 127: "PS", 128: "SS"}),
                          (_layer(2048, 20, 4096, 2, 1), {7: "SS", 8: "PS", 49: "PS", 50: "PP", 255: "PP"}),
                          (_layer(4096, 128, 1024, 4, 1), {47: "SS", 48: "PS", 255: "PS"}), (_layer(1024, 64, 4096, 8, 1), {37: "PS", 38: "PP"}),
                          (_layer(2048, 128, 768, 8, 1, (768,)), {15: "SS", 16: "PS", 17: "PP", 64: "PP", 65: "SP"}),
                          (_layer(2048, 256, 512, 8, 1, (512,)), {16: "SS", 17: "SP", 255: "SP"}),
                          (wl.CONFIGS["coarse8"], {8: "SS", 255: "SS"})):
        for T, want in expect.items():
            assert panels(layer.with_(T=T), True, False) == want, (layer, T)


def test_prefill_of_few_rows_streams_in_panels(panels):
    """Narrow formats of any size while the weights meet few token rows (fewer in smaller layers of many small experts), bf16
    only with few experts and where the tiles leave CUs idle."""
    few, many, small = wl.CONFIGS["coarse8"], wl.CONFIGS["fine60_decode"], _layer(512, 8, 512, 2, 256)
    many_small, smaller = _layer(2048, 64, 1024, 8, 256), _layer(1024, 64, 512, 8, 256)
    for cfg, dtype, expect in (
            (few, "bf16", {256: "PP", 319: "PP", 320: "TT", 4096: "WW"}), (many, "bf16", {256: "TT", 600: "TT"}), (small, "bf16", {256: "TT"}),
            (_layer(4096, 16, 1024, 2, 1), "bf16", {256: "PT", 639: "PT", 640: "TT"}), (_layer(4096, 16, 4096, 2, 1), "bf16", {256: "TT"}),
            (_layer(4096, 16, 1024, 2, 1, (1024,)), "bf16", {256: "TT"}),
            (few, "bf16w8", {277: "PP", 278: "PP2", 373: "PP2", 374: "TT"}), (many, "bf16w8", {256: "PP", 475: "PP", 476: "PP2", 767: "PP2", 768: "TT"}),
            (few, "bf16mx4", {144: "PP2", 143: "PP", 405: "PP2", 406: "TT"}), (many, "bf16mx4", {246: "PP", 247: "PP2", 767: "PP2", 768: "TT"}),
            (small, "bf16w8", {255: "SS", 256: "PP", 512: "TT"}), (small, "bf16mx4", {255: "SS", 256: "PP2", 405: "PP2", 512: "TT"}),
            (_layer(2048, 16, 1408, 2, 1), "bf16mx4", {597: "PP2", 598: "TP2", 810: "TP2", 811: "TT"}), (_layer(2048, 16, 1408, 2, 1), "bf16w8", {740: "PP2", 747: "TT"}),
            (many_small, "bf16w8", {383: "PP", 384: "TP", 660: "TP2", 662: "PP2", 810: "PP2", 811: "TT"}),
            (many_small, "bf16mx4", {287: "PP", 288: "PP2", 597: "PP2", 598: "TP2", 810: "TP2", 811: "TT"}),
            (_layer(4096, 64, 1024, 8, 1, (1024,)), "bf16w8", {340: "PP", 560: "PP2"}), (_layer(4096, 64, 1024, 8, 1, (1024,)), "bf16mx4", {680: "PP2"}),
            (_layer(2048, 20, 4096, 2, 1), "bf16w8", {1013: "PP2", 1014: "TT"}), (_layer(2048, 20, 4096, 2, 1), "bf16mx4", {933: "PP2", 934: "TP2", 1014: "TT"}),
            (smaller, "bf16w8", {383: "PP", 384: "TT", 600: "TT"}), (smaller, "bf16mx4", {383: "PP2", 384: "TT"}),
            (few, "fp32", {256: "SS"}), (_layer(512, 4096, 4096, 1, 1), "bf16w8", {65535: "PP", 65536: "TT"})):
        for T, want in expect.items():
            assert panels(cfg.with_(T=T, dtype=dtype)) == want, (cfg, dtype, T)
            assert "P" not in panels(cfg.with_(T=T, dtype=dtype), False, True)
            if T >= 256 and dtype != "fp32":       # a part: both launches wherever the step's rows allow it
                assert panels(cfg.with_(T=T, dtype=dtype), True, False)[:2] == ("PP" if "P" in want or (cfg.E, T) == (16, 256) else "TT")
    # a fallback pass: two tiles where they make one round over the CUs of two
    assert panels(_layer(528, 64, 272, 6, 256, (992,), "bf16w8"), True, False) == "PP2"
    assert panels(_layer(512, 64, 256, 4, 256, (1024,), "bf16w8"), True, False) == "PP"
    assert panels(few.with_(T=400, dtype="bf16mx4"), True, False) == "PP"


def test_gate_up_on_tiles_above_128_tokens(panels):
    """Whole bf16 steps of large layers of few experts, or of up to 64 beside shared ones; rows that are whole cache lines only.
    Parts stay streamed."""
    for layer in (_layer(2048, 64, 1408, 6, 1, (1408, 1408)), _layer(2048, 17, 8192, 2, 1, (8192,)), _layer(4096, 8, 8192, 2, 1, (8192,)),
                  _layer(4096, 64, 1536, 6, 1, (3072,)), wl.CONFIGS["coarse8"], wl.CONFIGS["fine60_decode"]):
        assert [panels(layer.with_(T=T))[0] == "T" for T in (65, 128, 129, 255)] == [False, False, True, True], layer
        assert "T" not in panels(layer.with_(T=200), True, False) + panels(layer.with_(T=200), False, True)
    for layer in (_layer(2048, 64, 1400, 6, 1, (2800,)), _layer(2048, 64, 1024, 8, 1), _layer(2048, 17, 8192, 2, 1), _layer(7168, 16, 2880, 1, 1), _layer(2048, 160, 1408, 8, 1, (1408, 1408)), _layer(2048, 24, 2048, 2, 1, (2048,))):
        assert "T" not in panels(layer.with_(T=65)) + panels(layer.with_(T=255))
