"""The rules that let a step of few token rows per expert stream its weights in panels (csrc/ffn_route.cpp) without a GPU."""
import pytest

from paper_2510_12357_amd import workloads as wl
from test_ffn_route_host import PANELS, TILED, route  # noqa: F401


@pytest.fixture(scope="module")
def panels(route):  # noqa: F811
    def ask(cfg, routed=True, shared=True):
        gate_up, down, _, _, _, wide, _, _ = route.raw(cfg, routed, shared)
        tiled = gate_up == TILED and down == PANELS
        assert not tiled or (cfg.dtype == "bf16" and 64 < cfg.T < 256 and routed and shared)
        assert not wide or cfg.dtype in ("bf16w8", "bf16mx4")
        return (down == PANELS) + wide + 4 * tiled
    return ask


def _layer(H, E, I, k, T, shared=(), dtype="bf16"):
    return wl.LayerConfig("r", T=T, H=H, E=E, I=I, k_big=k, k_little=max(1, k // 2), shared_I=shared, dtype=dtype)


def test_large_layers_stream_in_panels(panels):
    """Large layers (narrow formats: medium ones too); bf16 with few experts from 65 tokens on and where enough rows are
    hit, fallback passes from 8 tokens on; many experts from 8 (16) tokens on; never the shared experts alone."""
    few, many = wl.CONFIGS["coarse8"], wl.CONFIGS["fine60_decode"]
    for T in (1, 2, 64, 65, 255):
        assert panels(many.with_(T=T)) == (1 if T < 129 else 5) and panels(few.with_(T=T)) == (T > 64)
        assert panels(many.with_(T=T), True, False) == (T >= 8)
        assert not panels(many.with_(T=T), False, True) and not panels(many.with_(T=T, dtype="fp32"))
        for dtype in ("bf16w8", "bf16mx4"):
            assert panels(few.with_(T=T, dtype=dtype)) and panels(many.with_(T=T, dtype=dtype), True, False)
            assert panels(_layer(4096, 16, 1024, 2, T, (), dtype)) and not panels(_layer(2048, 8, 2048, 2, T, (2048,), dtype))
        assert not panels(_layer(4096, 16, 1024, 2, T))
        assert panels(_layer(2048, 256, 512, 8, T, (512,))) == (T >= 8)
    assert not panels(many.with_(T=256)) and not panels(_layer(2048, 20, 4096, 2, 1)) and panels(_layer(2048, 20, 4096, 2, 4))


def test_prefill_of_few_rows_streams_in_panels(panels):
    """0: tiled; 1, 2: panels of one and two tiles per wave.  Narrow formats of any size while the weights meet few token rows
    (fewer in smaller layers of many small experts), bf16 only with few experts; the same line for parts of a step."""
    few, many, small = wl.CONFIGS["coarse8"], wl.CONFIGS["fine60_decode"], _layer(512, 8, 512, 2, 256)
    many_small, smaller = _layer(2048, 64, 1024, 8, 256), _layer(1024, 64, 512, 8, 256)
    for cfg, dtype, expect in (
            (few, "bf16", ((256, 1), (319, 1), (320, 0), (4096, 0))), (many, "bf16", ((256, 0), (600, 0))),
            (small, "bf16", ((256, 0),)), (small.with_(T=256, H=65536), "bf16", ((256, 1),)),
            (few, "bf16w8", ((277, 1), (278, 2), (373, 2), (374, 0))), (many, "bf16w8", ((256, 1), (475, 1), (476, 2), (767, 2), (768, 0))),
            (few, "bf16mx4", ((144, 2), (143, 1), (405, 2), (406, 0))), (many, "bf16mx4", ((246, 1), (247, 2), (767, 2), (768, 0))),
            (small, "bf16w8", ((255, 0), (256, 1), (512, 0))), (small, "bf16mx4", ((255, 0), (256, 2), (512, 0))),
            (many_small, "bf16w8", ((383, 1), (384, 0), (575, 0), (576, 2), (810, 2), (811, 0))), (many_small, "bf16mx4", ((287, 1), (288, 2), (811, 0))),
            (smaller, "bf16w8", ((383, 1), (384, 0), (600, 0))), (smaller, "bf16mx4", ((383, 2), (384, 0))),
            (few, "fp32", ((256, 0),)), (_layer(512, 4096, 4096, 1, 1), "bf16w8", ((65535, 1), (65536, 0)))):
        for T, want in expect:
            assert panels(cfg.with_(T=T, dtype=dtype)) == want, (cfg, T)
            assert not panels(cfg.with_(T=T, dtype=dtype), False, True)
            if T >= 256:
                assert (panels(cfg.with_(T=T, dtype=dtype), True, False) > 0) == (want > 0)
    # a fallback pass: two tiles where they make one round over the CUs of two
    assert panels(_layer(528, 64, 272, 6, 256, (992,), "bf16w8"), True, False) == 2
    assert panels(_layer(512, 64, 256, 4, 256, (1024,), "bf16w8"), True, False) == 1
    assert panels(few.with_(T=400, dtype="bf16mx4"), True, False) == 1


def test_gate_up_on_tiles_where_the_panels_need_more_rounds(panels):
    """More than two rounds of panels over the CUs for one of tiles; rows that are whole cache lines only."""
    for layer, expect in ((_layer(2048, 64, 1408, 6, 1, (1408, 1408)), {64: 1, 128: 1, 129: 5, 255: 5}),
                          (_layer(2048, 64, 1408, 6, 1, (2816,)), {128: 1, 129: 5, 255: 5}),
                          (_layer(2048, 64, 1400, 6, 1, (2800,)), {255: 1}),                  # rows that are no whole cache lines
                          (_layer(2048, 64, 1024, 8, 1), {255: 1}), (_layer(4096, 64, 1536, 6, 1, (3072,)), {255: 1}),
                          (_layer(2048, 128, 768, 8, 1, (768,)), {255: 1})):
        for T, want in expect.items():
            assert panels(layer.with_(T=T)) == want, (layer, T)
