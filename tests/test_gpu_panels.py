"""Steps that moe_expert_ffn's own rules send to the panels of 256 tokens and more, or to gate/up on tiles below that, against
the oracle: ragged selections, mixed confidences, shared experts, both passes of a two-pass step."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_12357_amd import binding as mm
from paper_2510_12357_amd import workloads as wl
from gpu_util import TOL_OUT, DeviceLayer, out_to_f64, rel_err, run_gpu_layer, run_oracle_layer
from test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu
STREAMED, TILES = 0, 1                        # moe_profile_expert_ffn_kernel; from 256 tokens on streamed means panels


def _cfg(dtype, **kw):
    small = dict(H=256, I=128, shared_I=(128, 128)) if dtype == "bf16mx4" else dict(H=272, I=144, shared_I=(208, 48))
    base = dict(name="panels", T=300, E=48, k_big=5, k_little=2, dtype=dtype, gate_std=0.3, w_std=0.1, gate_bias_std=0.5,
                fallback_ratio=0.3, **small)
    base.update(kw)
    return wl.LayerConfig(**base)


def _gate_up(cfg, shared=True):
    return mm.moe_profile_expert_ffn_kernel(mm.make_config(cfg), True, shared)


@pytest.mark.parametrize("dtype", ["bf16w8", "bf16mx4"])
@pytest.mark.parametrize("kw", [dict(), dict(T=256, E=70, k_big=6, k_little=3, renorm=True), dict(T=400, E=20, k_big=2, k_little=1, shared_I=())])
def test_prefill_in_panels(dtype, kw):
    cfg = _cfg(dtype, **kw)
    assert _gate_up(cfg) == STREAMED
    check_layer(cfg, seed=cfg.T)


@pytest.mark.parametrize("dtype", ["bf16w8", "bf16mx4"])
def test_two_passes_in_panels(dtype):
    """The second pass has a fifth of the pairs: dispatch positions behind them belong to nobody."""
    cfg = _cfg(dtype, fallback_ratio=0.2)
    assert _gate_up(cfg) == _gate_up(cfg, False) == STREAMED
    layer = wl.make_layer(cfg, seed=8)
    dl = DeviceLayer(layer)
    logits = oracle.gate_logits(layer.x, layer.Wg, layer.gate_bias)
    b = mm.StepBuffers(cfg)
    b.logits.copy_(torch.from_numpy(logits))
    mm.layer_step(b, dl.x, dl.Wg, dl.gate_bias, torch.full((cfg.T,), 2.0, device="cuda"), dl.table, dl.shared, logits_given=True)
    mm.fallback_step(b, dl.x, dl.conf, dl.table)
    torch.cuda.synchronize()
    ref = run_oracle_layer(layer, logits=logits)
    assert rel_err(out_to_f64(b.out), ref["out"]) <= TOL_OUT


def test_gate_up_on_tiles_of_a_full_size_step():
    cfg = wl.CONFIGS["fine60_decode"].with_(T=200)
    assert _gate_up(cfg) == TILES and _gate_up(cfg, False) == STREAMED
    layer = wl.make_layer(cfg, seed=3)
    dl = DeviceLayer(layer)
    logits = oracle.gate_logits(layer.x, layer.Wg, layer.gate_bias)
    b = run_gpu_layer(dl, logits=logits)
    tokens = np.random.default_rng(3).choice(cfg.T, 24, replace=False)
    tokens[:3] = 0, 128, 199                  # both blocks of 128 rows and their ends
    ref = run_oracle_layer(layer, logits=logits, tokens=tokens)
    assert rel_err(out_to_f64(b.out)[tokens], ref["out"]) <= TOL_OUT
