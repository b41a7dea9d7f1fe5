"""Performance cases: what a user of the library has it do, through its public entry points.

One pass of a case is one step of one MoE layer (or one call of the confidence test), with the
weights, buffers and tables that a serving program keeps already on the device.  The layer shapes
are the package's own (``workloads.CONFIGS``); weights, activations and confidences have the
distributions of the package's synthetic workloads and are made on the GPU from the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2510_12357_amd import binding as mm
from paper_2510_12357_amd import workloads as wl

LAYERS = {"fine60": "fine60_decode", "fine64": "fine64_prefill", "shared2": "shared2_offload",
          "coarse8": "coarse8", "tiny": "tiny_fp32"}
CACHE_SLOTS = 16                       # HBM slots of the offloaded layer (a quarter of its experts)
WEIGHT_BYTES = {"fp32": 4, "bf16": 2, "bf16w8": 1, "bf16mx4": 0.5 + 1.0 / 32}


def listed():
    return [
        # One sequence generating: a single token through the 60-expert layer, latency only.
        _case("decode_b1", "decode", "fine60", 1),
        # A small decode batch, still through the one-launch step.
        _case("decode_b8", "decode", "fine60", 8),
        # The ordinary decode batch of a server: nearly every expert is touched once.
        _case("decode_b64", "step", "fine60", 64),
        # The same batch with 4-bit experts, the way to fit more layers and to read fewer bytes.
        _case("decode_b64_mxfp4", "step", "fine60", 64, "bf16mx4"),
        # A mixed batch: a short prompt chunk together with running sequences.
        _case("chunk_t200", "step", "fine60", 200),
        # Alg. 1 at layer level on a ragged batch: little pass, then the fallback pass.
        _case("two_pass_b33", "two_pass", "fine60", 33),
        # Prefill of many small experts with skewed loads (ordinary prompt).
        _case("prefill_fine64_t2048", "step", "fine64", 2048),
        # A ragged prompt with 8-bit experts.
        _case("prefill_fine64_w8_t777", "step", "fine64", 777, "bf16w8"),
        # Prefill of few wide experts: the largest products of the range.
        _case("prefill_coarse8_t4096", "step", "coarse8", 4096),
        # A tiny fp32 layer (tests, small models): launches and latency.
        _case("tiny_fp32_t64", "step", "tiny", 64, "fp32"),
        # The confidence test of Alg. 1 on the output distributions of a decode batch.
        {"name": "confidence_b64", "kind": "confidence", "tokens": 64, "vocab": 131072},
        # The paper's own setting: experts in pinned host memory behind a small HBM cache.
        _case("offload_b16", "offload", "shared2", 16),
    ]


def _case(name, kind, layer, tokens, dtype="bf16", ratio=0.2):
    """ratio: the share of tokens that fall back to the big selection (the package's headline value)."""
    return {"name": name, "kind": kind, "layer": layer, "tokens": tokens, "dtype": dtype, "ratio": ratio}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["decode", "decode", "step_small", "step_small", "step_small", "step_large", "step_large",
                       "two_pass", "tiny", "confidence"])
    narrow = lambda: rng.choice(["bf16", "bf16", "bf16w8", "bf16mx4"])  # noqa: E731
    if what == "decode":
        c = _case("", "decode", rng.choice(["fine60", "fine60", "shared2"]), _log_int(rng, 1, 32))
    elif what == "step_small":
        c = _case("", "step", rng.choice(["fine60", "fine60", "fine64", "shared2", "coarse8"]), _log_int(rng, 1, 255), narrow())
    elif what == "step_large":
        layer = rng.choice(["fine60", "fine64", "fine64", "shared2", "coarse8"])
        c = _case("", "step", layer, _log_int(rng, 256, 4000 if layer == "coarse8" else 4096), narrow())
        if layer == "coarse8" and c["dtype"] != "bf16":      # wide narrow-format layers cost more than the listed ones
            c["tokens"] = _log_int(rng, 256, 3000)
    elif what == "two_pass":
        c = _case("", "two_pass", rng.choice(["fine60", "shared2"]), _log_int(rng, 1, 256))
    elif what == "tiny":
        c = _case("", "step", "tiny", _log_int(rng, 1, 512), "fp32")
    else:
        c = {"kind": "confidence", "tokens": _log_int(rng, 1, 128), "vocab": _log_int(rng, 1000, 160000)}
    c.pop("name", None)
    if "ratio" in c:
        c["ratio"] = round(rng.uniform(0.05, 0.5), 3)
    return c


def _config(case):
    return wl.CONFIGS[LAYERS[case["layer"]]].with_(T=case["tokens"], dtype=case["dtype"], fallback_ratio=case["ratio"])


# ------------------------------------------------------------------------------------ inputs
def _blob(g, cfg, I):
    """One expert blob on the device, in the layer's storage format."""
    n = 3 * cfg.H * I
    if cfg.dtype == "bf16mx4":
        codes = torch.randint(0, 256, (n // 2,), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)
        scales = torch.randint(118, 122, (n // 32,), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)
        return torch.cat([codes, scales])
    w = torch.randn((n,), generator=g, device="cuda", dtype=torch.float32) * cfg.w_std
    if cfg.dtype != "bf16w8":
        return w.to(torch.float32 if cfg.dtype == "fp32" else torch.bfloat16)
    codes, scales = [], []
    for m in _matrices(w, cfg.H, I):
        s = m.abs().amax(dim=1) / 448.0
        codes.append((m / s[:, None]).to(torch.float8_e4m3fn).view(torch.uint8).reshape(-1))
        scales.append(s)
    return torch.cat(codes + [torch.cat(scales).view(torch.uint8)])


def _matrices(w, H, I):
    n = H * I
    return w[:n].view(I, H), w[n:2 * n].view(I, H), w[2 * n:3 * n].view(H, I)


class _Inputs:
    """Everything random of a layer case; the same for `prepare` and `exact`."""

    def __init__(self, case, seed):
        cfg = self.cfg = _config(case)
        g = self.g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        dt = torch.float32 if cfg.dtype == "fp32" else torch.bfloat16

        def randn(shape, std):
            return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dt)

        self.x = randn((cfg.T, cfg.H), 1.0)
        self.Wg = randn((cfg.E, cfg.H), cfg.gate_std)
        self.bias = torch.randn((cfg.E,), generator=g, device="cuda") * cfg.gate_bias_std if cfg.gate_bias_std > 0 else None
        self.conf = torch.from_numpy(wl.make_confidence(seed, cfg.T, cfg.gamma, cfg.fallback_ratio)).cuda()
        self.shared = [_blob(g, cfg, i) for i in cfg.shared_I]
        first = _blob(g, cfg, cfg.I)
        offload = case["kind"] == "offload"
        self.experts = torch.empty((cfg.E, first.numel()), dtype=first.dtype, device="cpu" if offload else "cuda",
                                   pin_memory=offload)
        self.experts[0].copy_(first)
        for e in range(1, cfg.E):
            self.experts[e].copy_(_blob(g, cfg, cfg.I))


class _Cache:
    """The expert cache of an offloaded layer with the memory that it uses."""

    def __init__(self, cfg, experts):
        self.experts = experts
        self.slots = torch.zeros((CACHE_SLOTS, experts.shape[1]), dtype=experts.dtype, device="cuda")
        self.handle = mm.moe_cache_create(cfg.E, experts.shape[1] * experts.element_size(), CACHE_SLOTS, experts, self.slots)

    def __del__(self):
        handle = getattr(self, "handle", None)
        if handle:
            torch.cuda.synchronize()
            mm.moe_cache_sync(handle)
            mm.moe_cache_destroy(handle)


def _lm_logits(case, seed):
    """Output logits: noise, and for most rows one dominant entry (the fraction the package's own
    generator gives for the paper's fallback ratios)."""
    T, V = case["tokens"], case["vocab"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    z = torch.randn((T, V), generator=g, device="cuda", dtype=torch.float32) * 3.0
    confident = torch.rand((T,), generator=g, device="cuda") >= 0.2
    hot = torch.randint(0, V, (T,), generator=g, device="cuda")
    z[torch.arange(T, device="cuda"), hot] += 16.0 * confident
    return z


def prepare(case, seed):
    if case["kind"] == "confidence":
        z = _lm_logits(case, seed)
        return {"case": case, "z": z, "conf": torch.empty((case["tokens"],), dtype=torch.float32, device="cuda")}
    s = _Inputs(case, seed)
    state = {"case": case, "inputs": s, "buffers": mm.StepBuffers(s.cfg)}
    if case["kind"] == "offload":
        state["cache"] = _Cache(s.cfg, s.experts)
    else:
        step = s.experts.stride(0) * s.experts.element_size()
        state["table"] = torch.tensor([s.experts.data_ptr() + e * step for e in range(s.cfg.E)], dtype=torch.int64, device="cuda")
    if case["kind"] == "two_pass":       # a confidence above gamma for every token: the little pass
        state["never"] = torch.full((s.cfg.T,), float("inf"), dtype=torch.float32, device="cuda")
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "confidence":
        mm.moe_token_confidence(state["z"], case["tokens"], case["vocab"], state["conf"])
        return state["conf"]
    s, b = state["inputs"], state["buffers"]
    if case["kind"] == "decode":
        mm.layer_decode_step(b, s.x, s.Wg, s.bias, s.conf, state["table"], s.shared)
    elif case["kind"] == "step":
        mm.layer_step(b, s.x, s.Wg, s.bias, s.conf, state["table"], s.shared)
    elif case["kind"] == "two_pass":
        mm.layer_step(b, s.x, s.Wg, s.bias, state["never"], state["table"], s.shared)
        mm.fallback_step(b, s.x, s.conf, state["table"])
    else:
        mm.layer_step_cached(b, s.x, s.Wg, s.bias, s.conf, state["cache"].handle, s.shared)
    return {"out": b.out, "logits": b.logits, "topk_w": b.topk_w, "topk_idx": b.topk_idx}


# ------------------------------------------------------------------------------------ what a pass is
def work(case):
    if case["kind"] == "confidence":
        n = case["tokens"] * case["vocab"]
        return {"bytes": 4.0 * n + 4.0 * case["tokens"], "flops": 3.0 * n}
    # the experts that a batch touches, from a batch of random tokens with the layer's gate statistics
    cfg = _config(case)
    rng = np.random.default_rng(1)
    D = P = 0.0
    trials = 16
    for _ in range(trials):
        z = rng.standard_normal((cfg.T, cfg.E)) * cfg.gate_std * math.sqrt(cfg.H) + rng.standard_normal(cfg.E) * cfg.gate_bias_std
        k = np.where(rng.random(cfg.T) < cfg.fallback_ratio, cfg.k_big, cfg.k_little)
        order = np.argsort(-z, axis=1)[:, :cfg.k_big]
        D += len(np.unique(order[np.arange(cfg.k_big)[None, :] < k[:, None]])) / trials
        P += float(k.sum()) / trials
    eb, wb, H, T = (4 if cfg.dtype == "fp32" else 2), WEIGHT_BYTES[cfg.dtype], cfg.H, cfg.T
    shared = sum(cfg.shared_I)
    return {"bytes": wb * 3 * H * (D * cfg.I + shared) + eb * cfg.E * H + 2 * eb * T * H + 4 * T * cfg.E,
            "flops": 6.0 * H * (P * cfg.I + T * shared) + 2.0 * T * cfg.E * H}


def tolerance(case):
    if case["kind"] == "confidence":     # fp32 sums of up to 160000 exponentials in any order
        return {"rel": 6e-6, "max": 4e-5}
    if case["dtype"] == "fp32":
        return {"rel": 2e-6, "max": 4e-5, "differ": 1e-3}
    # bf16 activations between the products and a bf16 result, fp32 sums
    return {"rel": 1e-2, "max": 0.3, "differ": 1e-3}


# ------------------------------------------------------------------------------------ 64 bits
_E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


def _weights64(cfg, blob, I):
    """The three matrices of a blob in 64 bits."""
    n = 3 * cfg.H * I
    if cfg.dtype in ("bf16", "fp32"):
        return _matrices(blob.double(), cfg.H, I)
    if cfg.dtype == "bf16w8":
        scale = blob[n:].view(torch.float32).double()
        scale = (scale[:I], scale[I:2 * I], scale[2 * I:])
        return tuple(m * s[:, None] for m, s in zip(_matrices(blob[:n].view(torch.float8_e4m3fn).double(), cfg.H, I), scale))
    table = torch.tensor(_E2M1 + tuple(-v for v in _E2M1), dtype=torch.float64, device=blob.device)
    codes = torch.stack([blob[:n // 2] & 15, blob[:n // 2] >> 4], dim=1).reshape(-1)
    scale = torch.exp2(blob[n // 2:].double() - 127.0)
    return _matrices((table[codes.long()].view(-1, 32) * scale[:, None]).reshape(-1), cfg.H, I)


def _ffn64(cfg, blob, I, x):
    gate, up, down = _weights64(cfg, blob, I)
    a = x @ gate.t()
    return (a * torch.sigmoid(a) * (x @ up.t())) @ down.t()


def exact(case, seed):
    if case["kind"] == "confidence":
        z = _lm_logits(case, seed).double()
        return 1.0 / torch.exp(z - z.amax(dim=1, keepdim=True)).sum(dim=1)
    s = _Inputs(case, seed)
    cfg, x = s.cfg, s.x.double()
    logits = x @ s.Wg.double().t() + (0.0 if s.bias is None else s.bias.double())
    k = torch.where(s.conf > cfg.gamma, cfg.k_little, cfg.k_big)
    idx = torch.argsort(logits, dim=1, descending=True, stable=True)[:, :cfg.k_big]
    used = torch.arange(cfg.k_big, device="cuda")[None, :] < k[:, None]
    w = torch.softmax(logits, dim=1).gather(1, idx) * used
    if cfg.renorm:
        w = w / w.sum(dim=1, keepdim=True)
    out = torch.zeros_like(x)
    for e in range(cfg.E):
        t, j = torch.nonzero((idx == e) & used, as_tuple=True)
        if len(t):
            out[t] += w[t, j][:, None] * _ffn64(cfg, s.experts[e].cuda(), cfg.I, x[t])
    for blob, i in zip(s.shared, cfg.shared_I):
        out += _ffn64(cfg, blob, i, x)
    return {"out": out, "logits": logits, "topk_w": w, "topk_idx": None}
