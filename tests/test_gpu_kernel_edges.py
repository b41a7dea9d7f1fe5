"""Edges of the kernels' tiles, remainders and dispatch rules, against plain torch or the oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2510_12357_amd import binding as mm
from paper_2510_12357_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [1, 3, 5, 1021, 8191, 8192, 8193, 32768, 40007])
def test_confidence_row_edges(V):
    """Row lengths around the 16-byte loads, one batch of loads and the two workgroup sizes; with
    odd V the rows start at every alignment.  A sum of exponentials below 1 added up in chains of at
    most V / 4096 + 64 terms, each off by a few 2^-24: 4e-6 covers V = 40007 with the exponentials' own error."""
    T = 5
    z = torch.randn((T, V), generator=torch.Generator().manual_seed(V)) * 3.0
    z[1, V // 2] += 16.0
    z[2] = -math.inf
    z[2, V - 1] = -1000.0                      # one possible value: probability 1
    z[3] = torch.finfo(torch.float32).min      # a fully masked row: uniform
    z[4, 0] = math.nan
    conf = torch.empty((T,), dtype=torch.float32, device="cuda")
    mm.moe_token_confidence(z.cuda(), T, V, conf)
    got = conf.cpu().numpy().astype(np.float64)
    ref = oracle.token_confidence(z[:2].numpy())
    assert np.all(np.abs(got[:2] / ref - 1.0) <= 4e-6)
    assert got[2] == 1.0 and abs(got[3] * V - 1.0) <= 4e-6 and np.isnan(got[4])


@pytest.mark.parametrize("V", [1000, 1001, 8192, 8193, 20000, 36864])
def test_confidence_of_short_rows_has_the_exponentials_full_precision(V):
    """Rows of one value d below the largest, d = 6 .. 10 in steps of 2^-7: the differences are exact, and the
    exponential of d, times up to 0.99 of the sum, is all that rounds much: within one unit in the last
    place, 2^-23 / sqrt 3 = 6.9e-8 in the mean square, with 3.4e-8 for the additions 7.7e-8.  A product
    d log2 e rounded once instead is off by up to 3.3e-7 by itself (1.0e-7 .. 2.0e-7 in the mean square)."""
    T = 512
    d = 6.0 + torch.arange(T, device="cuda") / 128.0
    z = (-d[:, None]).expand(T, V).contiguous()
    z[:, V // 2] = 0.0
    conf = torch.empty((T,), dtype=torch.float32, device="cuda")
    mm.moe_token_confidence(z, T, V, conf)
    err = conf.double() * torch.exp(z.double()).sum(1) - 1.0
    assert err.pow(2).mean().sqrt().item() <= 8.5e-8


def _assigned_layer(counts, H, I, shared, seed):
    """A bf16 layer in which expert e gets counts[e] tokens (one expert per token), through given logits."""
    E, T = len(counts), sum(counts)
    cfg = wl.LayerConfig("edge", T=T, H=H, E=E, I=I, k_big=1, k_little=1, shared_I=shared)
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    x = rnd(T, H).bfloat16()
    experts = (rnd(E, 3 * H * I) * 0.05).bfloat16()
    sh = [(rnd(3 * H * i) * 0.05).bfloat16() for i in shared]
    of = torch.repeat_interleave(torch.arange(E), torch.tensor(counts))[torch.randperm(T, generator=torch.Generator().manual_seed(seed))]
    b = mm.StepBuffers(cfg)
    b.logits.fill_(0.0)
    b.logits[torch.arange(T), of.cuda()] = 4.0
    table = torch.tensor([w.data_ptr() for w in experts], dtype=torch.int64, device="cuda")
    return cfg, x, experts, sh, table, b


def _ffn32(w, H, I, x):
    w = w.float()
    a = x.float() @ w[:H * I].view(I, H).t()
    h = (a * torch.sigmoid(a) * (x.float() @ w[H * I:2 * H * I].view(I, H).t())).bfloat16().float()
    return h @ w[2 * H * I:].view(H, I).t()


STREAM, TILED, WIDE = 0, 1, 2                  # moe_profile_expert_ffn


def _run_on(kernel, variant, b, x, table, sh, routed=True, shared=True):
    b.y.fill_(7.0)
    if b.shared_out is not None:
        b.shared_out.fill_(7.0)
    mm.moe_profile_expert_ffn(b.c, kernel, variant, x, b.expert_offsets, b.sorted_token, table, sh, routed, shared, b.y,
                              b.shared_out, b.fws, b.fws_bytes)
    return b.y.clone(), None if b.shared_out is None else b.shared_out.clone()


def _check_assigned(counts, H, I, shared, kernel, variants):
    """Every variant of the kernel on the layer, against fp32 products; the results of the last."""
    cfg, x, experts, sh, table, b = _assigned_layer(counts, H, I, shared, seed=len(counts) * 7 + H)
    mm.layer_step(b, x, None, None, None, table, sh, logits_given=True)
    off, st = b.expert_offsets.tolist(), b.sorted_token.long()
    assert [off[e + 1] - off[e] for e in range(cfg.E)] == list(counts)
    ref = torch.cat([_ffn32(experts[e], H, I, x[st[off[e]:off[e + 1]]]) for e in range(cfg.E)])
    for variant in variants:
        y, out = _run_on(kernel, variant, b, x, table, sh)
        assert ((y - ref).abs().max() / ref.pow(2).mean().sqrt()).item() <= 2e-2, variant
        if shared:
            ref_sh = sum(_ffn32(w, H, i, x) for w, i in zip(sh, shared))
            assert ((out.sum(0) - ref_sh).abs().max() / ref_sh.pow(2).mean().sqrt()).item() <= 2e-2, variant
    return x, sh, table, b, y, out


@pytest.mark.parametrize("counts,H,I,shared", [
    ([0, 1, 40, 128, 129, 193, 257, 520, 900], 200, 264, ()),      # every tile shape, ragged K and N
    ([0, 1, 40, 128, 129, 193, 257, 520, 900], 64, 328, (72,)),    # one chunk of K, padded to the ring's length
    ([400, 512, 31, 450], 576, 128, (1512, 8)),                     # shared experts cut along K; whole tiles
    ([1300], 128, 40, ()),                                          # one group, fewer panels than XCDs
    ([0, 1, 40, 128, 129, 193, 257, 300] + [3] * 10, 200, 264, (1512,)),  # few rows beside a shared expert
    ([400] * 15 + [900, 1, 0], 64, 296, ()),                        # many experts
    ([300], 64, 40, (72, 2048)),                                    # fewer tiles than workgroups
])
def test_wide_tiles(counts, H, I, shared):
    """256 x 256 tiles against fp32 products of the same bf16 operands: the activations h round to
    bf16 on both sides, where fp32 sums in another order may fall to the neighbouring value (2^-8 of one of
    I terms), so rows agree far inside the bf16 bar of 2e-2 of the tensor's RMS.  Both orders of the tiles; and
    either kernel adds up a row's products in the same order, so every bit is that of the 128 x 256
    tiles."""
    x, sh, table, b, y, out = _check_assigned(counts, H, I, shared, WIDE, (0, 1))
    y1, out1 = _run_on(TILED, 0, b, x, table, sh)
    assert torch.equal(y, y1) and (out is None or torch.equal(out, out1))


def _counts(n, rows, rest):
    """n experts with `rows` tokens each but for those named in `rest`."""
    return [rest.get(e, rows) for e in range(n)]


@pytest.mark.parametrize("counts,H,I,shared,null", [
    # 66 groups: the shared experts' first, then experts without rows on both sides of a word of 64 groups
    (_counts(64, 9, {0: 0, 61: 0, 62: 0, 63: 200, 5: 130, 40: 65}), 64, 40, (1512, 1512), [30, 63]),
    (_counts(64, 212, {3: 0, 61: 1, 62: 500, 63: 300}), 64, 40, (72, 40), [62]),
    # 130 and 256 groups
    (_counts(130, 360, {0: 1500, 62: 33, 63: 0, 64: 0, 65: 700, 127: 0, 128: 900, 129: 129}), 64, 40, (), [127, 129]),
    (_counts(256, 370, {0: 0, 63: 0, 64: 1000, 127: 64, 128: 0, 191: 0, 192: 257, 254: 700, 255: 1}), 72, 136, (), [64, 254]),
])
def test_wide_tiles_of_many_groups(counts, H, I, shared, null):
    """More groups than a wave has lanes: the tile list's words of 64 groups, experts without rows at their
    ends, experts without weights (their rows of y stay as they are).  Bar and bits as for the wide tiles."""
    cfg, x, experts, sh, table, b = _assigned_layer(counts, H, I, shared, seed=len(counts))
    table[torch.tensor(null)] = 0
    mm.layer_step(b, x, None, None, None, table, sh, logits_given=True)
    off, st = b.expert_offsets.tolist(), b.sorted_token.long()
    assert [off[e + 1] - off[e] for e in range(cfg.E)] == list(counts)
    y, out = _run_on(WIDE, 0, b, x, table, sh)
    for e in range(cfg.E):
        got = y[off[e]:off[e + 1]]
        if e in null:
            assert bool((got == 7.0).all())
        elif counts[e]:
            ref = _ffn32(experts[e], H, I, x[st[off[e]:off[e + 1]]])
            assert ((got - ref).abs().max() / ref.pow(2).mean().sqrt()).item() <= 2e-2, e
    if shared:
        ref = sum(_ffn32(w, H, i, x) for w, i in zip(sh, shared))
        assert ((out.sum(0) - ref).abs().max() / ref.pow(2).mean().sqrt()).item() <= 2e-2
    for kernel, variant in ((WIDE, 1), (TILED, 0), (TILED, 1)):
        y1, out1 = _run_on(kernel, variant, b, x, table, sh)
        assert torch.equal(y, y1) and (out is None or torch.equal(out, out1)), (kernel, variant)


@pytest.mark.parametrize("counts,H,I,shared", [
    ([0, 1, 40, 128, 129, 193, 257, 300] + [3] * 10, 200, 264, (1512,)),
    ([400] * 15 + [900, 1, 0], 64, 296, ()),
    ([0, 1, 40, 128, 129, 193, 257, 520, 900], 64, 328, (72,)),
])
@pytest.mark.parametrize("kernel,variant", [(TILED, 0), (TILED, 1), (WIDE, 0), (WIDE, 1)])
def test_parts_of_a_step_have_the_bits_of_the_whole(counts, H, I, shared, kernel, variant):
    """The routed part alone (as a fallback pass or a wave of an offloaded layer calls it) and the shared
    experts alone: the bits of a whole step, and nothing of the other part is written."""
    cfg, x, experts, sh, table, b = _assigned_layer(counts, H, I, shared, seed=3)
    mm.layer_step(b, x, None, None, None, table, sh, logits_given=True)
    y, out = b.y.clone(), None if b.shared_out is None else b.shared_out.clone()
    y1, out1 = _run_on(kernel, variant, b, x, table, (), shared=False)
    assert torch.equal(y1, y) and (out1 is None or bool((out1 == 7.0).all()))
    if shared:
        y1, out1 = _run_on(kernel, variant, b, x, None, sh, routed=False)
        assert torch.equal(out1, out) and bool((y1 == 7.0).all())


@pytest.mark.parametrize("counts,H,I,shared", [
    ([0, 1, 40, 127, 128, 129, 1], 200, 264, ()),                  # one token tile per panel, and two
    ([90, 64, 128, 31], 72, 136, (264,)),                          # a shared expert of three token tiles
])
def test_tiled_bf16_weights_read_once(counts, H, I, shared):
    """Prefill with few rows per expert: panels of one token tile load their weights past the caches, the
    others through them; the bits are the same.  Bar as for the wide tiles."""
    x, sh, table, b, y, out = _check_assigned(counts, H, I, shared, TILED, (0, 1, 2, 3))
    y0, out0 = _run_on(TILED, 0, b, x, table, sh)
    assert torch.equal(y, y0) and (out is None or torch.equal(out, out0))


@pytest.mark.parametrize("counts,H,I,shared", [
    ([0, 1, 40, 127, 128, 129, 1], 200, 264, ()),                  # less than a round: half the width, with remainders
    ([20] * 40, 520, 1032, ()),                                    # 360 tiles of gate/up: two rounds of 256 CUs, narrower by a quarter
    ([9] * 30 + [0, 130], 264, 1160, (2056, 72)),                  # shared experts of several token tiles
    ([300, 1, 2], 72, 136, (264,)),
])
def test_tiles_that_fill_their_rounds(counts, H, I, shared):
    """Tiles narrower than the kernel's (variants 2 and 3): every column once, and the bits of full ones."""
    _check_assigned(counts, H, I, shared, TILED, (2, 3))
    cfg, x, experts, sh, table, b = _assigned_layer(counts, H, I, shared, seed=5)
    mm.layer_step(b, x, None, None, None, table, sh, logits_given=True)
    y0, out0 = _run_on(TILED, 0, b, x, table, sh)
    for variant in (2, 3):
        y, out = _run_on(TILED, variant, b, x, table, sh)
        assert torch.equal(y, y0) and (out is None or torch.equal(out, out0)), variant
        y, out = _run_on(TILED, variant, b, x, table, (), shared=False)
        assert torch.equal(y, y0) and (out is None or bool((out == 7.0).all())), variant


@pytest.mark.parametrize("counts,H,I,shared", [
    ([0, 1, 32, 33, 64, 65, 50], 200, 264, ()),                    # items of 64 token rows, their remainders
    ([16, 17, 48, 49], 1032, 72, (520,)),                          # several chunks of K; a shared expert of 130 rows
    ([65], 64, 40, ()),
])
def test_streamed_items_of_64_rows(counts, H, I, shared):
    """Steps of 65 .. 255 tokens: groups of more than 32 rows in items of 64, and of 32.  Bar as for the wide
    tiles."""
    _check_assigned(counts, H, I, shared, STREAM, (2, 1))


def _coded_layer(counts, H, I, shared, dtype):
    """_assigned_layer's selection with random weights of any stored format, all of them finite."""
    T, E = sum(counts), len(counts)
    cfg = wl.LayerConfig("edge", T=T, H=H, E=E, I=I, k_big=1, k_little=1, shared_I=tuple(shared), dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(T + H)

    def blob(i):
        n = 3 * H * i
        codes = torch.randint(0, 256, (n,), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)
        if dtype == "bf16":
            return (torch.randn(n, generator=g, device="cuda") * 0.05).to(torch.bfloat16)
        if dtype == "bf16w8":
            scale = torch.rand(2 * i + H, generator=g, device="cuda") * 1e-3
            return torch.cat([codes & 0xf7, scale.view(torch.uint8)])                      # no NaN codes
        return torch.cat([codes[:n // 2], torch.randint(117, 122, (n // 32,), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)])

    experts, sh = [blob(I) for _ in range(E)], [blob(i) for i in shared]
    table = torch.tensor([w.data_ptr() for w in experts], dtype=torch.int64, device="cuda")
    x = torch.randn(T, H, generator=g, device="cuda").to(torch.bfloat16)
    of = torch.repeat_interleave(torch.arange(E), torch.tensor(counts))[torch.randperm(T, generator=torch.Generator().manual_seed(T))]
    return cfg, experts, sh, table, x, of.cuda()


def _assigned_step(cfg, x, table, sh, of):
    """Buffers of a step whose token t goes to expert of[t]."""
    b = mm.StepBuffers(cfg)
    b.logits.fill_(0.0)
    b.logits[torch.arange(cfg.T), of] = 4.0
    mm.layer_step(b, x, None, None, None, table, sh, logits_given=True)
    return b


@pytest.mark.parametrize("dtype", ["bf16", "bf16w8", "bf16mx4"])
@pytest.mark.parametrize("counts,H,I,shared", [
    ([0, 1, 2, 16, 17, 43, 44, 64], 128, 384, ()),                 # blocks of token rows, their remainders; one k unit and less
    ([65, 0, 129, 1], 1152, 256, (640, 128)),                      # several blocks; K in parts of a unit; shared experts cut along K
    ([1], 2048, 128, (128,)),                                      # more waves than rows
    ([3] * 63 + [0, 2, 1, 4] + [0] * 133 + [5], 128, 128, ()),     # experts behind every word of 64 lanes
    ([30] * 8, 256, 16384, ()),                                    # more rounds than one
    ([1] * 255 + [0], 128, 4224, (256,)),                          # more panels in a workgroup than lanes in a wave
])
def test_streamed_by_waves(counts, H, I, shared, dtype):
    """Every wave with rows of its own: the bits of the kernel with loader waves, which the tests against the oracle
    cover, in y and in the shared experts' outputs; rows that belong to nobody stay as they are."""
    cfg, experts, sh, table, x, of = _coded_layer(counts, H, I, shared, dtype)
    b = _assigned_step(cfg, x, table, sh, of)
    for routed, with_shared in ((True, True), (True, False)) + (((False, True),) if shared else ()):
        y1, out1 = _run_on(STREAM, 1, b, x, table, sh, routed, with_shared)
        for variant in (4,) if dtype == "bf16" else (4, 5):
            y4, out4 = _run_on(STREAM, variant, b, x, table, sh, routed, with_shared)
            assert torch.isfinite(y1).all() and torch.equal(y1, y4) and (out1 is None or torch.equal(out1, out4))


@pytest.mark.parametrize("T,kernel,variants", [(16, STREAM, (1, 4, 5)), (256, STREAM, (4, 5)), (256, TILED, (0, 1))])
def test_every_code_of_8_bits(T, kernel, variants):
    """Widening is exact: one activation h0 other than zero meets each code once, so a column is h0 times its value in one fp32 product (or NaN)."""
    H, I = 256, 16
    cfg = wl.LayerConfig("codes", T=T, H=H, E=1, I=I, k_big=1, k_little=1, dtype="bf16w8")
    codes = torch.arange(256, dtype=torch.int32, device="cuda").to(torch.uint8)
    gate, down = torch.zeros(I, H, dtype=torch.uint8, device="cuda"), torch.zeros(H, I, dtype=torch.uint8, device="cuda")
    gate[0], down[:, 0] = 0x38, codes                              # 1.0
    scale = torch.cat([torch.full((2 * I,), 2.0 ** -7, device="cuda"), torch.ones(H, device="cuda")])
    blob = torch.cat([gate.flatten(), gate.flatten(), down.flatten(), scale.view(torch.uint8)])
    table = torch.tensor([blob.data_ptr()], dtype=torch.int64, device="cuda")
    x = torch.ones(T, H, dtype=torch.bfloat16, device="cuda")
    b = _assigned_step(cfg, x, table, [], torch.zeros(T, dtype=torch.int64, device="cuda"))
    value = codes.view(torch.float8_e4m3fn).float()
    for variant in variants:
        y, _ = _run_on(kernel, variant, b, x, table, [])
        assert torch.equal(torch.nan_to_num(y, 1e9), torch.nan_to_num(y[:, 0x38:0x39] * value, 1e9)) and y[0, 0x38] > 3, variant


@pytest.mark.parametrize("dtype", ["bf16w8", "bf16mx4"])
@pytest.mark.parametrize("counts,H,I,shared", [
    ([200, 0, 1, 55], 32, 96, ()),                                 # K within a line, a line ends in its middle
    ([31, 32, 33, 64, 96, 127], 128, 256, (288,)),                 # whole lines, one of them; every number of token blocks
    ([129, 257, 2], 160, 544, (64, 1056)),                         # several token tiles; last line of one chunk or less
    ([300], 640, 352, (32,)),
    ([9] * 30, 1056, 736, ()),                                     # several tiles per workgroup
])
def test_narrow_weights_in_whole_lines(dtype, counts, H, I, shared):
    """Variant 1 loads whole lines: every bit is that of chunk after chunk, which the fp32 oracle checks."""
    if dtype == "bf16mx4":                                         # multiples of 128: lines of two chunks and four
        H, I, shared = -(-H // 128) * 128, -(-I // 128) * 128, [-(-i // 128) * 128 for i in shared]
    cfg, experts, sh, table, x, of = _coded_layer(counts, H, I, shared, dtype)
    b = _assigned_step(cfg, x, table, sh, of)
    ref, ref_out = _run_on(TILED, 0, b, x, table, sh)
    assert torch.isfinite(ref).all()
    y, out = _run_on(TILED, 1, b, x, table, sh)
    assert torch.equal(y, ref) and (not shared or torch.equal(out, ref_out))


@pytest.mark.parametrize("dtype,T,E,I,shared", [
    ("bf16mx4", 900, 64, 1024, ()),                                # lines, tiles in contiguous ranges
    ("bf16w8", 800, 64, 1040, (1040,)),                            # chunks, tiles by rows
    ("bf16w8", 1500, 64, 1024, ()), ("bf16mx4", 550, 60, 1408, (5632,)),   # lines, by rows
])
def test_narrow_tiles_as_the_rules_take_them(dtype, T, E, I, shared):
    """Order of the tiles and pieces of the weights are chosen each by itself, which variants 0 and 1 are not: the public call
    has every bit of variant 0 (contiguous, chunk after chunk)."""
    H = 2048
    cfg = wl.LayerConfig("rules", T=T, H=H, E=E, I=I, k_big=8, k_little=4, shared_I=shared, dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(T)
    c = mm.make_config(cfg)

    def blob(i):
        b = torch.randint(0, 256, (mm.moe_expert_blob_bytes(c, i),), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)
        n = 3 * H * i
        if dtype == "bf16mx4":
            b[n // 2:] = torch.randint(118, 122, (n // 32,), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)
        else:
            b[:n] &= 0xF7                                          # no NaN
            b[n:] = torch.full((2 * i + H,), 2e-4, device="cuda").view(torch.uint8)
        return b
    experts = [blob(I) for _ in range(3)]                           # three different experts, over and over
    table = torch.tensor([experts[e % 3].data_ptr() for e in range(E)], dtype=torch.int64, device="cuda")
    sh = [blob(i) for i in shared]
    x = torch.randn((T, H), generator=g, device="cuda").bfloat16()
    conf = torch.rand((T,), generator=g, device="cuda")
    b = mm.StepBuffers(cfg)
    b.logits.copy_(torch.randn((T, E), generator=g, device="cuda") * 1.5)
    mm.layer_step(b, x, None, None, conf, table, sh, logits_given=True)
    P = int(b.expert_offsets[-1])
    y, out = b.y[:P].clone(), None if b.shared_out is None else b.shared_out.clone()
    y0, out0 = _run_on(TILED, 0, b, x, table, sh)
    assert torch.isfinite(y).all() and torch.equal(y, y0[:P]) and (out is None or torch.equal(out, out0))


@pytest.mark.parametrize("dtype,counts,H,I,shared", [
    ("bf16", [5, 0, 20, 17, 1], 200, 264, ()),                     # K ends inside a unit of 256 bytes; quads that the waves do not divide
    ("bf16", [30, 2, 64, 65], 1032, 72, (520,)),                   # gate rows that end inside a tile; K in parts of a unit
    ("bf16", [1, 3], 136, 1480, (8,)),
    ("bf16w8", [5, 0, 20, 17, 1], 208, 272, ()),
    ("bf16w8", [30, 2, 64, 65], 1040, 80, (528, 48)),
    ("bf16w8", [1, 3], 144, 1488, (16,)),
    ("bf16w8", [43, 44, 0, 130, 66], 272, 336, (208,)),            # 256 tokens and more
    ("bf16w8", [260, 1, 3], 1040, 48, ()),
    ("bf16", [60, 66, 0, 130, 9], 200, 264, (1032,)),
    ("bf16", [300, 2], 72, 520, ()),
])
def test_streamed_by_waves_ragged(dtype, counts, H, I, shared):
    """Rows and columns of any size that the layer may have: the bits of the kernel that such a step has otherwise."""
    cfg, experts, sh, table, x, of = _coded_layer(counts, H, I, shared, dtype)
    b = _assigned_step(cfg, x, table, sh, of)
    ref, ref_out = _run_on(*((STREAM, 1) if cfg.T < 256 else (TILED, 0)), b, x, table, sh)
    assert torch.isfinite(ref).all()
    for variant in (4,) if dtype == "bf16" else (4, 5):
        y, out = _run_on(STREAM, variant, b, x, table, sh)
        assert torch.equal(y, ref) and (not shared or torch.equal(out, ref_out)), variant


@pytest.mark.parametrize("counts,H,I,shared", [
    ([0, 1, 32, 33, 64, 65, 50], 200, 264, ()),
    ([1, 127, 0, 1, 126], 1032, 72, (520,)),                       # 255 tokens: a shared expert of two row blocks
    ([129], 64, 40, (128, 72)),
])
def test_streamed_with_gate_up_on_tiles(counts, H, I, shared):
    """Gate/up on tiles of 128 token rows, the down projection streamed, fewer than 256 tokens.  Bar as for the wide tiles, and
    the bits of the streaming kernel."""
    x, sh, table, b, y, out = _check_assigned(counts, H, I, shared, STREAM, (6,))
    y1, out1 = _run_on(STREAM, 1, b, x, table, sh)
    assert torch.equal(y, y1) and (out is None or torch.equal(out, out1))


@pytest.mark.parametrize("dtype", ["bf16", "bf16w8", "bf16mx4"])
@pytest.mark.parametrize("counts,H,I,shared", [
    ([0, 1, 43, 44, 64, 65, 129, 200], 128, 384, ()),              # blocks of token rows, their remainders
    ([256, 0, 1], 1152, 256, (640, 128)),                          # more shared rows than a byte numbers; K in parts of a unit
    ([1] * 253 + [3, 0, 0], 256, 128, (128,)),                     # four groups of experts to look through
    ([300, 2400], 128, 4224, (256,)),                              # blocks of one expert in several rounds; many panels in a workgroup
])
def test_prefill_streamed_by_waves(counts, H, I, shared, dtype):
    """Steps of 256 tokens and more, one and two tiles of rows per wave: the bits of the tiled kernel, which the tests against
    the oracle cover; rows of the part not asked for stay as they are."""
    cfg, experts, sh, table, x, of = _coded_layer(counts, H, I, shared, dtype)
    b = _assigned_step(cfg, x, table, sh, of)
    ref, ref_out = _run_on(TILED, 0, b, x, table, sh)
    assert torch.isfinite(ref).all()
    for variant in (4,) if dtype == "bf16" else (4, 5):
        y, out = _run_on(STREAM, variant, b, x, table, sh)
        assert torch.equal(y, ref) and (not shared or torch.equal(out, ref_out)), variant
        y, out = _run_on(STREAM, variant, b, x, table, sh, shared=False)
        assert torch.equal(y, ref) and (out is None or bool((out == 7.0).all())), variant
        if shared:
            y, out = _run_on(STREAM, variant, b, x, table, sh, routed=False)
            assert torch.equal(out, ref_out) and bool((y == 7.0).all()), variant


@pytest.mark.parametrize("counts,H,I,shared,dtype", [
    ([32] * 8, 512, 512, (512,), "bf16w8"),                        # whole on panels, the shared expert alone on tiles
    ([32] * 8, 512, 512, (512,), "bf16mx4"),
    ([13] * 20 + [1, 0, 70, 40], 528, 272, (992, 48), "bf16w8"),
    ([3] * 50 + [5] * 10, 2048, 1408, (5632,), "bf16"),            # whole with gate/up on tiles, in parts streamed
])
def test_parts_through_the_rules_have_the_bits_of_the_whole(counts, H, I, shared, dtype):
    """A step issued in parts (shared experts on a stream of their own, an offloaded layer's waves) on whatever kernels the
    rules pick for them."""
    cfg, experts, sh, table, x, of = _coded_layer(counts, H, I, shared, dtype)
    b = _assigned_step(cfg, x, table, sh, of)

    def run(routed, with_shared):
        b.y.fill_(7.0)
        b.shared_out.fill_(7.0)
        mm.moe_expert_ffn(b.c, x, b.expert_offsets, b.sorted_token, table, sh, routed, with_shared, b.y, b.shared_out, b.fws, b.fws_bytes)
        return b.y.clone(), b.shared_out.clone()
    y, out = run(True, True)
    assert torch.isfinite(y).all() and torch.equal(run(True, False)[0], y) and torch.equal(run(False, True)[1], out)


@pytest.mark.parametrize("counts,H,I,shared,dtype", [
    ([3] * 40 + [4] * 20, 2048, 1408, (5632,), "bf16"),            # 200 tokens: whole with gate/up on tiles
    ([15] * 20, 512, 512, (512, 256), "bf16w8"),                   # 300 tokens: whole on panels
])
def test_side_stream_step_has_the_bits_of_the_whole(counts, H, I, shared, dtype):
    """The shared experts on a stream of their own, through layer_step."""
    cfg, experts, sh, table, x, of = _coded_layer(counts, H, I, shared, dtype)
    whole = _assigned_step(cfg, x, table, sh, of)
    b, side = mm.StepBuffers(cfg), torch.cuda.Stream()
    b.logits.copy_(whole.logits)
    torch.cuda.synchronize()
    for _ in range(2):
        mm.layer_step(b, x, None, None, None, table, sh, logits_given=True, side_stream=side)
    torch.cuda.synchronize()
    assert torch.equal(b.out.view(torch.int16), whole.out.view(torch.int16))


@pytest.mark.parametrize("counts,H,I", [
    ([0, 5, 128, 129, 1, 40, 64, 33], 256, 384),                   # few rows per expert
    ([300, 0, 290, 400], 128, 256),                                # many rows per expert
    ([1] * 200 + [100], 128, 128),                                 # more groups than a wave has lanes
])
def test_tiled_mxfp4_orders(counts, H, I):
    """Prefill with MXFP4 experts in both tile orders, against fp32 products with the dequantised
    weights (the kernel widens code x scale exactly); bar as for the wide tiles."""
    E, T = len(counts), sum(counts)
    assert T >= 256
    g = torch.Generator(device="cuda").manual_seed(T)
    n = 3 * H * I
    codes = torch.randint(0, 256, (E, n // 2), generator=g, device="cuda").to(torch.uint8)
    scales = torch.randint(117, 122, (E, n // 32), generator=g, device="cuda").to(torch.uint8)
    grid = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6], device="cuda")
    grid = torch.cat([grid, -grid])
    dense = torch.stack([grid[(codes & 15).long()], grid[(codes >> 4).long()]], dim=2).view(E, n // 32, 32)
    dense = (dense * torch.exp2(scales.float() - 127.0)[..., None]).view(E, n)
    cfg, x, _, _, _, b = _assigned_layer(counts, H, I, (), seed=T)
    cfg = cfg.with_(dtype="bf16mx4")
    blob = torch.cat([codes, scales], dim=1)
    table = torch.tensor([w.data_ptr() for w in blob], dtype=torch.int64, device="cuda")
    logits = b.logits
    b = mm.StepBuffers(cfg)
    b.logits.copy_(logits)
    mm.layer_step(b, x, None, None, None, table, [], logits_given=True)
    off, st = b.expert_offsets.tolist(), b.sorted_token.long()
    ref = torch.cat([_ffn32(dense[e], H, I, x[st[off[e]:off[e + 1]]]) for e in range(E)])
    y, _ = _run_on(TILED, 0, b, x, table, [])
    assert ((y - ref).abs().max() / ref.pow(2).mean().sqrt()).item() <= 2e-2
    assert torch.equal(y, _run_on(TILED, 1, b, x, table, [])[0])


@pytest.mark.parametrize("T,E,K", [(1, 1, 1), (63, 5, 3), (64, 60, 4), (65, 256, 16), (255, 7, 7), (256, 256, 16),
                                   (257, 64, 8), (300, 256, 16), (1024, 9, 2)])
@pytest.mark.parametrize("j_lo", [0, 1])
def test_dispatch_masks(T, E, K, j_lo):
    """Edges of the token masks (64 tokens a word), of the two shapes and of the thread-to-pair
    mapping, against a sort of the pairs; k_t from 0 to K."""
    rng = np.random.default_rng(T * 1000 + E)
    cfg = wl.LayerConfig("edge", T=T, H=64, E=E, I=64, k_big=K, k_little=1)
    idx = np.stack([rng.permutation(E)[:K] for _ in range(T)]).astype(np.int32)
    k_t = rng.integers(0, K + 1, T).astype(np.int32)
    idx[np.arange(K)[None, :] >= k_t[:, None]] = -1
    b = mm.StepBuffers(cfg)
    b.topk_idx.copy_(torch.from_numpy(idx))
    b.k_t.copy_(torch.from_numpy(k_t))
    mm.moe_dispatch_from(b.c, b.topk_idx, b.k_t, j_lo, b.expert_offsets, b.sorted_token, b.sorted_rank, b.inv_pos,
                         b.dws, b.dws_bytes)
    pairs = sorted((idx[t, j], t, j) for t in range(T) for j in range(j_lo, k_t[t]))
    off = np.searchsorted([p[0] for p in pairs], np.arange(E + 1)).astype(np.int32)
    tok, rank = np.full(T * K, -1, np.int32), np.full(T * K, -1, np.int32)
    inv = np.full((T, K), -1, np.int32)
    for p, (_, t, j) in enumerate(pairs):
        tok[p], rank[p], inv[t, j] = t, j, p
    assert np.array_equal(b.expert_offsets.cpu().numpy(), off)
    assert np.array_equal(b.sorted_token.cpu().numpy(), tok) and np.array_equal(b.sorted_rank.cpu().numpy(), rank)
    assert np.array_equal(b.inv_pos.cpu().numpy(), inv)


# ------------------------------------------------------------------ router
@pytest.mark.parametrize("E", [1, 63, 64, 65, 128, 129, 256])
def test_selection_with_ties_in_every_set_of_64_experts(E):
    """A round takes the first set bit of a ballot per 64 experts: equal logits within a set, across sets and in
    all of a row, and rows that run out of numbers."""
    K, T = min(E, 16), 9
    g = np.random.default_rng(E)
    z = np.round(g.standard_normal((T, E)) * 2).astype(np.float32)      # few distinct values: ties everywhere
    z[1] = 0.25
    z[2] = -np.inf
    z[3] = np.nan
    z[4, :] = -np.inf
    z[4, E - 1] = 1.0
    z[5, E // 2:] = np.nan
    cfg = wl.LayerConfig("r", T=T, H=8, E=E, I=8, k_big=K, k_little=1)
    b = mm.StepBuffers(cfg)
    b.logits.copy_(torch.from_numpy(z))
    mm.moe_route(b.c, None, None, None, None, b.logits, True, b.topk_idx, b.topk_w, b.important, b.k_t)
    torch.cuda.synchronize()
    idx, w, _, _ = oracle.route(z, None, cfg.gamma, K, 1, False)
    assert np.array_equal(b.topk_idx.cpu().numpy(), idx)
    assert np.abs(b.topk_w.cpu().numpy() - w).max() <= 2e-6


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,E,H", [(257, 1, 8), (257, 10, 40), (300, 16, 264), (1030, 17, 128), (272, 64, 136), (1100, 64, 2048), (4097, 33, 72),
                                   (258, 256, 520), (600, 133, 4104)])
def test_router_logits_of_many_tokens(dtype, T, E, H):
    """Tiles of 16 or 32 tokens and experts, k-steps left over, and a last one that is not full.  Products of bf16 are exact
    in fp32 and a sum of H terms in any order is off by at most H 2^-24 times the sum of their magnitudes (fp32: one rounding more)."""
    cfg = wl.LayerConfig("g", T=T, H=H, E=E, I=8, k_big=1, k_little=1, dtype=dtype, gate_std=0.1, gate_bias_std=1.0)
    layer = wl.make_layer(cfg, seed=T + E, experts=False)
    x, Wg = mm.to_device(layer.x, cfg), mm.to_device(layer.Wg, cfg)
    b = mm.StepBuffers(cfg)
    mm.moe_route(b.c, x, Wg, torch.from_numpy(layer.gate_bias).cuda(), None, b.logits, False, b.topk_idx, b.topk_w, b.important, b.k_t)
    x, Wg, bias = x.double().cpu(), Wg.double().cpu(), torch.from_numpy(layer.gate_bias).double()
    bound = (H + 2) * 2.0 ** -24 * (x.abs() @ Wg.abs().t() + bias.abs())
    assert bool(((b.logits.double().cpu() - (x @ Wg.t() + bias)).abs() <= bound).all())
    idx, _, _, _ = oracle.route(b.logits.cpu().numpy(), None, cfg.gamma, 1, 1, False)
    assert np.array_equal(b.topk_idx.cpu().numpy(), idx)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,E,H", [(4097, 1, 8), (4112, 16, 264), (4129, 9, 2048)])
def test_router_logits_of_many_tokens_and_few_experts(dtype, T, E, H):
    """Tiles of 32 tokens x 16 experts: more than 4096 tokens on 256 CUs, a last tile of 1 or 16 tokens."""
    test_router_logits_of_many_tokens(dtype, T, E, H)


# ------------------------------------------------------------------ a step in one call
@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("T,E,K,kl,I,shared", [(1, 8, 2, 1, 64, ()), (256, 60, 4, 2, 64, (72,)), (257, 1, 1, 1, 8, ()), (300, 64, 8, 4, 72, (64, 40)),
                                               (300, 256, 1, 1, 8, ()), (1111, 200, 3, 2, 40, ()), (2049, 7, 7, 3, 16, ())])
def test_step_in_one_call_equals_the_separate_calls(T, E, K, kl, I, shared, given):
    """Above 256 tokens the selection counts for the dispatch, while the table is small (1111 tokens, 200 experts: it is not) and fits the
    activations' workspace (300 tokens, 256 experts of 8: it does not).  Every output array is the same."""
    cfg = wl.LayerConfig("one", T=T, H=64, E=E, I=I, k_big=K, k_little=kl, shared_I=shared, gate_std=0.3, gate_bias_std=1.0,
                         w_std=0.1, fallback_ratio=0.4)
    layer = wl.make_layer(cfg, seed=T + E)
    x, Wg = mm.to_device(layer.x, cfg), mm.to_device(layer.Wg, cfg)
    bias, conf = torch.from_numpy(layer.gate_bias).cuda(), torch.from_numpy(layer.conf).cuda()
    experts = torch.stack([mm.to_device(e, cfg) for e in layer.expert_w])
    table = torch.tensor([e.data_ptr() for e in experts], dtype=torch.int64, device="cuda")
    sh = [mm.to_device(s, cfg) for s in layer.shared_w]
    b1, b2 = mm.StepBuffers(cfg), mm.StepBuffers(cfg)
    for b in (b1, b2):
        b.fws.fill_(0x5A)                                          # whatever the last step left there
        if given:
            b.logits.copy_(torch.from_numpy(oracle.gate_logits(layer.x, layer.Wg, layer.gate_bias)))
    arrays = ("logits", "topk_idx", "topk_w", "important", "k_t", "expert_offsets", "sorted_token", "sorted_rank", "inv_pos", "out")
    b = b2
    mm.layer_step(b1, x, Wg, bias, conf, table, sh, logits_given=given)
    mm.moe_route(b.c, x, Wg, bias, conf, b.logits, given, b.topk_idx, b.topk_w, b.important, b.k_t)
    mm.moe_dispatch(b.c, b.topk_idx, b.k_t, b.expert_offsets, b.sorted_token, b.sorted_rank, b.inv_pos, b.dws, b.dws_bytes)
    mm.moe_expert_ffn(b.c, x, b.expert_offsets, b.sorted_token, table, sh, True, True, b.y, b.shared_out, b.fws, b.fws_bytes)
    mm.moe_combine(b.c, b.y, b.topk_w, b.inv_pos, b.k_t, b.shared_out, b.out)
    assert [n for n in arrays if not torch.equal(getattr(b1, n), getattr(b2, n))] == []
    # the second pass, here on top of a mixed step: the same calls on both sides
    mm.fallback_step(b1, x, conf, table)
    mm.moe_route(b.c, x, None, None, conf, b.logits, True, b.topk_idx, b.topk_w, b.important, b.k_t)
    mm.moe_dispatch_from(b.c, b.topk_idx, b.k_t, kl, b.expert_offsets, b.sorted_token, b.sorted_rank, b.inv_pos, b.dws, b.dws_bytes)
    mm.moe_expert_ffn(b.c, x, b.expert_offsets, b.sorted_token, table, (), True, False, b.y, b.shared_out, b.fws, b.fws_bytes)
    mm.moe_combine_add(b.c, b.y, b.topk_w, b.inv_pos, b.k_t, kl, b.out)
    assert [n for n in arrays if not torch.equal(getattr(b1, n), getattr(b2, n))] == []


@pytest.mark.parametrize("T,E", [(512, 256), (513, 256), (1024, 128), (655, 200), (8192, 16), (8193, 16)])
def test_step_in_one_call_with_many_tokens_or_experts(T, E):
    """The largest steps whose selection counts, and steps just above them: every output array of the separate calls."""
    test_step_in_one_call_equals_the_separate_calls(T, E, 8, 4, 16, (), False)


@pytest.mark.parametrize("dtype,T,E,K,kl,H,I,shared", [
    ("bf16mx4", 8, 200, 16, 8, 1024, 384, (128,)), ("bf16mx4", 63, 256, 3, 1, 512, 640, ()), ("bf16mx4", 64, 200, 8, 4, 1024, 384, ()),
    ("bf16mx4", 65, 200, 16, 8, 1024, 384, (128, 256)), ("bf16mx4", 255, 200, 16, 8, 1024, 384, (128,)),
    ("bf16", 1, 60, 4, 2, 2048, 1408, (5632,)), ("bf16", 33, 60, 4, 2, 2048, 1408, (5632,)), ("bf16", 64, 60, 4, 2, 2048, 1408, (5632,)),
    ("bf16w8", 1, 40, 4, 2, 1024, 2064, (48,)), ("bf16w8", 64, 40, 8, 3, 1024, 2064, (48,)), ("bf16w8", 130, 65, 8, 4, 1040, 1040, ()), ("bf16w8", 255, 40, 2, 1, 1024, 2064, (48,))])
def test_dispatch_built_by_the_gate_up_launch(dtype, T, E, K, kl, H, I, shared):
    """Steps in panels below 256 tokens: one, two and eight pairs per thread, one to four words of a token mask, all sets of 64
    experts, an expert without weights; the pass and its fallback pass have every array and every bit of the separate calls."""
    cfg = wl.LayerConfig("fold", T=T, H=H, E=E, I=I, k_big=K, k_little=kl, shared_I=shared, dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(T + E)
    c = mm.make_config(cfg)

    def blob(i):
        n = mm.moe_expert_blob_bytes(c, i)
        b = torch.randint(0, 256, (n,), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)
        w = 3 * H * i
        if dtype == "bf16":
            return (torch.randn((w,), generator=g, device="cuda") * 0.02).bfloat16()
        if dtype == "bf16mx4":
            b[w // 2:] = torch.randint(118, 122, (n - w // 2,), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)
        else:
            b[:w] = (torch.randn((w,), generator=g, device="cuda") * 50).to(torch.float8_e4m3fn).view(torch.uint8)
            b[w:] = torch.full(((n - w) // 4,), 4e-4, device="cuda").view(torch.uint8)
        return b
    one = [blob(I) for _ in range(3)]                               # three different experts, over and over
    table = torch.tensor([one[e % 3].data_ptr() for e in range(E)], dtype=torch.int64, device="cuda")
    table[E // 2] = 0
    sh = [blob(i) for i in shared]
    x = torch.randn((T, H), generator=g, device="cuda").bfloat16()
    Wg = (torch.randn((E, H), generator=g, device="cuda") * 0.05).bfloat16()
    conf = torch.rand((T,), generator=g, device="cuda")
    b1, b = mm.StepBuffers(cfg), mm.StepBuffers(cfg)
    arrays = ("logits", "topk_idx", "topk_w", "important", "k_t", "expert_offsets", "sorted_token", "sorted_rank", "inv_pos", "out")

    def same():
        P = int(b.expert_offsets[-1])
        return [n for n in arrays if not torch.equal(getattr(b1, n), getattr(b, n))] == [] and torch.equal(b1.y[:P], b.y[:P])
    mm.layer_step(b1, x, Wg, None, conf, table, sh)
    mm.moe_route(b.c, x, Wg, None, conf, b.logits, False, b.topk_idx, b.topk_w, b.important, b.k_t)
    mm.moe_dispatch(b.c, b.topk_idx, b.k_t, b.expert_offsets, b.sorted_token, b.sorted_rank, b.inv_pos, b.dws, b.dws_bytes)
    mm.moe_expert_ffn(b.c, x, b.expert_offsets, b.sorted_token, table, sh, True, True, b.y, b.shared_out, b.fws, b.fws_bytes)
    mm.moe_combine(b.c, b.y, b.topk_w, b.inv_pos, b.k_t, b.shared_out, b.out)
    assert same() and bool(b.out.isfinite().all()) and b.out.float().abs().max() > 0
    if b1.lws is not None:                                          # the decode call takes the same launches
        for n in arrays + ("y",):
            getattr(b1, n).zero_()
        mm.layer_decode_step(b1, x, Wg, None, conf, table, sh)
        assert same() and mm.moe_layer_decode_status(b1.lws) == 0
    for a in (b1, b):
        a.fws.fill_(0x5A)
    mm.fallback_step(b1, x, conf, table)
    mm.moe_route(b.c, x, None, None, conf, b.logits, True, b.topk_idx, b.topk_w, b.important, b.k_t)
    mm.moe_dispatch_from(b.c, b.topk_idx, b.k_t, kl, b.expert_offsets, b.sorted_token, b.sorted_rank, b.inv_pos, b.dws, b.dws_bytes)
    mm.moe_expert_ffn(b.c, x, b.expert_offsets, b.sorted_token, table, (), True, False, b.y, b.shared_out, b.fws, b.fws_bytes)
    mm.moe_combine_add(b.c, b.y, b.topk_w, b.inv_pos, b.k_t, kl, b.out)
    assert same()
