"""Edges of the kernels' tiles, remainders and dispatch rules, against plain torch or the oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2510_12357_amd import binding as mm

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
