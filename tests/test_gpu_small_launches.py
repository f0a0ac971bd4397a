"""Launches with fewer tiles (or bundles of rows) than the chip has wavefronts, and with a few more than it has compute
units: every row must be written once, whatever the split, and LayerNorm's vectors may start at any float."""

import numpy as np
import pytest
import torch

from fb4_inputs import DEFAULT_FORMATBOOK, synth
from oracle import fb4_oracle as O

pytestmark = pytest.mark.gpu

SHAPES = [(1, 32), (1, 2080), (3, 96), (255, 64), (256, 64), (257, 64), (255, 2048), (257, 2048), (300, 1152), (1025, 512)]


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_02883_amd as F
    return F


@pytest.mark.parametrize("selector,block,g", [(1, 32, 8), (1, 16, 8), (0, 32, 8), (1, 32, 32)])
def test_quantize_and_gelu(F, selector, block, g):
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    for rows, cols in SHAPES:
        x = synth.vdit_activation(rows=rows, cols=cols, seed=rows + cols, device="cuda")
        o = F.opts(block=block, selector=selector, num_groups=g)
        c, m = F.fb4_quantize(luts, o, x)
        torch.cuda.synchronize()
        cr, mr = O.quantize(DEFAULT_FORMATBOOK, synth.bf16_bits(x), block=block, selector=selector, num_groups=g)
        assert np.array_equal(c.cpu().numpy(), cr) and np.array_equal(m.cpu().numpy().view(np.uint16), mr), (rows, cols)
        if selector == 1 and g == 8:
            c, m = F.fb4_gelu_quantize(luts, o, x, 1)
            torch.cuda.synchronize()
            cr, mr = O.quantize(DEFAULT_FORMATBOOK, O.gelu(synth.bf16_bits(x), 1), block=block)
            assert np.array_equal(c.cpu().numpy(), cr) and np.array_equal(m.cpu().numpy().view(np.uint16), mr), (rows, cols)
    luts.free()


@pytest.mark.parametrize("rows,cols", SHAPES + [(5, 4128), (5, 8192), (5, 10240), (5, 12288), (700, 3072), (700, 6176)])
def test_layernorm(F, rows, cols):
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    x = synth.vdit_activation(rows=rows, cols=cols, seed=rows + cols, device="cuda")
    rng = np.random.default_rng(cols)
    for shift, with_gamma, with_beta in ((0, True, True), (1, True, True), (3, True, False), (2, False, True), (0, False, False)):
        # vectors that start 4, 8 and 12 bytes past a 16-byte boundary
        gamma = torch.from_numpy(rng.normal(1.0, 0.2, cols + 8).astype(np.float32)).cuda()[shift:shift + cols]
        beta = torch.from_numpy(rng.normal(0.0, 0.2, cols + 8).astype(np.float32)).cuda()[shift:shift + cols]
        y = torch.empty_like(x)
        c, m = F.fb4_layernorm_quantize(luts, F.opts(), x, gamma if with_gamma else None, beta if with_beta else None, 1e-6, y_out=y)
        torch.cuda.synchronize()
        gr = gamma.cpu().numpy() if with_gamma else np.ones(cols, dtype=np.float32)
        br = beta.cpu().numpy() if with_beta else np.zeros(cols, dtype=np.float32)
        yb = synth.bf16_bits(y)
        yr, _, _ = O.layernorm(synth.bf16_bits(x), gr, br, 1e-6)
        order = lambda b: np.where(b & 0x8000, -(b & 0x7FFF).astype(np.int64), (b & 0x7FFF).astype(np.int64))
        off = np.abs(order(yb) - order(yr))
        # within one bf16 step, except where gamma t and beta cancel (then within 2^-17 of terms of a few units)
        far = off > 1
        f = lambda b: (b.astype(np.uint32) << 16).view(np.float32)
        assert np.abs(f(yb)[far] - f(yr)[far]).max(initial=0.0) <= 2.0 ** -12 and far.mean() < 1e-3, (rows, cols, shift)
        cr, mr = O.quantize(DEFAULT_FORMATBOOK, yb)
        assert np.array_equal(c.cpu().numpy(), cr) and np.array_equal(m.cpu().numpy().view(np.uint16), mr), (rows, cols, shift)
    luts.free()
