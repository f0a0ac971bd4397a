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


def layernorm_bundles(rows, cols, num_groups):
    """The launcher's choice: (chunks per lane, rows per bundle, whether every wavefront gets one bundle at most)."""
    nb, cu = cols // 32, torch.cuda.get_device_properties(0).multi_processor_count
    fewest = (nb + 63) // 64
    threads = lambda b: 768 if b <= 4 and not (num_groups > 8 and b >= 2) else 512
    wavefronts = lambda b: cu * (threads(b) // 64)
    if fewest <= 4 and -(-rows // (64 * fewest // nb)) <= wavefronts(fewest):
        return fewest, min(64 * fewest // nb, rows), True
    best, B = 0.0, 0
    for b in range(fewest, 5):
        r = 64 * b // nb
        chunk = ((1, 1.2, 1.17, 1.18) if num_groups > 8 else (1, 1.05, 1.01, 1.08))[b - 1]
        cost = (b + 0.05 * r) * chunk * (-(-rows // r) + 0.45 * wavefronts(b))
        if B == 0 or cost < best:
            best, B = cost, b
    B = B or fewest
    return B, min(64 * B // nb, rows), -(-rows // (64 * B // nb)) <= wavefronts(B)


@pytest.mark.parametrize("block,g", [(32, 8), (16, 8), (32, 16), (16, 16)])
@pytest.mark.parametrize("rows,cols,chunks,rows_per_bundle", [(9001, 960, 1, 2), (6501, 1600, 1, 1), (3301, 4096, 2, 1), (16001, 1152, 3, 5), (30001, 1152, 3, 5),
                                                              (6501, 3072, 3, 2), (3100, 6176, 4, 1), (2100, 9216, 5, 1), (2101, 12288, 6, 1)])
def test_layernorm_of_more_bundles_than_wavefronts(F, rows, cols, chunks, rows_per_bundle, block, g):
    assert layernorm_bundles(rows, cols, g) == (chunks, rows_per_bundle, False)
    layernorm_against_two_steps(F, rows, cols, block, g)


# (with 16 groups, whose kernels run fewer wavefronts from two chunks on; the last four on the short side of both choices)
@pytest.mark.parametrize("block", [32, 16])
@pytest.mark.parametrize("rows,cols,g,bundles", [(25001, 768, 8, (2, 5, False)), (25001, 768, 16, (1, 2, False)),
                                                 (20001, 2400, 8, (3, 2, False)), (20001, 2400, 16, (4, 3, False)),
                                                 (6501, 1024, 8, (1, 2, False)), (6501, 1024, 16, (1, 2, False)),
                                                 (3300, 2048, 8, (1, 1, False)), (3300, 2048, 16, (1, 1, False))])
def test_layernorm_where_the_groups_decide_the_bundles(F, rows, cols, g, bundles, block):
    assert layernorm_bundles(rows, cols, g) == bundles
    layernorm_against_two_steps(F, rows, cols, block, g)


def layernorm_against_two_steps(F, rows, cols, block, g):
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    x = synth.vdit_activation(rows=rows, cols=cols, seed=cols, device="cuda")
    gamma, beta = synth.layernorm_affine(cols, seed=cols)
    y = torch.empty_like(x)
    o = F.opts(block=block, num_groups=g)
    c, m = F.fb4_layernorm_quantize(luts, o, x, torch.from_numpy(gamma).cuda(), torch.from_numpy(beta).cuda(), 1e-6, y_out=y)
    c0, m0 = F.fb4_quantize(luts, o, y)                       # (against the oracle in tests of its own)
    torch.cuda.synchronize()
    assert torch.equal(c, c0) and torch.equal(m, m0)
    assert_layernorm(x, y, gamma, beta)
    luts.free()


# Every number of chunks per lane with one bundle per wavefront and with several, whose chunks -- and their rows' groups -- are
# requested during the bundle before
LISTED = [(9001, 960, 1), (9001, 2048, 1), (1500, 4096, 2), (3301, 4096, 2), (25001, 768, 2), (6501, 3072, 3), (3301, 5120, 3), (20001, 2400, 3),
          (300, 8192, 4), (3100, 6176, 4), (20001, 2400, 4), (2100, 9216, 5), (5001, 10240, 5), (300, 12288, 6), (5001, 12288, 6)]


@pytest.mark.parametrize("two_stage", [False, True])
@pytest.mark.parametrize("block,g", [(32, 8), (16, 8), (32, 16), (16, 16)])
@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 5, 6])
def test_layernorm_with_lists_over_bundles(F, chunks, block, g, two_stage):
    shapes = [s for s in LISTED if s[2] == chunks and layernorm_bundles(s[0], s[1], g)[0] == chunks]
    assert any(not layernorm_bundles(rows, cols, g)[2] for rows, cols, _ in shapes)
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    sub_h = synth.seda_sub_formatbooks(DEFAULT_FORMATBOOK, n_groups=7, seed=chunks)
    sub_h[2] = np.arange(24, 32)             # dialects of the upper ranges only: the range filter leaves nothing for most blocks
    sub = torch.from_numpy(sub_h).cuda()
    o = F.opts(block=block, num_groups=g, flags=F.FLAG_TWO_STAGE if two_stage else 0)
    for rows, cols, _ in shapes:
        x = synth.vdit_activation(rows=rows, cols=cols, seed=cols, device="cuda")
        x[5::97] += 30.0                     # some bundles take the walk over squared deviations as well
        # another group from row to row, the whole formatbook (-1) and one past the table among them
        tg = torch.from_numpy((np.random.default_rng(rows).integers(0, 9, size=rows) - 1).astype(np.int32)).cuda()
        gamma, beta = (torch.from_numpy(a).cuda() for a in synth.layernorm_affine(cols, seed=cols))
        y = torch.empty_like(x)
        F.fb4_layernorm_quantize(luts, o, x, gamma, beta, 1e-6, y_out=y)
        c, m = F.fb4_layernorm_quantize(luts, o, x, gamma, beta, 1e-6, token_group=tg, sub_formatbooks=sub)
        c0, m0 = F.fb4_quantize_seda(luts, o, y, tg, sub)    # (against the oracle in tests of its own)
        torch.cuda.synchronize()
        assert torch.equal(m, m0) and torch.equal(c, c0), (rows, cols)
    luts.free()


@pytest.mark.parametrize("rows,cols,chunks", [(9001, 960, 1), (25001, 768, 2), (20001, 2400, 3), (3301, 5120, 3), (3100, 6176, 4),
                                              (2100, 9216, 5), (2101, 12288, 6)])
def test_layernorm_of_large_means_and_overflowing_rows(F, rows, cols, chunks):
    # rows that take the walk over squared deviations, and some that are redone in double, between ordinary ones
    assert layernorm_bundles(rows, cols, 8)[0] == chunks
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    x = synth.vdit_activation(rows=rows, cols=cols, seed=cols, device="cuda").float()
    x[3::7] += 40.0
    x[11::1001] *= 2.0 ** 70
    x = x.bfloat16()
    gamma, beta = synth.layernorm_affine(cols, seed=cols)
    y = torch.empty_like(x)
    c, m = F.fb4_layernorm_quantize(luts, F.opts(), x, torch.from_numpy(gamma).cuda(), torch.from_numpy(beta).cuda(), 1e-6, y_out=y)
    c0, m0 = F.fb4_quantize(luts, F.opts(), y)
    torch.cuda.synchronize()
    assert torch.equal(c, c0) and torch.equal(m, m0)
    assert_layernorm(x, y, gamma, beta)
    luts.free()


def assert_layernorm(x, y, gamma, beta):
    """y is the LayerNorm of x within one bf16 step, or within 2^-19 (|gamma| (|t| + |mean| rstd + 1) + |beta|) where the
    terms cancel, t = (x - mean) rstd."""
    xd, g, b = x.double(), torch.from_numpy(gamma).cuda().double(), torch.from_numpy(beta).cuda().double()
    mean = xd.mean(dim=1, keepdim=True)
    rstd = ((xd - mean).square().mean(dim=1, keepdim=True) + 1e-6).rsqrt()
    t = (xd - mean) * rstd
    ref = t * g + b
    step = torch.ldexp(torch.ones_like(ref), torch.frexp(ref.abs().clamp_min(2.0 ** -126))[1] - 8)   # (8 significant bits)
    err = (y.double() - ref).abs()
    assert (err <= torch.maximum(step, 2.0 ** -19 * (g.abs() * (t.abs() + mean.abs() * rstd + 1) + b.abs()) + step / 2)).all()
    return (err <= step / 2).double().mean().item()


@pytest.mark.parametrize("cols", [1152, 3072])
def test_layernorm_of_the_same_rows_in_a_short_and_a_long_call(F, cols):
    # how many chunks a lane takes, and with it the order of a row's sums, goes with the number of rows: a value next to the
    # middle of two bf16 values may be rounded to either
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    x = synth.vdit_activation(rows=16384, cols=cols, seed=3, device="cuda")
    gamma, beta = (torch.from_numpy(a).cuda() for a in synth.layernorm_affine(cols))
    ys = []
    for rows in (16384, 300):
        y = torch.empty_like(x[:rows])
        F.fb4_layernorm_quantize(luts, F.opts(), x[:rows], gamma, beta, 1e-6, y_out=y)
        ys.append(y[:300].float())
    torch.cuda.synchronize()
    assert layernorm_bundles(300, cols, 8)[0] != layernorm_bundles(16384, cols, 8)[0]
    # one bf16 step apart, or (gamma t and beta cancel) within 2^-18 of terms of a few units
    off = (ys[0] - ys[1]).abs()
    assert (off <= torch.maximum(ys[0].abs() * 2.0 ** -7, torch.full_like(off, 2.0 ** -15))).all()
    assert (off != 0).float().mean() < 1e-4
    luts.free()
