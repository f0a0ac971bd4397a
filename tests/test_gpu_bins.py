"""Bins and fractions of the streaming kernel: every bf16 mantissa at every distance from the block's largest exponent that
can reach a bin, for block exponents over the whole range, against the oracle."""

import numpy as np
import pytest
import torch

from fb4_inputs import DEFAULT_FORMATBOOK, synth
from oracle import fb4_oracle as O

pytestmark = pytest.mark.gpu

EXPONENTS = [4, 5, 6, 7, 9, 12, 13, 18, 19, 20, 21, 40, 64, 100, 127, 128, 191, 240, 253, 254]


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_02883_amd as F
    return F


def patterns():
    """Rows of 64 bf16 patterns: two blocks of 32 (four of 16), each led by an element of the row's block exponent."""
    rng = np.random.default_rng(5)
    rows = []
    for e in EXPONENTS:
        p = np.concatenate([(np.arange(max(0, e - 8), e + 1)[:, None] * 128 + np.arange(128)).ravel(),
                            rng.integers(0, e * 128 + 128, 256)])   # ... and anything below
        p = rng.permutation(p)
        p = np.concatenate([p, np.zeros(-len(p) % 60, dtype=p.dtype)]).reshape(-1, 4, 15)
        lead = e * 128 + rng.integers(0, 128, (len(p), 4, 1))
        rows.append(np.concatenate([lead, p], axis=2).reshape(len(p), 64))
    x = np.concatenate(rows).astype(np.uint16)
    return x | (rng.integers(0, 2, x.shape).astype(np.uint16) << 15)


@pytest.mark.parametrize("two_stage", [False, True])
@pytest.mark.parametrize("block,selector,groups", [(32, "lut", 8), (32, "lut", 16), (32, "lut", 32), (32, "sse", 8),
                                                   (16, "lut", 8), (16, "lut", 16), (16, "sse", 8)])
def test_every_pattern_near_the_block_maximum(F, block, selector, groups, two_stage):
    bits = patterns()
    x = torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)
    sel = F.SEL_SSE if selector == "sse" else F.SEL_LUT
    o = F.opts(block=block, selector=sel, num_groups=groups, flags=F.FLAG_TWO_STAGE if two_stage else 0)
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    codes, meta = F.fb4_quantize(luts, o, x)
    # ... and under candidate lists: seven groups and rows outside any; the first list has dialects of the upper ranges only, so
    # that the range filter leaves none of them for most blocks
    rows = len(bits)
    tg = (np.arange(rows) % 8 - 1).astype(np.int32)
    sub = synth.seda_sub_formatbooks(DEFAULT_FORMATBOOK, n_groups=7, seed=3)
    sub[0] = np.arange(24, 32)
    cs, ms = F.fb4_quantize_seda(luts, o, x, torch.from_numpy(tg).cuda(), torch.from_numpy(sub).cuda())
    torch.cuda.synchronize()
    for got, kw in (((codes, meta), {}), ((cs, ms), dict(token_group=tg, sub_formatbooks=sub))):
        c, m = O.quantize(DEFAULT_FORMATBOOK, bits, block=block, selector=sel, num_groups=groups, flags=o.flags, **kw)
        assert np.array_equal(got[1].cpu().numpy().view(np.uint16), m)
        assert np.array_equal(got[0].cpu().numpy(), c)


@pytest.mark.parametrize("rows", [2000, 4551, 4552, 9000])
def test_block_16_lists_and_range_filter_on_both_sides_of_the_wavefront_rule(F, rows):
    # 36 chunks per row: 2560 tiles of 64 chunks are 10 per compute unit
    cols = 1152
    x = synth.mixture_activation(rows=rows, cols=cols, seed=rows, device="cuda", n_components=6)[0]
    tg = (np.arange(rows) % 7 - 1).astype(np.int32)
    sub = synth.seda_sub_formatbooks(DEFAULT_FORMATBOOK, n_groups=6, seed=2)
    o = F.opts(block=16, num_groups=8, flags=F.FLAG_TWO_STAGE)
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    codes, meta = F.fb4_quantize_seda(luts, o, x, torch.from_numpy(tg).cuda(), torch.from_numpy(sub).cuda())
    torch.cuda.synchronize()
    c, m = O.quantize(DEFAULT_FORMATBOOK, synth.bf16_bits(x), block=16, num_groups=8, flags=o.flags, token_group=tg, sub_formatbooks=sub)
    assert np.array_equal(meta.cpu().numpy().view(np.uint16), m) and np.array_equal(codes.cpu().numpy(), c)


@pytest.mark.parametrize("rows", [14563, 14564, 20024, 20025])
def test_block_16_lists_and_range_filter_where_eight_wavefronts_take_over_again(F, rows):
    # 32, 33, 44 and 45 tiles per compute unit of 256, against the same rows in calls of fewer than 10
    cols = 1152
    x = synth.mixture_activation(rows=rows, cols=cols, seed=rows, device="cuda", n_components=6)[0]
    tg = torch.from_numpy((np.arange(rows) % 7 - 1).astype(np.int32)).cuda()
    sub = torch.from_numpy(synth.seda_sub_formatbooks(DEFAULT_FORMATBOOK, n_groups=6, seed=2)).cuda()
    o = F.opts(block=16, num_groups=8, flags=F.FLAG_TWO_STAGE)
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    codes, meta = F.fb4_quantize_seda(luts, o, x, tg, sub)
    for r in range(0, rows, 2000):
        c, m = F.fb4_quantize_seda(luts, o, x[r:r + 2000], tg[r:r + 2000], sub)
        assert torch.equal(meta[r:r + 2000], m) and torch.equal(codes[r:r + 2000], c), r
    luts.free()
