"""Attention scores at the edges of the kernels' tiles: token counts around the blocks of 32 queries and 64 keys, rows of
every kind of length (odd and even numbers of 16-byte pieces), values that must not leave their row."""

import numpy as np
import pytest
import torch

from fb4_inputs import synth

pytestmark = pytest.mark.gpu

LONG_TOKENS = [65, 95, 96, 97, 127, 128, 129, 161, 192, 255, 257, 289, 513]
DIMS = [8, 16, 24, 32, 40, 56, 64, 72, 80, 96, 104, 112, 120, 128]


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_02883_amd as F
    return F


def reference(q, k, mode):
    """(scores, error bound) in float64.  The products of two bf16 are exact in fp32; at most dim + tokens + 8 additions
    and one division follow, each rounding by at most 2^-24 (chopping included: 2^-23) of the sum of absolute values."""
    s = torch.matmul(q.double().cpu(), k.double().cpu().transpose(1, 2))
    ref = (s.clamp_min(0) if mode else s.abs()).mean(dim=2)
    mass = torch.matmul(q.double().cpu().abs(), k.double().cpu().abs().transpose(1, 2)).mean(dim=2)
    return ref, mass * (q.shape[2] + q.shape[1] + 8) * 2.0 ** -23 + 1e-30


def check(F, q, k, mode):
    groups, tokens, dim = q.shape
    out = torch.full((groups * tokens + 64,), -7.0, device="cuda")       # what lies behind the scores stays
    F.fb4_attention_scores(q, k, mode, scores=out[:groups * tokens].view(groups, tokens))
    torch.cuda.synchronize()
    assert (out[groups * tokens:] == -7.0).all()
    got = out[:groups * tokens].view(groups, tokens).double().cpu()
    ref, bound = reference(q, k, mode)
    assert ((got - ref).abs() <= bound).all(), (groups, tokens, dim, mode)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("tokens", LONG_TOKENS)
def test_long_groups(F, tokens, mode):
    for i, dim in enumerate(DIMS):
        groups = (1, 3, 10)[i % 3]
        q, k = synth.attention_qk(groups, tokens, dim, seed=100 * tokens + dim, device="cuda")
        check(F, q, k, mode)


def query_blocks(groups, tokens):
    """The launcher's choice: blocks of 32 queries per wavefront, and those of the two wavefront pairs of the last
    workgroup of a group (0, 0 where the whole workgroups take all)."""
    n_blk, best, best_cost = (tokens + 31) // 32, 4, 0.0
    for b in (4, 3, 2, 1):
        full, rest = divmod(n_blk, 2 * b)
        units = full * (b + 0.7) + ((rest + 1) // 2 + 0.7 if rest else 0.0)
        load = groups * units / ((b + 0.7) * 256)
        cost = (b + 0.7) * (0.2 + 0.8 * (int(load + 0.999) if load > 1 else 1))
        if b == 4 or cost < best_cost:
            best, best_cost = b, cost
    rest = n_blk % (2 * best)
    return best, (rest + 1) // 2, rest // 2


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("groups,tokens,blocks", [(1, 97, (1, 0, 0)), (1, 65, (1, 1, 0)), (16, 390, (1, 1, 0)), (134, 97, (2, 0, 0)),
                                                  (92, 129, (2, 1, 0)), (92, 161, (2, 1, 1)), (134, 65, (2, 2, 1)), (24, 999, (2, 0, 0)),
                                                  (176, 161, (3, 0, 0)), (260, 97, (3, 2, 2)), (176, 129, (3, 3, 2)), (130, 480, (3, 2, 1)),
                                                  (197, 225, (4, 0, 0)), (155, 257, (4, 1, 0)), (386, 65, (4, 2, 1)), (260, 161, (4, 3, 3)),
                                                  (197, 193, (4, 4, 3))])
def test_long_groups_with_every_number_of_query_blocks(F, groups, tokens, blocks, mode):
    # whole workgroups of 1, 2, 3 and 4 blocks per wavefront and last workgroups with every number of them, in the variants
    # with three wavefronts per SIMD (up to 72 channels) and with two
    assert query_blocks(groups, tokens) == blocks
    for dim in (64, 72, 96, 128):
        q, k = synth.attention_qk(groups, tokens, dim, seed=groups + dim, device="cuda")
        check(F, q, k, mode)


@pytest.mark.parametrize("groups,tokens,dim", [(272, 1350, 72), (384, 1024, 128)])
def test_long_groups_of_a_whole_clip(F, groups, tokens, dim):
    assert query_blocks(groups, tokens)[0] == 4
    q, k = synth.attention_qk(groups, tokens, dim, seed=dim, device="cuda")
    got = F.fb4_attention_scores(q, k, 0)
    torch.cuda.synchronize()
    for g in (0, 1, groups // 2, groups - 2, groups - 1):
        ref, bound = reference(q[g:g + 1], k[g:g + 1], 0)
        assert ((got[g:g + 1].double().cpu() - ref).abs() <= bound).all(), g


@pytest.mark.parametrize("dim", [24, 64, 72, 128])
@pytest.mark.parametrize("tokens", [67, 130])
def test_infinities_and_nans_stay_in_their_rows(F, tokens, dim):
    q, k = synth.attention_qk(3, tokens, dim, seed=dim + tokens, device="cuda")
    clean = F.fb4_attention_scores(q, k, 0).clone()
    q2, k2 = q.clone(), k.clone()
    q2[0, 5, dim - 1] = float("nan")         # one query of group 0
    k2[2, tokens - 1, 0] = float("inf")      # the last key of group 2: every score of that group is infinite
    k2[2, tokens - 1, 1:] = 0.0
    q2[2, :, 0] = 1.0
    got = F.fb4_attention_scores(q2, k2, 0)
    torch.cuda.synchronize()
    assert torch.isnan(got[0, 5])
    keep = torch.ones(tokens, dtype=torch.bool, device="cuda")
    keep[5] = False
    assert torch.equal(got[0][keep], clean[0][keep]) and torch.equal(got[1], clean[1])
    assert torch.isinf(got[2]).all()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("tokens", [1, 2, 3, 5, 8, 11, 15, 16, 17, 21, 31, 32, 33, 40, 47, 63, 64])
def test_short_groups(F, tokens, mode):
    for i, dim in enumerate(DIMS + [136, 200, 248, 256]):
        groups = (1, 2, 7, 33, 1001)[i % 5]
        q, k = synth.attention_qk(groups, tokens, dim, seed=1000 * tokens + dim, device="cuda")
        check(F, q, k, mode)


@pytest.mark.parametrize("dim", [64, 72, 96, 128, 40])
def test_short_groups_over_many_tasks_per_wavefront(F, dim):
    for groups, tokens in ((40001, 16), (30003, 24), (9001, 50)):
        q, k = synth.attention_qk(groups, tokens, dim, seed=dim, device="cuda")
        out = F.fb4_attention_scores(q, k, 1)
        p = torch.matmul(q.float(), k.float().transpose(1, 2).contiguous())
        ref = p.clamp_min(0).mean(dim=2)
        # both sides round their sums in fp32: the bound of `reference` twice, with the products' mass from above
        mass = (q.float().norm(dim=2) * k.float().norm(dim=2).amax(dim=1, keepdim=True))
        assert ((out - ref).abs() <= mass * (dim + tokens + 8) * 2.0 ** -22).all(), (groups, tokens, dim)


def close_to_fp32(F, groups, tokens, dim, mode):
    q, k = synth.attention_qk(groups, tokens, dim, seed=groups + dim, device="cuda")
    out = torch.full((groups * tokens + 64,), -7.0, device="cuda")
    F.fb4_attention_scores(q, k, mode, scores=out[:groups * tokens].view(groups, tokens))
    assert (out[groups * tokens:] == -7.0).all()
    p = torch.matmul(q.float(), k.float().transpose(1, 2).contiguous())
    ref = (p.clamp_min(0) if mode else p.abs()).mean(dim=2)
    # both sides round their sums in fp32: the bound of `reference` twice, with the products' mass from above
    mass = (q.float().norm(dim=2) * k.float().norm(dim=2).amax(dim=1, keepdim=True))
    assert ((out[:groups * tokens].view(groups, tokens) - ref).abs() <= mass * (dim + tokens + 8) * 2.0 ** -22).all(), (groups, tokens, dim)


@pytest.mark.parametrize("dim", range(8, 257, 8))
def test_short_groups_of_every_row_length(F, dim):
    # one wavefront per task and several tasks per wavefront; up to 128 channels groups of 33 to 48 tokens on both sides of
    # the number of groups from which one wavefront takes a group, and always of 49 and more, which four take
    for groups, tokens in ((40, 32), (9001, 16), (1023, 48), (1024, 48), (5003, 33), (1100, 49), (1100, 64)):
        close_to_fp32(F, groups, tokens, dim, (dim // 8 + tokens) % 2)


def test_short_groups_keep_infinities_and_nans_in_their_group(F):
    for dim in (24, 64, 72):
        q, k = synth.attention_qk(9, 12, dim, seed=dim, device="cuda")
        clean = F.fb4_attention_scores(q, k, 0).clone()
        k2 = k.clone()
        k2[3, 11, :] = float("nan")
        k2[5, 0, dim - 1] = float("inf")
        got = F.fb4_attention_scores(q, k2, 0)
        torch.cuda.synchronize()
        assert torch.isnan(got[3]).all() and not torch.isfinite(got[5]).any()
        rest = [0, 1, 2, 4, 6, 7, 8]
        assert torch.equal(got[rest], clean[rest])


def query_blocks_80_to_96(groups, tokens):
    """As query_blocks, with up to six blocks per wavefront and the constants of those kernels."""
    n_blk, best, best_cost = (tokens + 31) // 32, 6, 0.0
    for b in (6, 5, 4, 3, 2, 1):
        full, rest = divmod(n_blk, 2 * b)
        units = full * (b + 1.05) + ((rest + 1) // 2 + 1.05 if rest else 0.0)
        load = groups * units / ((b + 1.05) * 256)
        rounds = -(-groups * (full + (rest > 0)) // 256)
        m = max(1.0, 0.48 * max(1, int(load + 0.999)) + 0.1 * rounds + 0.42 * load)
        cost = (b + 1.05) * (0.33 + 0.67 * m)
        if b == 6 or cost < best_cost:
            best, best_cost = b, cost
    rest = n_blk % (2 * best)
    return best, (rest + 1) // 2, rest // 2


@pytest.mark.parametrize("groups,tokens,blocks", [(205, 289, (5, 0, 0)), (51, 1281, (5, 1, 0)), (51, 1345, (5, 2, 1)), (79, 801, (5, 3, 3)),
                                                  (261, 193, (5, 4, 3)), (205, 257, (5, 5, 4)), (387, 353, (6, 0, 0)), (303, 769, (6, 1, 0)),
                                                  (289, 865, (6, 2, 2)), (121, 1281, (6, 3, 2)), (114, 1345, (6, 4, 3)), (296, 257, (6, 5, 4)), (296, 289, (6, 5, 5)),
                                                  (130, 480, (3, 2, 1)), (130, 1350, (4, 2, 1)), (310, 129, (4, 3, 2)), (261, 161, (2, 1, 1))])
def test_long_groups_with_five_and_six_query_blocks(F, groups, tokens, blocks):
    assert query_blocks_80_to_96(groups, tokens) == blocks
    for dim in (80, 88, 96):
        close_to_fp32(F, groups, tokens, dim, (dim // 8) % 2)
