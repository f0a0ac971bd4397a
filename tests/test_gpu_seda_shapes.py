"""The SeDA refresh at the edges of its kernels' tiles and rules, against the CPU oracle."""

import numpy as np
import pytest
import torch

from fb4_inputs import DEFAULT_FORMATBOOK, synth
from oracle import fb4_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_02883_amd as F
    return F


@pytest.mark.parametrize("window", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("dim,heads,joint,window_t", [(8, 1, False, 1), (72, 5, False, 1), (136, 3, True, 2), (256, 9, True, 3),
                                                          (8, 6, True, 2), (16, 4, False, 1), (24, 5, True, 2), (32, 9, False, 1), (40, 4, False, 1),
                                                          (64, 7, True, 3), (48, 2, False, 1), (128, 1, True, 2)])
def test_seda_assign_windows_and_row_lengths(F, window, dim, heads, joint, window_t):
    frames, gh, gw = 3, 7, 9
    tokens = gh * gw
    q, k = synth.attention_qk(frames * heads, tokens, dim, seed=window * 1000 + dim, device="cuda")
    shape = (heads, frames * tokens, dim) if joint else (frames, heads, tokens, dim)
    q, k = q.reshape(shape).contiguous(), k.reshape(shape).contiguous()
    anchors = np.random.default_rng(dim + window).choice(frames * tokens, size=23, replace=False).astype(np.int32)
    anchors[::5] = -1
    tgr, agr, sr = O.seda_assign(synth.bf16_bits(q), synth.bf16_bits(k), anchors, frames, gh, gw, window=window,
                                 window_t=window_t, threshold=0.0, joint=joint)
    inside = ~np.isnan(sr)
    threshold = float(np.median(sr[inside]))
    tgr, agr, sr = O.seda_assign(synth.bf16_bits(q), synth.bf16_bits(k), anchors, frames, gh, gw, window=window,
                                 window_t=window_t, threshold=threshold, joint=joint)
    tg, ag, sc = F.fb4_seda_assign(q, k, torch.from_numpy(anchors).cuda(), frames, gh, gw, window=window, window_t=window_t,
                                   threshold=threshold, joint=joint, want_scores=True)
    torch.cuda.synchronize()
    sc = sc.cpu().numpy()
    assert np.array_equal(np.isnan(sc), ~inside)
    # fp32 sums of exact products: at most dim * heads + 8 additions, 2^-23 each of the sum of absolute values, which is at
    # most the product of the largest row norms
    qn = float(q.float().norm(dim=-1).max() * k.float().norm(dim=-1).max())
    bound = (dim * heads + 8) * 2.0 ** -23 * qn
    assert np.abs(sc[inside] - sr[inside]).max() <= bound
    if (np.abs(sr[inside] - threshold) > bound).sum() >= inside.sum() - 1:   # (the median itself may fall on either side)
        near = np.abs(sr - threshold) <= bound
        if not near.any():
            assert np.array_equal(tg.cpu().numpy(), tgr)
    assert np.array_equal(ag.cpu().numpy(), agr)
    # the groups follow from the compared scores exactly
    expect = np.full(frames * tokens, -1, dtype=np.int32)
    for a, row in enumerate(anchors):
        if row < 0:
            continue
        f, t = divmod(int(row), tokens)
        g = (t // gw // 4) * ((gw + 3) // 4) + (t % gw) // 4
        for s in range(window_t * window * window):
            if sc[a, s] > np.float32(threshold):
                ft = f + s // (window * window) - window_t // 2
                y, x = t // gw + s % (window * window) // window - window // 2, t % gw + s % window - window // 2
                at = ft * tokens + y * gw + x
                expect[at] = max(expect[at], g)
    expect[agr >= 0] = agr[agr >= 0]
    assert np.array_equal(tg.cpu().numpy(), expect)


def test_seda_assign_with_very_many_anchor_entries(F):
    # more entries than the one-launch preparation takes: the same groups as from the list without repetitions
    frames, gh, gw, heads, dim = 8, 64, 64, 1, 8
    tokens = gh * gw
    q, k = synth.attention_qk(frames * heads, tokens, dim, seed=3, device="cuda")
    q, k = q.view(frames, heads, tokens, dim), k.view(frames, heads, tokens, dim)
    few = torch.from_numpy(np.random.default_rng(1).choice(frames * tokens, size=400, replace=False).astype(np.int32)).cuda()
    many = few.repeat(400)
    a = F.fb4_seda_assign(q, k, few, frames, gh, gw, window=3, threshold=1.0)
    b = F.fb4_seda_assign(q, k, many, frames, gh, gw, window=3, threshold=1.0)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert int((a[1] >= 0).sum()) == 400


@pytest.mark.parametrize("n_anchors", [0, 1, 255, 256, 257, 2047, 2048, 2049, 5000])
def test_seda_assign_own_groups_by_the_number_of_anchor_entries(F, n_anchors):
    frames, gh, gw, dim = 5, 21, 34, 8                       # 3570 rows: the last of four workgroups is short
    rows = frames * gh * gw
    q, k = synth.attention_qk(frames, gh * gw, dim, seed=4, device="cuda")
    q, k = q.view(frames, 1, gh * gw, dim), k.view(frames, 1, gh * gw, dim)
    anchors = np.random.default_rng(n_anchors).integers(-2, rows + 2, size=n_anchors).astype(np.int32)
    anchors[:3] = [0, rows - 1, 0x7FFFFFFF][:n_anchors]
    tg, ag = F.fb4_seda_assign(q, k, torch.from_numpy(anchors).cuda(), frames, gh, gw, window=1, threshold=1e30)
    torch.cuda.synchronize()
    want = np.full(rows, -1, dtype=np.int32)
    for r in anchors[(anchors >= 0) & (anchors < rows)]:
        y, x = divmod(int(r) % (gh * gw), gw)
        want[r] = (y // 4) * ((gw + 3) // 4) + x // 4
    assert np.array_equal(ag.cpu().numpy(), want) and np.array_equal(tg.cpu().numpy(), want)


@pytest.mark.parametrize("n_anchors", [150, 70000])
def test_seda_assign_into_one_buffer(F, n_anchors):
    # a caller without use for the anchors' groups may pass one buffer for both: it holds the tokens' groups
    frames, gh, gw, heads, dim = 3, 40, 41, 2, 16
    tokens = gh * gw
    q, k = synth.attention_qk(frames * heads, tokens, dim, seed=9, device="cuda")
    q, k = q.view(frames, heads, tokens, dim), k.view(frames, heads, tokens, dim)
    few = torch.from_numpy(np.random.default_rng(2).choice(frames * tokens, size=150, replace=False).astype(np.int32)).cuda()
    anchors = few.repeat(n_anchors // 150 + 1)[:max(n_anchors, 150)]
    want, _ = F.fb4_seda_assign(q, k, few, frames, gh, gw, window=8, threshold=-1e9)   # every window whole: marks meet everywhere
    one = torch.empty(frames * tokens, dtype=torch.int32, device="cuda")
    F.fb4_seda_assign(q, k, anchors, frames, gh, gw, window=8, threshold=-1e9, token_group=one, anchor_group=one)
    torch.cuda.synchronize()
    assert torch.equal(one, want)


@pytest.mark.parametrize("frames,heads,dim", [(1, 1, 8), (2, 70, 136), (17, 3, 72), (64, 2, 8), (70, 5, 16), (200, 1, 8)])
def test_seda_main_anchor_frames_heads_and_ties(F, frames, heads, dim):
    gh, gw = 4, 8                                            # two tiles
    tokens = gh * gw
    rng = np.random.default_rng(frames)
    ts = rng.integers(0, 3, size=(tokens, heads, frames)).astype(np.float32)       # few values: ties are the rule
    ts[rng.random(ts.shape) < 0.02] = np.nan
    cand = np.stack([np.array([f * tokens + rng.integers(0, 4), f * tokens + 4 + rng.integers(0, 4)]) for f in range(frames)])
    cand[rng.random(cand.shape) < 0.1] = -1
    qt, kt = synth.attention_qk(tokens * heads, frames, dim, seed=frames, device="cuda")
    qt, kt = qt.view(tokens, heads, frames, dim), kt.view(tokens, heads, frames, dim)
    cand = cand.astype(np.int32)
    main, kept, ps = F.fb4_seda_main_anchor(torch.from_numpy(ts).cuda(), qt, kt, torch.from_numpy(cand).cuda(), gh, gw,
                                            prune_threshold=1.0, want_scores=True)
    torch.cuda.synchronize()
    main_r, kept_r, ps_r = O.seda_main_anchor(ts, synth.bf16_bits(qt), synth.bf16_bits(kt), cand, gh, gw, prune_threshold=1.0)
    assert np.array_equal(main.cpu().numpy(), main_r)
    got = ps.cpu().numpy()
    inside = ~np.isnan(ps_r)
    assert np.array_equal(np.isnan(got), ~inside)
    bound = (dim * heads + 8) * 2.0 ** -23 * float(qt.float().norm(dim=-1).max() * kt.float().norm(dim=-1).max())
    if inside.any():
        assert np.abs(got[inside] - ps_r[inside]).max() <= bound
    # the kept list follows from the compared scores exactly
    for f in range(frames):
        for tile in range(2):
            if inside[f, tile]:
                keep = got[f, tile] > np.float32(1.0) or cand[f, tile] == main_r[tile]
                assert kept.cpu().numpy()[f, tile] == (cand[f, tile] if keep else -1)


def check_main_anchor(F, ts, qt, kt, cand, gh, gw, tile, threshold=1.0):
    """Main anchors as the oracle's, scores to fp32 sums, and every entry of the list -- written anew or over the candidates -- as it follows
    from the scores of the same call."""
    tokens, heads, frames, dim = qt.shape
    tiles_x = (gw + tile - 1) // tile
    with np.errstate(invalid="ignore"):
        main_r, kept_r, ps_r = O.seda_main_anchor(ts, synth.bf16_bits(qt), synth.bf16_bits(kt), cand, gh, gw, tile, tile, prune_threshold=threshold)
    # A lane adds up 8 products per 16 bytes of a row, 16 lanes a row, every fourth head; then six exchanges, up to 16 shares and the division.
    steps = 8 * ((dim + 127) // 128) * ((heads + 3) // 4) + 6 + 16 + 1
    bound = np.full(ps_r.shape, np.nan)
    at = np.flatnonzero(main_r >= 0)
    bf, p = (torch.from_numpy(v).long().cuda() for v in np.divmod(main_r[at], tokens))
    bound[:, at] = steps * 2.0 ** -24 / heads * (qt[p, :, bf].double().abs()[:, :, None] * kt[p].double().abs()).sum((1, 3)).t().cpu().numpy()
    # an entry's tile, -1 for one of another frame and for a later one of a tile that the frame's list has named
    tile_of = np.full(cand.shape, -1)
    for f in range(frames):
        seen = set()
        for j, row in enumerate(cand[f].tolist()):
            if f * tokens <= row < (f + 1) * tokens:
                y, x = divmod(row - f * tokens, gw)
                t = y // tile * tiles_x + x // tile
                if t not in seen:
                    tile_of[f, j] = t
                seen.add(t)
    main_frame = np.where(main_r >= 0, main_r // tokens, -1)
    ts = torch.from_numpy(ts).cuda()
    for in_place in (False, True):
        given = torch.from_numpy(cand).cuda()
        main, kept, ps = F.fb4_seda_main_anchor(ts, qt, kt, given, gh, gw, tile, tile, prune_threshold=threshold, want_scores=True,
                                                kept=given if in_place else torch.full_like(given, 77777))
        torch.cuda.synchronize()
        assert np.array_equal(main.cpu().numpy(), main_r)
        got, kept = ps.cpu().numpy(), kept.cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(ps_r)) and np.array_equal(got[np.isinf(ps_r)], ps_r[np.isinf(ps_r)])
        inside = np.isfinite(ps_r)
        assert (np.abs(got[inside] - ps_r[inside]) <= bound[inside]).all()
        score = np.take_along_axis(got, np.maximum(tile_of, 0), axis=1)
        keep = (tile_of >= 0) & ((score > np.float32(threshold)) | (main_frame[np.maximum(tile_of, 0)] == np.arange(frames)[:, None]))
        assert np.array_equal(kept, np.where(keep, cand, -1))
        far = ~(np.abs(ps_r - threshold) <= bound)      # (where rounding cannot put the score on the other side of the threshold)
        far = np.where(tile_of >= 0, np.take_along_axis(far, np.maximum(tile_of, 0), axis=1), True)
        assert np.array_equal(kept[far], kept_r[far])


# a tile's frames in 1 to 28 parts, one to six wavefronts per frame, a list that is overwritten
@pytest.mark.parametrize("gh,gw,tile,frames,heads,dim", [(4, 4, 4, 17, 24, 72), (8, 16, 4, 6, 9, 120), (32, 32, 4, 30, 40, 32), (16, 16, 4, 16, 9, 128),
                                                         (20, 20, 4, 40, 11, 96), (12, 12, 4, 70, 8, 128), (8, 8, 1, 80, 8, 128), (32, 32, 4, 16, 24, 128),
                                                         (44, 44, 4, 16, 3, 16), (8, 24, 4, 16, 5, 136)])
def test_seda_main_anchor_in_parts(F, gh, gw, tile, frames, heads, dim):
    tokens = gh * gw
    rng = np.random.default_rng(tokens + frames)
    ts = rng.random((tokens, heads, frames)).astype(np.float32)
    cand = F.fb4_select_salient_tokens(torch.from_numpy(rng.random((frames, 1, tokens)).astype(np.float32)).cuda(), gh, gw, tile, tile).cpu().numpy()
    cand[rng.random(cand.shape) < 0.1] = -1
    qt, kt = synth.attention_qk(tokens * heads, frames, dim, seed=tokens, device="cuda")
    check_main_anchor(F, ts, qt.view(tokens, heads, frames, dim), kt.view(tokens, heads, frames, dim), cand, gh, gw, tile)


# (ragged tiles at both edges, up to and from 32 tiles, more entries than a wavefront has lanes, both sides of the frames from which there
# are two parts; the last: one part)
@pytest.mark.parametrize("gh,gw,tile,frames,heads,dim", [(18, 19, 4, 20, 24, 72), (33, 30, 4, 7, 16, 64), (5, 3, 4, 33, 8, 128), (7, 62, 4, 3, 9, 256),
                                                         (1, 9, 2, 2, 43, 24), (29, 50, 4, 11, 8, 128), (29, 50, 4, 12, 8, 128), (37, 35, 4, 6, 24, 72)])
def test_seda_main_anchor_in_parts_of_lists_with_other_entries(F, gh, gw, tile, frames, heads, dim):
    # several entries of a tile in a frame, entries of other frames, before the first row and beyond the last, tiles that no frame names;
    # ties and NaN among the temporal scores, NaN and infinities in Q and K
    tokens = gh * gw
    rng = np.random.default_rng(tokens + frames)
    n = 2 * ((gh + tile - 1) // tile) * ((gw + tile - 1) // tile) + 3
    cand = (np.arange(frames)[:, None] * tokens + rng.integers(0, tokens, size=(frames, n))).astype(np.int64)
    tile_of = cand % tokens // gw // tile * ((gw + tile - 1) // tile) + cand % tokens % gw // tile
    cand = np.where(rng.random(cand.shape) < 0.15, rng.integers(-3, frames * tokens + 3, size=cand.shape), cand)
    cand = np.where((tile_of == 1) & (cand >= 0), rng.choice([-1, frames * tokens, 0x7FFFFFFF, -0x80000000], size=cand.shape), cand).astype(np.int32)
    ts = rng.integers(0, 3, size=(tokens, heads, frames)).astype(np.float32)
    ts[rng.random(ts.shape) < 0.1 / heads] = np.nan
    qt, kt = synth.attention_qk(tokens * heads, frames, dim, seed=tokens, device="cuda")
    qt, kt = qt.view(tokens, heads, frames, dim), kt.view(tokens, heads, frames, dim)
    for x, seed in ((qt, 1), (kt, 2)):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        at = torch.rand(x.shape, device="cuda", generator=g) * heads * dim
        x[at < 0.03] = float("inf")
        x[(at >= 0.03) & (at < 0.06)] = -float("inf")
        x[(at >= 0.06) & (at < 0.09)] = float("nan")
    check_main_anchor(F, ts, qt, kt, cand, gh, gw, tile)


@pytest.mark.parametrize("gh,gw", [(16, 32), (19, 27), (2049, 2048)])
def test_seda_main_anchor_with_many_tiles(F, gh, gw):
    # on both sides of the number of tiles that two workgroups per compute unit hold, and (16 frames) more tiles than a
    # launch takes workgroups of 1024 threads
    frames, heads, dim = 16, 1, 8
    tokens = gh * gw
    rng = np.random.default_rng(gw)
    at = rng.choice(tokens, size=5, replace=False)                                  # tiles of one token
    cand = np.array([f * tokens + at for f in range(frames)], dtype=np.int32)
    qt, kt = torch.ones((tokens, heads, frames, dim), dtype=torch.bfloat16, device="cuda"), torch.ones((tokens, heads, frames, dim), dtype=torch.bfloat16, device="cuda")
    kt[torch.from_numpy(at).cuda(), :, 3] = 0.25                                    # frame 3: score 2, the others 8
    ts = torch.zeros((tokens, heads, frames), device="cuda")
    best = rng.integers(0, frames, size=5)
    ts[torch.from_numpy(at).cuda(), 0, torch.from_numpy(best).cuda()] = 1.0
    main, kept = F.fb4_seda_main_anchor(ts, qt, kt, torch.from_numpy(cand).cuda(), gh, gw, 1, 1, prune_threshold=3.0)
    torch.cuda.synchronize()
    want = np.full(tokens, -1, dtype=np.int32)
    want[at] = best * tokens + at
    assert np.array_equal(main.cpu().numpy(), want)
    cand[3] = np.where(best == 3, cand[3], -1)
    assert np.array_equal(kept.cpu().numpy(), cand)


@pytest.mark.parametrize("frames,heads,gh,gw,th,tw", [(1, 1, 1, 1, 4, 4), (3, 24, 32, 32, 4, 4), (2, 25, 7, 9, 4, 4), (2, 33, 64, 128, 4, 4),
                                                      (2, 7, 90, 91, 5, 7), (1, 3, 33, 31, 40, 40), (2, 50, 13, 17, 1, 1), (2, 2, 64, 64, 64, 1),
                                                      (256, 3, 18, 20, 4, 4), (257, 25, 18, 20, 4, 4), (257, 9, 16, 16, 4, 4), (1, 9, 16, 17, 4, 4),
                                                      (300, 2, 65, 66, 3, 2), (3, 5, 9, 9, 2, 2)])
def test_salient_token_choice_shapes_ties_and_nans(F, frames, heads, gh, gw, th, tw):
    rng = np.random.default_rng(gh * gw + heads)
    s = rng.integers(0, 4, size=(frames, heads, gh * gw)).astype(np.float32)       # few values: ties are the rule
    s[rng.random(s.shape) < 0.3 / heads] = np.nan
    got = F.fb4_select_salient_tokens(torch.from_numpy(s).cuda(), gh, gw, th, tw)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), O.select_salient_tokens(s, gh, gw, th, tw))


# (several rows of tiles per workgroup with a ragged last one, one row of 128 / 512 / 1024 threads with both LDS sizes, a thread
# per tile, and both sides of the number of workgroups from which each takes a frame)
@pytest.mark.parametrize("frames,heads,gh,gw,th,tw", [(5, 3, 40, 6, 4, 4), (7, 9, 13, 3, 4, 4), (2, 2, 30, 100, 4, 4), (3, 2, 40, 200, 4, 4),
                                                      (1, 2, 90, 91, 30, 7), (2, 2, 64, 128, 1, 2), (2, 3, 16, 500, 2, 2),
                                                      (200, 2, 32, 32, 4, 4), (201, 2, 32, 32, 4, 4), (1700, 2, 5, 5, 4, 4)])
def test_salient_token_choice_of_rows_of_tiles(F, frames, heads, gh, gw, th, tw):
    test_salient_token_choice_shapes_ties_and_nans(F, frames, heads, gh, gw, th, tw)


# (both sides of the limits on frames, threads and tiles from which a workgroup takes a frame; large frames with a thread per
# tile and fewer heads than are added at once, as many, and one more)
@pytest.mark.parametrize("frames,heads,gh,gw,th,tw", [(384, 2, 13, 61, 8, 8), (385, 2, 13, 61, 8, 8), (128, 3, 16, 16, 8, 8), (129, 3, 16, 16, 8, 8),
                                                      (129, 3, 16, 16, 2, 2), (85, 1, 90, 90, 8, 8), (86, 1, 90, 90, 8, 8),
                                                      (260, 23, 47, 46, 2, 2), (260, 24, 47, 46, 2, 2), (260, 25, 47, 46, 2, 2), (2, 8, 4, 1030, 4, 1)])
def test_salient_token_choice_where_a_workgroup_takes_a_frame(F, frames, heads, gh, gw, th, tw):
    test_salient_token_choice_shapes_ties_and_nans(F, frames, heads, gh, gw, th, tw)


def test_salient_token_choice_of_as_many_frames_as_a_launch_of_large_workgroups_refuses(F):
    # (a workgroup of 1024 threads per frame would be 2^32 threads here, one more than a launch takes)
    frames = 1 << 22
    got = F.fb4_select_salient_tokens(torch.zeros((frames, 1, 1), device="cuda"), 1, 1)
    torch.cuda.synchronize()
    assert torch.equal(got.view(-1), torch.arange(frames, dtype=torch.int32, device="cuda"))


def test_salient_token_choice_of_more_frames_than_one_launch_takes(F):
    # (a launch has fewer than 2^32 threads, 256 of them per frame here)
    frames = (1 << 24) + 3
    got = F.fb4_select_salient_tokens(torch.zeros((frames, 1, 1), device="cuda"), 1, 1, rows_out=torch.full((frames, 1), -1, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    assert torch.equal(got.view(-1), torch.arange(frames, dtype=torch.int32, device="cuda"))


# Both sides of the limits of the kernel with a workgroup per group (rows, rows x groups, groups, blocks per row for 8, 4, 2
# and 1 metadata words per load), more rows than it looks through at a time, every row in one group, one dialect everywhere
@pytest.mark.parametrize("rows,nb,groups,share", [(1, 1, 1, 1.0), (16385, 8, 3, 1.0), (32768, 136, 256, 0.05), (32768, 144, 8, 0.05), (32769, 96, 5, 0.2),
                                                  (16384, 8, 512, 0.3), (16384, 8, 513, 0.3), (3000, 104, 9, 0.5), (3000, 108, 9, 0.5), (999, 70, 2, 0.9),
                                                  (999, 74, 2, 0.9), (777, 43, 4, 0.6), (777, 45, 4, 0.6), (5000, 36, 1, 1.0), (40, 41, 60, 0.5)])
def test_seda_profile_by_group(F, rows, nb, groups, share):
    test_seda_profile_shapes(F, rows, nb, groups, share)


# (one to sixteen rows per thread, a ragged last one, two looks; as many threads of a wavefront with anchors as get their places one by
# one, one more, and all; one anchor of a thread or all of its rows)
@pytest.mark.parametrize("rows", [64, 1023, 1024, 1025, 3071, 15361, 16384, 16447, 20000])
def test_seda_profile_by_group_places_in_the_list(F, rows):
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    reads, nb = min((rows + 1023) // 1024, 16), 5
    meta = np.random.default_rng(rows).integers(0, 32, size=(rows, nb)).astype(np.uint16)
    r = np.arange(rows)
    for lanes in sorted({1, min(2 * reads, 64), min(2 * reads + 1, 64), 64}):
        for every in (False, True):
            group = np.where((r % 64 >= 64 - lanes) & (every | (r // 1024 % reads == r % 64 % reads)), 1, 7 * (r % 2) - 1).astype(np.int32)
            counts, _ = F.fb4_seda_profile(luts, torch.from_numpy(meta.view(np.int16)).cuda(), torch.from_numpy(group).cuda(), 2)
            torch.cuda.synchronize()
            assert counts[0].sum().item() == 0
            assert np.array_equal(counts[1].cpu().numpy(), np.bincount(meta[group == 1].ravel(), minlength=32)), (lanes, every)
    luts.free()


@pytest.mark.parametrize("offset", [0, 1, 2, 4])
def test_seda_profile_alignment_and_concentration(F, offset):
    # metadata that start 0, 2, 4 and 8 bytes past a 16-byte boundary; every block the same dialect, every row the same group
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    rows, nb = 2000, 96
    buf = torch.full((rows * nb + 8,), 9 | (130 << 8), dtype=torch.int32).to(torch.int16).cuda()
    group = torch.full((rows,), 3, dtype=torch.int32, device="cuda")
    counts, sub = F.fb4_seda_profile(luts, buf[offset:offset + rows * nb].view(rows, nb), group, 5)
    torch.cuda.synchronize()
    assert int(counts[3, 9]) == rows * nb and int(counts.sum()) == rows * nb
    want = [min(d for d in range(32) if DEFAULT_FORMATBOOK[d][7] == 8 + k) for k in range(8)]
    want[DEFAULT_FORMATBOOK[9][7] - 8] = 9
    assert sub[3].tolist() == want
    luts.free()


# (rows, blocks per row, groups, share of anchors)
@pytest.mark.parametrize("rows,nb,groups,share", [(0, 5, 8, 1.0), (1, 1, 8, 1.0), (63, 7, 8, 1.0), (1030, 129, 9, 0.7), (8193, 96, 64, 0.1),
                                                  (32768, 3, 256, 0.1), (32769, 3, 16, 0.1), (300, 40, 7, 0.5), (4096, 1025, 16, 0.05)])
def test_seda_profile_shapes(F, rows, nb, groups, share):
    rng = np.random.default_rng(rows + nb)
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    meta = (rng.integers(0, 34, size=(rows, nb)) | (rng.integers(0, 255, size=(rows, nb)) << 8)).astype(np.uint16)   # (32, 33: no dialect)
    group = rng.integers(0, groups, size=rows).astype(np.int32)
    group[rng.random(rows) >= share] = rng.choice([-1, groups, groups + 100])
    counts = torch.full((groups, 32), 77, dtype=torch.int32, device="cuda")
    counts, sub = F.fb4_seda_profile(luts, torch.from_numpy(meta.view(np.int16)).cuda(), torch.from_numpy(group).cuda(), groups, counts=counts)
    torch.cuda.synchronize()
    cr = np.zeros((groups, 32), dtype=np.int64)
    for g in range(groups):
        d = (meta[group == g] & 0xFF).ravel()
        cr[g] = np.bincount(d[d < 32], minlength=32)
    assert np.array_equal(counts.cpu().numpy(), cr)
    for g in range(groups):
        for k in range(8):
            ds = [d for d in range(32) if DEFAULT_FORMATBOOK[d][7] == 8 + k]
            best = min(ds, key=lambda d: (-cr[g][d], d)) if ds else 255
            assert int(sub[g, k]) == best
    luts.free()


@pytest.mark.parametrize("rows", [0, 1])
def test_seda_profile_with_as_many_groups_as_a_launch_of_large_workgroups_refuses(F, rows):
    # (a workgroup of 1024 threads per group would be 2^32 threads here, one more than a launch takes)
    groups = 1 << 22
    luts = F.fb4_build_luts(DEFAULT_FORMATBOOK)
    meta = torch.full((rows, 3), 5, dtype=torch.int16, device="cuda")
    group = torch.full((rows,), groups - 1, dtype=torch.int32, device="cuda")
    counts = torch.full((groups, 32), 77, dtype=torch.int32, device="cuda")
    counts, sub = F.fb4_seda_profile(luts, meta, group, groups, counts=counts)
    torch.cuda.synchronize()
    assert int(counts.sum()) == 3 * rows and int(counts[-1, 5]) == 3 * rows
    # without anchors the lowest dialect of every range
    lowest = [min(d for d in range(32) if DEFAULT_FORMATBOOK[d][7] == 8 + k) for k in range(8)]
    assert (sub[:-1] == torch.tensor(lowest, dtype=torch.uint8, device="cuda")).all()
    luts.free()
