"""The score and statistics walks (stationary window queries, keys streamed in ranges) at the edges of their cut: tiles of
32 keys, ranges of 1 to 12 tiles, row blocks of 32 window rows paired within a KV head's group, tasks split over
wavefronts and workgroups.  Against the float64 oracle; the scores tighter than the parity tolerance: a logit of magnitude x
carries at most 130 roundings of the fp32 accumulation and its row's denominator as many, so x = 8 bounds the
relative error of a probability by 260 * 2^-24 * 8 ~ 1.3e-4 and in the mean (rounding errors of either sign) far below it."""
import numpy as np
import pytest

from paper_2405_12532_amd import synth
from tests import parity, test_gpu_decode, test_gpu_layer
from tests.routes import COUNTED, EQUAL, PLACES, SEQ_PER_XCD, launches, route

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
SCORE_RTOL = 1.3e-4


def _wl(lens, Hq, Hkv, d, w):
    return synth.shrunk(synth.workload("cfg2"), lens, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, w=w, hidden_dim=0)


SHAPES = [
    ((31, 32, 33, 63, 64, 65, 96, 97), 4, 4, 128, 32),          # one row block per head, tiles and their remainders
    ((383, 384, 385, 767, 768, 769), 2, 2, 128, 33),            # around ranges of 12 tiles; a row block of one row
    ((200, 1, 90), 6, 2, 128, 20),                              # group of 3: pairs span query heads, one row block is left over
    ((500, 130), 12, 4, 64, 96),                                # nine row blocks per KV head
    ((260,), 40, 40, 128, 64),                                  # rows not a power of two apart; tasks split over workgroups
    ((1300,), 5, 5, 64, 100),                                   # fewer tasks than wavefronts; four row blocks, the last of four rows
    ((150,) * 16, 8, 8, 128, 64),                               # a sequence per XCD
]


def _one_launch(lib, lens, Hq, Hkv, d, w, **device):
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32))
    return lib.diag_layer(lib.make_shape(len(lens), sum(lens), max(lens), Hq, Hkv, d), off, w, **device)


@pytest.mark.parametrize("lens,Hq,Hkv,d,w", SHAPES)
@pytest.mark.parametrize("weighted", [False, True])
def test_prefill_scores(lib, lens, Hq, Hkv, d, w, weighted):
    """A layer of these takes its scores in the attention's launch (the strip walk by itself: tests/test_gpu_layer_launch.py)."""
    assert _one_launch(lib, lens, Hq, Hkv, d, w) > 0
    rw = np.linspace(0.0, 1.0, w, dtype=np.float32) if weighted and w > 1 else None      # (the first weight is zero)
    res, ref, _ = test_gpu_layer.run_and_check(lib, _wl(lens, Hq, Hkv, d, w), row_weights=rw)
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)


def _spread(n, lo, hi, seed):
    return tuple(int(x) for x in np.random.default_rng(seed).integers(lo, hi + 1, size=n))


SPLIT = [                                                       # layers whose strip walk is split: order of the ranges, workgroups of a range
    ((2100, 33, 700), 16, 8, 128, 64, COUNTED, 2),
    ((2500, 130), 12, 4, 64, 96, COUNTED, 4),                   # nine row blocks per KV head: pairs span query heads, one is left over
    ((2300,), 5, 5, 64, 100, EQUAL, 2),                         # five KV heads; four row blocks, the last of four rows
    ((2060,), 40, 40, 128, 64, EQUAL, 8),                       # rows not a power of two apart
    ((64,) * 60, 40, 40, 128, 64, EQUAL, 4),                    # many short ones
    ((300,) * 14, 64, 8, 128, 100, EQUAL, 16),                  # as many workgroups as there can be
    ((64,) * 64, 32, 32, 64, 16, SEQ_PER_XCD, 4),
    ((520,) * 16, 2, 1, 128, 300, SEQ_PER_XCD, 2),              # twenty row blocks of one KV head, whose share no workgroup begins at
    (_spread(200, 1, 100, 6), 12, 4, 64, 100, PLACES, 2),
    (_spread(200, 1, 100, 6), 40, 40, 64, 64, PLACES, 2),
    (_spread(150, 1, 150, 6), 2, 1, 128, 256, PLACES, 2),       # windows longer than the sequences
]


@pytest.mark.parametrize("lens,Hq,Hkv,d,w,order,groups", SPLIT)
@pytest.mark.parametrize("weighted", [False, True])
def test_split_walk_of_a_layer(lib, lens, Hq, Hkv, d, w, order, groups, weighted):
    r = route(lib, lens, Hq, Hkv, d, w)
    assert (_one_launch(lib, lens, Hq, Hkv, d, w), r.score_order, r.score_groups) == (0, order, groups)
    rw = np.linspace(0.25, 1.0, w, dtype=np.float32) if weighted else None
    res, ref, _ = test_gpu_layer.run_and_check(lib, _wl(lens, Hq, Hkv, d, w), row_weights=rw)
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)


@pytest.mark.parametrize("lens,Hq,Hkv,d,w", SHAPES)
def test_decode_scores(lib, lens, Hq, Hkv, d, w):
    res, ref, _ = test_gpu_decode.run_and_check(lib, _wl(lens, Hq, Hkv, d, w), with_pos=True)
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)


def test_decode_long_cache(lib):
    """More ranges than the fold keeps in flight, and a context the selection cannot stage in LDS."""
    res, ref, _ = test_gpu_decode.run_and_check(lib, _wl((40000,), 8, 2, 64, 40))
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)


LOOSE = ((64,) * 64, 32, 64, 16)


def test_loose_max_seqlen(lib):
    """A caller whose max_seqlen is far above the longest sequence gets no more workspace than it asked for: the score pass, which does
    split this batch into partial sums where there is room for them, may not do so there.  The guard behind the workspace stays
    as it was."""
    lens, H, d, w = LOOSE
    assert route(lib, lens, H, H, d, w).score_groups > 1 and _one_launch(lib, lens, H, H, d, w) == 0
    wl = _wl(lens, H, H, d, w)
    x = parity.inputs(wl, lib, want_hidden=False)
    q, k, v = (lib.to_device_bf16(x[n]) for n in ("q", "k", "v"))
    T = sum(lens)
    off_h = torch.from_numpy(np.ascontiguousarray(x["seq_offsets"], dtype=np.int32))
    keep_h = torch.from_numpy(np.ascontiguousarray(x["keep_len"], dtype=np.int32))
    off_d, keep_d = off_h.cuda(), keep_h.cuda()
    n_kept = int(keep_h.sum())
    results = []
    for claimed in (64, T):
        shape = lib.make_shape(len(lens), T, claimed, H, H, d)
        ws_bytes = lib.workspace_bytes(shape, w)
        ws = torch.full((ws_bytes + 4 * 16 * T,), 0x5A, dtype=torch.uint8, device="cuda")
        out, scores = torch.empty_like(q), torch.empty(T, dtype=torch.float32, device="cuda")
        kept, out_off = torch.empty(n_kept, dtype=torch.int32, device="cuda"), torch.empty(len(lens) + 1, dtype=torch.int32, device="cuda")
        lib.prefill_layer(q, k, v, off_d, off_h, shape, w, 0.0, keep_d, keep_h, out, scores, kept, out_off, None, None, ws, ws_bytes)
        torch.cuda.synchronize()
        assert bool((ws[ws_bytes:] == 0x5A).all())
        parts = ws_bytes - 4 * 16 * T                      # (where the partial sums begin, if there is room for them)
        assert claimed == T or bool((ws[parts:ws_bytes] != 0x5A).any())
        results.append(scores.cpu().numpy())
    np.testing.assert_allclose(results[0], results[1], rtol=2e-6, atol=1e-12)


ORDERS = [                                                      # order of the score walk's ranges, whether a layer takes its scores in the attention's launch
    ((900,) * 7, 4, 4, 64, 32, EQUAL, True),                    # as many ranges in every sequence, not a multiple of the XCDs
    ((380, 370, 384, 361), 4, 2, 128, 16, EQUAL, True),         # ... of lengths that differ
    ((0, 700, 0, 0, 33, 1), 4, 2, 128, 32, COUNTED, True),      # counted by the workgroup: empty sequences in front and between
    (_spread(64, 1, 400, 1), 2, 2, 64, 16, COUNTED, True),      # one round of the count
    (_spread(65, 1, 400, 2) + (0,), 2, 1, 128, 16, COUNTED, True),    # two
    (_spread(255, 0, 300, 3) + (600,), 2, 2, 64, 16, COUNTED, False), # four, the last sequence the longest
    (_spread(257, 0, 300, 4), 2, 2, 64, 16, PLACES, False),     # places for every sequence
    (_spread(129, 1, 250, 5), 2, 2, 128, 16, PLACES, True),     # ... more than 128 short ones
    ((700,) * 7, 2, 2, 64, 400, EQUAL, True),                   # half a sequence in the window: each starts at another range
    ((520,) * 16, 2, 1, 128, 300, SEQ_PER_XCD, False),          # ... on one XCD each
    ((2100,) * 3, 2, 1, 64, 16, EQUAL, False),                  # too long for one launch
    ((2100, 2098, 2112), 4, 2, 128, 33, EQUAL, False),
    ((2100,) * 8, 2, 1, 64, 16, SEQ_PER_XCD, False),
    ((0, 2100, 0, 0, 33, 1), 4, 2, 128, 32, COUNTED, False),
    (_spread(64, 1, 400, 1) + (0, 2100), 2, 2, 64, 16, COUNTED, False),
    (_spread(257, 0, 300, 4) + (2100,), 2, 2, 64, 16, PLACES, False),
]


@pytest.mark.parametrize("lens,Hq,Hkv,d,w,order,one", ORDERS)
def test_order_of_the_ranges(lib, lens, Hq, Hkv, d, w, order, one):
    """Every range is taken by exactly one workgroup, whichever way the grid is laid out: scores of the prefill step, where it does not take
    them in the attention's launch (the score walk of all of these by itself: tests/test_gpu_layer_launch.py); and the cache update of
    the same batches (test_order_of_the_updates_ranges has its two walks)."""
    assert (route(lib, lens, Hq, Hkv, d, w).score_order, _one_launch(lib, lens, Hq, Hkv, d, w) > 0) == (order, one)
    wl = _wl(lens, Hq, Hkv, d, w)
    for run in (test_gpu_layer.run_and_check, test_gpu_decode.run_and_check):
        res, ref, _ = run(lib, wl)
        np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)


UPDATE_ORDERS = [                                               # statistics and scores, two walks
    ((2100,) * 3, 2, 1, 64, 16, EQUAL, EQUAL),
    ((2100, 2098, 2112), 4, 2, 128, 33, EQUAL, EQUAL),          # lengths that differ, as many ranges
    ((2100,) * 8, 2, 1, 64, 16, SEQ_PER_XCD, SEQ_PER_XCD),
    ((0, 2100, 0, 0, 33, 1), 4, 2, 128, 32, COUNTED, COUNTED),  # empty sequences in front and between
    (_spread(64, 1, 400, 1) + (0, 2100), 2, 2, 64, 16, COUNTED, COUNTED),
    (_spread(255, 0, 300, 3) + (2100,), 2, 2, 64, 16, COUNTED, COUNTED),
    (_spread(257, 0, 300, 4) + (2100,), 2, 2, 64, 16, PLACES, PLACES),
    ((2100,) * 7, 2, 2, 64, 1100, EQUAL, EQUAL),                # half a sequence in the window: each starts at another range
    ((2060,) * 8, 1, 1, 64, 1030, SEQ_PER_XCD, SEQ_PER_XCD),    # ... on one XCD each
]


@pytest.mark.parametrize("lens,Hq,Hkv,d,w,stats,scores", UPDATE_ORDERS)
@pytest.mark.parametrize("weighted", [False, True])
def test_order_of_the_updates_ranges(lib, lens, Hq, Hkv, d, w, stats, scores, weighted):
    r = launches(lib, lens, Hq, Hkv, d, w, generation=True)
    assert (r.stats_order, r.window_order) == (stats, scores)
    rw = np.linspace(0.25, 1.0, w, dtype=np.float32) if weighted else None
    res, ref, _ = test_gpu_decode.run_and_check(lib, _wl(lens, Hq, Hkv, d, w), row_weights=rw)
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)


FOLDS = [                                                       # the ranges of the longest sequence, then of the others
    ((257,) * 24, 32, 1, 128, 100, [1] * 24),                   # one lane folds a row of up to four ranges
    ((500,) * 28 + (1, 33, 128, 129, 384, 385), 16, 1, 64, 33, [4] * 28 + [1, 1, 1, 2, 3, 4]),
    ((600,) * 32 + (1, 33, 128, 129, 256, 257), 16, 1, 64, 33, [5] * 32 + [1, 1, 1, 2, 2, 3]),           # eight lanes share it from five on
    ((513, 512), 2, 2, 128, 16, [9, 8]),                        # ... and one of them has a second one
    ((2100, 1, 64, 65, 256, 257, 512, 513), 4, 2, 128, 40, [33, 1, 1, 2, 4, 5, 8, 9]),
    ((40, 2900), 4, 4, 64, 64, [1, 46]),                        # more than the fold keeps in flight; a sequence shorter than the window
]


def fold_ranges(lib, lens, Hq, Hkv, d, w, **device):
    tiles = route(lib, lens, Hq, Hkv, d, w, **device).stats_tiles
    return [-(-S // (32 * tiles)) for S in lens] if tiles else None


@pytest.mark.parametrize("lens,Hq,Hkv,d,w,ranges", FOLDS)
def test_fold_of_the_statistics(lib, lens, Hq, Hkv, d, w, ranges):
    """A row's ranges, folded by one lane where there are four at most in the longest sequence, else by eight."""
    assert fold_ranges(lib, lens, Hq, Hkv, d, w) == ranges
    res, ref, _ = test_gpu_decode.run_and_check(lib, _wl(lens, Hq, Hkv, d, w))
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)


@pytest.mark.parametrize("S", [1, 64, 256, 257, 512, 513, 2100])
def test_update_of_one_cache(lib, S):
    """One walk up to 2048 rows, two beyond."""
    assert (route(lib, (S,), 4, 2, 128, 40).stats_waves > 0) == (S > 2048)
    res, ref, _ = test_gpu_decode.run_and_check(lib, _wl((S,), 4, 2, 128, 40))
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)
