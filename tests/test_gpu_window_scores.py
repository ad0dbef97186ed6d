"""The generation phase's one walk over K (csrc/window_device.h): logits of a window's row block kept in registers, eight 32-key tiles per
wavefront at most.  At the edges of tiles, of wavefronts and of the longest sequence it takes, against the float64 oracle with the
tolerance of the two walks (tests/test_gpu_score_ranges.py); every batch asserts that it goes there.  The two walks it stands in for at these
lengths are reached by batches that assert that instead."""
import numpy as np
import pytest

from paper_2405_12532_amd import synth
from tests import parity, test_gpu_decode
from tests.routes import route
from tests.test_gpu_large_logits import F64, shaped_inputs
from tests.test_gpu_decode import window_queries
from oracle import pyr_oracle as orc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
SCORE_RTOL = 1.3e-4                                             # (derived in tests/test_gpu_score_ranges.py)


def _wl(lens, Hq, Hkv, d, w):
    return synth.shrunk(synth.workload("cfg2"), lens, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, w=w, hidden_dim=0)


ONE_WALK = [
    ((1, 2, 31, 32), 4, 4, 128, 16),                            # one tile, one wavefront
    ((33, 64, 65, 255), 4, 4, 64, 32),                          # a second tile of one row; no key left for some wavefronts
    ((256, 257, 0, 1), 6, 3, 128, 33),                          # row block of one row; empty sequence; groups without a task
    ((511, 512, 513), 4, 2, 64, 40),                            # two tiles per wavefront and one more
    ((1023, 1025), 8, 8, 128, 32),                              # four and five: the next register layout
    ((2047, 2048, 2020, 2017, 1999, 2047), 16, 16, 64, 32),     # the longest sequences
    ((2048,) * 8, 16, 16, 128, 16),
    ((300,) * 16, 8, 8, 128, 64),                               # a sequence's workgroups on one XCD
    ((1030,), 32, 32, 64, 64),                                  # 64 rows of partial sums, added by a launch of their own
    ((70, 0, 513, 3), 24, 24, 64, 64),                          # ... 48, their number not a multiple of 64 tokens
    ((1537, 1100), 9, 9, 64, 128),                              # ... fewer, but of many tokens
    ((200,) * 90, 16, 16, 64, 32),                              # several rounds of workgroups, several tasks each
]
BY_KV_HEAD = [                                                  # tasks in turn over the KV heads (window.hip, by_kv_head) ..., tasks of a workgroup
    ((300, 290), 8, 8, 128, 33, 2),                             # two row blocks a head
    ((700, 33, 0), 32, 8, 64, 32, 1),                           # GQA 4
    ((260,) * 50, 16, 8, 64, 40, 2),
    ((800,) * 5, 12, 4, 64, 40, 2),                             # KV heads that do not divide over the XCDs; six row blocks each
    ((1500, 5), 16, 8, 128, 128, 1),                            # eight
    ((256, 200), 8, 8, 64, 64, 1),                              # the shortest
    ((300,), 32, 8, 64, 128, 1),                                # sixteen row blocks
    ((300,) * 7 + (299,), 8, 8, 64, 64, 1),                     # eight sequences, not equal
    ((768,), 8, 4, 64, 64, 1),                                  # the shortest where KV heads do not divide over the XCDs, with four row blocks
]
BY_QUERY_HEAD = [                                               # ... on the other side of each limit
    ((255, 200), 8, 8, 64, 64, 1),
    ((300,), 8, 8, 64, 32, 1),                                  # one row block
    ((300,), 40, 8, 64, 128, 1),                                # twenty
    ((300,) * 8, 8, 8, 64, 64, 1),                              # equal: a sequence's workgroups on one XCD
    ((767,), 8, 4, 64, 64, 1),
    ((800,), 4, 4, 64, 96, 1),                                  # three
]
TWO_WALKS = [
    ((2049,), 4, 4, 64, 16),                                    # a key too many
    ((120,) * 60, 32, 1, 128, 128),                             # many row blocks per KV head: one lane folds a row's one range
    ((250,) * 30, 32, 1, 128, 256),
    ((1200, 700), 8, 8, 64, 40),                                # few heads
    ((2081, 200, 1, 90), 6, 2, 128, 20),                        # group of 3: pairs of row blocks span query heads, one is left over
    ((2500, 130), 12, 4, 64, 96),                               # nine row blocks per KV head
    ((2300,), 5, 5, 64, 100),                                   # fewer tasks than wavefronts; four row blocks, the last of four rows
    ((2052, 33, 64), 40, 40, 128, 64),                          # rows not a power of two apart; tasks split over workgroups
]


def task_order(lib, lens, Hq, Hkv, d, w, **device):
    """Order of the one walk's tasks (-1: two walks), the most tasks of a workgroup."""
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32))
    order = lib.diag_update(lib.make_shape(len(lens), int(sum(lens)), max(lens), Hq, Hkv, d), off, w, **device)
    return order, -(-Hq * -(-min(w, max(lens)) // 32) // route(lib, lens, Hq, Hkv, d, w, **device).window_groups)


@pytest.mark.parametrize("by_kv_head", [True, False])
def test_order_of_the_tasks(lib, by_kv_head):
    for *batch, tasks in BY_KV_HEAD if by_kv_head else BY_QUERY_HEAD:
        assert task_order(lib, *batch) == (int(by_kv_head), tasks), batch


@pytest.mark.parametrize("lens,Hq,Hkv,d,w", ONE_WALK + [batch[:5] for batch in BY_KV_HEAD + BY_QUERY_HEAD])
@pytest.mark.parametrize("weighted", [False, True])
def test_one_walk(lib, lens, Hq, Hkv, d, w, weighted):
    assert route(lib, lens, Hq, Hkv, d, w).stats_waves == 0
    rw = np.linspace(0.0, 1.0, w, dtype=np.float32) if weighted else None            # (the first weight is zero)
    if weighted and min(S for S in lens if S) == 1:
        rw = rw + np.float32(0.25)
    res, ref, _ = test_gpu_decode.run_and_check(lib, _wl(lens, Hq, Hkv, d, w), row_weights=rw)
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)


@pytest.mark.parametrize("lens,Hq,Hkv,d,w", TWO_WALKS)
@pytest.mark.parametrize("weighted", [False, True])
def test_two_walks(lib, lens, Hq, Hkv, d, w, weighted):
    assert route(lib, lens, Hq, Hkv, d, w).stats_waves > 0
    rw = np.linspace(0.0, 1.0, w, dtype=np.float32) if weighted else None            # (the first weight is zero)
    if weighted and min(S for S in lens if S) == 1:
        rw = rw + np.float32(0.25)
    res, ref, _ = test_gpu_decode.run_and_check(lib, _wl(lens, Hq, Hkv, d, w), row_weights=rw)
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=SCORE_RTOL, atol=1e-12)


@pytest.mark.parametrize("kind", ["ramp", "low_start_overflow"])
@pytest.mark.parametrize("lens,Hq,Hkv,d,w", [((900, 300), 8, 4, 128, 32), ((1100, 130), 16, 16, 64, 32)])
def test_moved_references(lib, kind, lens, Hq, Hkv, d, w):
    """Rows that outgrow a wavefront's reference, its first key's logit, by more than 2^40 in later tiles."""
    r = route(lib, lens, Hq, Hkv, d, w)
    assert r.stats_waves == 0
    wl = _wl(lens, Hq, Hkv, d, w)
    x = shaped_inputs(kind, wl, lib, seed=2)
    q, k, S = F64(x["q"]), F64(x["k"]), lens[0]
    moved = 0
    for h in range(Hq):
        lg = q[S - w:S, h] @ k[:S, h // (Hq // Hkv)].T / np.sqrt(d)
        for wave in range(r.window_waves):
            keys = np.arange(32 * wave, S - w)
            keys = keys[(keys // 32 - wave) % r.window_waves == 0]
            moved += int(np.sum(lg[:, keys[32:]].max(axis=1, initial=-np.inf) - lg[:, keys[0]] > 41 * np.log(2.0)))
    assert moved > 30, moved
    off, keep = x["seq_offsets"], x["keep_len"]
    q_win = window_queries(x["q"], off, wl.w)
    res = lib.decode_update_from_numpy(q_win, x["k"], x["v"], off, keep, wl.w)
    ref = orc.decode_update(F64(q_win.reshape(-1)).reshape(q_win.shape), F64(x["k"]), F64(x["v"]), off, wl.w, keep)
    parity.check_scores(res["scores"], ref)
    parity.check_index_sets(res["kept_idx"], ref, off, keep, wl.w)


def _planted(lens, Hq, Hkv, d, w, lib):
    """Inputs whose logits are the first component of the keys, in nats, for every row and head."""
    wl = _wl(lens, Hq, Hkv, d, w)
    x = parity.inputs(wl, lib)
    x["q"][:], x["k"][:] = 0, 0
    x["q"][:, :, 0] = synth.f32_to_bf16_bits(np.float32([np.sqrt(d)]))[0]
    return wl, x


def _set_logits(x, rows, log2s):
    x["k"][rows, :, 0] = synth.f32_to_bf16_bits(np.float32(np.asarray(log2s) * np.log(2.0)))[..., None]


def _update(lib, wl, x, row_weights=None):
    off, keep = x["seq_offsets"], x["keep_len"]
    q_win = window_queries(x["q"], off, wl.w)
    res = lib.decode_update_from_numpy(q_win, x["k"], x["v"], off, keep, wl.w, row_weights=row_weights)
    return res, orc.decode_update(F64(q_win.reshape(-1)).reshape(q_win.shape), F64(x["k"]), F64(x["v"]), off, wl.w, keep, row_weights=row_weights)


@pytest.mark.parametrize("weights", [None, 1.0, 2.0 ** 40])
def test_probabilities_down_to_the_smallest_normal_number(lib, weights):
    """Keys of probability 2^-101 in wavefronts whose first key lies below 2^-126: as the wavefront's last reference (its factor is then
    below the normal numbers), and in front of a tile that moves the reference by more than 126.  A logit of 102 (base 2) carries at most 130 roundings of its
    own, its denominator as many of logits near zero: 130 * 2^-24 * 102 ~ 8e-4."""
    lens, H, d, w = (1030,), 16, 64, 32
    r = route(lib, lens, H, H, d, w)
    assert r.stats_waves == 0 and r.window_waves >= 3 and r.window_tiles >= 2
    wl, x = _planted(lens, H, H, d, w, lib)
    tile, wave = np.arange(1030) // 32, (np.arange(1030) // 32) % r.window_waves
    logits = np.where(wave == 1, -100.0, 0.0)
    logits[tile == 2] = -100.0
    logits[32], logits[64] = -130.0, -135.0
    _set_logits(x, np.arange(1030), logits)
    rw = None if weights is None else np.linspace(0.0, weights, w, dtype=np.float32)
    res, ref = _update(lib, wl, x, rw)
    far = ref["scores"] < 2.0 ** -100
    assert far.sum() > 100
    far[[32, 64]] = False
    np.testing.assert_allclose(res["scores"][far], ref["scores"][far], rtol=8e-4, atol=0)
    np.testing.assert_allclose(res["scores"][~far], ref["scores"][~far], rtol=SCORE_RTOL, atol=2.0 ** -126)


@pytest.mark.parametrize("lens,Hq,Hkv,d,w", [((300,), 8, 4, 128, 40), ((700, 90), 16, 16, 64, 64)])
@pytest.mark.parametrize("kind", ["nan", "all_keys_minus_inf"])
def test_rows_without_a_sum_leave_later_keys_alone(lib, kind, lens, Hq, Hkv, d, w):
    """A window row that is NaN, or one that sees logits of -inf only, makes the scores of the keys it sees NaN and no others'."""
    assert route(lib, lens, Hq, Hkv, d, w).stats_waves == 0
    wl, x = _planted(lens, Hq, Hkv, d, w, lib)
    rng = np.random.default_rng(5)
    _set_logits(x, np.arange(sum(lens)), rng.normal(size=sum(lens)))
    S, bad = lens[0], lens[0] - w // 2 - 3
    if kind == "nan":
        x["q"][bad] = 0x7FC1
    else:                                                        # keys up to `bad`, which every row then finds at -inf
        x["q"][:, :, 1], x["k"][:bad + 1, :, 1] = 0x3F80, 0xFF80
    off, keep = x["seq_offsets"], x["keep_len"]
    res = lib.decode_update_from_numpy(window_queries(x["q"], off, wl.w), x["k"], x["v"], off, keep, wl.w)
    logits = F64(x["k"][:S, 0, 0]) * F64(x["q"][:1, 0, 0])[0] / np.sqrt(d)
    if kind != "nan":
        logits[:bad + 1] = -np.inf
    ref = np.zeros(S)
    for i in range(bad + 1, S):                                  # (the rows that later keys depend on)
        e = np.exp(logits[:i + 1] - logits[bad + 1:i + 1].max())
        ref[:i + 1] += e / e.sum() / w
    assert np.isnan(res["scores"][:bad + 1]).all()
    np.testing.assert_allclose(res["scores"][bad + 1:S], ref[bad + 1:], rtol=SCORE_RTOL, atol=1e-12)
    assert np.isfinite(res["scores"][S:]).all()
