"""Attention and scores of a small prefill batch in one launch (pyr_diag_layer says for which), at the edges of its cut: tiles of 32 keys, two, four
and eight of them a wavefront, in four wavefronts (one group of the attention tile) and eight (two groups), fewer rows of partial sums than tasks and as many,
more of them than the strip walk has.  And the strip walk, which the same batches no longer reach through a layer, by itself.  Against the float64 oracle;
scores to the bound derived in test_gpu_score_ranges."""
import itertools

import numpy as np
import pytest

from oracle import pyr_oracle as orc
from paper_2405_12532_amd import binding, synth
from tests import parity, test_gpu_layer, test_gpu_score_ranges as ranges
from tests.routes import LISTS, MI355X, ONE_GROUP, TWO_GROUPS, route

torch = pytest.importorskip("torch")

BATCHES = [                                                # ..., attention kernel, rows of partial sums
    ((40,), 1, 1, 64, 16, TWO_GROUPS, 1),                  # one task
    ((300, 0, 120, 1), 4, 4, 64, 16, TWO_GROUPS, 4),       # an empty sequence, one shorter than a tile
    ((512,), 4, 4, 128, 32, TWO_GROUPS, 4),                # two tiles a wavefront at most
    ((513,), 4, 2, 128, 33, TWO_GROUPS, 8),                # ... more; a row block of one row
    ((1024,), 4, 4, 64, 16, TWO_GROUPS, 4),
    ((1025, 31), 4, 4, 64, 16, TWO_GROUPS, 4),
    ((2047,), 4, 2, 128, 20, TWO_GROUPS, 4),
    ((2048,), 4, 2, 64, 64, TWO_GROUPS, 8),                # the longest
    ((1900,), 32, 32, 128, 64, TWO_GROUPS, 32),            # rows where the row statistics would lie; two tasks each
    ((256,) * 24, 8, 8, 128, 32, ONE_GROUP, 8),
    ((257,) * 24, 8, 8, 128, 32, ONE_GROUP, 8),
    ((512,) * 40, 4, 4, 64, 20, ONE_GROUP, 4),
    ((513,) * 40, 4, 4, 64, 20, ONE_GROUP, 4),
    ((1024,) * 8, 8, 8, 128, 16, ONE_GROUP, 8),            # the longest with one group
    ((900, 1024, 500) * 6, 4, 4, 128, 16, ONE_GROUP, 4),
    ((90, 33, 64), 40, 40, 128, 48, ONE_GROUP, 40),        # a sequence shorter than the window
    ((200,) * 3, 24, 24, 128, 128, ONE_GROUP, 32),
    ((400, 300, 500), 8, 2, 64, 100, TWO_GROUPS, 16),      # GQA 4: tasks in turn over two KV heads
    ((700, 650), 6, 2, 128, 70, TWO_GROUPS, 18),           # ... GQA 3, a row per task
]
APART = [((2049,), 4, 4, 64, 16), ((64,) * 64 + (2049,), 4, 4, 64, 16), ((359,) * 64, 32, 32, 128, 64), ((2048,), 32, 32, 128, 64), ((700,) * 100, 8, 8, 64, 16)]


def _rows(lens, Hq, Hkv, d, w, **device):
    off = torch.tensor([0] + list(itertools.accumulate(lens)), dtype=torch.int32)
    return binding.diag_layer(binding.make_shape(len(lens), sum(lens), max(lens), Hq, Hkv, d), off, w, **device)


def test_which_batches():
    for *batch, kernel, rows in BATCHES:
        assert (route(binding, *batch, **MI355X).attention, _rows(*batch, **MI355X)) == (kernel, rows), batch
    for batch in APART:
        assert _rows(*batch, **MI355X) == 0, batch
    for *batch, kernel, rows in ODD_ROWS:
        assert (route(binding, *batch, **MI355X).attention, _rows(*batch, **MI355X)) == (kernel, rows), batch
    off = torch.tensor([0, 5000], dtype=torch.int32)       # a max_seqlen without room for partial sums
    assert binding.diag_layer(binding.make_shape(1, 5000, 5000, 4, 4, 64), off, 16, **MI355X) == 0
    with pytest.raises(binding.PyrError):
        binding.diag_layer(binding.make_shape(1, 5000, 5000, 4, 4, 64), off, 0, **MI355X)


@pytest.mark.gpu
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("lens,Hq,Hkv,d,w,kernel,rows", BATCHES)
def test_one_launch_against_the_oracle(lib, lens, Hq, Hkv, d, w, kernel, rows, weighted):
    assert _rows(lens, Hq, Hkv, d, w) == rows
    rw = np.linspace(0.0, 1.0, w, dtype=np.float32) if weighted else None
    wl = ranges._wl(lens, Hq, Hkv, d, w)
    out_rows = test_gpu_layer.sample_rows(wl, 24, 3) if sum(lens) * Hq > 30000 else None
    res, ref, _ = test_gpu_layer.run_and_check(lib, wl, row_weights=rw, out_rows=out_rows)
    np.testing.assert_allclose(res["scores"], ref["scores"], rtol=ranges.SCORE_RTOL, atol=1e-12)


@pytest.mark.gpu
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("lens,Hq,Hkv,d,w", ranges.SHAPES + [batch[:5] for batch in ranges.ORDERS])
def test_strip_walk_by_itself(lib, lens, Hq, Hkv, d, w, weighted):
    x = parity.inputs(ranges._wl(lens, Hq, Hkv, d, w), lib, want_hidden=False)
    q, k, v = (lib.to_device_bf16(x[n]) for n in ("q", "k", "v"))
    off_h = torch.from_numpy(np.ascontiguousarray(x["seq_offsets"], dtype=np.int32))
    shape = lib.make_shape(len(lens), sum(lens), max(lens), Hq, Hkv, d)
    lse = torch.empty(sum(lens), Hq, dtype=torch.float32, device="cuda")
    scores = torch.empty(sum(lens), dtype=torch.float32, device="cuda")
    lib.attention(q, k, v, off_h.cuda(), off_h, shape, 0.0, torch.empty_like(q), lse, torch.empty(len(lens) + 1, dtype=torch.int32, device="cuda"))
    rw = np.linspace(0.0, 1.0, w, dtype=np.float32) if weighted else None
    if weighted:
        lib.score_weighted(q, k, lse, off_h.cuda(), off_h, shape, w, 0.0, torch.from_numpy(rw).cuda(), scores)
    else:
        lib.score(q, k, lse, off_h.cuda(), off_h, shape, w, 0.0, scores)
    ref = orc.prefill_layer(*(synth.bf16_bits_to_f64(x[n]) for n in ("q", "k", "v")), x["seq_offsets"], w, x["keep_len"], row_weights=rw)
    np.testing.assert_allclose(scores.cpu().numpy(), ref["scores"], rtol=ranges.SCORE_RTOL, atol=1e-12)


ODD_ROWS = [BATCHES[i] for i in (1, 3, 8, 9, 15, 18)] + [(*APART[2], ONE_GROUP, 0), (*APART[3], TWO_GROUPS, 0), ((1024,) * 16, 16, 16, 128, 48, LISTS, 0)]


def _attention_and_scores(lib, x, lens, d, w):
    """the layer's scores and output, and those of the separate calls"""
    q, k, v = (lib.to_device_bf16(x[n]) for n in ("q", "k", "v"))
    off_h, keep_h = (torch.from_numpy(np.ascontiguousarray(x[n], dtype=np.int32)) for n in ("seq_offsets", "keep_len"))
    off_d, T, n_kept = off_h.cuda(), sum(lens), int(keep_h.sum())
    shape = lib.make_shape(len(lens), T, max(lens), q.shape[1], k.shape[1], d)
    ws_bytes = lib.workspace_bytes(shape, w)
    scores, apart = (torch.empty(T, dtype=torch.float32, device="cuda") for _ in range(2))
    out, out_apart, lse = torch.empty_like(q), torch.empty_like(q), torch.empty(T, q.shape[1], dtype=torch.float32, device="cuda")
    kept, out_off = torch.empty(n_kept, dtype=torch.int32, device="cuda"), torch.empty(len(lens) + 1, dtype=torch.int32, device="cuda")
    lib.prefill_layer(q, k, v, off_d, off_h, shape, w, 0.0, keep_h.cuda(), keep_h, out, scores, kept, out_off, None, None,
                      torch.empty(ws_bytes, dtype=torch.uint8, device="cuda"), ws_bytes)
    lib.attention(q, k, v, off_d, off_h, shape, 0.0, out_apart, lse, torch.empty(len(lens) + 1, dtype=torch.int32, device="cuda"))
    lib.score(q, k, lse, off_d, off_h, shape, w, 0.0, apart)
    assert torch.equal(out.view(torch.int16), out_apart.view(torch.int16))
    return scores.cpu().numpy(), apart.cpu().numpy(), out.float().cpu().numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["keys_in_front_minus_inf", "nan_row", "row_of_minus_inf"])
@pytest.mark.parametrize("lens,Hq,Hkv,d,w,kernel,rows", ODD_ROWS)
def test_one_launch_and_two_agree_on_odd_rows(lib, lens, Hq, Hkv, d, w, kernel, rows, kind):
    """Logits of -inf at the keys in front, one or more tiles of them, are keys without weight, and a window row that is NaN, or that sees
    logits of -inf only, makes the scores of the keys it sees NaN and no others': in a layer of one launch, of two, and in the separate calls."""
    assert (route(lib, lens, Hq, Hkv, d, w).attention, _rows(lens, Hq, Hkv, d, w)) == (kernel, rows)
    wl = ranges._wl(lens, Hq, Hkv, d, w)
    x = parity.inputs(wl, lib, want_hidden=False)
    off = x["seq_offsets"]
    x["q"][:, :, 1], x["k"][:, :, 1] = 0x3F80, 0                       # 1, 0
    S = lens[0]
    bad = S - w // 2 - 3                                               # a window row of the first sequence
    if kind == "keys_in_front_minus_inf":
        for r0, n in zip(off, lens):
            x["k"][r0:r0 + max(0, min(n - w, 77)), :, 1] = 0xFF80
    elif kind == "nan_row":
        x["q"][bad] = 0x7FC1
    else:
        x["k"][:bad + 1, :, 1] = 0xFF80
    scores, apart, out = _attention_and_scores(lib, x, lens, d, w)
    if kind == "keys_in_front_minus_inf":
        with np.errstate(invalid="ignore"):
            ref = orc.prefill_layer(*(synth.bf16_bits_to_f64(x[n]) for n in ("q", "k", "v")), off, w, x["keep_len"], out_rows=[np.arange(max(0, n - 8), n) for n in lens])
        np.testing.assert_allclose(scores, ref["scores"], rtol=ranges.SCORE_RTOL, atol=1e-12)
        parity.check_out(synth.f32_to_bf16_bits(out), ref, off, synth.bf16_bits_to_f64)
    else:
        assert np.isnan(scores[:bad + 1]).all() and np.isfinite(scores[bad + 1:]).all()
    np.testing.assert_allclose(scores, apart, rtol=ranges.SCORE_RTOL, atol=1e-12)
