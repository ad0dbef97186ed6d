"""The batches of the GPU tests get the kernels those tests are for on an MI355X (host only: pyr_diag_route)."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2405_12532_amd import binding
from tests import test_gpu_attention_kernels as att, test_gpu_score_ranges as ranges
from tests.routes import COUNTED, EQUAL, LISTS, MI355X, ONE_GROUP, PLACES, SEQ_PER_XCD, TWO_GROUPS, launches, route


def _kernel(lens, Hq, Hkv, d):
    return route(binding, lens, Hq, Hkv, d, **MI355X)


def test_attention_kernels():
    for lens, d in att.TWO_GROUP_EDGES:
        assert _kernel(lens, 4, 2, d).attention == TWO_GROUPS, (lens, d)
    for batch in att.ONE_GROUP_EDGES:
        assert _kernel(*batch).attention == ONE_GROUP, batch
    for *batch, kernel in att.TILE_BATCHES + att.MASKED_BATCHES:
        assert _kernel(*batch).attention == kernel, batch
    for lens, Hq, Hkv in att.LONG_BATCHES:
        r = _kernel(lens, Hq, Hkv, 128)
        assert r.attention == LISTS and (r.attention_items > att.TABLE) == (len(lens) > 600), (len(lens), r.attention_items)
    for lens, Hq, d, kernel in att.RENEWAL_BATCHES:
        assert _kernel(lens, Hq, Hq, d).attention == kernel, (lens, Hq, d)
    for batch in att.LISTED_BATCHES:
        assert _kernel(*batch).attention_listed == 1, batch[1:]


def test_score_walks():
    for *batch, order, one in ranges.ORDERS:
        assert (route(binding, *batch, **MI355X).score_order, ranges._one_launch(binding, *batch, **MI355X) > 0) == (order, one), (len(batch[0]), batch[1:])
    for *batch, order, groups in ranges.SPLIT:
        r = route(binding, *batch, **MI355X)
        assert (ranges._one_launch(binding, *batch, **MI355X), r.score_order, r.score_groups) == (0, order, groups), (len(batch[0]), batch[1:])
    assert all(ranges._one_launch(binding, *batch, **MI355X) > 0 for batch in ranges.SHAPES)
    for *batch, stats, scores in ranges.UPDATE_ORDERS:
        r = launches(binding, *batch, generation=True, **MI355X)
        assert (r.stats_order, r.window_order) == (stats, scores), (len(batch[0]), batch[1:], r.stats_order, r.window_order)
    for *batch, counts in ranges.FOLDS:
        assert ranges.fold_ranges(binding, *batch, **MI355X) == counts, (batch, ranges.fold_ranges(binding, *batch, **MI355X))
    lens, H, d, w = ranges.LOOSE
    assert route(binding, lens, H, H, d, w, **MI355X).score_groups > 1


def test_route_arguments():
    off = torch.tensor([0, 100], dtype=torch.int32)
    shape = binding.make_shape(1, 100, 100, 4, 2, 64)
    assert binding.diag_route(shape, off, 16, 256, 8).score_groups >= 1
    for args in ((shape, off, 0, 256, 8), (shape, off, 16, 256, 0), (shape, off, 16, -1, 8)):
        with pytest.raises(binding.PyrError):
            binding.diag_route(*args)
    lib = binding.load()
    assert lib.pyr_diag_route(ctypes.byref(shape), off.data_ptr(), 16, 256, 8, None) == -1
    assert lib.pyr_diag_route(ctypes.byref(shape), None, 16, 256, 8, ctypes.byref(binding.PyrRoute())) == -1
    keep = torch.tensor([101], dtype=torch.int32)
    for args in ((shape, off, 16, 0, None, 0, 256, 0), (shape, off, 0, 0, None, 0, 256, 8), (shape, off, 16, 1, keep, 256, 256, 8),
                 (shape, off, 16, 1, None, 8, 256, 8)):
        with pytest.raises(binding.PyrError):
            binding.diag_launches(*args)
    assert lib.pyr_diag_launches(ctypes.byref(shape), off.data_ptr(), 16, 0, None, 0, 256, 8, None) == -1
    with pytest.raises(binding.PyrError):
        binding.diag_update(shape, off, 0, 256, 8)
    assert lib.pyr_diag_update(ctypes.byref(shape), off.data_ptr(), 16, 256, 8, None) == -1
    empty = binding.make_shape(0, 0, 0, 4, 2, 64)
    assert binding.diag_update(empty, torch.zeros(1, dtype=torch.int32), 16, 256, 8) == -1
    assert binding.diag_launches(empty, torch.zeros(1, dtype=torch.int32), 16, 1, None, 0, 256, 8).attention_units == 0
    assert binding.diag_route(empty, torch.zeros(1, dtype=torch.int32), 16, 256, 8).score_tiles == 0


@pytest.mark.parametrize("lens,Hq,Hkv,one", [
    ((1500,) * 24, 12, 12, False),                               # equal
    ((1500,) * 23 + (1499,), 12, 12, False),                     # nearly: as equal ones go
    (tuple(range(1477, 1501)), 12, 12, False),
    ((330,) * 20 + (264,) * 13, 8, 8, False),
    ((1280,) * 19 + (640,) * 4 + (512,), 12, 12, False),         # the longest has just under 9/8 of the mean's tiles ...
    ((1280,) * 19 + (640,) * 3 + (512,) * 2, 12, 12, True),      # ... and just over
    ((1500,) * 18 + (1499,), 12, 12, False),                     # 29 units an XCD, 28, ...
    ((1500,) * 27 + (1499,), 8, 8, True),
    (tuple(range(609, 3418, 175)), 8, 8, True),                  # unequal
    ((900,) * 30 + (300,) * 8, 8, 8, True),                      # 38 units
    ((900,) * 30 + (300,) * 9, 8, 8, False),                     # 39
])
def test_chunks_of_units_at_d64(lens, Hq, Hkv, one):
    """The units of an XCD go in one chunk by how unequal the sequences are, not by whether one of them differs from the rest."""
    assert _kernel(lens, Hq, Hkv, 64).attention != LISTS
    r = launches(binding, lens, Hq, Hkv, 64, **MI355X)
    assert r.attention_units == -(-len(lens) * Hkv // 8) and (r.attention_chunk == r.attention_units) == one


def test_generation_walks():
    from tests import test_gpu_window_scores as window
    for batch in window.ONE_WALK:
        r = route(binding, *batch, **MI355X)
        assert r.stats_waves == r.stats_tiles == r.stats_groups == 0, batch
    for batch in window.TWO_WALKS:
        assert route(binding, *batch, **MI355X).stats_waves > 0, batch
        assert window.task_order(binding, *batch, **MI355X)[0] == -1, batch
    for batches, order in ((window.BY_KV_HEAD, 1), (window.BY_QUERY_HEAD, 0)):
        for *batch, tasks in batches:
            assert window.task_order(binding, *batch, **MI355X) == (order, tasks), batch
    # measured, two walks / one (us): 115 / 127, 66 / 71, 145 / 159, and with other numbers of row blocks per KV head 34 / 31, 1073 / 900
    for *batch, walks in (((793,) * 10, 40, 40, 128, 100, 2), ((300,) * 52, 64, 8, 128, 32, 2), ((1518,) * 69, 32, 8, 64, 32, 2),
                          ((1537,), 32, 32, 128, 64, 1), ((2048,) * 64, 32, 32, 128, 64, 1)):
        assert (route(binding, *batch, **MI355X).stats_waves > 0) == (walks == 2), batch


def test_fused_steps():
    from tests import test_gpu_fused as fused
    for *batch, merged, split in fused.FUSED:
        assert fused.kinds(binding, *batch, **MI355X) == (merged, split), batch


def test_selection_and_gather():
    from tests import test_gpu_select_gather as small
    for lens, Hkv, d, w, plain, with_hidden in small.LAYERS:
        assert [small.merged(binding, lens, Hkv, d, w, hidden, **MI355X) for hidden in (0, 72)] == [plain, with_hidden], (lens, Hkv, d)
    for *batch, rows, sums, one in small.UPDATES:
        assert small.update_launches(binding, *batch, **MI355X) == (rows, sums, one), batch
