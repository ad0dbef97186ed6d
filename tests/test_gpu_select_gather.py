"""The launch that selects and gathers a small batch (and the two launches around its limits): the kept rows are exactly what the
oracle selects on the scores the step returned, and every gathered byte is a copy."""
import numpy as np
import pytest

from oracle import pyr_oracle as orc
from paper_2405_12532_amd import synth
from tests import parity

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("hidden,pos", [(0, False), (72, True)])
@pytest.mark.parametrize("lens,Hkv,d,w", [
    ((1,), 1, 64, 1),                          # one row for 192 workgroups
    ((97,), 2, 64, 16),
    ((3, 0, 250, 64, 1), 2, 128, 48),          # sequences shorter than the window, an empty one
    ((40,) * 200, 1, 64, 16),                  # more sequences than workgroups wanted: one each
    ((4096,), 1, 64, 32),                      # eight keys a lane
    ((4097,), 1, 64, 32),                      # one token too long for the one launch
    ((366,) * 16, 4, 64, 20),                  # about as many bytes as it takes
    ((1200, 40, 700, 900), 8, 128, 64),        # more: two launches
])
def test_small_batches_select_and_gather(lib, lens, Hkv, d, w, hidden, pos):
    wl = synth.shrunk(synth.workload("cfg2"), lens, n_q_heads=2 * Hkv, n_kv_heads=Hkv, head_dim=d, w=w, hidden_dim=max(hidden, 8))
    x = parity.inputs(wl, lib)
    ids = np.random.default_rng(3).integers(0, 1 << 28, sum(lens)).astype(np.int32) if pos else None
    r = lib.prefill_layer_from_numpy(x, wl.w, hidden=x["hidden"] if hidden else None, pos=ids)
    off = x["seq_offsets"]
    ref = [orc.select_pvc(r["scores"][off[b]:off[b + 1]], w, x["keep_len"][b]) + off[b] for b in range(len(lens))]
    kept = np.concatenate(ref)
    assert np.array_equal(r["kept_idx"], kept)
    assert r["out_offsets"].tolist() == np.concatenate([[0], np.cumsum(x["keep_len"])]).tolist()
    assert np.array_equal(r["k_out"], x["k"][kept]) and np.array_equal(r["v_out"], x["v"][kept])
    if hidden:
        assert np.array_equal(r["hidden_out"], x["hidden"][kept])
    if pos:
        assert np.array_equal(r["pos_out"], ids[kept])
