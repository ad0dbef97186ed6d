"""The launch that selects and gathers a small batch (and the two launches around its limits): the kept rows are exactly what the
oracle selects on the scores the step returned, and every gathered byte is a copy.  Every batch asserts which of the two it gets."""
import numpy as np
import pytest

from oracle import pyr_oracle as orc
from paper_2405_12532_amd import synth
from tests import parity, test_gpu_decode
from tests.routes import launches, route

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LAYERS = [                                     # whether one launch does both, without and with hidden rows of 144 bytes
    ((1,), 1, 64, 1, True, True),                          # one row for 192 workgroups
    ((97,), 2, 64, 16, True, True),
    ((3, 0, 250, 64, 1), 2, 128, 48, True, True),          # sequences shorter than the window, an empty one
    ((40,) * 200, 1, 64, 16, True, True),                  # more sequences than workgroups wanted: one each
    ((4096,), 1, 64, 32, True, True),                      # eight keys a lane
    ((4097,), 1, 64, 32, False, False),                    # one token too long for the one launch
    ((229,) * 16, 4, 64, 20, True, True),                  # 12 workgroups per sequence; 160 rows each, 2.62 and 2.99 MB
    ((230,) * 16, 4, 64, 20, True, False),                 # 161 rows: 3.01 MB with the hidden rows
    ((261,) * 16, 4, 64, 20, True, False),                 # 183 rows, 2.998 MB
    ((263,) * 16, 4, 64, 20, False, False),                # 184 rows, 3.015 MB
    ((263,) + (20,) * 15, 4, 64, 20, False, False),        # ... counted as if all kept as many
    ((1200, 40, 700, 900), 8, 128, 64, False, False),
]
UPDATES = [                                    # rows of partial sums: some, added in their own launch; one launch or two behind them
    ((300, 97), 4, 2, 64, 32, True, False, True),
    ((40, 3, 0, 64), 16, 4, 128, 48, True, False, True),
    ((2000, 1100), 8, 2, 64, 64, True, False, True),
    ((200, 150), 48, 2, 64, 64, True, True, True),
    ((1500,), 16, 1, 64, 64, True, True, True),
    ((1030,), 32, 32, 64, 64, True, True, False),
    ((2049,), 4, 4, 64, 16, False, False, True),           # two walks
    ((2500, 300), 64, 1, 64, 64, True, False, True),       # ... their score pass split
]


def workload(lens, Hq, Hkv, d, w, hidden=0):
    return synth.shrunk(synth.workload("cfg2"), lens, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, w=w, hidden_dim=max(hidden, 8))


def merged(lib, lens, Hkv, d, w, hidden, **device):
    keep = parity.keep_lens(workload(lens, 2 * Hkv, Hkv, d, w))
    return launches(lib, lens, 2 * Hkv, Hkv, d, w, False, keep, 4 * Hkv * d + 2 * hidden, **device).select_split > 0


def update_launches(lib, lens, Hq, Hkv, d, w, **device):
    keep = parity.keep_lens(workload(lens, Hq, Hkv, d, w))
    r = launches(lib, lens, Hq, Hkv, d, w, True, keep, 4 * Hkv * d, **device)
    return route(lib, lens, Hq, Hkv, d, w, **device).window_groups > 1, bool(r.sums), r.select_split > 0


@pytest.mark.parametrize("hidden,pos", [(0, False), (72, True)])      # 144 bytes: lanes of a wavefront in several rows and sources
@pytest.mark.parametrize("lens,Hkv,d,w,plain,with_hidden", LAYERS)
def test_small_batches_select_and_gather(lib, lens, Hkv, d, w, plain, with_hidden, hidden, pos):
    assert merged(lib, lens, Hkv, d, w, hidden) == (with_hidden if hidden else plain)
    wl = workload(lens, 2 * Hkv, Hkv, d, w, hidden)
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


@pytest.mark.parametrize("hidden", [8, 72, 4104])                      # rows of one 16-byte piece, of nine, of 513
@pytest.mark.parametrize("lens", [(300,), (100, 7, 220), (5,) * 100])
def test_rows_of_any_length_by_themselves(lib, lens, hidden):
    """Hidden rows without K and V: one source, whose rows are shorter or longer than what a wavefront moves at a time."""
    wl = workload(lens, 4, 2, 64, 16, hidden)
    x = parity.inputs(wl, lib)
    n_kept, T = int(x["keep_len"].sum()), sum(lens)
    assert (launches(lib, lens, 4, 2, 64, 16, False, x["keep_len"], 2 * hidden).select_split > 0) == (max(x["keep_len"]) * len(lens) * 2 * hidden <= 3000000)
    q, k, v, h = (lib.to_device_bf16(x[n]) for n in ("q", "k", "v", "hidden"))
    off_h, keep_h = (torch.from_numpy(np.ascontiguousarray(x[n], dtype=np.int32)) for n in ("seq_offsets", "keep_len"))
    shape = lib.make_shape(len(lens), T, max(lens), 4, 2, 64)
    ws = torch.empty(lib.workspace_bytes(shape, 16), dtype=torch.uint8, device="cuda")
    out, scores = torch.empty_like(q), torch.empty(T, dtype=torch.float32, device="cuda")
    kept, out_off = torch.empty(n_kept, dtype=torch.int32, device="cuda"), torch.empty(len(lens) + 1, dtype=torch.int32, device="cuda")
    h_out = torch.full((n_kept + 1, hidden), -7.0, dtype=torch.bfloat16, device="cuda")
    lib.prefill_layer_fused(q, k, v, off_h.cuda(), off_h, shape, 16, 0.0, keep_h.cuda(), keep_h, None, h, 2 * hidden, None, out, scores, kept, out_off,
                            None, None, h_out, None, ws, ws.numel())
    torch.cuda.synchronize()
    assert np.array_equal(lib.to_host_bits(h_out)[:n_kept], x["hidden"][kept.cpu().numpy()])
    assert bool((h_out[n_kept] == -7.0).all()), "nothing is written past the kept rows"


@pytest.mark.parametrize("lens,Hq,Hkv,d,w,rows,sums,one", UPDATES)
def test_updates_add_select_and_gather(lib, lens, Hq, Hkv, d, w, rows, sums, one):
    assert update_launches(lib, lens, Hq, Hkv, d, w) == (rows, sums, one)
    res, _, x = test_gpu_decode.run_and_check(lib, workload(lens, Hq, Hkv, d, w), with_pos=True)
    off = x["seq_offsets"]
    kept = [orc.select_pvc(res["scores"][off[b]:off[b + 1]], w, x["keep_len"][b]) + off[b] for b in range(len(lens))]
    assert np.array_equal(res["kept_idx"], np.concatenate(kept))


def test_offsets_written_in_place(lib):
    """One sequence whose offsets are replaced by the kept rows': workgroups that share the selection must not find them already replaced."""
    lens, Hkv, d, w = (900,), 2, 64, 32
    x = parity.inputs(workload(lens, 2 * Hkv, Hkv, d, w), lib)
    want = lib.prefill_layer_from_numpy(x, w)
    q, k, v = (lib.to_device_bf16(x[n]) for n in ("q", "k", "v"))
    off_h, keep_h = (torch.from_numpy(np.ascontiguousarray(x[n], dtype=np.int32)) for n in ("seq_offsets", "keep_len"))
    n_kept, shape = int(keep_h.sum()), lib.make_shape(1, 900, 900, 2 * Hkv, Hkv, d)
    off_d, keep_d = off_h.cuda(), keep_h.cuda()
    ws = torch.empty(lib.workspace_bytes(shape, w), dtype=torch.uint8, device="cuda")
    out, scores = torch.empty_like(q), torch.empty(900, dtype=torch.float32, device="cuda")
    kept, k_out = torch.empty(n_kept, dtype=torch.int32, device="cuda"), torch.empty(n_kept, Hkv, d, dtype=torch.bfloat16, device="cuda")
    v_out = torch.empty_like(k_out)
    for _ in range(20):
        off_d.copy_(off_h)
        lib.prefill_layer(q, k, v, off_d, off_h, shape, w, 0.0, keep_d, keep_h, out, scores, kept, off_d, k_out, v_out, ws, ws.numel())
        assert off_d.tolist() == [0, n_kept]
        assert np.array_equal(kept.cpu().numpy(), want["kept_idx"])
        assert np.array_equal(lib.to_host_bits(k_out), want["k_out"]) and np.array_equal(lib.to_host_bits(v_out), want["v_out"])
