"""The attention kernels one by one against plain PyTorch in float64: a 128-row tile per workgroup with its keys in one group
(many tiles) or two (few tiles), and the 256-row kernel that walks lists of paired tiles (d = 128, long tiles).  Which of them
runs follows from the batch alone (pick_kernel in attention.hip); every test asserts that its batch gets the one it is for."""
import math

import numpy as np
import pytest

from paper_2405_12532_amd import synth
from tests import test_gpu_large_logits, test_gpu_layer
from tests.routes import LISTS, ONE_GROUP, TWO_GROUPS, route

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _batch(lens, Hq, Hkv, d, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    T = sum(lens)
    return [torch.randn((T, h, d), generator=gen, device="cuda").to(torch.bfloat16) for h in (Hq, Hkv, Hkv)]


def _reference(q, k, v, scale=None):
    """Causal attention of one sequence in float64: out [S, Hq, d], log2 of the denominators [S, Hq]."""
    S, Hq, d = q.shape
    Hkv = k.shape[1]
    g = Hq // Hkv
    qh = q.double().permute(1, 0, 2).reshape(Hkv, g * S, d).contiguous()
    kh, vh = k.double().permute(1, 2, 0).contiguous(), v.double().permute(1, 0, 2).contiguous()
    x = (torch.bmm(qh, kh) * (scale or 1 / math.sqrt(d))).reshape(Hkv, g, S, S)
    x.masked_fill_(torch.ones(S, S, dtype=torch.bool, device=q.device).triu(1), -math.inf)
    out = torch.bmm(torch.softmax(x, dim=3).reshape(Hkv, g * S, S), vh).reshape(Hq, S, d).permute(1, 0, 2)
    return out, (torch.logsumexp(x, dim=3) / math.log(2.0)).reshape(Hq, S).t()


def _check(lib, lens, Hq, Hkv, d, seed=1, every=1, masked=(), scale=None):
    """masked: positions of every sequence whose keys nobody may see, a logit of -inf by way of one head dimension."""
    q, k, v = _batch(lens, Hq, Hkv, d, seed)
    if scale:
        q *= 1 / (scale * math.sqrt(d))            # (the same logits)
    T = sum(lens)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    if len(masked):
        q[:, :, 0], k[:, :, 0] = 1.0, 0.0
        for r0, r1 in zip(off[:-1], off[1:]):
            k[[int(r0) + j for j in masked if r0 + j < r1], :, 0] = -math.inf
    off_h = torch.from_numpy(off)
    shape = lib.make_shape(len(lens), T, max(lens), Hq, Hkv, d)
    out, lse = torch.full_like(q, 7.0), torch.full((T, Hq), 7.0, dtype=torch.float32, device="cuda")
    lib.attention(q, k, v, off_h.cuda(), off_h, shape, scale or 0.0, out, lse, torch.empty(len(lens) + 1, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    vmax = float(v.abs().max())
    for b in range(0, len(lens), every):
        r0, r1 = int(off[b]), int(off[b + 1])
        if r0 == r1:
            continue
        o, den = _reference(q[r0:r1], k[r0:r1], v[r0:r1], scale)
        if 0 in masked:                            # rows that see none but masked keys have no output
            blind = next(j for j in range(r1 - r0 + 1) if j not in masked)
            assert bool(out[r0:r0 + blind].isnan().all()) and bool((lse[r0:r0 + blind] == -math.inf).all())
            r0, o, den = r0 + blind, o[blind:], den[blind:]
            if r0 >= r1:
                continue
        # one rounding of the result to bf16, bf16 probabilities that sum to one, fp32 sums
        err = (out[r0:r1].double() - o).abs()
        assert bool((err <= 2.0 ** -8 * (o.abs() + vmax) + 1e-3).all()), (b, float(err.max()))
        # logits of at most about 10: 128 fp32 products and sums, times log2(e)
        assert float((lse[r0:r1].double() - den).abs().max()) < 128 * 2.0 ** -24 * 10 * 1.5, b


EDGES = (1, 2, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 160, 191, 192, 193, 255, 256, 257, 320, 383, 384, 385)


TWO_GROUP_EDGES = [([S], 64) for S in EDGES] + [([S, 700], 128) for S in EDGES]      # (at d = 128 short prompts alone get one group)


@pytest.mark.parametrize("lens,d", TWO_GROUP_EDGES, ids=lambda x: str(x))
def test_two_groups_edges(lib, lens, d):
    """A few tiles only: two groups of four wavefronts share a tile's keys (the second has none up to 64)."""
    assert route(lib, lens, 4, 2, d).attention == TWO_GROUPS
    _check(lib, lens, 4, 2, d, seed=lens[0])


ONE_GROUP_EDGES = [(list(EDGES) * 4 + [0, 500, 0], Hq, Hkv, d) for d, Hq, Hkv in ((64, 24, 8), (128, 24, 8), (64, 11, 11), (128, 36, 12))]
ONE_GROUP_EDGES += [([S], 4, 2, 128) for S in (1, 32, 33, 64, 65, 128, 129, 192, 320)]


@pytest.mark.parametrize("lens,Hq,Hkv,d", ONE_GROUP_EDGES)
def test_one_group_edges(lib, lens, Hq, Hkv, d):
    """All edge lengths in one ragged batch, several times over (and empty sequences): enough tiles for one group each; and the short
    prompts that two groups are too many for."""
    assert route(lib, lens, Hq, Hkv, d).attention == ONE_GROUP
    _check(lib, lens, Hq, Hkv, d, seed=d + Hq, every=3)


TILE_BATCHES = [
    ([300] * 40, 16, 16, 64, ONE_GROUP),       # equal lengths: no offsets read
    ([2500] * 2, 8, 8, 64, TWO_GROUPS),        # 20 tiles
    ([3000, 1, 1700], 8, 2, 64, TWO_GROUPS),
    ([1100] * 6, 32, 8, 128, ONE_GROUP),       # grouped heads
    ([200] * 64, 32, 32, 128, ONE_GROUP),
    ([2048], 32, 32, 128, TWO_GROUPS),         # two workgroups in turn on a compute unit
    ([1900, 700, 64], 12, 12, 128, TWO_GROUPS),     # heads that do not divide over the XCDs
]


@pytest.mark.parametrize("lens,Hq,Hkv,d,kernel", TILE_BATCHES)
def test_tile_kernels(lib, lens, Hq, Hkv, d, kernel):
    assert route(lib, lens, Hq, Hkv, d).attention == kernel
    _check(lib, lens, Hq, Hkv, d, every=max(1, len(lens) // 6))


LONG_BATCHES = [
    ([512] * 64, 32, 32),                      # two tiles: one pair
    ([700] * 24, 32, 32),                      # three: a pair and the one in the middle, places that move on by one
    ([1200] * 16, 32, 8),                      # five, grouped heads
    ([1700] * 16, 16, 16),                     # seven
    ([4096], 32, 32),
    ([6000, 5000, 300, 8000, 200, 0, 1], 32, 8),    # ragged, sequences of one tile and of none
    ([1500] * 700, 8, 8),                      # more than 64 items per workgroup: its table of items is moved along
    ([1792, 1536] * 350, 8, 8),                # ... of a ragged batch
]
TABLE = 64                                     # items a workgroup's table holds


@pytest.mark.parametrize("lens,Hq,Hkv", LONG_BATCHES)
def test_long_tile_kernel(lib, lens, Hq, Hkv):
    r = route(lib, lens, Hq, Hkv, 128)
    assert r.attention == LISTS and (r.attention_items > TABLE) == (len(lens) > 600)
    _check(lib, lens, Hq, Hkv, 128, every=max(1, len(lens) // 30))


RENEWAL_BATCHES = [((1024,) * 16, 16, 128, LISTS), ((800,), 4, 128, TWO_GROUPS), ((300,) * 60, 8, 64, ONE_GROUP), ((1024,) * 3, 32, 128, ONE_GROUP)]


@pytest.mark.parametrize("kind", ["ramp", "low_start", "low_start_overflow"])
@pytest.mark.parametrize("lens,Hq,d,kernel", RENEWAL_BATCHES)
def test_exponent_reference_renewal(lib, kind, lens, Hq, d, kernel):
    """Rows that outgrow the exponent reference taken from their first 32 keys, in each kernel (long tiles, two groups - which renew it
    one by one -, one group), against the oracle."""
    assert route(lib, lens, Hq, Hq, d).attention == kernel
    wl = synth.shrunk(synth.workload("cfg1"), lens, n_q_heads=Hq, n_kv_heads=Hq, head_dim=d, w=32, keep_fixed=0,
                      keep_num=7, keep_den=10, hidden_dim=0)
    x = test_gpu_large_logits.shaped_inputs(kind, wl, lib)
    assert test_gpu_large_logits.rows_outgrowing_the_reference(x, wl) > 100
    test_gpu_layer.run_and_check(lib, wl, x=x, hidden=False)


LISTED_BATCHES = [
    ([3000] + [17, 0, 130] * 100, 8, 8, 64),   # 301 sequences: two rounds of the search, empty ones among them
    ([40] * 63 + [0, 6000], 12, 12, 64),       # 65, heads that take turns over the XCDs
    ([1] * 4200 + [700] + [0] * 70 + [129], 36, 12, 64),      # three rounds, empty sequences in a row
    ([9000] + [100] * 63, 6, 2, 64),           # 64: one round; fewer heads than XCDs
    ([4000] + [64] * 260, 16, 8, 128),
    ([8000, 8000] + [33] * 500, 4, 1, 128),
]


@pytest.mark.parametrize("lens,Hq,Hkv,d", LISTED_BATCHES)
def test_list_of_tiles(lib, lens, Hq, Hkv, d):
    """One long sequence among many short ones: the tile kernel's grid would be mostly empty, and it works on a list."""
    assert route(lib, lens, Hq, Hkv, d).attention_listed == 1
    _check(lib, lens, Hq, Hkv, d, every=1 if len(lens) < 100 else 97)


MASKED_BATCHES = [
    ([300], 4, 2, 64, TWO_GROUPS),             # all the second group has seen of a row may be masked keys
    ([800], 4, 4, 128, TWO_GROUPS),
    ([2048], 32, 32, 128, TWO_GROUPS),
    ([300] * 60, 8, 8, 64, ONE_GROUP),
    ([1100] * 6, 32, 8, 128, ONE_GROUP),
    ([2048] * 32, 32, 32, 128, LISTS),
]


@pytest.mark.parametrize("lens,Hq,Hkv,d,kernel", MASKED_BATCHES)
def test_masked_keys(lib, lens, Hq, Hkv, d, kernel):
    """Infinitely negative logits weigh nothing wherever they lie beyond a row's first 32 keys: a group's whole first tile, a half
    of a tile, every other key."""
    assert route(lib, lens, Hq, Hkv, d).attention == kernel
    masked = [*range(40, 200), *range(256, 288), *range(301, 700, 2)]
    _check(lib, lens, Hq, Hkv, d, masked=masked, every=max(1, len(lens) // 4))


@pytest.mark.parametrize("first", [32, 70, 200])
@pytest.mark.parametrize("lens,Hq,Hkv,d,kernel", MASKED_BATCHES)
def test_masked_keys_in_front(lib, lens, Hq, Hkv, d, kernel, first):
    """... and where they are all of a row's first 32 keys, which the exponent reference is taken from.  Also with a softmax scale whose
    product with the lowest finite reference is no finite number."""
    assert route(lib, lens, Hq, Hkv, d).attention == kernel
    masked = [*range(first), *range(256, 288)]
    for scale in (None, 1.0):
        _check(lib, lens, Hq, Hkv, d, masked=masked, every=max(1, len(lens) // 4), scale=scale)
