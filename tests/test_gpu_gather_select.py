"""GPU parity of the gather and selection kernels in isolation (bit-exact), through the C ABI."""
import numpy as np
import pytest

from oracle import pyr_oracle as orc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _gather_case(lib, n_src, n_kept, row_bytes, seed, two=False):
    rng = np.random.default_rng(seed)
    src = rng.integers(0, 256, size=(n_src, row_bytes), dtype=np.uint8)
    idx = np.sort(rng.choice(n_src, size=n_kept, replace=False)).astype(np.int32) if n_kept <= n_src else None
    d_src = torch.from_numpy(src).cuda()
    d_idx = torch.from_numpy(idx).cuda()
    d_dst = torch.full((max(n_kept, 1) + 1, row_bytes), 0xAB, dtype=torch.uint8, device="cuda")
    if two:
        src1 = rng.integers(0, 256, size=(n_src, row_bytes), dtype=np.uint8)
        d_src1 = torch.from_numpy(src1).cuda()
        d_dst1 = torch.full_like(d_dst, 0xCD)
        lib.compact2(d_src, d_dst, d_src1, d_dst1, row_bytes, d_idx, n_kept)
        torch.cuda.synchronize()
        assert np.array_equal(d_dst1.cpu().numpy()[:n_kept], orc.gather_rows(src1, idx))
        assert np.all(d_dst1.cpu().numpy()[n_kept:] == 0xCD)
    else:
        lib.compact(d_src, row_bytes, d_idx, n_kept, d_dst)
        torch.cuda.synchronize()
    got = d_dst.cpu().numpy()
    assert np.array_equal(got[:n_kept], orc.gather_rows(src, idx))
    assert np.all(got[n_kept:] == 0xAB), "nothing may be written past the kept rows"


@pytest.mark.parametrize("n_src,n_kept,row_bytes", [
    (1, 1, 16), (7, 3, 16), (100, 100, 48), (1000, 613, 1024), (513, 200, 2048), (300, 299, 8192),
    (257, 129, 10240), (64, 17, 16 * 1027),            # rows longer than one unrolled sweep, ragged tail
])
def test_gather_bit_exact(lib, n_src, n_kept, row_bytes):
    _gather_case(lib, n_src, n_kept, row_bytes, seed=n_src + row_bytes)


def test_gather_two_sources_one_launch(lib):
    _gather_case(lib, 700, 431, 8192, seed=5, two=True)
    _gather_case(lib, 9, 4, 32, seed=6, two=True)


def test_gather_many_rows_uses_the_stride_loop(lib):
    _gather_case(lib, 200000, 150001, 64, seed=7)


def test_gather_unsorted_and_repeated_indices(lib):
    rng = np.random.default_rng(11)
    src = rng.integers(0, 256, size=(50, 256), dtype=np.uint8)
    idx = rng.integers(0, 50, size=120).astype(np.int32)
    d_dst = torch.empty((120, 256), dtype=torch.uint8, device="cuda")
    lib.compact(torch.from_numpy(src).cuda(), 256, torch.from_numpy(idx).cuda(), 120, d_dst)
    torch.cuda.synchronize()
    assert np.array_equal(d_dst.cpu().numpy(), src[idx])


# --------------------------------------------------------------------------- select
def _select_case(lib, lens, w, keep, scores):
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    keep = np.asarray(keep, dtype=np.int32)
    off_h, keep_h = torch.from_numpy(off), torch.from_numpy(keep)
    n_kept = int(keep.sum())
    kept = torch.full((n_kept + 8,), -7, dtype=torch.int32, device="cuda")
    out_off = torch.full((len(lens) + 1,), -1, dtype=torch.int32, device="cuda")
    lib.select(torch.from_numpy(scores).cuda(), off_h.cuda(), off_h, keep_h.cuda(), keep_h, len(lens), w, kept, out_off)
    torch.cuda.synchronize()
    got = kept.cpu().numpy()
    assert np.all(got[n_kept:] == -7), "nothing may be written past sum(keep_len)"
    ref = [orc.select_pvc(scores[off[b]:off[b + 1]], w, keep[b]) + off[b] for b in range(len(lens))]
    ref = np.concatenate(ref) if ref else np.zeros(0, dtype=np.int64)
    assert np.array_equal(got[:n_kept].astype(np.int64), ref), "selection must be exact on the given fp32 scores"
    assert out_off.cpu().numpy().tolist() == np.concatenate([[0], np.cumsum(keep)]).tolist()


@pytest.mark.parametrize("seed", range(6))
def test_select_exact_random(lib, seed):
    rng = np.random.default_rng(seed)
    B = int(rng.integers(1, 9))
    lens = rng.integers(1, 3000, size=B)
    w = int(rng.integers(1, 100))
    keep = [int(rng.integers(min(w, S), S + 1)) for S in lens]
    scores = rng.random(int(lens.sum()), dtype=np.float32) ** 4
    _select_case(lib, lens, w, keep, scores)


def test_select_heavy_ties_lower_position_wins(lib):
    rng = np.random.default_rng(3)
    lens = [2048, 777, 64, 5000]
    scores = (rng.integers(0, 5, size=sum(lens)) / 8.0).astype(np.float32)        # 5 distinct values
    _select_case(lib, lens, 64, [1434, 500, 64, 2500], scores)
    const = np.full(sum(lens), 0.25, dtype=np.float32)                          # one value only
    _select_case(lib, lens, 64, [1434, 500, 64, 2500], const)
    zeros = np.zeros(sum(lens), dtype=np.float32)
    zeros[::7] = -0.0
    _select_case(lib, lens, 64, [1000, 65, 64, 4999], zeros)


def test_select_edges(lib):
    rng = np.random.default_rng(4)
    lens = [1, 16, 17, 300, 300, 300]
    scores = rng.random(sum(lens), dtype=np.float32)
    _select_case(lib, lens, 16, [1, 16, 17, 16, 300, 17], scores)   # S<w, S==w, keep all, local only, identity, one ctx
    _select_case(lib, [300], 16, [299], scores[:300])               # evict exactly one


def test_select_long_sequences_staged_and_unstaged(lib):
    rng = np.random.default_rng(5)
    lens = [32768, 36864 + 128, 50000]                  # in LDS / just over the LDS capacity / far over
    scores = (rng.random(sum(lens), dtype=np.float32) * np.float32(1e-3)).astype(np.float32)
    scores[::5] = scores[3]                             # a big tie class as well
    _select_case(lib, lens, 128, [16384, 20000, 128 + 1], scores)


def test_select_tiny_and_denormal_scores(lib):
    rng = np.random.default_rng(6)
    scores = rng.random(4096, dtype=np.float32) * np.float32(1e-38)
    scores[100:200] = 0.0
    _select_case(lib, [4096], 64, [2000], scores.astype(np.float32))


def _ulps_above(base, steps):
    return (np.float32(base).view(np.uint32) + np.asarray(steps, dtype=np.uint32)).astype(np.uint32).view(np.float32)


@pytest.mark.parametrize("n", [300, 4096, 4097])                     # 512 lanes up to 4096 tokens, 1024 beyond
@pytest.mark.parametrize("spread", ["few_ulps", "few_to_a_bin", "outlier", "clusters", "bin_256", "bin_257"])
def test_select_search_passes(lib, n, spread):
    """Score distributions that end the search for the threshold in its different ways (bins divide the span of the keys in 1024 parts with 512
    lanes, in 2048 with 1024): a bin for every value; bins of one, two and four values; all keys but one in the first bin, so
    that a second pass, and at 4096 keys a third, divides it; four clusters; a bin of 256 keys (ranked directly) and of 257 (another pass)."""
    rng = np.random.default_rng(n)
    steps = {
        "few_ulps": lambda: rng.integers(0, 40, n),
        "few_to_a_bin": lambda: rng.integers(0, 1 << int(rng.integers(11, 13)), n),
        "outlier": lambda: np.where(np.arange(n) == n // 2, 0x08000000, rng.integers(0, 3000, n)),
        "clusters": lambda: rng.integers(0, 4, n) * 0x00400000 + rng.integers(0, 1 << 20, n),
        "bin_256": lambda: np.where(np.arange(n) < 256, rng.integers(0, 1 << 12, n), 0x00800000 + np.arange(n) * 8192),
        "bin_257": lambda: np.where(np.arange(n) < 257, rng.integers(0, 1 << 12, n), 0x00800000 + np.arange(n) * 8192),
    }[spread]()
    scores = _ulps_above(1e-4, steps)
    w = 16
    for keep in (w + 1, n - 100, n // 2, n - 1):
        _select_case(lib, [n], w, [keep], scores)


@pytest.mark.parametrize("n_src,n_kept", [(1, 1), (1000, 777), (3_000_000, 2_500_001)])
def test_gather_positions_bit_exact(lib, n_src, n_kept):
    rng = np.random.default_rng(n_kept)
    pos = rng.integers(-(1 << 31), 1 << 31, n_src, dtype=np.int64).astype(np.int32)
    idx = np.sort(rng.choice(n_src, n_kept, replace=False)).astype(np.int32)
    pos_d, idx_d = torch.from_numpy(pos).cuda(), torch.from_numpy(idx).cuda()
    out = torch.full((n_kept + 8,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    lib.gather_positions(pos_d, idx_d, n_kept, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.array_equal(got[:n_kept], pos[idx])
    assert np.all(got[n_kept:] == 0x5A5A5A5A), "nothing is written past n_kept"


@pytest.mark.parametrize("dist", ["spread", "tied", "outlier", "signed"])
@pytest.mark.parametrize("longest", [63, 512, 4096, 4097, 8192, 8193, 36864, 36865])
def test_select_key_sources_and_search(lib, longest, dist):
    """Sizes at the ends of the ranges a lane keeps its keys in registers, LDS or memory for, with scores that end the search in its first
    bin, in a bin of more equal keys than are ranked, and after further passes."""
    lens = [longest, max(longest - 61, 1), longest // 2 + 1, 3]
    rng = np.random.default_rng(longest)
    scores = np.exp(rng.normal(size=sum(lens))).astype(np.float32)
    if dist == "tied":                                      # six values: hundreds of keys equal the threshold
        scores = (np.minimum(scores, 5.0).astype(np.int32) * 0.125).astype(np.float32)
    elif dist == "outlier":                                 # all but two keys share the top bin's neighbourhood
        scores = (1.0 + 1e-4 * rng.random(sum(lens))).astype(np.float32)
        scores[0], scores[lens[0]] = 1e-38, 3e38
    elif dist == "signed":
        scores = (scores * rng.choice([-1.0, 1.0, 0.0], size=len(scores))).astype(np.float32)
        scores[1], scores[lens[0] + 1] = np.inf, -np.inf
    for share in (0.02, 0.5, 0.98):
        _select_case(lib, lens, 2, [max(min(2, S), int(share * S)) for S in lens], scores)


@pytest.mark.parametrize("longest", [700, 4096, 8192, 9000, 40000])          # keys in registers (512 and 1024 lanes), LDS, memory
@pytest.mark.parametrize("equal", [47, 48, 49, 256, 257])
def test_select_equal_keys(lib, longest, equal):
    """Neighbouring fp32 numbers, each the score of so many tokens: equal keys of the threshold's bin are ranked or counted in order."""
    rng = np.random.default_rng(longest + equal)
    lens, w = [longest, longest - 63, equal + 5], 5
    scores = np.concatenate([_ulps_above(0.25, rng.permutation(np.arange(S) // equal)) for S in lens])
    for k in (1, equal - 1, equal, equal + 1, longest // 2):
        _select_case(lib, lens, w, [w + min(k, S - w) for S in lens], scores)
