"""Which kernels a batch gets, from the library's own answer (pyr_diag_route): a test asserts that it reaches the path it is written
for, on the GPU for the device at hand and on the CPU (test_routes.py) for one of 256 compute units in 8 XCDs."""
import numpy as np

LISTS, ONE_GROUP, TWO_GROUPS = 0, 1, 2                               # pyr_route.attention
SEQ_PER_XCD, EQUAL, COUNTED, PLACES = 0, 1, 2, 3                     # pyr_route.score_order
MI355X = dict(compute_units=256, xcds=8)


def route(lib, lens, Hq, Hkv, d, w=32, **device):
    import torch
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32))
    shape = lib.make_shape(len(lens), int(sum(lens)), max(lens, default=0), Hq, Hkv, d)
    return lib.diag_route(shape, off, w, **device)


def launches(lib, lens, Hq, Hkv, d, w=32, generation=False, keep=None, row_bytes=0, **device):
    import torch
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32))
    keep = None if keep is None else torch.from_numpy(np.asarray(keep, dtype=np.int32))
    return lib.diag_launches(lib.make_shape(len(lens), int(sum(lens)), max(lens, default=0), Hq, Hkv, d), off, w, generation, keep, row_bytes, **device)
