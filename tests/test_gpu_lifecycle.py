"""What the library keeps between calls: the report of the last batch across a
change of the database's regions, and buffers that hold their size."""
import ctypes

import numpy as np
import pytest

from paper_2006_08861_amd import hloc

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _feats(n, d, seed):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((n, d)).astype(np.float32), rng.uniform(0, 40, size=(n, 2))


@pytest.mark.parametrize("n_after", [2, 6, 400])
def test_last_regions_after_new_regions(torch_cuda, n_after):
    # an exhaustive batch over five non-empty regions of six, then fewer, as
    # many and more regions: the report is still the batch's, and nothing is
    # written past the nq x n_regions entries it announces (the buffer holds
    # as many as the new regions would fill)
    feats, xy = _feats(1200, 32, 3)
    region_of = (np.arange(1200) % 6).astype(np.int32)
    region_of[region_of == 2] = 4
    db = hloc.HlocDB(feats, xy)
    db.set_regions(region_of, 6)
    db.query(torch_cuda.from_numpy(feats[:3]).cuda(), 4, 6)
    say(f"[case] 5 regions kept by 3 frames, then {n_after} regions")
    db.set_regions((np.arange(1200) % n_after).astype(np.int32), n_after)
    buf = np.full(3 * 5 + 3 * n_after, -7, np.int32)
    nq, nr = ctypes.c_int32(), ctypes.c_int32()
    assert hloc.load_library().hloc_last_regions(
        db._h, buf.ctypes.data_as(ctypes.c_void_p), ctypes.byref(nq), ctypes.byref(nr)) == 0
    assert (nq.value, nr.value) == (3, 5)
    assert buf[:15].reshape(3, 5).tolist() == [[0, 1, 3, 4, 5]] * 3
    assert (buf[15:] == -7).all()
    db.close()
