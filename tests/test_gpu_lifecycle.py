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


@pytest.mark.parametrize("n_reg", [3, 6])
def test_info_after_new_regions(torch_cuda, n_reg):
    # counters of a batch without an item list, on the database's workspace and
    # on one of the caller's, after the database went from 6 to 1,200 regions
    # (more than its per-region buffers hold): the batch's, as before
    feats, xy = _feats(1200, 32, 4)
    q = torch_cuda.from_numpy(feats[:40]).cuda()
    db = hloc.HlocDB(feats, xy)
    db.set_regions((np.arange(1200) % 6).astype(np.int32), 6)
    ws = hloc.Workspace(db)
    out = ws.outputs(40, 40, 4, "cuda")
    ws.query_async(q, 4, n_reg, None, out, torch_cuda.cuda.current_stream())
    db.query(q, 4, n_reg)
    before = db.info()
    say(f"[case] {n_reg} of 6 regions, then 1,200: {before}")
    # every region has 200 rows: 13 blocks, against groups of 16 of its frames
    assert before["items"] >= 13 * n_reg and before["candidates"] == 40 * 200 * n_reg
    assert ws.info() == before
    db.set_regions(np.arange(1200, dtype=np.int32), 1200)
    assert db.info() == before and ws.info() == before
    ws.close()
    db.close()
