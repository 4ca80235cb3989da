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


def _line_db(precision, R, rows, d, seed=5):
    feats, xy = _feats(R * rows, d, seed)
    mirrors = {"fp32": 0, "bf16": hloc.MIRROR_BF16, "fp8": hloc.MIRROR_FP8}[precision]
    db = hloc.HlocDB(feats, xy, mirrors=mirrors)
    db.set_regions(np.repeat(np.arange(R), rows).astype(np.int32), R)
    rng = np.random.default_rng(seed + 1)
    q = feats[rng.integers(0, len(feats), 2048)]
    return db, (q + 0.1 * rng.standard_normal(q.shape)).astype(np.float32)


@pytest.mark.parametrize("precision,captured,R,n_reg,first,later", [
    # 64 frames have dense coarse words; a handful takes the key lists
    ("bf16", "bf16", 200, 5, 64, (1, 5)),
    ("fp8", "fp8", 200, 5, 64, (1, 5)),
    # 2,048 frames have an item list; 1,900 the frame lists of the direct
    # screen, which take more behind fewer words
    ("fp32", "fp32", 512, 60, 2048, (1900, 17)),
    # an fp32 batch of an fp8 database leaves room for one vector per frame
    ("fp8", "fp32", 200, 5, 300, (300, 2)),
])
def test_smaller_batch_keeps_the_captured_graph(torch_cuda, precision, captured, R, n_reg, first,
                                                later):
    db, q = _line_db(precision, R, 100, 64)
    qd = torch_cuda.from_numpy(q).cuda()
    s = torch_cuda.cuda.current_stream()
    ws = hloc.Workspace(db)
    out = ws.outputs(first, first, 8, "cuda")
    ws.capture(qd[:first], 8, n_reg, None, out, captured)
    for nq in later:
        say(f"[case] {precision}, R {R}: {first} frames captured, then {nq}")
        part = ws.outputs(nq, nq, 8, "cuda")
        ws.query_async(qd[:nq], 8, n_reg, None, part, s, precision)
        ref = db.query(qd[:nq], 8, n_reg, precision=precision)
        for key in part:
            assert torch_cuda.equal(part[key], ref[key]), (nq, key)
        for v in out.values():
            v.zero_()
        ws.replay(s)  # raises if a buffer grew and the graph was dropped
        ref = db.query(qd[:first], 8, n_reg, precision=captured)
        torch_cuda.cuda.synchronize()
        for key in out:
            assert torch_cuda.equal(out[key], ref[key]), (nq, key)
    ws.close()
    db.close()


@pytest.mark.parametrize("precision", ["bf16", "fp8"])
def test_server_slot_takes_small_batches(torch_cuda, precision):
    # a slot sized for 64 frames x 200 regions (dense coarse words) has no key
    # lists for requests of 1 to 5 frames: they take words too, and give the
    # direct call's results
    db, q = _line_db(precision, 200, 100, 64)
    srv = hloc.Server(db, 8, 5, precision, max_batch_frames=64, max_slots=2)
    for f in (64, 1, 3, 5, 64):
        say(f"[case] {precision} request of {f}")
        got = srv.wait(srv.submit(q[:f]), f)
        ref = db.query(q[:f], 8, 5, np.array([0, f], np.int32), precision)
        assert (got["idx"] == ref["idx"]).all() and (got["dist"] == ref["dist"]).all()
        assert (got["xy"] == ref["xy"][0]).all() and got["flags"] == ref["flags"][0]
    srv.close()
    db.close()


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp8"])
def test_reserve_covers_smaller_calls(torch_cuda, precision):
    # reserved for 2,048 frames and every region: within that, calls with fewer
    # regions (dense coarse words, or key lists at full size: 2,048 x 6,400
    # words), fewer frames (frame lists of the direct screen; a handful) and
    # every region allocate nothing (each of these forms takes megabytes that
    # were missing), and give the results of a workspace sized by each call
    R = 6400
    db, q = _line_db(precision, R, 2, 64)
    qd = torch_cuda.from_numpy(q).cuda()
    s = torch_cuda.cuda.current_stream()
    calls = [(2048, 8), (2048, 64), (600, 8), (300, 60), (1, 8), (40, R)]
    refs = [db.query(qd[:nq], 8, nr, precision=precision) for nq, nr in calls]
    ws = hloc.Workspace(db)
    outs = [ws.outputs(nq, nq, 8, "cuda") for nq, _ in calls]
    torch_cuda.cuda.synchronize()
    ws.reserve(2048, 2048, 8, R)
    free = torch_cuda.cuda.mem_get_info()[0]
    for (nq, nr), out in zip(calls, outs):
        ws.query_async(qd[:nq], 8, nr, None, out, s, precision)
        say(f"[case] {precision} {nq} frames, {nr} regions: "
            f"free {torch_cuda.cuda.mem_get_info()[0] - free:+d}")
        assert torch_cuda.cuda.mem_get_info()[0] == free, (nq, nr)
    for ref, out in zip(refs, outs):
        for key in out:
            assert torch_cuda.equal(out[key], ref[key]), key
    ws.close()
    db.close()


def test_static_batch_that_fills_the_array(torch_cuda):
    # 188,166 frames of 32 values against 40 regions of 40 rows, one searched:
    # 67,108,864 bytes of scratch memory without the wide screen's item counters
    db, q = _line_db("fp32", 40, 40, 32)
    rng = np.random.default_rng(8)
    q = np.tile(q, (92, 1))[:188_166]
    q += 0.01 * rng.standard_normal(q.shape, dtype=np.float32)
    qd = torch_cuda.from_numpy(q).cuda()
    say(f"[case] static batch of {len(q)} frames")
    out = db.query_static(qd, 8, 1)
    ref = db.query(qd, 8, 1)
    torch_cuda.cuda.synchronize()
    for key in out:
        assert torch_cuda.equal(out[key], ref[key]), key
    db.close()


@pytest.mark.parametrize("precision", ["bf16", "fp8"])
def test_key_lists_where_memory_is_short(torch_cuda, precision):
    # 300 frames against 40,000 regions: 48 MB of coarse words, with the key lists
    # beside them more than the static array. Both the call on that array and a
    # server whose budget is just below a slot with the lists run on the words
    rng = np.random.default_rng(12)
    R, rows, d, k, n_reg, nq = 40_000, 2, 64, 8, 5, 300
    feats = rng.standard_normal((R * rows, d)).astype(np.float32)
    q = (feats[rng.integers(0, len(feats), nq)]
         + 0.05 * rng.standard_normal((nq, d))).astype(np.float32)
    db = hloc.HlocDB(feats, rng.uniform(0, 40, size=(len(feats), 2)),
                     mirrors=hloc.MIRROR_BF16 | hloc.MIRROR_FP8)
    db.set_regions(np.repeat(np.arange(R), rows).astype(np.int32), R)
    qd = torch_cuda.from_numpy(q).cuda()
    ref = db.query(qd, k, n_reg, precision=precision)
    say(f"[case] {precision} static batch of {nq} frames")
    out = db.query_static(qd, k, n_reg, precision=precision)
    torch_cuda.cuda.synchronize()
    for key in out:
        assert torch_cuda.equal(out[key], ref[key]), key
    cfg = dict(max_batch_frames=nq, max_slots=1)
    srv = hloc.Server(db, k, n_reg, precision, **cfg)
    slot = srv.stats()["slot_bytes"]
    srv.close()
    srv = hloc.Server(db, k, n_reg, precision, hbm_budget_bytes=slot - 1, **cfg)
    assert srv.stats()["slots"] == 1 and srv.stats()["slot_bytes"] < slot
    say(f"[case] {precision} server requests")
    for f in (nq, 7):
        got = srv.wait(srv.submit(q[:f]), f)
        assert (got["idx"] == ref["idx"][:f].cpu().numpy()).all()
        assert (got["dist"] == ref["dist"][:f].cpu().numpy()).all()
    srv.close()
    db.close()


def test_binding_inputs_on_another_stream(torch_cuda):
    # calls on a side stream with inputs that the binding copies (strided
    # frames, int64 offsets and lists) while the current stream is busy: the
    # copies belong to the side stream, so they are made before its kernels
    # read them and not reused under them; outputs likewise
    torch = torch_cuda
    db, q = _line_db("fp32", 64, 100, 64)
    db.set_region_labels((np.arange(64) % 2).astype(np.int32), 2)
    wide = torch.from_numpy(np.repeat(q[:256], 2, axis=1)).cuda()
    sig = torch.randn(64, 512, device="cuda")
    frames, strided, sig2 = wide[:, ::2], wide[:, ::2].contiguous(), sig.t().contiguous().t()
    offs = torch.arange(0, 257, 8, device="cuda")
    lists = torch.arange(256, device="cuda")
    st = [hloc.Streams(db, 256, 3, 8, 256) for _ in range(4)]
    one = torch.arange(257, device="cuda")

    def calls(f, sg, i, **kw):
        return [db.query(f, 8, 5, offs, **kw), db.query_static(f, 8, 5, offs, **kw),
                db.query_labels(f, 8, 5, 2, offs, **kw),
                db.query_windows(f, 8, 5, offs, lists, **kw),
                st[i].query(f, one, one[:256], 5, **kw),
                {"out": hloc.fft_features(sg, 200, **kw)}]

    ref = calls(strided, sig, 0)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    calls(frames, sig2, 1, stream=side)  # (memory of the side stream)
    torch.cuda.synchronize()
    # copies made earlier hold other values by now
    calls(frames.flip(1).t().contiguous().t(), -2 * sig2, 2)
    a = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    for _ in range(100):
        a = (a @ a).clamp_(-1, 1)
    say("[case] six calls on a side stream beside a busy current stream")
    got = calls(frames, sig2, 3, stream=side)
    side.synchronize()
    say(f"[ok] current stream still busy after them: {not torch.cuda.current_stream().query()}")
    for r, g in zip(ref, got):
        for key in r:
            assert np.array_equal(g[key].cpu().numpy(), r[key].cpu().numpy(), equal_nan=True), key
    for s in st:
        s.close()
    db.close()
