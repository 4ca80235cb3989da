"""Forms that a batch may take (two fp8 vectors or one, key lists or dense
words, the lists of the selection) at the sizes where one gives way to another:
bitwise the same results, and the oracle's."""
import numpy as np
import pytest

import oracle
from parity import judge_frames
from paper_2006_08861_amd import hloc, workload

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("d,n_reg", [(640, 9), (740, 9), (768, 9), (1000, 9), (1024, 9),
                                     (640, 3), (768, 3), (1000, 3)])
def test_fp8_long_rows_in_wide_items(torch_cuda, d, n_reg):
    # fp8 frames as two vectors (up to 768 padded values, where the register-row
    # kernel takes more than 64 KB of LDS) and as one (above), past the direct
    # screen's work: regions kept by every frame, in chunks with remainders,
    # give wide items; with three regions kept, the coarse screen has no bf16
    # kernel of this length and runs on fp8 copies too, for many frames and for
    # 20; the same bits as the fp32 screens, and the first 40 frames match the
    # oracle
    rng = np.random.default_rng(41)
    sizes = np.array([333, 129, 64, 40, 1, 40, 15, 40, 17])
    region_of = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    n, R = len(region_of), len(sizes)
    feats = rng.standard_normal((n, d)).astype(np.float32)
    feats[:526] *= 0.2
    feats[526:] += 0.6
    xy = rng.uniform(0, 40, size=(n, 2))
    rows = n if n_reg == R else n_reg * float((sizes ** 2).sum()) / n
    nq = int(1.6e9 / (2 * rows * ((d + 31) // 32 * 32))) + 300
    q = (feats[rng.integers(0, 526, nq)] + 0.05 * rng.standard_normal((nq, d))).astype(np.float32)
    say(f"[case] {nq} frames, d {d}, n_reg {n_reg}")
    db = hloc.HlocDB(feats, xy, mirrors=hloc.MIRROR_FP8)
    db.set_regions(region_of, R)
    qd = torch_cuda.from_numpy(q).cuda()
    outs = {p: db.query(qd, 9, n_reg, precision=p) for p in ("fp32", "fp8")}
    info = db.info()
    say(f"[ok] {info}")
    assert info["items"] > info["narrow_items"]
    for key in outs["fp8"]:
        assert torch_cuda.equal(outs["fp8"][key], outs["fp32"][key]), key
    few = db.query(qd[:20], 9, n_reg, precision="fp8")
    for key in few:
        assert torch_cuda.equal(few[key], outs["fp32"][key][:20]), key
    db.close()
    ora = oracle.localize(feats, xy, region_of, R, q[:40], np.arange(41), 9, n_reg,
                          (0.5, 1, 0.0, 0))
    idx, dist = (outs["fp8"][key][:40].cpu().numpy() for key in ("idx", "dist"))
    st = judge_frames(idx, dist, None, ora, feats, region_of, R, q[:40], 9)
    assert st["recall"] == 1.0


@pytest.mark.parametrize("rows,precision,k,n_reg", [
    (60, "fp32", 240, 28), (60, "fp32", 241, 28), (60, "fp32", 256, 60), (60, "bf16", 85, 28),
    (60, "bf16", 86, 28), (60, "fp8", 85, 28), (60, "fp8", 107, 28), (60, "fp8", 171, 28),
    (600, "bf16", 86, 130), (600, "fp32", 256, 130)])
def test_selection_past_sixteen_survivor_blocks(torch_cuda, rows, precision, k, n_reg):
    # up to 16 survivor blocks (frame kernel), 17 to 32 (either, by the frames
    # and the length of their lists: about 10 blocks a region, and every one of
    # 5,000) and 33 (block kernel), in batches of 1, 300, 520 and 4,100 frames:
    # bitwise the fp32 screens' results of one batch, and 12 frames against the
    # oracle
    rng = np.random.default_rng(42)
    sizes = rng.integers(1, 2 * rows, 130)
    region_of = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    n, d, R = len(region_of), 64, len(sizes)
    feats = rng.standard_normal((n, d)).astype(np.float32)
    xy = rng.uniform(0, 40, size=(n, 2))
    most = 4100 if rows == 60 else 520
    q = feats[rng.integers(0, n, most)] + 0.2 * rng.standard_normal((most, d), dtype=np.float32)
    say(f"[case] k={k} {precision}, {n_reg} of {R} regions, {n} rows")
    db = hloc.HlocDB(feats, xy, mirrors=hloc.MIRROR_BF16 | hloc.MIRROR_FP8)
    db.set_regions(region_of, R)
    qd = torch_cuda.from_numpy(q).cuda()
    ref = db.query(qd, k, n_reg)
    for nq in (1, 300, 520, 4100):
        got = db.query(qd[:nq], k, n_reg, precision=precision)
        for key in got:
            assert torch_cuda.equal(got[key], ref[key][:nq]), (nq, key)
    db.close()
    ora = oracle.localize(feats, xy, region_of, R, q[:12], np.arange(13), k, n_reg,
                          (0.5, 1, 0.0, 0))
    idx, dist = (ref[key][:12].cpu().numpy() for key in ("idx", "dist"))
    st = judge_frames(idx, dist, None, ora, feats, region_of, R, q[:12], k)
    assert st["recall"] == 1.0


@pytest.mark.parametrize("precision,k", [("fp32", 10), ("fp32", 50), ("bf16", 10), ("fp8", 10)])
def test_survivors_of_short_blocks(torch_cuda, precision, k):
    # regions of 20 rows (blocks of 16 and of 4), every row searched: the
    # survivor blocks nearly always hold k rows, so few frames re-score their
    # whole list of 2,000 blocks (a frame in forty of them would be 800 row
    # slots a frame; with ceil((k + 16) / 16) survivors it is a frame in four);
    # bitwise the fp32 screens' results, and 12 frames against the oracle
    rng = np.random.default_rng(43)
    n, d, R, nq = 20_000, 64, 1000, 600
    feats = workload.walk_features(n, d, rng)
    xy = workload.corridor_xy(n)
    region_of = np.repeat(np.arange(R), n // R).astype(np.int32)
    q = (feats[rng.integers(0, n, nq)] + 0.03 * rng.standard_normal((nq, d))).astype(np.float32)
    db = hloc.HlocDB(feats, xy, mirrors=hloc.MIRROR_BF16 | hloc.MIRROR_FP8)
    db.set_regions(region_of, R)
    qd = torch_cuda.from_numpy(q).cuda()
    ref = db.query(qd, k, R)
    got = db.query(qd, k, R, precision=precision)
    info = db.info()
    say(f"[case] {precision} k={k}: {info}")
    for key in got:
        assert torch_cuda.equal(got[key], ref[key]), key
    assert info["rerank_rows"] <= 2000 * nq
    db.close()
    ora = oracle.localize(feats, xy, region_of, R, q[:12], np.arange(13), k, R,
                          (0.5, 1, 0.0, 0))
    idx, dist = (ref[key][:12].cpu().numpy() for key in ("idx", "dist"))
    st = judge_frames(idx, dist, None, ora, feats, region_of, R, q[:12], k)
    assert st["recall"] == 1.0


@pytest.mark.parametrize("precision", ["bf16", "fp8"])
@pytest.mark.parametrize("labels", [0, 3])
def test_key_lists_and_words_agree(torch_cuda, precision, labels):
    # more than 12 M frame x representative words take the fused coarse product
    # (1,601 frames x 8,192 regions; 600 frames under 3 labels, whose regions it
    # masks: last tiles of 65 and 8 of 128 frames, several splits), batches of
    # 100 frames dense words: the same bits, also as the fp32 screens. 120
    # regions hold the same rows, so the keys cannot decide the frames near them
    # (every tenth) and those take the words. 12 frames against the oracle.
    rng = np.random.default_rng(44)
    R, rows, d, k, n_reg, nq = 8192, 2, 64, 6, 3, 600 if labels else 1601
    feats = rng.standard_normal((R * rows, d)).astype(np.float32)
    feats[:120 * rows] = np.tile(feats[:rows], (120, 1))
    region_of = np.repeat(np.arange(R), rows).astype(np.int32)
    xy = rng.uniform(0, 40, size=(len(feats), 2))
    src = rng.integers(120 * rows, len(feats), nq)
    src[::10] = 0
    q = (feats[src] + 0.05 * rng.standard_normal((nq, d))).astype(np.float32)
    of = (np.arange(R) * 3 // R).astype(np.int32)
    db = hloc.HlocDB(feats, xy, mirrors=hloc.MIRROR_BF16 | hloc.MIRROR_FP8)
    db.set_regions(region_of, R)
    if labels:
        db.set_region_labels(of, labels)

    def run(frames, prec):
        fd = torch_cuda.from_numpy(frames).cuda()
        if labels:
            offs = torch_cuda.arange(len(frames) + 1, dtype=torch_cuda.int32, device="cuda")
            out = db.query_labels(fd, k, n_reg, labels, offs, precision=prec)
        else:
            out = db.query(fd, k, n_reg, precision=prec)
        return {key: v.cpu() for key, v in out.items()}, db.info()

    say(f"[case] {precision}, {nq} frames, {labels} labels")
    full, info = run(q, precision)
    say(f"[ok] {info}")
    assert info["coarse_deferred"] >= len(src[::10])
    fp32, _ = run(q, "fp32")
    for key in full:
        assert torch_cuda.equal(full[key], fp32[key]), key
    for a in range(0, nq, 100):
        part, info = run(q[a:a + 100], precision)
        if len(q[a:a + 100]) == 100:
            assert info["coarse_deferred"] == 0
        for key in part:
            per_label = labels and key in ("idx", "dist")
            want = full[key][:, a:a + 100] if per_label else full[key][a:a + 100]
            assert torch_cuda.equal(part[key], want), (a, key)
    db.close()
    if labels:
        ora = oracle.localize_labels(feats, xy, region_of, R, of, q[:12], np.arange(13), k, n_reg,
                                     (0.5, 1, 0.0, 0))
        for p in range(labels):
            st = judge_frames(full["idx"][p, :12].numpy(), full["dist"][p, :12].numpy(), None,
                              ora["per_label"][p], feats, region_of, R, q[:12], k)
            assert st["recall"] == 1.0
    else:
        ora = oracle.localize(feats, xy, region_of, R, q[:12], np.arange(13), k, n_reg,
                              (0.5, 1, 0.0, 0))
        st = judge_frames(full["idx"][:12].numpy(), full["dist"][:12].numpy(), None, ora, feats,
                          region_of, R, q[:12], k)
        assert st["recall"] == 1.0


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("rows,k,n_reg", [(2, 50, 1500), (1, 17, 20), (2, 10, 3), (3, 200, 60)])
def test_survivor_blocks_of_fewer_rows_than_k(torch_cuda, rows, k, n_reg, precision):
    # no 16 blocks of one to three rows hold k: the k-th smallest word of a block
    # and the error bound say what can still be among the k nearest, not half of the
    # 1,500 blocks (16 row slots each) of the exhaustive search even behind fp8; a
    # list of fewer blocks than k is re-scored whole. 8, 4 and 2 waves a frame:
    # bitwise the fp32 screens' results, and 12 frames against the oracle
    rng = np.random.default_rng(46)
    R, d, nq = 1500, 64, 4100
    feats = rng.standard_normal((R * rows, d)).astype(np.float32)
    region_of = np.repeat(np.arange(R), rows).astype(np.int32)
    xy = rng.uniform(0, 40, size=(len(feats), 2))
    q = feats[rng.integers(0, len(feats), nq)] + 0.3 * rng.standard_normal((nq, d), dtype=np.float32)
    db = hloc.HlocDB(feats, xy, mirrors=hloc.MIRROR_BF16 | hloc.MIRROR_FP8)
    db.set_regions(region_of, R)
    qd = torch_cuda.from_numpy(q).cuda()
    ref = db.query(qd, k, n_reg)
    for frames in (40, 1600, nq):
        got = db.query(qd[:frames], k, n_reg, precision=precision)
        info = db.info()
        say(f"[case] {precision} {frames} frames: {info}")
        for key in got:
            assert torch_cuda.equal(got[key], ref[key][:frames]), (frames, key)
        assert n_reg < R or info["rerank_rows"] <= 750 * 16 * frames
    db.close()
    ora = oracle.localize(feats, xy, region_of, R, q[:12], np.arange(13), k, n_reg,
                          (0.5, 1, 0.0, 0))
    idx, dist = (ref[key][:12].cpu().numpy() for key in ("idx", "dist"))
    st = judge_frames(idx, dist, None, ora, feats, region_of, R, q[:12], k)
    assert st["recall"] == 1.0


@pytest.mark.parametrize("R,n_reg,nqs,labels", [
    (40_000, 8, (1, 300), 2), (32_768, 8, (40,), 2), (900, 28, (40, 600), 0),
    (900, 29, (40, 512, 513), 3), (900, 37, (513,), 0), (900, 60, (600,), 3), (900, 61, (40,), 3)])
def test_coarse_words_of_long_lists_and_many_survivors(torch_cuda, R, n_reg, nqs, labels):
    # regions where the coarse selection goes from the frame kernel to the block
    # kernel: 32,768 words and more, 32 / 33 / 41 / 64 / 65 survivors, 512 and 513
    # frames, with labels (looked up by the one, masked ahead of the other):
    # bitwise the results of bf16 screens and of halves of the batch, and 8
    # frames against the oracle
    rng = np.random.default_rng(45)
    rows, d, k = 3, 64, 10
    feats = rng.standard_normal((R * rows, d)).astype(np.float32)
    region_of = np.repeat(np.arange(R), rows).astype(np.int32)
    xy = rng.uniform(0, 40, size=(len(feats), 2))
    q = (feats[rng.integers(0, len(feats), max(nqs))]
         + 0.3 * rng.standard_normal((max(nqs), d))).astype(np.float32)
    of = (np.arange(R) % max(labels, 1)).astype(np.int32)
    db = hloc.HlocDB(feats, xy, mirrors=hloc.MIRROR_BF16)
    db.set_regions(region_of, R)
    if labels:
        db.set_region_labels(of, labels)

    def run(frames, prec):
        fd = torch_cuda.from_numpy(frames).cuda()
        if labels:
            offs = torch_cuda.arange(len(frames) + 1, dtype=torch_cuda.int32, device="cuda")
            return [db.query_labels(fd, k, n_reg, labels, offs, precision=prec),
                    db.query(fd, k, n_reg, precision=prec)]
        return [db.query(fd, k, n_reg, precision=prec)]

    for nq in nqs:
        say(f"[case] {nq} frames, {n_reg} of {R} regions, {labels} labels")
        full = run(q[:nq], "fp32")
        cut = (nq + 1) // 2
        parts = [run(q[:cut], "fp32"), run(q[cut:nq], "fp32")] if nq > 1 else [full]
        for i, (f, b) in enumerate(zip(full, run(q[:nq], "bf16"))):
            per_label = labels and i == 0
            for key in f:
                assert torch_cuda.equal(f[key], b[key]), (nq, i, key)
                dim = 1 if per_label and key in ("idx", "dist") else 0
                whole = torch_cuda.cat([p[i][key] for p in parts], dim=dim)
                assert torch_cuda.equal(f[key], whole), (nq, i, key)
    db.close()
    m = min(8, max(nqs))
    ora = oracle.localize(feats, xy, region_of, R, q[:m], np.arange(m + 1), k, n_reg,
                          (0.5, 1, 0.0, 0))
    idx, dist = (full[-1][key][:m].cpu().numpy() for key in ("idx", "dist"))
    st = judge_frames(idx, dist, None, ora, feats, region_of, R, q[:m], k)
    assert st["recall"] == 1.0


@pytest.mark.parametrize("precision,n_reg,labels", [
    ("bf16", 3, 0), ("bf16", 44, 0), ("fp8", 44, 0), ("bf16", 3, 3), ("bf16", 44, 3)])
def test_coarse_keys_of_long_lists(torch_cuda, precision, n_reg, labels):
    # 40,000 regions: 104 frames take dense words, 105 and 300 (and three labels of
    # 35) the key lists, and those of them near the regions that hold the same
    # rows, every tenth, the words: bitwise the fp32 screens' results, and 12
    # frames against the oracle
    rng = np.random.default_rng(47)
    R, rows, d, k, nq = 40_000, 2, 64, 10, 300
    feats = rng.standard_normal((R * rows, d)).astype(np.float32)
    feats[:120 * rows] = np.tile(feats[:rows], (120, 1))
    region_of = np.repeat(np.arange(R), rows).astype(np.int32)
    xy = rng.uniform(0, 40, size=(len(feats), 2))
    src = rng.integers(120 * rows, len(feats), nq)
    src[::10] = 0
    q = (feats[src] + 0.05 * rng.standard_normal((nq, d))).astype(np.float32)
    of = (np.arange(R) * 3 // R).astype(np.int32)
    db = hloc.HlocDB(feats, xy, mirrors=hloc.MIRROR_BF16 | hloc.MIRROR_FP8)
    db.set_regions(region_of, R)
    if labels:
        db.set_region_labels(of, labels)

    def run(frames, prec):
        fd = torch_cuda.from_numpy(frames).cuda()
        if labels:
            offs = torch_cuda.arange(len(frames) + 1, dtype=torch_cuda.int32, device="cuda")
            return db.query_labels(fd, k, n_reg, labels, offs, precision=prec)
        return db.query(fd, k, n_reg, precision=prec)

    for frames in (34, 35, 100) if labels else (104, 105, 300):
        got = run(q[:frames], precision)
        info = db.info()
        say(f"[case] {precision} {frames} frames, {labels} labels: {info}")
        ref = run(q[:frames], "fp32")
        for key in got:
            assert torch_cuda.equal(got[key], ref[key]), (frames, key)
        assert (info["coarse_deferred"] >= len(src[:frames:10])) == (frames not in (34, 104))
    db.close()
    if labels:
        ora = oracle.localize_labels(feats, xy, region_of, R, of, q[:12], np.arange(13), k, n_reg,
                                     (0.5, 1, 0.0, 0))["per_label"]
        sides = [(ref["idx"][p, :12], ref["dist"][p, :12]) for p in range(labels)]
    else:
        ora = [oracle.localize(feats, xy, region_of, R, q[:12], np.arange(13), k, n_reg,
                               (0.5, 1, 0.0, 0))]
        sides = [(ref["idx"][:12], ref["dist"][:12])]
    for o, (idx, dist) in zip(ora, sides):
        st = judge_frames(idx.cpu().numpy(), dist.cpu().numpy(), None, o, feats, region_of, R,
                          q[:12], k)
        assert st["recall"] == 1.0
