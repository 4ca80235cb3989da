"""Forms that a batch may take (two fp8 vectors or one, key lists or dense
words, the lists of the selection) at the sizes where one gives way to another:
bitwise the same results, and the oracle's."""
import numpy as np
import pytest

import oracle
from parity import judge_frames
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
