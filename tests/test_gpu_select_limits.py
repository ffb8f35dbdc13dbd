"""Segment maxima at the ends of the int32 ranges: segments that end at the last of 2^31 - 1
scores (8 and 64 lanes per segment), and more segments than a launch has groups of threads."""
import numpy as np
import pytest

from helpers import weights

pytestmark = pytest.mark.gpu

LAST = 2 ** 31 - 1


def _scorer():
    from paper_2104_04547_amd import Scorer
    arch, w = weights("tiny")
    return Scorer(arch, w, "bf16")


@pytest.mark.parametrize("n_seg", [3, LAST // 128 + 2])
def test_segments_at_the_end_of_the_index_range(n_seg):
    import torch
    print(f"\n[gpu-case] cf_compound_max {n_seg} segments at the end of {LAST} scores", flush=True)
    s = _scorer()
    scores = torch.empty(LAST, dtype=torch.float32, device="cuda")
    tail = np.random.default_rng(1).normal(size=300).astype(np.float32)
    scores[LAST - 300:] = torch.from_numpy(tail).cuda()
    off = torch.full((n_seg + 1,), LAST - 300, dtype=torch.int32, device="cuda")
    off[n_seg - 1], off[n_seg] = LAST - 7, LAST        # the last but one of 293, the last of 7
    best, idx = s.compound_max(scores, off)
    s.check()
    for k, (a, b) in ((n_seg - 2, (0, 293)), (n_seg - 1, (293, 300))):
        assert idx[k].item() == LAST - 300 + a + int(np.argmax(tail[a:b]))
        assert best[k].item() == tail[a:b].max()
    assert (idx[:n_seg - 2] == -1).all().item() and torch.isinf(best[:n_seg - 2]).all().item()
    s.close()


def test_more_segments_than_one_launch_has_threads_for():
    import torch
    n = 2 ** 29 + 3       # 8 lanes each: 2^32 threads and 24
    print(f"\n[gpu-case] cf_compound_max {n} segments", flush=True)
    s = _scorer()
    off = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    off[n // 2:] = 2
    off[n - 1], off[n] = 3, 8
    scores = torch.tensor([1.0, -2.0, 0.5, 7.0, 9.0, 9.0, -1.0, 4.0], device="cuda")
    best, idx = s.compound_max(scores, off)
    s.check()
    assert [idx[k].item() for k in (0, n // 2 - 1, n // 2, n - 2, n - 1)] == [-1, 0, -1, 2, 4]
    assert [best[k].item() for k in (n // 2 - 1, n - 2, n - 1)] == [1.0, 0.5, 9.0]
    assert int((idx >= 0).sum()) == 3
    s.close()
