"""Selection at the edges of its kernels: value counts around the single-workgroup limit and
its register widths, values that defeat its bound (all equal, two levels, NaNs), k up to
1024; segments of one to thousands of scores with ties across the lanes that share one."""
import numpy as np
import pytest

import oracle
from helpers import weights

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scorer():
    from paper_2104_04547_amd import Scorer
    arch, w = weights("tiny")
    s = Scorer(arch, w, "fp32")
    yield s
    s.close()


def _values(kind, n, rng):
    if kind == "normal":
        return rng.normal(0, 2, n).astype(np.float32)
    if kind == "equal":
        return np.full(n, -1.5, np.float32)
    if kind == "levels":     # two values, signed zeros and infinities among them
        return rng.choice(np.array([0.0, -0.0, 3.25, -np.inf, np.inf], np.float32), n)
    if kind == "nan":
        v = np.full(n, np.nan, np.float32)
        v[rng.permutation(n)[:n // 3]] = 2.0
        return v
    return np.sort(rng.normal(0, 2, n).astype(np.float32))[::-1].copy()


@pytest.mark.parametrize("kind", ["normal", "equal", "levels", "nan", "sorted"])
@pytest.mark.parametrize("n", [2, 1023, 4096, 4097, 16385, 65536, 65537, 300_000])
def test_top_k_paths_bit_exact(scorer, kind, n):
    import torch
    rng = np.random.default_rng(n)
    v = _values(kind, n, rng)
    t = torch.from_numpy(v).cuda()
    want = oracle.top_k(v.astype(np.float64), min(n, 1024))
    for k in sorted({1, min(n, 100), min(n, 1024)}):
        print(f"\n[gpu-case] cf_top_k {kind} n={n} k={k}", flush=True)
        idx, val = scorer.top_k(t, k)
        np.testing.assert_array_equal(idx.cpu().numpy(), want[:k])
        np.testing.assert_array_equal(val.cpu().numpy(), v[want[:k]])


@pytest.mark.parametrize("lens", [[1], [0, 1, 7, 8, 9, 31, 32, 33, 0], [3000, 1, 0, 257], [40] * 300])
def test_compound_max_paths_bit_exact(scorer, lens):
    import torch
    print(f"\n[gpu-case] cf_compound_max lengths {lens[:9]}", flush=True)
    rng = np.random.default_rng(len(lens))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    v = rng.choice(np.array([0.0, -0.0, 1.5, -2.0, np.nan, -np.inf], np.float32), int(off[-1]))
    best, idx = scorer.compound_max(torch.from_numpy(v).cuda(), torch.from_numpy(off))
    scorer.check()
    wb, wi = oracle.compound_best(v, off)
    np.testing.assert_array_equal(idx.cpu().numpy(), wi)
    np.testing.assert_array_equal(best.cpu().numpy().astype(np.float64), wb)
