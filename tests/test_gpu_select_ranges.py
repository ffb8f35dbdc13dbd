"""Top-k in one workgroup where more than 2048 values reach its first bound: large k, ties at
the k-th value, one thread holding all large values, and ranges from -inf to inf."""
import numpy as np
import pytest

import oracle
from helpers import weights

pytestmark = pytest.mark.gpu


def _values(kind, n, rng):
    v = rng.normal(0, 2, n).astype(np.float32)
    if kind == "ascending":
        v.sort()
    elif kind == "mostly -inf":           # fewer finite values than k
        v[rng.permutation(n)[900:]] = -np.inf
    elif kind == "one column":            # the large values at indices that one thread reads, ties below
        v = np.round(v)
        v[5::1024] = np.linspace(50, 90, len(v[5::1024]), dtype=np.float32)
    elif kind == "whole range":           # -inf, NaN, signed zeros, subnormals, +inf, each many times
        v = rng.choice(np.array([-np.inf, np.inf, np.nan, 0.0, -0.0, 1e-45, -1e-45, 3e38, -3e38], np.float32), n,
                       p=[.3, .0005, .1, .3, .1, .0995, .05, .01, .04])
    elif kind == "near ties":             # images a few units apart: the range narrows to its last bits
        v = (1.0 + rng.integers(0, 3, n) * 2.0 ** -23).astype(np.float32)
    return v


@pytest.mark.parametrize("kind", ["normal", "ascending", "mostly -inf", "one column", "whole range", "near ties"])
@pytest.mark.parametrize("n", [2048, 2049, 10000, 16384, 16385, 50000, 65536])
def test_top_k_beyond_the_first_bound(kind, n):
    import torch
    from paper_2104_04547_amd import Scorer
    arch, w = weights("tiny")
    s = Scorer(arch, w, "bf16")
    v = _values(kind, n, np.random.default_rng(n))
    t = torch.from_numpy(v).cuda()
    want = oracle.top_k(v.astype(np.float64), 1024)
    for k in (1, 63, 500, 1000, 1024):
        print(f"\n[gpu-case] cf_top_k {kind} n={n} k={k}", flush=True)
        idx, val = s.top_k(t, k)
        np.testing.assert_array_equal(idx.cpu().numpy(), want[:k])
        np.testing.assert_array_equal(val.cpu().numpy(), v[want[:k]])
    s.close()
