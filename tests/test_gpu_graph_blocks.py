"""Neighbour lists at the edges of the block split: poses around the 64-atom blocks
and the 1024-atom tile, one pose far above the batch's mean, pose counts around the
switch of the totals' kernel, and cutoffs around the 32-bit form's limit."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from helpers import weights

pytestmark = pytest.mark.gpu


def _batch(sizes, box, seed):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(off[-1])
    x = rng.integers(-box, box, size=(n, 3)).astype(np.int32)
    return synth.PoseBatch(off, x, np.zeros((n, 19), np.float32), np.ones(n, np.uint8), np.asarray(sizes, np.int32))


def _clipped_graph(b, r):
    """radius_graph_batch for coordinates whose squared differences exceed 64 bits:
    an axis beyond r decides alone, so differences are clipped to r + 1."""
    rows, cols = [np.zeros(1, np.int64)], []
    for a, e in zip(b.atom_off[:-1], b.atom_off[1:]):
        x = b.xyz[a:e].astype(np.int64)
        d = np.minimum(np.abs(x[:, None] - x[None]), r + 1)
        near = (d * d).sum(-1) <= r * r
        np.fill_diagonal(near, False)
        rows.append(rows[-1][-1] + np.cumsum(near.sum(1)))
        cols.append(np.nonzero(near)[1] + a)
    return np.concatenate(rows), np.concatenate(cols)


def _check(scorer, b, r_cov, r_nc, graph=oracle.radius_graph_batch):
    import torch
    from paper_2104_04547_amd import cfabi
    wc = graph(b, r_cov)
    wn = graph(b, r_nc)
    t = scorer.build_graphs(cfabi.DeviceBatch.from_pose_batch(b), len(wc[1]), len(wn[1]))
    assert scorer.status()[0] == 0
    torch.cuda.synchronize()
    for k, (rp, col) in (("cov", wc), ("nc", wn)):
        assert np.array_equal(t[k + "_row"].cpu().numpy(), rp)
        assert np.array_equal(t[k + "_col"].cpu().numpy()[:len(col)], col)


@pytest.mark.parametrize("sizes", [[1], [64], [65, 63], [1024, 1025, 1], [4096], [3] * 31 + [700], [3] * 32 + [700],
                                   list(range(1, 200, 3))])
def test_graph_blocks_bit_exact(sizes):
    from paper_2104_04547_amd import Scorer
    print(f"\n[gpu-case] cf_build_graphs sizes {sizes[:4]}.. x{len(sizes)}", flush=True)
    arch, w = weights("full")
    s = Scorer(arch, w, "fp32")
    _check(s, _batch(sizes, 9000, len(sizes)), arch.r_cov_u, arch.r_nc_u)
    s.close()


@pytest.mark.parametrize("r_nc", [37836, 37837, 65536])
def test_graph_cutoffs_around_the_32_bit_form(r_nc):
    from paper_2104_04547_amd import Scorer
    print(f"\n[gpu-case] cf_build_graphs cutoff {r_nc} u", flush=True)
    arch, w = weights("tiny")
    arch = dataclasses.replace(arch, r_cov_u=r_nc - 1, r_nc_u=r_nc)
    s = Scorer(arch, w, "fp32")
    b = _batch([150, 40], 60000, r_nc)
    b.xyz[0], b.xyz[1], b.xyz[2] = (0, 0, 0), (r_nc, 0, 0), (0, r_nc + 1, 0)       # ties at the cutoff
    b.xyz[3], b.xyz[4] = (-2 ** 31, 7, 7), (2 ** 31 - 1, 7, 7)                     # the whole int32 span apart
    _check(s, b, r_nc - 1, r_nc, _clipped_graph)
    s.close()
