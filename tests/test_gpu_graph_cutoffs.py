"""Neighbour lists at cutoffs beyond 16 bits: blocks whose atoms share one place (a pose of
64 m + 1 atoms always ends in one, with a single atom) beside atoms inside, at and just
outside the cutoff, and beyond the 16-bit range."""
import dataclasses

import numpy as np
import pytest

from helpers import weights
from test_gpu_graph_blocks import _batch, _check, _clipped_graph

pytestmark = pytest.mark.gpu


def _cutoff_batch(r, seed):
    """Poses of 64 m + 1 atoms and one with a whole block at a single place."""
    sizes = [1, 65, 129, 128, 65]
    b = _batch(sizes, 60000, seed)
    off = b.atom_off
    b.xyz[off[3] + 64:off[3] + 128] = (17, -3, 5)                     # the block at one place
    for p in (1, 2, 3, 4):
        last = b.xyz[off[p + 1] - 1].astype(np.int64)                  # the atom of the one-place block
        for k, d in enumerate((r - 1, r, r + 1, 100, 32766, 32767, 32768, 50000)):
            for sign in (1, -1):
                v = np.zeros(3, np.int64)
                v[k % 3] = sign * d
                b.xyz[off[p] + 2 * k + (sign > 0)] = last + v
    b.xyz[off[4]] = (2 ** 31 - 1, 2 ** 31 - 1, -2 ** 31)
    return b


@pytest.mark.parametrize("r_nc", [4608, 32765, 32766, 32767, 34000, 37836, 37837, 65535, 65536])
def test_graph_cutoffs_beyond_16_bits(r_nc):
    from paper_2104_04547_amd import Scorer
    print(f"\n[gpu-case] cf_build_graphs, blocks at one place, cutoff {r_nc} u", flush=True)
    arch, w = weights("tiny")
    arch = dataclasses.replace(arch, r_cov_u=r_nc // 2, r_nc_u=r_nc)
    s = Scorer(arch, w, "fp32")
    _check(s, _cutoff_batch(r_nc, r_nc), r_nc // 2, r_nc, _clipped_graph)
    s.close()
