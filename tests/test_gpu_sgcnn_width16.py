"""The width-16 SG-CNN against the oracle at the edges of its 32-atom blocks, with blocks of
fewer and of more neighbours than a workgroup stages (64 a row)."""
import dataclasses

import numpy as np
import pytest

import oracle
from helpers import weights
from test_gpu_sgcnn_blocks import N_LIG, SIZES, _batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 0.6])      # 0.6: some 100 neighbours an atom
def test_width16_blocks_match_oracle(scale):
    from paper_2104_04547_amd import Scorer, cfabi
    arch, w = weights("tiny")
    assert arch.H == 16
    w = {k: v * np.float32(1 / 32) if ".msg" in k else v for k, v in w.items()}     # dense sums stay O(1)
    b = _batch(SIZES, N_LIG, 13)
    b.xyz[:] = (b.xyz * scale).astype(np.int32)
    print(f"\n[gpu-case] cf_sgcnn_fwd tiny, coordinates x {scale}", flush=True)
    s = Scorer(arch, w, "fp32")
    db = cfabi.DeviceBatch.from_pose_batch(b)
    g = s.build_graphs(db, 256 * b.n_atoms, 256 * b.n_atoms)
    if scale < 1:
        assert int(g["nc_row"][-1]) - int(g["nc_row"][-2 - 600]) > 64 * 600
    got = s.sgcnn(db, g).cpu().numpy()
    assert s.status()[0] == 0
    want = oracle.sgcnn_batch(b, w, arch)
    np.testing.assert_allclose(got, want, rtol=1e-4, atol=2e-5 * np.abs(want).max())
    s.close()
