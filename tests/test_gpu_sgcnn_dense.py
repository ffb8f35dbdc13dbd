"""SG-CNN blocks with more edges than a workgroup stages: an atom with 6,000 edges that no
other atom has as a neighbour and no readout sees pushes the rows after it past the staged
range.  The other atoms' sums, and so the latents, keep their bits."""
import dataclasses

import numpy as np
import pytest

import synth
from helpers import weights
from test_gpu_sgcnn_blocks import _batch

pytestmark = pytest.mark.gpu

SIZES = [40, 150, 70]
LONE = [20, 45, 100, 170, 195]      # one or two in every block of 32, 64 or 128 atoms


def _graphs(rows):
    """cf_csr of both graphs from lists of neighbours per atom."""
    import torch
    from paper_2104_04547_amd import cfabi
    t = {}
    for key, lists in rows.items():
        row = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32)
        t[key + "_row"] = torch.from_numpy(row).cuda()
        t[key + "_col"] = torch.from_numpy(np.concatenate(lists).astype(np.int32)).cuda()
        t[key] = cfabi.cf_csr(t[key + "_row"].data_ptr(), t[key + "_col"].data_ptr(), int(row[-1]))
    return t


@pytest.mark.parametrize("name,prec", [("full", "fp32"), ("full", "bf16"), ("paper", "fp32"), ("paper", "bf16"),
                                       ("h32", "fp32"), ("h32", "bf16"), ("tiny", "fp32")])
def test_rows_past_the_staged_edges_keep_their_bits(name, prec):
    from paper_2104_04547_amd import Scorer, cfabi
    print(f"\n[gpu-case] cf_sgcnn_fwd rows past the staged edges {name} {prec}", flush=True)
    if name == "h32":
        arch = dataclasses.replace(synth.ARCHS["tiny"], H=32)
        w = synth.make_weights(arch)
    else:
        arch, w = weights(name)
    b = _batch(SIZES, [9, 30, 12], 12)
    b.is_lig[LONE] = 0
    s = Scorer(arch, w, prec)
    db = cfabi.DeviceBatch.from_pose_batch(b)
    g = s.build_graphs(db)
    plain, crowded = {}, {}
    for key in ("cov", "nc"):
        row, col = g[key + "_row"].cpu().numpy(), g[key + "_col"].cpu().numpy()
        lists = [col[row[i]:row[i + 1]] for i in range(len(row) - 1)]
        lists = [x[~np.isin(x, LONE)] if i not in LONE else x[:0] for i, x in enumerate(lists)]
        plain[key] = lists
        crowded[key] = [np.full(6000, i) if i in LONE else x for i, x in enumerate(lists)]
    got = s.sgcnn(db, _graphs(plain)).cpu().numpy()
    more = s.sgcnn(db, _graphs(crowded)).cpu().numpy()
    assert s.status()[0] == 0 and np.isfinite(got).all() and got.any()
    np.testing.assert_array_equal(more, got)
    s.close()
