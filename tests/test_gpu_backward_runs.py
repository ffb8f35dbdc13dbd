"""Weight gradients of conv layers whose input rows are wider than the registers that hold
the next run: 256 channels (16-byte loads) and 150 (4-byte loads), stride 2."""
import dataclasses

import numpy as np
import pytest

import synth
from test_gpu_backward import _check_grads, _oracle_grads

pytestmark = pytest.mark.gpu

SHAPES = {
    "vec": (((19, 256, 3, 2, -1), (256, 40, 7, 2, -1)), 12, 1),
    "scalar": (((19, 150, 5, 2, -1), (150, 24, 5, 2, -1)), 16, 2),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_weight_gradients_of_wide_rows(name):
    import torch
    from paper_2104_04547_amd import Scorer, cfabi
    conv, G, n = SHAPES[name]
    print(f"\n[gpu-case] cf_backward wide rows {name} G={G} poses={n}", flush=True)
    arch = dataclasses.replace(synth.ARCHS["tiny"], name=name, conv=conv)
    w = synth.make_weights(arch)
    b = synth.make_poses("c1", n)
    dscore = np.random.default_rng(6).standard_normal(n)
    s = Scorer(arch, w, "fp32")
    grad, _ = s.backward(cfabi.DeviceBatch.from_pose_batch(b), G, torch.from_numpy(dscore.astype(np.float32)))
    s.check()
    got = s.unpack_params(grad)
    s.close()
    want, kink = _oracle_grads(b, w, arch, G, dscore)
    _check_grads(got, want, kink, name)
