"""Gradients of conv shapes at the edges of the gradient kernels' tiles: channel counts
that are not multiples of 32, odd grids, one to three poses, strides 1 and 2 with every
kernel size, and a long output row (more than one run of 24 voxels)."""
import dataclasses

import numpy as np
import pytest

import synth
from test_gpu_backward import _check_grads, _oracle_grads

pytestmark = pytest.mark.gpu

SHAPES = {
    # stride-2 layers of 3^3 and 7^3, odd channel counts
    "odd": (((19, 40, 3, 2, -1), (40, 24, 5, 1, -1), (24, 36, 7, 2, -1)), 20, 1),
    # 3^3 after 7^3, a residual add, more than 64 channels, 5^3 stride 2
    "wide": (((19, 100, 7, 2, -1), (100, 100, 3, 1, -1), (100, 100, 3, 1, 1), (100, 34, 5, 2, -1)), 12, 2),
    # stride 1 on the grid: rows of 28 voxels
    "long": (((19, 40, 3, 1, -1), (40, 8, 5, 1, -1)), 28, 3),
    # the frequency-domain gradients: 7^3 at 16^3 with a residual add; 3^3 and 5^3 at 24^3
    # between 32 and 64 channels; 7^3 on an odd 13^3 grid
    "spectral7": (((19, 64, 5, 2, -1), (64, 64, 7, 1, -1), (64, 64, 7, 1, 1)), 32, 2),
    "spectral35": (((19, 32, 5, 2, -1), (32, 64, 3, 1, -1), (64, 32, 5, 1, -1)), 48, 2),
    "spectral_odd": (((19, 32, 5, 2, -1), (32, 32, 5, 2, -1), (32, 32, 7, 1, -1)), 52, 2),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_conv_gradients_of_odd_shapes(name):
    import torch
    from paper_2104_04547_amd import Scorer, cfabi
    conv, G, n = SHAPES[name]
    print(f"\n[gpu-case] cf_backward shapes {name} G={G} poses={n}", flush=True)
    arch = dataclasses.replace(synth.ARCHS["tiny"], name=name, conv=conv)
    w = synth.make_weights(arch)
    b = synth.make_poses("c1", n)
    dscore = np.random.default_rng(5).standard_normal(n)
    s = Scorer(arch, w, "fp32")
    grad, _ = s.backward(cfabi.DeviceBatch.from_pose_batch(b), G, torch.from_numpy(dscore.astype(np.float32)))
    s.check()
    got = s.unpack_params(grad)
    s.close()
    want, kink = _oracle_grads(b, w, arch, G, dscore)
    _check_grads(got, want, kink, name)
