"""Gradients and the context's HBM budget: the same bits whatever the context ran before,
no refusal at a budget above one that is accepted, and the direct kernels, which a small
budget selects, against the oracle."""
import dataclasses

import numpy as np
import pytest

import synth
from helpers import weights
from test_gpu_backward import _check_grads, _oracle_grads

pytestmark = pytest.mark.gpu


def _batch(n, cfg="c2"):
    from paper_2104_04547_amd import cfabi
    return cfabi.DeviceBatch.from_pose_batch(synth.make_poses(cfg, n))


def _dscore(n):
    import torch
    return torch.from_numpy(np.random.default_rng(5).standard_normal(n).astype(np.float32))


@pytest.mark.parametrize("large", [60, 200])
def test_gradients_do_not_depend_on_earlier_calls(large):
    """A budget of 5 GiB holds the frequency-domain gradients of two poses twice over; 60
    scored poses of 32^3 take more than half of it together with the weights, 200 fill it."""
    import torch
    from paper_2104_04547_amd import Scorer
    arch, w = weights("full")
    G, n, budget = 32, 2, 5 << 30
    db, dbl, ds = _batch(n), _batch(large), _dscore(n)
    print(f"\n[gpu-case] cf_backward full G={G} poses={n}, score of {large} poses between", flush=True)
    s = Scorer(arch, w, "fp32", budget)
    first, _ = s.backward(db, G, ds)
    s.score(dbl, G)
    again, _ = s.backward(db, G, ds)
    s.check()
    assert torch.equal(first, again)
    s.close()
    if large == 60:          # the large call first, with room left beside it
        s = Scorer(arch, w, "fp32", budget)
        s.score(dbl, G)
        after, _ = s.backward(db, G, ds)
        s.check()
        assert torch.equal(first, after)
        s.close()


ARCH = dict(conv=((19, 32, 5, 2, -1), (32, 32, 7, 1, -1), (32, 64, 7, 2, -1)), cnn_dense=0)


def test_a_larger_budget_is_not_refused():
    from paper_2104_04547_amd import Scorer, cfabi
    arch = dataclasses.replace(synth.ARCHS["tiny"], name="budget_probe", **ARCH)
    w = synth.make_weights(arch)
    db, ds = _batch(1, "c1"), _dscore(1)
    accepted = []
    for mib in range(60, 200, 2):
        s = Scorer(arch, w, "fp32", mib << 20)
        try:
            s.backward(db, 48, ds)
            s.check()
            accepted.append(True)
        except cfabi.CfError as e:
            assert e.code == cfabi.CF_ERR_OOM
            accepted.append(False)
        s.close()
    print("\n[gpu-case] cf_backward accepted from", 60 + 2 * accepted.index(True), "MiB on", flush=True)
    assert accepted == sorted(accepted), accepted
    assert not accepted[0] and accepted[-1]


@pytest.mark.parametrize("mib", [400, 4000])
def test_direct_and_spectral_gradients_match_the_oracle(mib):
    """400 MiB refuse the frequency domain (its buffers alone need 200 beside the weights)."""
    import torch
    from paper_2104_04547_amd import Scorer
    arch = dataclasses.replace(synth.ARCHS["tiny"], name="budget_probe",
                               conv=((19, 64, 5, 2, -1), (64, 64, 5, 1, -1)))
    w = synth.make_weights(arch)
    G, n = 32, 2
    print(f"\n[gpu-case] cf_backward budget {mib} MiB", flush=True)
    s = Scorer(arch, w, "fp32", mib << 20)
    grad, _ = s.backward(_batch(n, "c1"), G, _dscore(n))
    s.check()
    got = s.unpack_params(grad)
    s.close()
    want, kink = _oracle_grads(synth.make_poses("c1", n), w, arch, G, _dscore(n).numpy().astype(np.float64))
    _check_grads(got, want, kink, f"budget {mib}")
