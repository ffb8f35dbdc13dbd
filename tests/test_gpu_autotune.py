"""Autotuned conv layers run the kernels that were measured: the ids it reports are the
tiles that run at the tuned batch (by the per-kernel timing's names), the small tiles are
among the candidates, and no batch size changes a pose's latent."""
import pytest

import synth
from helpers import weights

pytestmark = pytest.mark.gpu


def _ran(s, grid, G):
    """Names of the direct kernels that one 3D-CNN call of the grid ran, per layer."""
    import torch
    from paper_2104_04547_amd import cfabi
    cfabi.cf_timing_enable(s.ctx, True)
    out = s.cnn3d(grid, G)
    torch.cuda.synchronize()
    stats = cfabi.cf_timing_read(s.ctx)
    cfabi.cf_timing_enable(s.ctx, False)
    return out, {k.split(".")[0]: k.split(".")[1] for k in stats if k.startswith("conv") and ".fft32" not in k}


def _grid(s, n, G):
    from paper_2104_04547_amd import cfabi
    return s.voxelize(cfabi.DeviceBatch.from_pose_batch(synth.make_poses("c2", n)), G)


@pytest.mark.parametrize("prec,n_tuned", [("fp32", 2), ("fp32", 6), ("bf16", 1), ("bf16", 24)])
def test_the_tuned_variants_are_the_ones_that_run(prec, n_tuned):
    import torch
    from paper_2104_04547_amd import Scorer, cfabi
    arch, w = weights("full")
    G = 32
    s, plain = Scorer(arch, w, prec), Scorer(arch, w, prec)
    names = cfabi.cf_conv_variant_names()
    print(f"\n[gpu-case] cf_autotune full {prec} G={G} poses={n_tuned}", flush=True)
    v = s.autotune(G, n_tuned)
    tuned = {f"conv{i}": names[k] for i, k in enumerate(v) if names[k] != "fft32"}
    for n in (n_tuned, n_tuned + 7):
        _, ran = _ran(s, _grid(s, n, G), G)
        assert ran == tuned, (n, ran, tuned)
    if prec == "fp32":     # two and more times faster than the large tiles at these sizes
        assert tuned["conv0"].startswith("f32k7s2") and tuned["conv5"].startswith("f32k7s2"), tuned
    # the last layer's two-pose tile leaves the chip idle for one pose; the tile that runs is named
    _, ran = _ran(plain, _grid(plain, 1, G), G)
    assert not ran["conv5"].endswith("_p2") and ran["conv5"] != names[plain.variants(G)[5]], ran
    # any batch size, smaller than the tuned one or not: the same latents
    grid = _grid(s, 12, G)
    all12, _ = _ran(s, grid, G)
    for n in (1, 5):
        part, _ = _ran(s, grid[:n].contiguous(), G)
        assert torch.equal(part, all12[:n])
    s.close()
    plain.close()


def test_pinned_variants_run_at_any_size():
    from paper_2104_04547_amd import Scorer, cfabi
    arch, w = weights("full")
    s = Scorer(arch, w, "bf16")
    names = cfabi.cf_conv_variant_names()
    s.autotune(32, 3)
    s.set_variants(32, Scorer(arch, w, "bf16").variants(32))
    want = {f"conv{i}": names[k] for i, k in enumerate(s.variants(32)) if names[k] != "fft32"}
    for n in (1, 9):
        print(f"\n[gpu-case] cf_cnn3d_fwd pinned default variants, {n} poses", flush=True)
        assert _ran(s, _grid(s, n, 32), 32)[1] == want
    s.close()
