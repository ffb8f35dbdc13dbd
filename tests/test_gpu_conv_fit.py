"""Conv tiles fitted to the batch (and the plain form's small tiles): whatever tile a batch
size takes, the latents are bit for bit those of the variant itself (pinned, so that exactly
it runs)."""
import pytest

import synth
from helpers import weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch_name,G", [("full", 48), ("full", 40), ("full", 64), ("paper", 48), ("paper", 36), ("tiny", 24)])
@pytest.mark.parametrize("prec", ["bf16", "fp32"])
def test_small_batches_equal_the_pinned_variants(arch_name, G, prec):
    import torch
    from paper_2104_04547_amd import Scorer, cfabi
    arch, w = weights(arch_name)
    s, pinned = Scorer(arch, w, prec), Scorer(arch, w, prec)
    pinned.set_variants(G, s.variants(G))
    for n in (1, 2, 5, 12, 40):
        print(f"\n[gpu-case] cf_cnn3d_fwd {arch_name} {prec} G={G} poses={n}, fitted against pinned tiles", flush=True)
        grid = s.voxelize(cfabi.DeviceBatch.from_pose_batch(synth.make_poses("c1" if G < 32 else "c2", n)), G)
        a, b = s.cnn3d(grid, G), pinned.cnn3d(grid, G)
        torch.cuda.synchronize()
        assert torch.isfinite(a).all() and a.abs().max() > 0
        assert torch.equal(a, b)
    s.close()
    pinned.close()
