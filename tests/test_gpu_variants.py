"""Kernel variants that a launch size picks: each against the other variant, bit for bit, or against the oracle, at the
sizes where the choice changes and where tiles have remainders."""
from dataclasses import replace

import numpy as np
import pytest

from synthetic import dit_inputs as I

pytestmark = pytest.mark.gpu


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("hidden,heads,mlp,hw,B", [(1152, 16, 4608, (32, 32), 3),      # both tile sizes of the float32 linear
                                                   (80, 4, 176, (10, 14), 5),          # remainders in rows, columns and k
                                                   (48, 4, 112, (64, 64), 2)])         # a whole group is one sample
def test_reference_forward_does_not_depend_on_the_batch(hidden, heads, mlp, hw, B):
    """The un-quantised forward of a batch (samples in groups, larger tiles) equals that of each latent alone."""
    import torch
    import paper_2503_02508_amd as qc
    m = I.ModelDesc(depth=1, hidden=hidden, heads=heads, mlp_dim=mlp, patch=2, latent_c=4, latent_h=hw[0], latent_w=hw[1])
    w = I.make_weights(m, 11)
    ctx = qc.Context(m, B, 1)
    ctx.load_weights(w, keep_fp32=True)
    x, lab = _cuda(I.make_latents(B, m, 12)), _cuda(I.make_labels(B, m, 13))
    eps, one = torch.empty_like(x), torch.empty_like(x)
    ctx.denoise_f32(x, 345, lab, B, eps)
    for b in range(B):
        ctx.denoise_f32(x[b:b + 1], 345, lab[b:b + 1], 1, one[b:b + 1])
    assert torch.equal(eps, one)
    assert float(eps.abs().max()) > 0
