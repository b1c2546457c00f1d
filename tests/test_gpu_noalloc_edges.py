"""The allocation-free forward at the edges of its scratch, bit for bit against the forward
with a workspace of its own: activations of one sample that fill LFS_NOALLOC_SCRATCH_BYTES by
the documented rule (channels of each width, so that the kernels' padding adds to it), batches
that go through in parts, and networks whose weight fragments leave no room for all layers or
for one."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from paper_2208_08903_amd import lfs

from .gpu_util import dev, host, run_forward

pytestmark = pytest.mark.gpu

F, H = lfs.LFS_PLAIN_FP32, lfs.LFS_BF16_CONV

# dim, L, N, C, kernel, hidden_sizes, precision, B
CASES = [
    # one sample's activations within 8 MiB, its padded planes beyond
    (3, 64, 1, 0, 3, (5,), F, 1),
    (3, 64, 1, 0, 1, (1, 1), H, 1),
    (3, 62, 1, 0, 7, (5, 1), F, 1),
    (3, 54, 1, 0, 3, (5, 5), H, 1),
    (3, 46, 2, 0, 3, (9, 9), F, 1),
    (3, 40, 2, 16, 3, None, H, 1),
    (3, 50, 1, 8, 3, None, H, 1),
    (2, 180, 2, 32, 3, None, H, 1),
    (2, 254, 2, 16, 3, None, F, 1),
    (2, 256, 1, 0, 3, (13, 13), H, 1),
    # batches within 8 MiB by the rule, the planes beyond the array: in parts
    (2, 64, 2, 0, 3, (1, 1), F, 100),
    (2, 48, 3, 8, 3, None, H, 56),
    # fragments: a few layers at a time, one at a time, less than one
    (2, 8, 150, 0, 3, (16, 16, 16), F, 130),
    (2, 4, 90, 0, 5, (24, 24), H, 300),
    (3, 4, 2, 0, 7, (64, 64, 64), H, 5),
    (3, 4, 2, 0, 7, (64, 64), F, 5),
    (3, 4, 2, 0, 7, (64, 64, 64), F, 3),
    (2, 34, 130, 0, 5, (20, 20), F, 3),
]


@pytest.mark.parametrize("case", CASES)
def test_noalloc_matches_forward(case):
    dim, L, N, C, K, hs, precision, B = case
    print(f"noalloc forward {case}", flush=True)
    V = L ** dim
    desc = lfs.make_desc(dim, L, N, C, precision=precision, kernel=K, hidden_sizes=hs)
    params = (0.5 / (sum(hs or (C, C)) * K ** dim) ** 0.5) * si.flow_params(
        dim, N, C, seed=3, w_std=1.0, b_std=1.0, kernel=K, hidden_sizes=hs)
    z = si.normal_fields(60, B, V)
    ref = run_forward(desc, params, z)
    assert np.all(np.isfinite(host(ref["phi"])))
    phi = torch.full((B, V), float("nan"), device="cuda")
    logq = torch.full((B,), float("nan"), device="cuda", dtype=torch.float64)
    logdet = torch.full_like(logq, float("nan"))
    saved = torch.full(((N + 1) * B * V,), float("nan"), device="cuda")
    pt, zt = dev(params, torch.float32), dev(z, torch.float32)
    lfs.flow_forward_noalloc(desc, pt, zt, phi, logq, logdet, saved)
    torch.cuda.synchronize()
    for name, t in (("phi", phi), ("logq", logq), ("logdet", logdet), ("saved", saved)):
        np.testing.assert_array_equal(host(t).ravel(), host(ref[name]).ravel(), err_msg=name)
    lfs.flow_forward_noalloc(desc, pt, zt, zt, logq)  # phi may alias z
    torch.cuda.synchronize()
    np.testing.assert_array_equal(host(zt), host(ref["phi"]))
