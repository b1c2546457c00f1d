"""The fused kernels where a launch rule or a loop changes with the batch: the forward with and
without weights fetched a layer ahead (same bits), the sums over 1, 16, 17 and more
workgroups' weight-gradient partials (against the general kernels: both FP32, so within the
gradient tolerance of each against FP64, 1e-4 per block in the 2-norm)."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from paper_2208_08903_amd import lfs

from .gpu_util import host, run_backward, run_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,C", [(8, 8), (8, 16), (16, 8), (16, 16)])
def test_forward_batches_give_the_same_bits(L, C):
    desc = lfs.make_desc(2, L, 3, C, precision=lfs.LFS_PLAIN_FP32)
    params = si.flow_params(2, 3, C, seed=4, w_std=0.1, b_std=0.1)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    z = si.normal_fields(2, 4 * cus + 3, L * L)
    ref = run_forward(desc, params, z)
    for B in (1, 2 * cus, 2 * cus + 1):
        out = run_forward(desc, params, z[:B])
        for k in ("phi", "logq", "logdet"):
            np.testing.assert_array_equal(host(out[k]), host(ref[k])[:B], err_msg=f"{k} of batch {B}")


@pytest.mark.parametrize("B", [1, 2, 15, 16, 17, 33, 130])
@pytest.mark.parametrize("dim,L,C", [(2, 8, 8), (2, 16, 16), (3, 8, 16)])
def test_gradients_of_few_workgroups(dim, L, C, B):
    print(f"fused gradients dim={dim} L={L} C={C} B={B}", flush=True)
    params = si.flow_params(dim, 2, C, seed=6, w_std=0.05, b_std=0.05)
    z = si.normal_fields(3, B, L ** dim)
    gp = np.random.default_rng(1).standard_normal(z.shape).astype(np.float32)
    g = []
    for algo in (lfs.ALGO_FUSED, lfs.ALGO_GENERIC):
        desc = lfs.make_desc(dim, L, 2, C, precision=lfs.LFS_PLAIN_FP32, algo=algo)
        g.append(run_backward(desc, run_forward(desc, params, z), gp, 0.3)[0].astype(np.float64).reshape(2, -1))
    sizes, off = [C * 3 ** dim, C, C * C * 3 ** dim, C, 2 * C * 3 ** dim, 2], 0
    for n in sizes:
        a, b = (v[:, off:off + n] for v in g)
        assert np.linalg.norm(a - b) <= 2e-4 * np.linalg.norm(b)
        off += n
