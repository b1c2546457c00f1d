"""A sample's field, log q, log-det and g_z do not depend on the batch it is in: the same bits
from batches that run on eight waves a sample, on a few, on one, and, in FP32 on lattices of
at least 512 sites, by a launch per convolution up to 64 samples and in LDS above."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from paper_2208_08903_amd import lfs

from .gpu_util import dev, host, run_forward

pytestmark = pytest.mark.gpu

F, H = lfs.LFS_PLAIN_FP32, lfs.LFS_BF16_CONV

# dim, L, N, C, kernel, hidden_sizes, batches
CASES = [
    (2, 2, 3, 8, 3, None, (3, 600, 9000)),
    (2, 4, 3, 0, 3, (4, 4), (5, 300, 1300, 5000)),
    (2, 6, 3, 16, 3, None, (5, 700, 5000)),
    (2, 8, 3, 0, 3, (20, 6), (7, 513, 2500)),
    (3, 4, 2, 0, 3, (16, 16), (2, 257, 1100)),
    (2, 12, 2, 8, 3, None, (3, 1025)),
    (2, 24, 2, 0, 3, (6, 5), (1, 64, 65, 300)),
    (2, 24, 2, 16, 3, None, (2, 70)),
    (3, 8, 2, 0, 1, (3,), (3, 66, 600)),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("precision", [F, H])
def test_batch_does_not_change_a_sample(case, precision):
    dim, L, N, C, K, hs, batches = case
    print(f"batches {case} precision={precision}", flush=True)
    V = L ** dim
    desc = lfs.make_desc(dim, L, N, C, precision=precision, kernel=K, hidden_sizes=hs, algo=lfs.ALGO_GENERIC)
    params = si.flow_params(dim, N, C, seed=9, w_std=0.1, b_std=0.1, kernel=K, hidden_sizes=hs)
    z = si.normal_fields(8, batches[-1], V)
    gp = np.random.default_rng(5).standard_normal(z.shape).astype(np.float32)
    ref = None
    for B in batches:
        out = run_forward(desc, params, z[:B])
        gz = torch.full((B, V), float("nan"), device="cuda")
        g = torch.empty_like(out["params"])
        ws = torch.empty(lfs.workspace_bytes(desc, B, True), device="cuda", dtype=torch.uint8)
        lfs.flow_backward(desc, out["params"], out["saved"], dev(gp[:B], torch.float32), 0.3, g, gz, ws)
        torch.cuda.synchronize()
        got = {k: host(out[k])[:batches[0]] for k in ("phi", "logq", "logdet")}
        got["gz"] = host(gz)[:batches[0]]
        ref = ref or got
        for k, v in got.items():
            assert np.all(np.isfinite(v))
            np.testing.assert_array_equal(v, ref[k], err_msg=f"{k} of batch {B}")
