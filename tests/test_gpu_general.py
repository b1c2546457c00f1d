"""The general kernels at the sizes where they can go wrong, against the FP64 oracle with
the tolerances of the default network's tests: kernels wider than the lattice, several
row tiles with channels that are no multiple of four, fragments too large for the LDS,
samples too large for it (one launch per convolution), several layer groups, and the
allocation-free forward whose scratch has no room for all fragments."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from oracle import flow as of
from paper_2208_08903_amd import lfs

from .gpu_util import dev, host, run_forward
from .test_gpu_parity import _check_backward, _check_forward

pytestmark = pytest.mark.gpu

CASES = [
    # dim, L, N, kernel, hidden_sizes, B
    (2, 2, 2, 7, (5,), 3),            # every tap wraps more than once
    (2, 6, 2, 3, (20, 33), 2),        # two and three row tiles, ragged channels
    (2, 10, 1, 3, (64, 2, 17), 2),
    (3, 4, 2, 5, (24, 24), 2),        # a layer's fragments exceed the LDS
    (2, 34, 2, 3, (16, 16), 2),       # a sample's state exceeds the LDS
    (3, 10, 2, 3, (32, 8), 3),
    (2, 8, 17, 3, (12, 12), 5),       # odd number of layers
]


def _case(dim, L, N, K, hs, B, precision):
    desc = lfs.make_desc(dim, L, N, 0, precision=precision, kernel=K, hidden_sizes=hs)
    params = si.flow_params(dim, N, 0, seed=900 + L + K, w_std=0.05, b_std=0.05, kernel=K, hidden_sizes=hs)
    z = si.normal_fields(700 + L, B, L ** dim)
    return desc, params, z, of.FlowShape(dim, L, N, 0, kernel=K, hidden_sizes=hs)


@pytest.mark.parametrize("case", CASES)
def test_general_forward_backward(case):
    print(f"general kernels {case}", flush=True)
    desc, params, z, fs = _case(*case, lfs.LFS_PLAIN_FP32)
    out, _ = _check_forward(desc, params, z, fs, lfs.LFS_PLAIN_FP32)
    _check_backward(desc, params, z, fs, out, lfs.LFS_PLAIN_FP32)


@pytest.mark.parametrize("case", [CASES[1], CASES[4], CASES[5]])
def test_general_forward_bf16(case):
    print(f"general kernels, BF16, {case}", flush=True)
    desc, params, z, fs = _case(*case, lfs.LFS_BF16_CONV)
    _check_forward(desc, params, z, fs, lfs.LFS_BF16_CONV, rho=0.6)


@pytest.mark.parametrize("B", [1, 7])
def test_noalloc_without_room_for_fragments(B):
    """343 taps of 64 x 64 channels: 5.5 MB of fragments per convolution in 8 MiB of scratch."""
    desc, params, z, fs = _case(3, 4, 2, 7, (64, 64), B, lfs.LFS_PLAIN_FP32)
    assert lfs.workspace_bytes(desc, B, False) > lfs.NOALLOC_SCRATCH_BYTES
    ref = run_forward(desc, params, z)
    phi = torch.full((B, 64), float("nan"), device="cuda")
    logq = torch.full((B,), float("nan"), device="cuda", dtype=torch.float64)
    saved = torch.full((3 * B * 64,), float("nan"), device="cuda")
    lfs.flow_forward_noalloc(desc, dev(params, torch.float32), dev(z, torch.float32), phi, logq, None, saved)
    torch.cuda.synchronize()
    p, r = host(phi), host(ref["phi"])
    bound = 1e-5 * (343 / 9) * (1 + np.abs(r))
    assert np.all(np.abs(p - r) <= bound)
    assert np.all(np.abs(host(logq) - host(ref["logq"])) <= 1e-4 * 64)
    s = host(saved).reshape(3, B, 64)
    np.testing.assert_array_equal(s[0], z)
    np.testing.assert_array_equal(s[2], p)


@pytest.mark.parametrize("L,hs,B", [(8, (20, 6), 9), (8, (8, 8), 300), (34, (16, 16), 2)])
@pytest.mark.parametrize("mode", [lfs.BN_BATCH, lfs.BN_RUNNING])
def test_batch_norm_shapes(L, hs, B, mode):
    """Batch norm with several row tiles and ragged channels, with more samples than
    workgroups, and with a sample too large for the LDS: the tolerances of the batch-norm
    tests."""
    from . import test_gpu_bn as bn
    print(f"batch norm L={L} hidden={hs} B={B} mode={mode}", flush=True)
    desc, params, z, stats, fs = bn._case(2, L, 2, 3, hs, B, lfs.LFS_PLAIN_FP32)
    out = bn._forward(desc, params, z, mode, stats)
    f = of.flow_forward(params.astype(np.float64), z.astype(np.float64), fs,
                        bn_stats=None if mode == lfs.BN_BATCH else of.unpack_bn_stats(stats.astype(np.float64), fs))
    ref = f["phi"].reshape(B, -1)
    assert np.all(np.abs(host(out["phi"]) - ref) <= 1e-5 * (1 + np.abs(ref)))
    g_phi = np.random.default_rng(4).standard_normal(z.shape).astype(np.float32)
    gp, gz = bn._backward(desc, out, g_phi, 0.37, mode)
    go, zo = of.flow_vjp(params.astype(np.float64), z.astype(np.float64), fs, g_phi.astype(np.float64), 0.37,
                         bn_stats=None if mode == lfs.BN_BATCH else of.unpack_bn_stats(stats.astype(np.float64), fs))
    assert np.linalg.norm(gp - go) <= 1e-4 * np.linalg.norm(go)
    assert np.linalg.norm(gz - zo) <= 1e-4 * np.linalg.norm(zo)


@pytest.mark.parametrize("case", [
    (3, 12, 1, 3, (16, 16), 3),       # default network, slabs of a few slices
    (3, 6, 1, 3, (32, 32), 2),        # default network, two row tiles and column blocks
    (3, 4, 1, 7, (5, 18), 2),         # several groups of column tiles
    (2, 6, 1, 5, (33, 6), 3),         # slabs whose sites are no multiple of four
    (3, 50, 1, 3, (4,), 1),           # a slab of one slice exceeds the LDS
])
def test_weight_gradient_slabs(case):
    print(f"weight gradients {case}", flush=True)
    desc, params, z, fs = _case(*case, lfs.LFS_PLAIN_FP32)
    out, _ = _check_forward(desc, params, z, fs, lfs.LFS_PLAIN_FP32)
    _check_backward(desc, params, z, fs, out, lfs.LFS_PLAIN_FP32)


@pytest.mark.parametrize("dim,L,N,C,hs,B", [
    (2, 12, 12, 8, None, 3),          # the default network, a sample in LDS, a ragged last tile
    (3, 8, 16, 0, (5,), 2),           # many tiles per wave
    (2, 2, 5, 0, (3, 3), 4),          # one tile, two active sites
    (2, 68, 16, 16, None, 2),         # a launch per convolution
    (3, 10, 16, 0, (16, 6), 3),
])
@pytest.mark.parametrize("precision", [lfs.LFS_PLAIN_FP32, lfs.LFS_BF16_CONV])
def test_log_det_keeps_every_bit_of_s(dim, L, N, C, hs, B, precision):
    """With s = b exactly at every active site the log-det is N (V / 2) b: sums of s in FP64 are
    within (terms + layers) roundings of it, and sums over layers in FP32 are not."""
    print(f"log-det dim={dim} L={L} N={N} C={C} hidden={hs} precision={precision}", flush=True)
    V = L ** dim
    desc = lfs.make_desc(dim, L, N, C, final_tanh=False, precision=precision, hidden_sizes=hs)
    params = np.zeros((N, lfs.param_count(desc) // N), np.float32)
    params[:, -2] = b = np.float32(-0.1)
    out = run_forward(desc, params.ravel(), si.normal_fields(5, B, V))
    exact = N * (V // 2) * float(b)
    bound = (V // 2 + N) * 2.0 ** -53 * abs(exact)
    assert np.all(np.abs(host(out["logdet"]) - exact) <= bound)


@pytest.mark.parametrize("case", [
    (2, 10, 2, 3, (6, 5), 100),       # samples cut in uneven parts
    (2, 6, 1, 3, (3,), 1),            # a slice a part
    (2, 34, 1, 5, (9,), 1),           # parts thinner than a slab, more than 64 chunks
    (3, 8, 1, 1, (2,), 70),
    (2, 4, 2, 3, (4, 4), 1100),       # more samples than chunks
])
def test_weight_gradient_parts(case):
    print(f"weight gradients of parts of samples {case}", flush=True)
    desc, params, z, fs = _case(*case, lfs.LFS_PLAIN_FP32)
    out, _ = _check_forward(desc, params, z, fs, lfs.LFS_PLAIN_FP32)
    _check_backward(desc, params, z, fs, out, lfs.LFS_PLAIN_FP32)


@pytest.mark.parametrize("L,hs,B", [(4, (5, 4), 700), (4, (8, 3), 4097), (2, (20,), 4100)])
def test_batch_norm_workgroups(L, hs, B):
    """More samples than workgroups, at two eight-wave workgroups a CU and at four of four
    waves, against the oracle; log q too."""
    from . import test_gpu_bn as bn
    print(f"batch norm L={L} hidden={hs} B={B}", flush=True)
    desc, params, z, stats, fs = bn._case(2, L, 2, 3, hs, B, lfs.LFS_PLAIN_FP32)
    out = bn._forward(desc, params, z, lfs.BN_BATCH, stats)
    f = of.flow_forward(params.astype(np.float64), z.astype(np.float64), fs)
    ref = f["phi"].reshape(B, -1)
    assert np.all(np.abs(host(out["phi"]) - ref) <= 1e-5 * (1 + np.abs(ref)))
    assert np.all(np.abs(host(out["logq"]) - f["logq"]) <= 1e-4 * L * L)
    g_phi = np.random.default_rng(4).standard_normal(z.shape).astype(np.float32)
    gp, gz = bn._backward(desc, out, g_phi, 0.37, lfs.BN_BATCH)
    go, zo = of.flow_vjp(params.astype(np.float64), z.astype(np.float64), fs, g_phi.astype(np.float64), 0.37)
    assert np.linalg.norm(gp - go) <= 1e-4 * np.linalg.norm(go)
    assert np.linalg.norm(gz - zo) <= 1e-4 * np.linalg.norm(zo)


@pytest.mark.parametrize("case", [
    (2, 8, 3, 1, (64, 64, 64, 64), 1000),    # 132 MB of planes a layer: two layers, then one
    (2, 64, 3, 1, (64, 64, 64, 64), 16),     # as much, by a launch per convolution
    (2, 8, 2, 1, (64, 64, 64, 64), 1300),    # one layer a group
])
def test_layer_groups(case):
    """More planes than are kept at once for the weight gradients."""
    print(f"layer groups {case}", flush=True)
    desc, params, z, fs = _case(*case, lfs.LFS_PLAIN_FP32)
    assert lfs.workspace_bytes(desc, case[5], True) < 400 << 20
    out, _ = _check_forward(desc, params, z, fs, lfs.LFS_PLAIN_FP32)
    _check_backward(desc, params, z, fs, out, lfs.LFS_PLAIN_FP32)


def test_layer_groups_batch_norm():
    """The same with batch norm, whose store has three planes a hidden one: two layers, then one."""
    from . import test_gpu_bn as bn
    hs, B = (64, 64, 64, 64), 700
    desc, params, z, stats, fs = bn._case(2, 8, 3, 1, hs, B, lfs.LFS_PLAIN_FP32)
    params *= np.float32(0.5)
    out = bn._forward(desc, params, z, lfs.BN_BATCH, stats)
    g_phi = np.random.default_rng(4).standard_normal(z.shape).astype(np.float32)
    gp, gz = bn._backward(desc, out, g_phi, 0.37, lfs.BN_BATCH)
    go, zo = of.flow_vjp(params.astype(np.float64), z.astype(np.float64), fs, g_phi.astype(np.float64), 0.37)
    assert np.linalg.norm(gp - go) <= 1e-4 * np.linalg.norm(go)
    assert np.linalg.norm(gz - zo) <= 1e-4 * np.linalg.norm(zo)


def test_default_network_beyond_slabs():
    """The default network in FP32 on a lattice of which a slab of one slice exceeds the LDS."""
    case = (3, 38, 1, 3, (16, 16), 1)
    print(f"large default network {case}", flush=True)
    desc, params, z, fs = _case(*case, lfs.LFS_PLAIN_FP32)
    out, _ = _check_forward(desc, params, z, fs, lfs.LFS_PLAIN_FP32)
    _check_backward(desc, params, z, fs, out, lfs.LFS_PLAIN_FP32)
