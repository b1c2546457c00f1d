"""The chain and analysis kernels at the edges of their chunks, against the oracle: MH chains
around the length from which two launches are used and around whole chunks of 64, with
log-weights that compare in every way (infinities, NaN, ties, none and all accepted),
continued over calls; autocorrelation around its chunks and lag groups.  Decisions are
bit-exact; FP64 sums in another order: 1e-12 relative, as in the analysis tests."""
import numpy as np
import pytest
import torch

import seeded_inputs as si
from oracle import analysis as an
from oracle import mh as om
from paper_2208_08903_amd import lfs

from .gpu_util import dev, host

pytestmark = pytest.mark.gpu


def _weights(kind, n, seed):
    w = si.logw_stream(seed, n, 1.0)
    lu = si.log_uniforms(seed + 1, n)
    if kind == "wild":
        r = np.random.default_rng(seed + 2)
        for v in (np.inf, -np.inf, np.nan, 0.0, -0.0):
            w[r.integers(0, n, max(1, n // 40))] = v
        lu[r.integers(0, n, max(1, n // 40))] = -np.inf
    elif kind == "ties":
        w = np.round(w * 2) / 2
        lu = np.round(lu * 2) / 2
    elif kind == "rising":
        w = np.arange(n, dtype=np.float64)
    elif kind == "falling":
        w = -1e6 * np.arange(n, dtype=np.float64)
    return w, lu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 130, 511, 512, 513, 1024, 1300])
@pytest.mark.parametrize("kind", ["normal", "wild", "ties", "rising", "falling"])
def test_mh_chain_edges(n, kind):
    print(f"mh chain n={n} {kind}", flush=True)
    chains = 3
    W, U = zip(*(_weights(kind, 2 * n, 50 + 10 * c) for c in range(chains)))
    W, U = np.stack(W), np.stack(U)
    state = lfs.new_chain_state(chains)
    cur = np.empty((chains, 2 * n), np.int64)
    acc = np.empty((chains, 2 * n), np.uint8)
    for k in range(2):  # the chain goes on over two calls
        sl = slice(k * n, (k + 1) * n)
        c = torch.empty(chains, n, dtype=torch.int64, device="cuda")
        a = torch.empty(chains, n, dtype=torch.uint8, device="cuda")
        lfs.mh_chain(dev(W[:, sl], torch.float64), dev(U[:, sl], torch.float64), state, c, a)
        cur[:, sl], acc[:, sl] = host(c), host(a)
    st = lfs.decode_chain_state(state)
    for i in range(chains):
        with np.errstate(invalid="ignore"):
            co, ao, _ = om.mh_chain(W[i], U[i])
        np.testing.assert_array_equal(cur[i], co)
        np.testing.assert_array_equal(acc[i], np.asarray(ao, np.uint8))
        assert st[i]["n_seen"] == 2 * n and st[i]["n_acc"] == int(np.sum(ao)) - 1 and st[i]["idx_cur"] == co[-1]


@pytest.mark.parametrize("n,w_max", [(511, 100), (512, 511), (513, 600), (1500, 1023), (2600, 1024), (5000, 2047),
                                     (140000, 300)])
def test_autocorr_edges(n, w_max):
    print(f"autocorr n={n} w_max={w_max}", flush=True)
    x = si.correlated_series(70, 2, n, 0.7)
    gamma = torch.empty(2, w_max + 1, dtype=torch.float64, device="cuda")
    tau = torch.empty(2, dtype=torch.float64, device="cuda")
    lfs.autocorr(dev(x, torch.float64), w_max, 6.0, tau, gamma=gamma)
    torch.cuda.synchronize()
    g = host(gamma)
    for s in range(2):
        d = x[s] - x[s].mean()
        T = min(w_max, n - 1)
        for t in {0, 1, 3, 4, 7, T - 1, T} | ({255, 256, 1023, 1024} & set(range(T + 1))):
            assert abs(g[s, t] - d[:n - t] @ d[t:] / (n - t)) <= 1e-12 * g[s, 0]
        assert np.all(np.isnan(g[s, T + 1:]))


@pytest.mark.parametrize("n", [1, 1023, 1024, 8191, 8192, 8193, 20000])
def test_ess_edges(n):
    w = si.logw_stream(80, n, 2.0) - 700.0
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    lfs.ess(dev(w, torch.float64), out)
    assert abs(float(out.item()) - an.ess(w)) <= 1e-12


@pytest.mark.parametrize("n,ragged", [(2 ** 31 - 1, False), (2 ** 31 - 1025, False), (2 ** 31 - 1, True)])
def test_longest_chain(n, ragged):
    """2^31 - 1 proposals, the most a call can name, where what is looked up past the end lies
    past the largest int, and the most that two launches take.  Accepted at a few positions
    only, so the record is known."""
    at = [0, 5, 2 ** 30 + 17, n - 66, n - 1]
    logw = torch.zeros(1, n, dtype=torch.float64, device="cuda")
    lu = torch.ones(1, n, dtype=torch.float64, device="cuda")
    lu[0, at[1:]] = -1.0
    cur = torch.full((1, n), -7, dtype=torch.int64, device="cuda")
    acc = torch.full((1, n), 9, dtype=torch.uint8, device="cuda")
    state = lfs.new_chain_state(1)
    print(f"longest chain n={n} ragged={ragged}", flush=True)
    if ragged:
        lfs.mh_chain_ragged(torch.tensor([0, n], device="cuda"), logw.view(-1), lu.view(-1), state,
                            torch.zeros(1, dtype=torch.int32, device="cuda"), cur.view(-1), acc.view(-1))
    else:
        lfs.mh_chain(logw, lu, state, cur, acc)
    torch.cuda.synchronize()
    print("done", flush=True)
    del logw, lu
    for a, b in zip(at, at[1:] + [n]):
        assert bool((cur[0, a:b] == a).all()) and int(acc[0, a]) == 1
    assert int(acc.sum(dtype=torch.int64)) == len(at)
    st = lfs.decode_chain_state(state)[0]
    assert st["n_seen"] == n and st["n_acc"] == len(at) - 1 and st["idx_cur"] == n - 1 and st["w_cur"] == 0.0
    del cur, acc
    torch.cuda.empty_cache()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n,at", [(600, 300), (600, 0), (1500, 800)])
def test_autocorr_of_infinities(n, at, value):
    """A lag's average is over its own pairs only: it is infinite where no pair holds the
    element whose deviation is NaN, and NaN where one does."""
    x = si.correlated_series(71, 1, n, 0.7)
    x[0, at] = value
    gamma = torch.empty(1, n, dtype=torch.float64, device="cuda")
    tau = torch.empty(1, dtype=torch.float64, device="cuda")
    lfs.autocorr(dev(x, torch.float64), n - 1, 6.0, tau, gamma=gamma)
    with np.errstate(invalid="ignore"):
        d = x[0] - x[0].mean()
        ref = np.array([np.sum(d[:n - t] * d[t:]) / (n - t) for t in range(n)])
    np.testing.assert_array_equal(host(gamma)[0], ref)
    assert np.isnan(float(tau.item()))


@pytest.mark.parametrize("n", [1, 2, 3, 5, 64, 100, 127, 128, 129, 513, 1001, 2047, 2048, 2049])
@pytest.mark.parametrize("w_max", [0, 1, 63, 2000])
def test_autocorr_short_series(n, w_max):
    """Chunks as long as the series, and around the length up to which the chunks are added in
    the last launch; windows shorter and longer than the series."""
    print(f"autocorr n={n} w_max={w_max}", flush=True)
    S = 5
    x = si.correlated_series(72, S, n, 0.7) if n > 1 else np.array([[1.0], [2.0], [-3.0], [0.5], [0.25]])
    gamma = torch.full((S, w_max + 1), 7.0, dtype=torch.float64, device="cuda")
    tau = torch.empty(S, dtype=torch.float64, device="cuda")
    window = torch.empty(S, dtype=torch.int32, device="cuda")
    index = torch.arange(n - 1, -1, -1, device="cuda").repeat(S, 1)  # read backwards
    lfs.autocorr(dev(x, torch.float64), w_max, 6.0, tau, window=window, gamma=gamma, index=index)
    g, T = host(gamma), min(w_max, n - 1)
    for s in range(S):
        y = x[s, ::-1]
        d = y - y.mean()
        ref = np.array([d[:n - t] @ d[t:] / (n - t) for t in range(T + 1)])
        assert np.all(np.abs(g[s, :T + 1] - ref) <= 1e-12 * ref[0])
        assert np.all(np.isnan(g[s, T + 1:]))
        if ref[0] == 0:
            assert np.isnan(host(tau)[s])
            continue
        t, W = 0.5, 0
        for W in range(1, T + 1):
            t += ref[W] / ref[0]
            if W >= 6.0 * t:
                break
        assert abs(host(tau)[s] - t) <= 1e-9 * abs(t) + 1e-12 and host(window)[s] == min(W, T)


@pytest.mark.parametrize("n,S", [(2, 300), (255, 300), (2047, 300), (2048, 300), (2049, 300), (2049, 513)])
def test_ess_of_several_series(n, S):
    w = np.stack([si.logw_stream(80 + k, n, 2.0) for k in range(S)])
    out = torch.empty(S, dtype=torch.float64, device="cuda")
    lfs.ess(dev(w, torch.float64), out)
    assert np.all(np.abs(host(out) - [an.ess(v) for v in w]) <= 1e-12)
