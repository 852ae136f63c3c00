"""Calibration on the device at the sizes where its kernels can go wrong: K-means
with exact distance ties, duplicate tokens, odd token counts, squares below the
normal range and NaN or infinite tokens against the oracle's Lloyd rounds (bit for
bit), the token-order statistics at the edges of a
staged run, and the principal basis of degenerate second moments (low rank, equal
eigenvalues) against its defining equations."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_26425_amd import quantwm as qw

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _calibrate(cfg, q, k, v, iters):
    calib = torch.zeros(qw.quantwm_calib_bytes(cfg), dtype=torch.uint8, device=DEV)
    nh, n = (0 if q is None else q.shape[1]), k.shape[1]
    ws = torch.empty(qw.quantwm_calibrate_workspace_bytes(cfg, nh, n), dtype=torch.uint8, device=DEV)
    qw.quantwm_calibrate(cfg, q, nh, k, v, n, iters, calib, ws)
    off, bh = qw.quantwm_calib_offsets(cfg), cfg.batch * cfg.heads
    flat = calib.cpu().numpy().reshape(bh, off.slab_bytes)

    def field(at, dtype, *shape):
        size = int(np.prod(shape)) * np.dtype(dtype).itemsize
        return np.ascontiguousarray(flat[:, at:at + size]).view(dtype).reshape(bh, *shape)

    d, kc, r = cfg.head_dim, cfg.n_centroids, cfg.rank
    e = np.uint16 if cfg.dtype == qw.BF16 else np.float32
    return dict(mu_k=field(off.mu_k, e, kc, d), mu_v=field(off.mu_v, e, kc, d), w=field(off.w, np.float32, d),
                u=field(off.u_t, e, r, d), lam=field(off.lam, np.float32, r))


def _bits16(x):
    return (np.ascontiguousarray(x, np.float32).view(np.uint32) >> 16).astype(np.uint16)


def _tokens(kind, n, d, rng):
    if kind == "ties":      # small integers: exact ties between many centroids, duplicate tokens
        return rng.integers(-1, 2, (1, n, 2, d)).astype(np.float32)
    if kind == "close":     # one point and tokens a few BF16 ulps around it: every centroid inside the bound
        return (1.0 + rng.integers(-2, 3, (1, n, 2, d)) / 128.0).astype(np.float32)
    if kind == "tiny":      # squares below the normal range
        return torch.from_numpy((rng.standard_normal((1, n, 2, d)) * 1e-22).astype(np.float32)).bfloat16().float().numpy()
    if kind == "nan":       # NaN and infinite centroids among the first and later ids of both lane halves
        x = (rng.integers(-64, 65, (1, n, 2, d)) / 8.0).astype(np.float32)
        x[0, [4 * n // 48, 12 * n // 48, 33 * n // 48], 0, 3] = np.nan
        x[0, [0, 5 * n // 48], 1, 7], x[0, 20 * n // 48, 1, 2] = np.nan, np.inf
        return x
    x = rng.standard_normal((1, n, 2, d)) * np.exp(rng.standard_normal(d))
    return torch.from_numpy(x.astype(np.float32)).bfloat16().float().numpy()


# token counts around a wave (32), a workgroup (128), and past one list run
# (8192) of the update; centroid counts around a matrix-core block (32)
@pytest.mark.parametrize("kind,d,n,kc", [("plain", 128, 8200, 33), ("plain", 64, 129, 17), ("ties", 64, 300, 33),
                                         ("ties", 128, 127, 256), ("close", 128, 333, 64), ("close", 64, 31, 1),
                                         ("plain", 128, 1, 32), ("plain", 64, 8193, 64), ("tiny", 128, 200, 20),
                                         ("tiny", 64, 300, 64), ("nan", 128, 480, 48), ("nan", 64, 96, 48)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_kmeans_bits(kind, d, n, kc, dtype):
    if dtype == "f32" and n > 1000:
        pytest.skip("the fp32 assignment has no filter; its small cases cover it")
    rng = np.random.default_rng(n * kc + d)
    k, v = _tokens(kind, n, d, rng), _tokens(kind, n, d, rng)
    cfg = qw.make_config(1, 2, d, kc, 32, 4, 4, max(n, 64), dtype)
    ocfg = oracle.cfg_of(1, 2, d, kc, 32, 4, 4, max(n, 64), dtype == "bf16")
    ref = oracle.calibrate(ocfg, None, k, v, 4)
    dev = [torch.from_numpy(x).to(DEV, cfg.torch_dtype) for x in (k, v)]
    got = _calibrate(cfg, None, *dev, 4)
    for name, r in (("mu_k", ref[0]), ("mu_v", ref[1])):
        r = np.asarray(r).reshape(2, kc, d)
        # NaN payloads differ between the two machines
        g, r = (got[name], r.astype(np.float32)) if dtype == "f32" else (got[name].astype(np.uint32) << 16, r.astype(np.float32))
        g = g.view(np.float32)
        assert np.array_equal(np.isnan(g), np.isnan(r)), name
        assert np.array_equal(np.where(np.isnan(r), 0, g).view(np.uint32), np.where(np.isnan(r), 0, r).view(np.uint32)), name


@pytest.mark.parametrize("d,n,dtype", [(128, 1, "bf16"), (64, 63, "bf16"), (128, 64, "f32"), (64, 65, "f32"),
                                       (128, 130, "bf16")])
def test_statistics_are_token_order_sums(d, n, dtype):
    # fp64 fma in token order from stored (not symmetric) sums: numpy products of
    # these inputs are exact in fp64, so a plain multiply and add gives the same bits
    rng = np.random.default_rng(n)
    q = torch.from_numpy(rng.standard_normal((2, n, 3, d)).astype(np.float32)).bfloat16().float()
    cfg = qw.make_config(2, 3, d, 16, 32, 4, 4, 64, dtype)
    stats = torch.zeros(qw.quantwm_stats_bytes(cfg), dtype=torch.uint8, device=DEV)
    start = rng.standard_normal((6, d, d))
    stats[256:].view(torch.float64).copy_(torch.from_numpy(start.reshape(-1)))
    stats[:8].view(torch.int64).fill_(5)
    qw.quantwm_stats_update(cfg, q.to(DEV, cfg.torch_dtype), n, stats)
    ref = start.copy()
    qn = q.numpy().astype(np.float64)
    for b in range(2):
        for h in range(3):
            for t in range(n):
                ref[3 * b + h] += np.outer(qn[b, t, h], qn[b, t, h])
    got = stats.cpu()
    assert int(got[:8].view(torch.int64)) == 5 + n
    assert np.array_equal(got[256:].view(torch.float64).numpy().reshape(6, d, d), ref)


def _moment_queries(kind, d, rng):
    if kind == "rank1":
        return rng.standard_normal((1, d))
    if kind == "rank5":     # five Queries for 32 eigenpairs: 27 of them zero
        return rng.standard_normal((5, d))
    if kind == "equal":     # M = I / d: every eigenvalue the same
        return np.eye(d)
    if kind == "pairs":     # diagonal with every eigenvalue twice
        return np.diag(np.repeat(2.0 ** -np.arange(d // 2), 2))
    if kind == "close":     # a cluster of 40 eigenvalues a few 1e-7 apart above a spread
        a = np.linalg.qr(rng.standard_normal((d, d)))[0]
        s = np.concatenate([1.0 + 1e-7 * np.arange(40), 0.1 * rng.random(d - 40)])
        return np.sqrt(s)[:, None] * a.T
    if kind == "scales":    # channel scales over 24 decades
        return rng.standard_normal((200, d)) * 10.0 ** np.linspace(-12, 12, d)
    return rng.standard_normal((300, d)) @ rng.standard_normal((d, d))


@pytest.mark.parametrize("kind", ["rank1", "rank5", "equal", "pairs", "close", "scales", "plain"])
@pytest.mark.parametrize("d,r", [(128, 32), (64, 32), (128, 1), (64, 17)])
def test_basis_of_degenerate_moments(kind, d, r):
    rng = np.random.default_rng(d + r)
    q = np.ascontiguousarray(_moment_queries(kind, d, rng), np.float32)
    cfg = qw.make_config(1, 1, d, 4, 32, r, 4, 64, "f32")
    k = torch.from_numpy(rng.standard_normal((1, 64, 1, d)).astype(np.float32)).to(DEV)
    got = _calibrate(cfg, torch.from_numpy(q[None, :, None, :]).to(DEV), k, k, 0)
    m = q.astype(np.float64).T @ q.astype(np.float64) / q.shape[0]
    norm = np.linalg.norm(m, 2)
    u, lam = got["u"][0].astype(np.float64), got["lam"][0].astype(np.float64)
    ref = np.linalg.eigvalsh(m)[::-1][:r]
    # fp32 storage rounds entries of unit vectors and eigenvalues by 2^-24 each,
    # so sums over d entries by at most sqrt(d) 2^-24; four times that
    tol = 4 * np.sqrt(d) * 2.0 ** -24
    assert np.abs(lam - ref).max() <= 2.0 ** -23 * norm
    assert np.abs(u @ u.T - np.eye(r)).max() <= tol
    assert np.linalg.norm(u @ m - lam[:, None] * u, axis=1).max() <= tol * norm
    big = np.abs(u).argmax(1)
    assert (u[np.arange(r), big] > 0).all()
    assert np.array_equal(got["w"][0], (np.diag(m) / np.diag(m).mean()).astype(np.float32)) or \
        np.allclose(got["w"][0], np.diag(m) / np.diag(m).mean(), rtol=2e-7)
