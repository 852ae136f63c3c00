"""BF16 append where its workgroups and candidate selection can go wrong: one to
eight waves per workgroup with idle waves and ragged token counts, centroid
counts around the 32-row blocks and past the four-block instance, every candidate
count, and equal distances at the M-th place (duplicate centroids, resolved to
the lower ids), against the oracle's bytes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_26425_amd import quantwm as qw

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# name: heads, tokens, head_dim, centroids, group, rank, M, copies of each centroid, storage
CASES = {
    "one-token": (1, 1, 128, 32, 32, 8, 4, 1, 0),
    "one-wave": (3, 33, 128, 33, 32, 16, 4, 1, 1),
    "two-waves": (70, 230, 64, 64, 32, 4, 4, 1, 0),
    "four-waves": (130, 200, 64, 16, 64, 12, 4, 1, 1),
    "idle-waves": (130, 129, 64, 24, 16, 8, 3, 1, 0),
    "eight-waves": (260, 225, 64, 160, 32, 20, 4, 1, 0),
    "256-rows": (2, 300, 128, 256, 64, 32, 4, 1, 0),
    "129-rows": (2, 70, 128, 129, 16, 5, 2, 1, 1),
    "m8": (3, 90, 128, 100, 32, 16, 8, 1, 0),
    "m5-few": (3, 90, 64, 6, 32, 0, 5, 1, 0),
    "m8-128": (3, 70, 128, 128, 32, 16, 8, 1, 1),
    "m6-129": (2, 70, 64, 129, 16, 4, 6, 1, 0),
    "m5-129-waves": (130, 200, 64, 129, 64, 12, 5, 1, 1),
    "m-all": (2, 64, 128, 3, 32, 4, 4, 1, 0),
    "dup-m4": (2, 150, 128, 60, 32, 8, 4, 5, 0),
    "dup-m1": (2, 150, 64, 40, 32, 8, 1, 2, 0),
    "dup-m8": (2, 100, 128, 200, 32, 16, 8, 9, 1),
    "all-equal": (1, 64, 128, 70, 32, 8, 4, 70, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_append_bytes(name):
    H, n, d, kc, g, r, m, dup, st = CASES[name]
    rng = np.random.default_rng(H * n + kc)
    bf = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.float32)).bfloat16().float().numpy()  # noqa: E731
    rows = -(-kc // dup)
    # Keys on a coarse grid times a power of two per channel: sums are exact in
    # fp32, so distances tie exactly (in any summation order) or differ clearly
    scale = 2.0 ** rng.integers(-2, 3, d)
    grid = lambda *s: rng.integers(-8, 9, s) / 4.0  # noqa: E731
    mu_k = np.repeat(grid(1, H, rows, d) * scale, dup, axis=2)[:, :, rng.permutation(rows * dup)[:kc]]
    mu_v = np.repeat(grid(1, H, rows, d), dup, axis=2)[:, :, :kc]
    k, v = bf(grid(1, n, H, d) * scale), bf(grid(1, n, H, d))
    mu_k, mu_v = bf(mu_k), bf(mu_v)
    w = (2.0 ** rng.integers(-1, 2, (1, H, d))).astype(np.float32)
    u = bf(np.stack([np.linalg.qr(rng.standard_normal((d, d)))[0][:r] for _ in range(H)])[None])
    lam = np.ones((1, H, r), np.float32)
    start = 13
    ocfg = oracle.cfg_of(1, H, d, kc, g, r, m, start + n, True, st)
    ref = oracle.new_cache(ocfg)
    oracle.append(ocfg, (mu_k, mu_v, w, u, lam), ref, start, k, v)
    cfg = qw.make_config(1, H, d, kc, g, r, m, start + n, "bf16", st)
    T = lambda x, t=torch.bfloat16: torch.from_numpy(np.ascontiguousarray(x)).to(DEV, t)  # noqa: E731
    calib = torch.zeros(qw.quantwm_calib_bytes(cfg), dtype=torch.uint8, device=DEV)
    qw.quantwm_calib_pack(cfg, T(mu_k), T(mu_v), T(w, torch.float32), T(u) if r else None,
                          T(lam, torch.float32) if r else None, calib)
    cache = torch.zeros(qw.quantwm_cache_bytes(cfg), dtype=torch.uint8, device=DEV)
    coef = torch.full((1, H, n, max(r, 1)), 7.0, dtype=torch.float32, device=DEV)
    qw.quantwm_append(cfg, calib, cache, start, T(k), T(v), n, coef if r else None)
    got = cache.cpu().numpy()
    # every byte but INT8 codes (and their row scales) at a rounding midpoint: the
    # kernel sums C in fp32, the oracle in fp64
    assert np.mean(got != ref) <= 2e-4, np.flatnonzero(got != ref)[:20]
    if r:
        e = np.zeros((1, H, n, r))
        for h in range(H):
            kh = oracle.decode(ocfg, (mu_k, mu_v, w, u, lam), ref, 0, h, start + n)[0][start:]
            e[0, h] = (k[0, :, h].astype(np.float64) - kh) @ u[0, h].astype(np.float64).T
        # fp32 sums of d exact products: d 2^-24 of the terms' magnitudes, about |e| |u|
        tol = d * 2.0 ** -24 * np.abs(e).max() * 8 + 1e-6
        assert np.abs(coef.cpu().numpy() - e).max() <= tol


@pytest.mark.parametrize("d,g", [(128, 16), (64, 32), (128, 64)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_zero_step_groups_store_zero_codes(d, g, dtype):
    """8-bit scales: a group whose step rounds to code 0 stores zero codes, also when
    its wave holds tokens whose quotients are exact halves (the wave then divides
    instead of multiplying by the reciprocal, with a residual of 0.9 over no step)."""
    H, n, kc = 2, 64, 1
    rng = np.random.default_rng(d + g)
    x = np.zeros((1, n, H, d), np.float32)
    # even tokens: one group with a step of about 200, the others within [0, 0.875]
    x[:, ::2] = rng.choice([0.0, 0.5, 0.625, 0.875], (1, n // 2, H, d))
    x[:, ::2, :, 0], x[:, ::2, :, 1] = -304.0, 304.0
    # odd tokens: every group has the step 255 (sigma = 1) and quotients at +-1/2
    x[:, 1::2] = rng.choice([-127.5, 127.5], (1, n // 2, H, d))
    x[:, 1::2, :, ::g], x[:, 1::2, :, 1::g] = 512.0, -253.0
    mu = np.zeros((1, H, kc, d), np.float32)
    tables = (mu, mu, np.ones((1, H, d), np.float32), None, None)
    ocfg = oracle.cfg_of(1, H, d, kc, g, 0, 1, n, dtype == "bf16", 1)
    ref = oracle.new_cache(ocfg)
    oracle.append(ocfg, tables, ref, 0, x, x)
    assert (ref[:H * n * d // 4].reshape(H, n, d // 4)[:, ::2, g // 4:] == 0).all()
    cfg = qw.make_config(1, H, d, kc, g, 0, 1, n, dtype, 1)
    T = lambda x, t=cfg.torch_dtype: torch.from_numpy(np.ascontiguousarray(x)).to(DEV, t)  # noqa: E731
    calib = torch.zeros(qw.quantwm_calib_bytes(cfg), dtype=torch.uint8, device=DEV)
    qw.quantwm_calib_pack(cfg, T(mu), T(mu), T(tables[2], torch.float32), None, None, calib)
    cache = torch.zeros(qw.quantwm_cache_bytes(cfg), dtype=torch.uint8, device=DEV)
    qw.quantwm_append(cfg, calib, cache, 0, T(x), T(x), n)
    assert np.array_equal(cache.cpu().numpy(), ref)


@pytest.mark.parametrize("d,g,m,kc,st", [(128, 32, 4, 40, 0), (128, 16, 8, 20, 1), (64, 64, 1, 16, 0), (64, 16, 4, 150, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_keys_whose_scores_overflow(d, g, m, kc, st, dtype):
    """One channel at 3e19: W_g R^2 is infinite for every candidate, and so is the
    literal distance, so the choice is centroid 0. The outlier's group saturates and
    the token's other groups keep their residual (with 8-bit scales the shared scale
    saturates, and their steps are 0)."""
    H, n = 3, 70
    rng = np.random.default_rng(d + g + kc)
    bf = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.float32)).bfloat16().float().numpy()  # noqa: E731
    k, v = bf(rng.integers(-8, 9, (1, n, H, d)) / 4.0), bf(rng.integers(-8, 9, (1, n, H, d)) / 4.0)
    k[:, ::3, :, 5], k[:, 1::3, :, d - 1] = bf(np.float32(3e19)), bf(np.float32(-3e19))
    mu_k, mu_v = (bf(rng.integers(-8, 9, (1, H, kc, d)) / 4.0) for _ in range(2))
    tables = (mu_k, mu_v, np.ones((1, H, d), np.float32), None, None)
    ocfg = oracle.cfg_of(1, H, d, kc, g, 0, m, n, dtype == "bf16", st)
    ref = oracle.new_cache(ocfg)
    diag = oracle.append(ocfg, tables, ref, 0, k, v, diagnostics=True)
    big = np.abs(k).max(axis=3) > 1e19
    ids = diag["k_ids"].transpose(0, 2, 1)
    assert (ids[big] == 0).all() and (ids[~big] != 0).any()
    cfg = qw.make_config(1, H, d, kc, g, 0, m, n, dtype, st)
    T = lambda x, t=cfg.torch_dtype: torch.from_numpy(np.ascontiguousarray(x)).to(DEV, t)  # noqa: E731
    calib = torch.zeros(qw.quantwm_calib_bytes(cfg), dtype=torch.uint8, device=DEV)
    qw.quantwm_calib_pack(cfg, T(mu_k), T(mu_v), T(tables[2], torch.float32), None, None, calib)
    cache = torch.zeros(qw.quantwm_cache_bytes(cfg), dtype=torch.uint8, device=DEV)
    qw.quantwm_append(cfg, calib, cache, 0, T(k), T(v), n)
    assert np.array_equal(cache.cpu().numpy(), ref)
