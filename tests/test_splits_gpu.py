"""Key splits of small attention launches: parts of four tiles (BF16) or one (fp32)
and workspaces that hold fewer parts than the launch would take, against the
unsplit call."""
import numpy as np
import pytest
import torch

from paper_2609_26425_amd import quantwm as qw

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _call(dtype, d, n, nq, H):
    """A seeded call: attend(workspace bytes) -> (out, lse), planes(parts) -> bytes, config."""
    kc, r, frame = 24, 8, 16
    g = torch.Generator(device=DEV).manual_seed(n)
    cfg = qw.make_config(1, H, d, kc, 32, r, 4, n, dtype)
    dt = cfg.torch_dtype
    rnd = lambda *s, t=dt: torch.randn(*s, generator=g, device=DEV).to(t)  # noqa: E731
    calib = torch.zeros(qw.quantwm_calib_bytes(cfg), dtype=torch.uint8, device=DEV)
    u = torch.linalg.qr(torch.randn(H, d, r, generator=g, device=DEV).cpu())[0].transpose(1, 2).contiguous().to(DEV, dt)
    qw.quantwm_calib_pack(cfg, rnd(1, H, kc, d), rnd(1, H, kc, d), torch.ones(1, H, d, device=DEV), u,
                          torch.ones(1, H, r, device=DEV), calib)
    cache = torch.zeros(qw.quantwm_cache_bytes(cfg), dtype=torch.uint8, device=DEV)
    qw.quantwm_append(cfg, calib, cache, 0, rnd(1, n, H, d), rnd(1, n, H, d), n)
    q = rnd(1, nq, H, d)

    def attend(nb):
        ws = torch.full((nb,), 255, dtype=torch.uint8, device=DEV) if nb else None  # NaN planes
        out, lse = torch.empty_like(q), torch.empty(1, H, nq, dtype=torch.float32, device=DEV)
        qw.quantwm_attend(cfg, calib, cache, n, q, nq, n - nq if n > nq else 0, frame, out, lse, ws)
        return out.float().cpu().numpy(), lse.cpu().numpy()

    def planes(ns):
        return (ns * H * nq * d * 4 + 255) // 256 * 256 + ns * H * nq * 8
    return attend, planes, cfg


@pytest.mark.parametrize("dtype,d,n,nq", [("bf16", 128, 1400, 64), ("bf16", 64, 515, 33), ("f32", 64, 1000, 70),
                                          ("f32", 128, 130, 300)])
def test_splits_match_the_unsplit_call(dtype, d, n, nq):
    attend, planes, cfg = _call(dtype, d, n, nq, 2)
    full = qw.quantwm_attend_workspace_bytes(cfg, n, nq)
    parts = next(ns for ns in range(2, 17) if planes(ns) == full)
    tiles = (n + 63) // 64
    assert parts == (min(16, tiles) if dtype == "f32" else max(ns for ns in range(1, 17) if tiles // ns >= 4))
    ref, rlse = attend(0)
    # BF16: outputs round to 2^-9 and so do the weights, whose scale a split changes;
    # fp32: sums of n terms, 2^-24 each
    tol = 4 * 2.0 ** -8 if dtype == "bf16" else n * 2.0 ** -23
    for nb in (full, full - 1, planes(2), planes(2) - 1):
        out, lse = attend(nb)
        assert np.abs(out - ref).max() <= tol * np.abs(ref).max(), nb
        assert np.abs(lse - rlse).max() <= (2e-3 if dtype == "bf16" else 1e-5) * (1 + np.abs(rlse).max()), nb
    # one byte short of two parts: the unsplit launch, bit for bit
    assert np.array_equal(attend(planes(2) - 1)[0], ref)


def test_a_workspace_for_fewer_parts_takes_the_cheapest_count_that_fits():
    """33 heads x 5 Query blocks over 128 key tiles want three parts (2 rounds of
    workgroups over 43 + 32 tiles against one over 128 + 32); two parts (2 rounds over
    64 + 32) would take longer than none, so a workspace for two runs unsplit."""
    attend, planes, cfg = _call("bf16", 64, 8192, 1280, 33)
    assert qw.quantwm_attend_workspace_bytes(cfg, 8192, 1280) == planes(3)
    ref, rlse = attend(0)
    out, lse = attend(planes(3) - 1)
    assert np.array_equal(out, ref) and np.array_equal(lse, rlse)
    assert not np.array_equal(attend(planes(3))[1], rlse)
