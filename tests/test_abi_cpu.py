"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every entry point that include/quantwm.h declares, and its size queries and
argument validation behave as documented (no kernel is launched)."""
import ctypes
import subprocess
import os
import re

import pytest

import oracle
from paper_2609_26425_amd import quantwm as qw

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "quantwm.h")).read()
    return sorted(set(re.findall(r"\b(quantwm_[a-z_0-9]+)\s*\(", text)))


def _declared_param_counts():
    """Entry point -> number of parameters, from the declarations in quantwm.h."""
    text = open(os.path.join(ROOT, "include", "quantwm.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    out = {}
    for m in re.finditer(r"\b(quantwm_[a-z_0-9]+)\s*\(([^;{]*?)\)\s*;", text):
        params = m.group(2).strip()
        out[m.group(1)] = 0 if params in ("", "void") else params.count(",") + 1
    return out


def test_binding_argtypes_match_the_header():
    # every ctypes signature in the binding has as many arguments as the C declaration
    counts = _declared_param_counts()
    lib = qw.library()
    for name in qw.EXPORTED:
        assert len(getattr(lib, name).argtypes) == counts[name], name


def test_header_symbols_are_exported():
    names = declared_symbols()
    assert len(names) >= 10
    lib = ctypes.CDLL(qw.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), f"{n} declared in quantwm.h but not exported"
    assert set(names) == set(qw.EXPORTED)


@pytest.mark.parametrize("shape", [(1, 2, 64, 16, 32, 4, 4, 1024, "f32"), (1, 12, 128, 64, 32, 8, 4, 13200, "bf16"),
                                   (1, 40, 128, 128, 32, 16, 4, 32760, "bf16"),
                                   (4, 30, 128, 256, 64, 32, 4, 24960, "bf16"), (2, 3, 128, 37, 32, 12, 3, 1000, "bf16"),
                                   (1, 2, 64, 24, 16, 20, 8, 700, "bf16"), (1, 2, 128, 5, 64, 0, 1, 513, "bf16")])
@pytest.mark.parametrize("storage", [0, 1, 2, 3])
def test_sizes_agree_with_the_oracle_format(shape, storage):
    B, H, d, K, G, r, M, cap, dt = shape
    cfg = qw.make_config(B, H, d, K, G, r, M, cap, dt, storage)
    ocfg = oracle.cfg_of(B, H, d, K, G, r, M, cap, dt == "bf16", storage)
    assert qw.quantwm_cache_bytes(cfg) == oracle.cache_bytes(ocfg)
    assert qw.quantwm_token_bytes(cfg) == oracle.token_bytes(ocfg)
    L = qw.quantwm_calib_offsets(cfg)
    assert qw.quantwm_calib_bytes(cfg) == L.slab_bytes * B * H
    offs = [L.mu_k, L.mu_v, L.a_k, L.b_k, L.a_v, L.b_v, L.w, L.wg, L.u_t, L.lam, L.u_dr]
    assert all(o % 256 == 0 for o in offs) and offs == sorted(offs) and L.slab_bytes % 256 == 0


@pytest.mark.parametrize("d", [64, 128])
def test_full_metric_adds_the_matrix_to_the_calibration_block(d):
    # QWM_METRIC_FULL keeps the cache format and adds Mn ([d][d] fp32) to the slab,
    # after U_r and before the binary16 table copies.
    diag = qw.make_config(1, 3, d, 32, 32, 8, 4, 500, "bf16")
    full = qw.make_config(1, 3, d, 32, 32, 8, 4, 500, "bf16", metric=qw.METRIC_FULL)
    assert qw.quantwm_cache_bytes(full) == qw.quantwm_cache_bytes(diag)
    Ld, Lf = qw.quantwm_calib_offsets(diag), qw.quantwm_calib_offsets(full)
    assert Lf.m == Ld.m and Lf.mu_k16 == Lf.m + d * d * 4 and Lf.slab_bytes == Ld.slab_bytes + d * d * 4
    assert all(getattr(Lf, n) == getattr(Ld, n) for n in ("mu_k", "a_k", "b_k", "w", "u_t", "lam", "u_dr"))
    assert Ld.m == Ld.mu_k16  # no bytes without the full metric
    # the binary16 copies of the centroid tables and their two exponents (BF16 configs)
    assert Ld.mu_v16 - Ld.mu_k16 == (32 * d * 2 + 255) // 256 * 256 and Ld.a_k3 == Ld.e16 + 256
    # the three BF16 planes of a_k for the matrix-core search (BF16 configs)
    assert Ld.slab_bytes == Ld.a_k3 + (3 * 32 * d * 2 + 255) // 256 * 256
    f32 = qw.quantwm_calib_offsets(qw.make_config(1, 3, d, 32, 32, 8, 4, 500, "f32"))
    assert f32.mu_k16 == f32.mu_v16 == f32.e16 == f32.a_k3 == f32.slab_bytes  # none for fp32 tables
    with pytest.raises(qw.QuantwmError) as e:
        qw.quantwm_token_bytes(qw.make_config(1, 3, d, 32, 32, 8, 4, 500, "bf16", metric=2))
    assert e.value.status == qw.ERR_INVALID_ARG and "metric" in qw.quantwm_last_error()
    # the full metric needs its matrix
    P = ctypes.c_void_p
    with pytest.raises(qw.QuantwmError) as e:
        qw._check(qw.library().quantwm_calib_pack(ctypes.byref(full), P(0x1000), P(0x2000), P(0x3000), P(0x4000), None,
                                                  None, P(0x5000), None))
    assert e.value.status == qw.ERR_INVALID_ARG and "m is null" in qw.quantwm_last_error()


def test_coef_record_sizes_and_validation():
    # App. D.1 chunk records: the buffer bound is the dense size (at least the
    # header and counts); bad shapes and short buffers fail before device work.
    cfg = qw.make_config(2, 3, 128, 37, 32, 12, 3, 1000, "bf16")
    assert qw.quantwm_coef_record_max_bytes(cfg, 700) == 16 + 6 * 700 * 14
    assert qw.quantwm_coef_record_max_bytes(cfg, 0) == 16 + 4 * 6
    assert qw.quantwm_coef_record_max_bytes(cfg, 65537) == 0
    assert qw.quantwm_coef_record_max_bytes(qw.make_config(2, 3, 128, 37, 32, 0, 3, 1000, "bf16"), 10) == 0
    P = ctypes.c_void_p
    lib = qw.library()
    wr, lay = ctypes.c_int64(), ctypes.c_int32()
    cases = [(qw.make_config(2, 3, 128, 37, 32, 0, 3, 1000, "bf16"), 0, 10, 10 ** 6, "rank 0"),
             (cfg, 900, 200, 10 ** 6, "capacity"),
             (cfg, 0, 700, 100, "too small")]
    for c, start, n, nbytes, msg in cases:
        st = lib.quantwm_coef_pack(ctypes.byref(c), P(0x1000), start, n, P(0x2000), nbytes, ctypes.byref(wr),
                                   ctypes.byref(lay), None)
        assert st == qw.ERR_INVALID_ARG and msg in qw.quantwm_last_error(), qw.quantwm_last_error()
    assert lib.quantwm_coef_pack(ctypes.byref(cfg), P(0x1000), 0, 5, P(0x2000), 10 ** 6, None, None,
                                 None) == qw.ERR_INVALID_ARG
    assert lib.quantwm_coef_unpack(ctypes.byref(cfg), P(0x2000), 8, P(0x1000), 0, 5, None) == qw.ERR_INVALID_ARG
    assert "header" in qw.quantwm_last_error()


def test_validation_without_a_gpu():
    good = qw.make_config(1, 2, 128, 16, 32, 8, 4, 100, "bf16")
    for bad, status in [(qw.make_config(1, 2, 96, 16, 32, 8, 4, 100, "bf16"), qw.ERR_UNSUPPORTED),
                        (qw.make_config(1, 2, 128, 300, 32, 8, 4, 100, "bf16"), qw.ERR_INVALID_ARG),
                        (qw.make_config(1, 2, 128, 16, 48, 8, 4, 100, "bf16"), qw.ERR_INVALID_ARG),
                        (qw.make_config(1, 2, 128, 16, 32, 40, 4, 100, "bf16"), qw.ERR_UNSUPPORTED),
                        (qw.make_config(1, 2, 128, 16, 32, 8, 9, 100, "bf16"), qw.ERR_UNSUPPORTED),
                        (qw.make_config(0, 2, 128, 16, 32, 8, 4, 100, "bf16"), qw.ERR_INVALID_ARG)]:
        with pytest.raises(qw.QuantwmError) as e:
            qw.quantwm_token_bytes(bad)
        assert e.value.status == status
        assert qw.quantwm_cache_bytes(bad) == 0
    # unknown storage flags
    with pytest.raises(qw.QuantwmError) as e:
        qw.quantwm_token_bytes(qw.make_config(1, 2, 128, 16, 32, 8, 4, 100, "bf16", 4))
    assert e.value.status == qw.ERR_INVALID_ARG
    # 8-bit group scales are taken by the streaming forms: the checks that fire
    # are those of any config (here the null calibration block)
    i8 = qw.make_config(1, 2, 128, 16, 32, 8, 4, 100, "bf16", qw.STORE_SCALE_I8)
    with pytest.raises(qw.QuantwmError) as e:
        qw.quantwm_attend_active(i8, None, None, 50, None, None, 10, None, 4, 55, 1, None)
    assert e.value.status == qw.ERR_INVALID_ARG and "calib" in qw.quantwm_last_error()
    # checks that fire before any device work
    with pytest.raises(qw.QuantwmError) as e:
        qw._check(qw.library().quantwm_append(ctypes.byref(good), None, None, 90, None, None, 20, None, None))
    assert e.value.status == qw.ERR_CAPACITY
    with pytest.raises(qw.QuantwmError) as e:
        qw._check(qw.library().quantwm_append(ctypes.byref(good), None, None, 0, None, None, 5, None, None))
    assert e.value.status == qw.ERR_INVALID_ARG and "calib" in qw.quantwm_last_error()
    with pytest.raises(qw.QuantwmError) as e:
        qw._check(qw.library().quantwm_append(ctypes.byref(good), ctypes.c_void_p(0x1008), ctypes.c_void_p(0x2000),
                                              0, ctypes.c_void_p(0x3000), ctypes.c_void_p(0x4000), 5, None, None))
    assert "aligned" in qw.quantwm_last_error()
    # the BF16 append launches one workgroup per 128 tokens of a (b, h): a call
    # of 2^24 workgroups or more is refused before any device work
    big = qw.make_config(64, 2048, 128, 16, 32, 8, 4, 1 << 14, "bf16")
    dev = [ctypes.c_void_p(0x1000 * (i + 1)) for i in range(4)]
    with pytest.raises(qw.QuantwmError) as e:
        qw._check(qw.library().quantwm_append(ctypes.byref(big), dev[0], dev[1], 0, dev[2], dev[3], 1 << 14, None, None))
    assert e.value.status == qw.ERR_UNSUPPORTED and "2^24" in qw.quantwm_last_error()
    with pytest.raises(qw.QuantwmError) as e:
        qw._check(qw.library().quantwm_attend(ctypes.byref(good), None, None, 50, None, 4, 60, 1, None, None, None, 0, None))
    assert e.value.status == qw.ERR_INVALID_ARG
    with pytest.raises(qw.QuantwmError) as e:
        qw._check(qw.library().quantwm_attend(ctypes.byref(good), None, None, 50, None, 4, 10, 0, None, None, None, 0, None))
    assert "frame_tokens" in qw.quantwm_last_error()
    # empty calls are OK no-ops and touch nothing
    assert qw.library().quantwm_append(ctypes.byref(good), None, None, 0, None, None, 0, None, None) == qw.OK
    assert qw.library().quantwm_attend(ctypes.byref(good), None, None, 0, None, 0, 0, 1, None, None, None, 0, None) == qw.OK
    assert qw.quantwm_last_error() == ""


def test_streaming_workspace_sizes():
    """The streaming calls run in one launch and ask for its key split only: that of
    quantwm_attend over all their keys."""
    starts = [4680 * i for i in range(7)]
    for storage in (0, qw.STORE_SCALE_I8):
        ling = qw.make_config(1, 40, 128, 128, 32, 16, 4, 32760, "bf16", storage)
        assert qw.quantwm_attend_active_workspace_bytes(ling, 28080, 4680, 4680) == 0  # 760 workgroups: no split
        assert qw.quantwm_attend_epochs_workspace_bytes(ling, starts, 32760, 0, 4680) == 0
        for n_pk, n_act in ((28080, 1560), (32760, 0), (0, 1560), (40, 1560)):
            want = qw.quantwm_attend_workspace_bytes(ling, n_pk + n_act, 1560)
            assert want > 0 or n_pk == 0 or n_pk == 40
            assert qw.quantwm_attend_active_workspace_bytes(ling, n_pk, n_act, 1560) == want
            if n_pk >= 28080:
                assert qw.quantwm_attend_epochs_workspace_bytes(ling, starts[:6], n_pk, n_act, 1560) == want
                assert qw.quantwm_attend_epochs_workspace_bytes(ling, [0], n_pk, n_act, 1560) == 0


def test_attend_workspace_sizes():
    """A launch that under-fills the GPU asks for split workspace; a full one does not."""
    # 40 heads x 7 Query blocks of 256 = 280 workgroups < 2 per CU on 256 CUs. The
    # split count minimises rounds x (tiles per split + 32): over 1,875 key tiles
    # 7 splits (8 rounds of 268 + 32) beat 4 (5 rounds of 469 + 32); over 469
    # tiles 4 splits (5 x 150) beat 5 (6 x 126) and 8 (9 x 91)
    roll = qw.make_config(1, 40, 128, 128, 32, 16, 4, 120000, "bf16")

    def split_bytes(ns, n_q, heads=40):
        rows = ns * heads * n_q
        return (rows * 128 * 4 + 255) // 256 * 256 + rows * 8

    assert qw.quantwm_attend_workspace_bytes(roll, 120000, 1560) == split_bytes(7, 1560)
    assert qw.quantwm_attend_workspace_bytes(roll, 30000, 1560) == split_bytes(4, 1560)
    # 12 heads x 11 Query blocks = 132 workgroups over 207 tiles: 3 splits (2 rounds of 69 + 32)
    mg2 = qw.make_config(1, 12, 128, 64, 32, 8, 4, 13200, "bf16")
    assert qw.quantwm_attend_workspace_bytes(mg2, 13200, 2640) == split_bytes(3, 2640, 12)
    # 40 heads x 19 Query blocks = 760 workgroups: no split
    ling = qw.make_config(1, 40, 128, 128, 32, 16, 4, 32760, "bf16")
    assert qw.quantwm_attend_workspace_bytes(ling, 32760, 4680) == 0
    # too few key tiles to split (fewer than 8 per split)
    assert qw.quantwm_attend_workspace_bytes(roll, 64 * 15, 1560) == 0
    assert qw.quantwm_attend_workspace_bytes(roll, 120000, 0) == 0


@pytest.mark.parametrize("rows,stage", [(0, 300), (640, 300), (200, 4680)])
def test_sparse_row_sizes_agree_with_the_oracle_format(rows, stage):
    # QWM_STORE_SPARSE: pools of coef_rows rows, the tile directory, overflow
    # counters and the staging rows, laid out as the oracle lays them out
    for storage in (4, 5, 6, 7):
        cfg = qw.make_config(2, 3, 128, 37, 32, 12, 3, 1000, "bf16", storage, coef_rows=rows, coef_stage=stage)
        ocfg = oracle.cfg_of(2, 3, 128, 37, 32, 12, 3, 1000, True, storage, coef_rows=rows, coef_stage=stage)
        assert qw.quantwm_cache_bytes(cfg) == oracle.cache_bytes(ocfg) > 0


def test_sparse_row_argument_errors():
    for bad in (qw.make_config(1, 2, 128, 16, 32, 0, 4, 100, "bf16", 4, coef_stage=10),   # no PSAC rows
                qw.make_config(1, 2, 128, 16, 32, 8, 4, 100, "bf16", 4),                  # no staging rows
                qw.make_config(1, 2, 128, 16, 32, 8, 4, 100, "bf16", 4, coef_rows=-1, coef_stage=10)):
        with pytest.raises(qw.QuantwmError) as e:
            qw.quantwm_token_bytes(bad)
        assert e.value.status == qw.ERR_INVALID_ARG
    cfg = qw.make_config(1, 2, 128, 16, 32, 8, 4, 100, "bf16", 4, coef_stage=10)
    # an append of more tokens than the staging rows hold
    with pytest.raises(qw.QuantwmError) as e:
        qw._check(qw.library().quantwm_append(ctypes.byref(cfg), None, None, 0, None, None, 11, None, None))
    assert e.value.status == qw.ERR_CAPACITY and "coef_stage" in qw.quantwm_last_error()
    # the chunk records read slot-addressed rows
    with pytest.raises(qw.QuantwmError) as e:
        qw._check(qw.library().quantwm_coef_pack(ctypes.byref(cfg), None, 0, 10, None, 0, None, None, None))
    assert e.value.status == qw.ERR_INVALID_ARG and "sparse" in qw.quantwm_last_error()



def test_xcd_task_order_is_a_bijection(tmp_path):
    # The attention kernel maps workgroup L of n to task qwm_xcd_task(L, n)
    # (csrc/xcd_order.h, shared with the kernel); every grid size must cover
    # every task once. Compiled here with the host C compiler.
    src = tmp_path / "xcd.c"
    src.write_text('#include <stdio.h>\n#include <stdlib.h>\n#include "xcd_order.h"\n'
                   'int main(void) {\n'
                   '  for (uint32_t n = 1; n <= 5000; ++n) {\n'
                   '    unsigned char* seen = calloc(n, 1);\n'
                   '    for (uint32_t L = 0; L < n; ++L) {\n'
                   '      uint32_t t = qwm_xcd_task(L, n);\n'
                   '      if (t >= n || seen[t]) { printf("bad %u %u\\n", n, L); return 1; }\n'
                   '      seen[t] = 1;\n'
                   '      /* consecutive tasks of one XCD: L and L + 8 map to t and t + 1 */\n'
                   '      if (L + 8 < n && qwm_xcd_task(L + 8, n) != t + 1) { printf("run %u %u\\n", n, L); return 1; }\n'
                   '    }\n'
                   '    free(seen);\n'
                   '  }\n'
                   '  puts("ok");\n  return 0;\n}\n')
    exe = tmp_path / "xcd"
    inc = os.path.join(ROOT, "paper_2609_26425_amd", "csrc")
    subprocess.run(["gcc", "-O2", "-std=c11", "-I", inc, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
