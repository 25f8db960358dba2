"""Host-only checks of the C ABI: the library loads without a GPU, exports every entry
point the header declares, and validates its arguments before touching a device."""
import os
import re

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def nt():
    from paper_2109_08008_amd import nt as _nt
    if not os.path.exists(_nt.LIB_PATH):
        from paper_2109_08008_amd.build import build_library
        build_library()
    _nt.load_library()
    return _nt


def header_functions():
    src = open(os.path.join(ROOT, "include", "nt.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(nt_[a-z0-9_]+)\s*\(", src)))


def test_every_declared_function_is_exported(nt):
    declared = header_functions()
    assert len(declared) >= 16
    lib = nt.load_library()
    for name in declared:
        assert hasattr(lib, name), name
    assert sorted(nt.EXPORTS) == declared


def header_struct_fields(name):
    """(field, C type) of `typedef struct { ... } name;` in nt.h, in declaration order."""
    src = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "nt.h")).read(), flags=re.S)
    body = re.search(r"typedef struct \{([^}]*)\}\s*" + name + r"\s*;", src).group(1)
    out = []
    for decl in body.split(";"):
        decl = decl.strip()
        if not decl:
            continue
        ctype, names = decl.split(None, 1)
        out += [(n.strip(), ctype) for n in names.split(",")]
    return out


@pytest.mark.parametrize("name", ["nt_model_cfg", "nt_search_cfg"])
def test_struct_layouts_match_header(nt, name):
    import ctypes
    cmap = {"int32_t": ctypes.c_int32, "float": ctypes.c_float}
    fields = header_struct_fields(name)
    binding = getattr(nt, name)._fields_
    assert [f for f, _ in fields] == [f for f, _ in binding]
    assert [cmap[t] for _, t in fields] == [t for _, t in binding]
    assert ctypes.sizeof(getattr(nt, name)) == 4 * len(fields)


@pytest.mark.parametrize("name", list(synth.WORKLOADS))
def test_weights_size_matches_canonical_blob(nt, name):
    w = synth.WORKLOADS[name]
    for dt in ("f32", "f16", "bf16"):
        hf, db = nt.nt_weights_size(nt.model_cfg(w.model, dt))
        assert hf == synth.blob_size(w.model)
        elem = 4 if dt == "f32" else 2
        mats = sum(e.size for e in synth.weight_layout(w.model) if e.name == "E" or ".W_" in e.name)
        assert db >= mats * elem


@pytest.mark.parametrize("shape,code", [
    (synth.ModelShape(100, 4, 256, 1, 1, 50), 2),        # d % 64
    (synth.ModelShape(128, 8, 256, 1, 1, 50), 2),        # head size 16
    (synth.ModelShape(128, 4, 100, 1, 1, 50), 2),        # d_ffn % 64
    (synth.ModelShape(128, 4, 256, 1, 0, 50), 1),        # no decoder layer
    (synth.ModelShape(128, 4, 256, 1, 1, 3), 1),         # vocab without a word
    (synth.ModelShape(128, 4, 256, 1, 1, 50, max_positions=2048), 2),
])
def test_invalid_configs_are_rejected(nt, shape, code):
    with pytest.raises(nt.NTError) as e:
        nt.nt_weights_size(nt.model_cfg(shape))
    assert e.value.status == code
    assert e.value.message
    assert nt.load_library().nt_last_error().decode() == e.value.message


def test_null_arguments_are_errors_not_crashes(nt):
    import ctypes
    lib = nt.load_library()
    assert lib.nt_weights_size(None, None, None) == nt.NT_E_INVALID
    assert lib.nt_translate(None, None, None, None, 0, None, 0, None, None, None, None, 0, None) == nt.NT_E_INVALID
    assert lib.nt_decode_step(None, None, None, None, None) == nt.NT_E_INVALID
    assert lib.nt_dec_state_info(None, *([None] * 6)) == nt.NT_E_INVALID
    assert lib.nt_prof_get(99, None, None, None, None) == nt.NT_E_INVALID
    n = ctypes.c_int64()
    assert lib.nt_prof_get(0, ctypes.byref(n), None, None, None) == nt.NT_OK
    lib.nt_free_state(None)
    lib.nt_free_model(None)


def test_ensemble_arguments_are_checked_on_the_host(nt):
    import ctypes
    lib = nt.load_library()
    out = ctypes.c_void_p()
    arr = (ctypes.c_void_p * 2)(None, None)
    assert lib.nt_ensemble(None, 1, 0, ctypes.byref(out)) == nt.NT_E_INVALID
    assert lib.nt_ensemble(arr, 1, 0, None) == nt.NT_E_INVALID
    for n, rule in [(0, 0), (9, 0), (1, 2), (1, -1)]:
        assert lib.nt_ensemble(arr, n, rule, ctypes.byref(out)) == nt.NT_E_INVALID, (n, rule)
    assert lib.nt_ensemble(arr, 2, 1, ctypes.byref(out)) == nt.NT_E_INVALID
    assert "null" in lib.nt_last_error().decode()
    assert out.value is None


def test_library_fp8_quantizer_matches_the_oracle(nt):
    """The host quantization nt_load_weights applies (fp8_weights) gives the oracle's
    codes and scales bit for bit: random columns, a zero column, an outlier column, a
    column of hand-placed ties and subnormals (scale exactly 1), a tiny-valued column."""
    import oracle
    import torch
    rng = np.random.default_rng(2)
    w = rng.normal(0, 0.02, size=(96, 40)).astype(np.float32)
    w[:, 3] = 0.0
    w[5, 7] = 3.0
    w[:, 9] *= np.float32(1e-30)
    ties = np.array([448.0, 1.0625, 1.1875, 232.0, 1.5 * 2.0 ** -9, 0.5 * 2.0 ** -9, -3.3, -1.0625, 2.5 * 2.0 ** -9],
                    dtype=np.float32)
    w[:, 11] = 0.0
    w[:len(ties), 11] = ties
    q, sc = nt.nt_quantize_fp8(w)
    oq, osc = oracle.quantize_fp8_columns(w)
    np.testing.assert_array_equal(sc.view(np.uint32), osc.view(np.uint32))
    decoded = torch.from_numpy(q).view(torch.float8_e4m3fn).to(torch.float64).numpy()
    np.testing.assert_array_equal(decoded, oq.T)
    assert sc[11] == 1.0
    np.testing.assert_array_equal(decoded[11, :len(ties)], [448, 1.0, 1.25, 224, 2.0 ** -8, 0, -3.25, -1.0, 2.0 ** -8])


def test_fp8_weight_configs(nt):
    shape = synth.ModelShape(128, 4, 256, 1, 1, 50)
    for dt in ("f32", "bf16"):
        cfg = nt.model_cfg(shape, dt)
        cfg.fp8_weights = 1
        with pytest.raises(nt.NTError) as e:
            nt.nt_weights_size(cfg)
        assert e.value.status == nt.NT_E_UNSUPPORTED
    cfg = nt.model_cfg(shape, "f16")
    cfg.fp8_weights = 2
    with pytest.raises(nt.NTError) as e:
        nt.nt_weights_size(cfg)
    assert e.value.status == nt.NT_E_INVALID
    for dt in ("f32", "bf16"):
        cfg = nt.model_cfg(shape, dt)
        cfg.fp8_kv = 1
        with pytest.raises(nt.NTError) as e:
            nt.nt_weights_size(cfg)
        assert e.value.status == nt.NT_E_UNSUPPORTED
    cfg = nt.model_cfg(shape, "f16")
    cfg.fp8_kv = -1
    with pytest.raises(nt.NTError) as e:
        nt.nt_weights_size(cfg)
    assert e.value.status == nt.NT_E_INVALID
    assert (nt.model_cfg(shape, "f8").fp8_kv, nt.model_cfg(shape, "f8w").fp8_kv) == (1, 0)
    assert nt.model_cfg(shape, "f8w").fp8_weights == 1
    assert nt.nt_weights_size(nt.model_cfg(shape, "f8w")) == nt.nt_weights_size(nt.model_cfg(shape, "f8"))
    hf8, db8 = nt.nt_weights_size(nt.model_cfg(shape, "f8"))
    hf16, db16 = nt.nt_weights_size(nt.model_cfg(shape, "f16"))
    mats = sum(e.size for e in synth.weight_layout(shape) if ".W_" in e.name)
    assert hf8 == hf16 and db16 - db8 >= mats - 4 * 2 * 1024 * 16
    lib = nt.load_library()
    assert lib.nt_quantize_fp8(None, 4, 4, None, None) == nt.NT_E_INVALID


def test_library_e4m3_rounding_over_the_whole_range(nt):
    """The E4M3 rounding the library shares between its weight quantizer and its FP8
    key/value cache, reached through the quantizer with columns whose largest magnitude is
    448 (scale exactly 1): every midpoint between neighbouring E4M3 values (ties to even),
    every E4M3 value, and random magnitudes from 2^-14 to 448 of both signs, against
    torch's float8_e4m3fn cast."""
    import torch
    grid = torch.arange(256, dtype=torch.uint8).view(torch.float8_e4m3fn).to(torch.float64).numpy()
    grid = np.unique(grid[np.isfinite(grid)])
    mids = (grid[1:] + grid[:-1]) / 2
    rng = np.random.default_rng(9)
    rand = np.ldexp(rng.uniform(1.0, 2.0, 3000), rng.integers(-14, 9, 3000)) * rng.choice([-1.0, 1.0], 3000)
    vals = np.concatenate([grid, mids, rand[np.abs(rand) <= 448.0]]).astype(np.float32)
    w = np.zeros((len(vals), 2), dtype=np.float32)
    w[:, 0] = vals
    w[:, 1] = -vals
    w[0, :] = 448.0   # the column maximum: scale 1
    q, sc = nt.nt_quantize_fp8(w)
    np.testing.assert_array_equal(sc, [1.0, 1.0])
    decoded = torch.from_numpy(q).view(torch.float8_e4m3fn).to(torch.float64).numpy()
    want = torch.from_numpy(w.T.copy()).to(torch.float8_e4m3fn).to(torch.float64).numpy()
    np.testing.assert_array_equal(decoded, want)


def test_tiled_gemm_cases_reach_their_tiles(nt):
    """The sizes at which the GPU tests compare the tiles are still formed on them."""
    from tests import test_gpu_gemm_phased as t
    seen = {d: set() for d in t.TILES}
    for cases, ln in ((t.PROJ, False), (t.FOLDED, True)):
        for c in cases:
            for d, want in zip(t.TILES, c[3:]):
                for dt in ("f16", "bf16") if d == "16-bit" else ("f16",) if d == "f8" else ("f32",):
                    assert nt.nt_op_gemm_rows(dt, *c[:3], ln=ln, f8=d == "f8") == want, (c, dt, ln)
                seen[d].add((ln, want))
    assert seen == {"16-bit": {(False, 0), (False, 32), (False, 64), (False, 128), (False, 256), (True, 32), (True, 64),
                               (True, 128)},
                    "f8": {(False, 0), (False, 128), (True, 0), (True, 128)},
                    "f32": {(False, 0), (False, 32), (False, 64), (True, 0), (True, 32)}}
    # refused sizes and types; operands past 32-bit offsets
    for args, kw in ((("f16", 8, 8, 96), {}), (("f32", 8, 8, 64), {"f8": True}), (("f16", 8, 0, 64), {}),
                     (("f16", 8, 8, 128), {"lda": 64}), (("f16", 8, 8, 64), {"lda": 68}),
                     (("f16", 8, 8, 64), {"ln": True, "out_f32": True})):
        assert nt.nt_op_gemm_rows(*args, **kw) == -1
    assert nt.nt_op_gemm_rows("f16", 1 << 20, 1024, 2048) == 0
    assert nt.nt_op_gemm_rows("f16", 1 << 20, 1024, 1024) == 256
