"""GPU: the phased GEMM tiles, which gemm() picks by shape, against the 64x32 tile.

Both sum an element's products over K through the same MFMAs in the same order, so the
results are equal bit for bit; the 64x32 tile itself is held to an fp64 product in
test_gpu_gemm.py and test_gpu_gemm_ln.py.  The shapes sit on either side of each tile's
edges: the first and last rows and columns of a tile, one k-step pair, ragged N with rows
that vector stores cannot take, an output that starts unaligned.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

EPS = 1e-5


def _bits(t):
    import torch
    return t.view(torch.int32 if t.element_size() == 4 else torch.int16)


def _inputs(dtype, M, N, K, seed):
    import torch
    from paper_2109_08008_amd import nt
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    tdt = {"bf16": torch.bfloat16, "f32": torch.float32}.get(dtype, torch.float16)
    a = (r(M, K) + 0.3 * r(M, 1)).to(tdt)
    w, scale = 0.1 * r(N, K), None
    if dtype == "f8":
        q, sc = nt.nt_quantize_fp8(w.T.cpu().numpy())
        w, scale = torch.from_numpy(q).cuda(), torch.from_numpy(sc).cuda()
    else:
        w = w.to(tdt)
    return a, w, scale, r(N), r(M, N).to(tdt)


# sizes and what tile 0 runs them on, by kind of weight: 32 is the 64x32 phased tile, 64 the 64x128
# (fp32: 64x64), 128 and 256 the square ones, 0 a tile of nt_gemm.hip
TILES = ("16-bit", "f8", "f32")
PROJ = [
    (1, 8, 64, 32, 0, 32),              # one row, one k-step
    (65, 100, 192, 32, 0, 32),          # two rows of tiles, an odd number of k-steps, ragged N
    (128, 2050, 2048, 32, 0, 32),       # more k-steps than LDS holds, two columns in the last tile
    (450, 2048, 128, 0, 0, 32),         # 512 tiles of 64x32, the last row of two rows; four k-steps or fewer
    (450, 2048, 320, 32, 0, 32),        # five k-steps
    (2049, 250, 256, 0, 0, 32),         # 264 tiles
    (2048, 250, 256, 32, 0, 32),        # 256 tiles
    (2049, 250, 64, 0, 0, 0),           # two fp32 k-steps
    (897, 1024, 384, 32, 0, 32),        # one row in the last tile
    (577, 2048, 128, 64, 0, 64),        # 64x128: one row in the last tile, the shortest k-loop
    (1089, 1024, 384, 64, 0, 64),       # three pairs of k-steps
    (1090, 1024, 2048, 64, 0, 64),      # a long k-loop
    (641, 2051, 256, 64, 0, 64),        # rows of 2051 elements: no vector access
    (1100, 1000, 512, 64, 0, 64),       # N ending inside a tile
    (1089, 1024, 192, 0, 0, 64),        # an odd number of k-steps
    (2176, 1024, 384, 128, 0, 64),      # FP8: the last size on the older tiles
    (2177, 1024, 384, 128, 128, 64),    # one row in the last tile
    (4095, 1000, 512, 64, 128, 64),     # N ending inside a tile: 512 tiles of 64x128
    (4097, 1000, 512, 128, 128, 64),    # 520
    (2177, 1000, 1088, 0, 0, 64),       # an odd number of k-steps again
    (2177, 1000, 1152, 128, 128, 64),   # N ending inside a tile, a long k-loop
    (4225, 1031, 256, 128, 128, 64),    # 128x128, rows of 1031 elements: no vector access
    (4225, 1031, 128, 128, 128, 0),     # fp32 rows that no vector store takes, a short k-loop
    (4081, 4091, 256, 128, 128, 64),    # 256x256 but for its rows
    (4081, 4091, 384, 256, 128, 64),    # 256x256 in spite of its rows
    (4097, 4096, 256, 128, 128, 64),    # 128x128 where 256x256 would leave a round nearly empty
    (4096, 4096, 128, 256, 128, 64),    # 256x256, whole tiles
    (4081, 4092, 640, 256, 128, 64),    # 256x256, ragged in both directions
]
FOLDED = [
    (3, 40, 64, 32, 0, 32),
    (65, 1000, 448, 32, 0, 32),
    (200, 72, 128, 32, 0, 32),          # columns of tiles that do not divide among the XCDs: three
    (2600, 384, 128, 32, 0, 32),        # twelve
    (129, 1152, 192, 32, 0, 32),        # 36
    (513, 1024, 128, 32, 0, 32),
    (449, 2048, 512, 32, 0, 32),
    (577, 2048, 512, 64, 0, 0),         # 64x128: one row in the last tile, whole columns
    (1089, 1024, 128, 64, 0, 0),        # the shortest k-loop
    (1025, 1030, 384, 64, 0, 0),        # rows of 1030 elements: no vector access
    (2177, 1030, 256, 64, 128, 0),      # the same for FP8
    (1300, 3072, 128, 64, 0, 0),        # FP8: 264 tiles of 128x128, 504 of 64x128
    (2177, 1024, 256, 64, 128, 0),      # FP8: one row in the last tile
    (2111, 3072, 256, 128, 128, 0),     # 128x128
]


def _rows(dtype, case):
    return case[3 + TILES.index(dtype if dtype in TILES else "16-bit")]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f8", "f32"])
@pytest.mark.parametrize("case", PROJ, ids=str)
def test_projection_equals_small_tile(dtype, case):
    import torch
    from paper_2109_08008_amd import nt
    M, N, K = case[:3]
    assert nt.nt_op_gemm_rows("f16" if dtype == "f8" else dtype, M, N, K, f8=dtype == "f8") == _rows(dtype, case)
    a, w, scale, bias, resid = _inputs(dtype, M, N, K, M + N + K)
    for mode in ("store", "relu", "resid", "in place", "f32", "unaligned"):
        got = []
        for tile in (0, 1):
            out = torch.full((M * N + 1,), float("nan"), device="cuda",
                             dtype=torch.float32 if mode == "f32" else a.dtype)
            at = out[1:] if mode == "unaligned" else out[:-1]
            if mode == "in place":      # the residual is what the output overwrites
                at.copy_(resid.view(-1))
            add = at if mode == "in place" else resid if mode == "resid" else None
            nt.nt_op_gemm("f16" if dtype == "f8" else dtype, a.data_ptr(), K, w.data_ptr(), M, N, K, bias.data_ptr(),
                          add.data_ptr() if add is not None else None, at.data_ptr(), N, out_f32=mode == "f32",
                          relu=mode == "relu", tile=tile, d_bscale=scale.data_ptr() if scale is not None else None)
            torch.cuda.synchronize()
            edge = out[0] if mode == "unaligned" else out[-1]
            assert torch.isnan(edge), "stored past the output"
            got.append(at)
        assert torch.equal(_bits(got[0]), _bits(got[1])), mode


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f8", "f32"])
@pytest.mark.parametrize("case", FOLDED, ids=str)
def test_folded_layernorm_equals_small_tile(dtype, case):
    import torch
    from paper_2109_08008_amd import nt
    M, N, K = case[:3]
    assert nt.nt_op_gemm_rows("f16" if dtype == "f8" else dtype, M, N, K, ln=True, f8=dtype == "f8") == _rows(dtype, case)
    a, w, scale, bias, _ = _inputs(dtype, M, N, K, M + N + K)
    wf = w.view(torch.float8_e4m3fn).double() * scale.double()[:, None] if dtype == "f8" else w.double()
    colsum = wf.sum(1).float()
    for relu in (False, True):
        got = []
        for tile in (0, 1):
            out = torch.full((M, N), float("nan"), dtype=a.dtype, device="cuda")
            nt.nt_op_gemm_ln("f16" if dtype == "f8" else dtype, a.data_ptr(), K, w.data_ptr(), M, N, K,
                             colsum.data_ptr(), EPS, bias.data_ptr(), out.data_ptr(), N, relu=relu, tile=tile,
                             d_bscale=scale.data_ptr() if scale is not None else None)
            torch.cuda.synchronize()
            got.append(out)
        assert torch.equal(_bits(got[0]), _bits(got[1])), relu


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f8", "f32"])
@pytest.mark.parametrize("n", [160, 420])
def test_batch_size_does_not_change_a_translation(dtype, n):
    """640 and 1680 rows a step (phased tiles: cross keys/values, QKV with the cache scatter, FFN,
    the selection records; at 640 the 64x32 ones past two a CU, at 1680 64x128 for QKV and FFN1)
    against batches of eight sentences (small tiles throughout)."""
    from paper_2109_08008_amd import nt
    shape = synth.ModelShape(512, 8, 2048, 2, 2, 1100)
    blob = synth.make_weights(shape, seed=5, lively=True)
    rng = np.random.default_rng(6)
    lens = rng.integers(20, 31, size=n)
    offs = np.concatenate(([0], np.cumsum(lens))).astype(np.int64)
    ids = rng.integers(4, shape.vocab, size=int(offs[-1])).astype(np.int32)
    model = nt.Model(shape, blob, dtype)
    base = synth.SearchSetup(beam=4, max_len_a=0.0, max_len_b=8, token_budget=0)
    ref = model.translate(ids, offs, base)
    got = model.translate(ids, offs, synth.replace(base, max_batch_sents=8))
    for a, b in zip(ref[0], got[0]):
        np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(ref[1], got[1])
    for a, b in zip(ref[2], got[2]):
        np.testing.assert_array_equal(a, b)
    model.close()
