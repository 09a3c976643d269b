"""GPU parity of hdf_fc_reduce (the generic dense fc reducer, Sec. 2.2 / Table 1)
against the oracle: bf16 outputs within the bf16 storage tolerance, fp32 within 1e-4
relative per row."""
import numpy as np
import pytest
import torch

import synth
from oracle.fc_reducer import fc_reduce as ref_fc
from oracle.numerics import as_f64
from paper_2606_26744_amd import hdf
from tests._plans import deep_tile, gemm_plan
from tests._tol import assert_bf16_close, assert_f32_rows_close

pytestmark = pytest.mark.gpu


def _case(n, m, d, dtype, seed, bias=True):
    print(f"[fc_reduce] n={n} m={m} d={d} dtype={dtype} bias={bias}", flush=True)
    H = synth.normal([n, m, d], 1.0, seed, 70, dtype=dtype, device="cuda")
    W = synth.normal([d, m * d], 0.02, seed, 71, dtype=dtype, device="cuda")
    b = synth.normal([d], 0.1, seed, 72, dtype="f32", device="cuda") if bias else None
    Y = hdf.fc_reduce(H, hdf.pack_weight(W), b)
    torch.cuda.synchronize()
    ref = ref_fc(synth.to_numpy_bits(H), synth.to_numpy_bits(W),
                 None if b is None else b.cpu().numpy(), dtype=dtype)
    got = synth.to_numpy_bits(Y)
    if dtype == "bf16":
        assert_bf16_close(as_f64(got), ref, "Y")
    else:
        assert_f32_rows_close(got, ref, "Y")


def test_warm_step_rows():
    """The full-size step's 128 new rows: 4 paths x 4096 (a 67M-parameter projection)."""
    _case(128, 4, 4096, "bf16", 1)


@pytest.mark.parametrize("n,m,d,dtype,bias", [(37, 4, 256, "f32", True), (300, 3, 1024, "bf16", False),
                                              (1, 8, 512, "bf16", True), (2050, 2, 128, "bf16", True),
                                              # more than 128 rows on the matrix-core tiles with
                                              # K = 64 and 128: fewer 32-wide K units than the
                                              # weight ring holds, and exactly as many
                                              (257, 1, 64, "bf16", False), (300, 2, 64, "bf16", True)])
def test_shapes(n, m, d, dtype, bias):
    _case(n, m, d, dtype, n + m, bias)


def test_rows_past_one_chunk():
    """More rows than one projection launch takes (16384): the chunks line up."""
    _case(16384 + 100, 2, 256, "bf16", 3)


@pytest.mark.parametrize("rest,m,d,dtype", [(8634, 4, 64, "f32"), (5724, 4, 576, "bf16")])
def test_last_chunk_stays_in_the_workspace(rest, m, d, dtype):
    """A last chunk whose own plan takes more split partials than the whole chunks' workspace
    holds: nothing is written past the workspace's stated size."""
    n = 16384 + rest
    code = hdf.HDF_F32 if dtype == "f32" else hdf.HDF_BF16
    need = int(hdf.lib().hdf_fc_reduce_workspace(n, m, d, code))
    assert int(hdf.lib().hdf_fc_reduce_workspace(rest, m, d, code)) > need   # the case is that case
    H = synth.normal([n, m, d], 1.0, 5, 70, dtype=dtype, device="cuda")
    W = synth.normal([d, m * d], 0.02, 5, 71, dtype=dtype, device="cuda")
    buf = torch.full((need * 4,), 0x5A, dtype=torch.uint8, device="cuda")   # ends past any plan
    Y = hdf.fc_reduce(H, hdf.pack_weight(W), ws=buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0x5A).all())
    ref = ref_fc(synth.to_numpy_bits(H), synth.to_numpy_bits(W), None, dtype=dtype)
    got = synth.to_numpy_bits(Y)
    if dtype == "bf16":
        assert_bf16_close(as_f64(got), ref, "Y")
    else:
        assert_f32_rows_close(got, ref, "Y")


def test_block_identity_weights_sum_the_paths():
    """W_fc = [I I I I] sums the paths exactly as the gated reducer with unit gates."""
    n, m, d = 64, 4, 512
    H = synth.normal([n, m, d], 1.0, 9, 70, dtype="f32", device="cuda")
    W = torch.cat([torch.eye(d, device="cuda")] * m, dim=1).contiguous()
    Y = hdf.fc_reduce(H, hdf.pack_weight(W))
    torch.cuda.synchronize()
    assert torch.allclose(Y, H.sum(dim=1), rtol=1e-6, atol=1e-5)


def test_empty():
    H = torch.empty((0, 4, 256), dtype=torch.bfloat16, device="cuda")
    W = torch.zeros((256, 1024), dtype=torch.bfloat16, device="cuda")
    assert hdf.fc_reduce(H, hdf.pack_weight(W)).shape == (0, 256)


@pytest.mark.parametrize("n,m,d", [(1, 1, 16), (31, 4, 36), (33, 3, 48), (64, 1, 80), (65, 4, 132),
                                   (129, 5, 112), (300, 4, 1024), (3, 8, 1000)])
def test_fp32_k_steps(n, m, d):
    """fp32 tiles with whole and half last K steps (m*d a multiple of 16 only), K below one
    step, K splits, and row counts around 32, 64 and 128."""
    _case(n, m, d, "f32", n + m, n % 2 == 1)


@pytest.mark.parametrize("n,m,d", [(129, 3, 64), (256, 5, 64), (255, 1, 576), (513, 7, 192), (1025, 2, 1088),
                                   (2049, 3, 320), (2177, 5, 64), (4100, 1, 704)])
def test_matrix_core_tiles(n, m, d):
    """The 128 x 256 matrix-core bound tiles around their row and column edges, and K of one,
    three, five, seven and more 64-K steps (a part of the loop's unrolled units)."""
    _case(n, m, d, "bf16", n + m, n % 2 == 0)


@pytest.mark.parametrize("n,m,d", [(1024, 4, 1280), (900, 2, 2304), (700, 4, 640), (513, 2, 1920)])
def test_matrix_core_small_tiles(n, m, d):
    """Shapes whose plan takes the 128 x 256 tiles, with and without K splits."""
    _case(n, m, d, "bf16", n + m, n % 2 == 0)


@pytest.mark.parametrize("n,m,d,tile,splits", [(2026, 1, 4160, (256, 256), 1), (4622, 1, 1600, (128, 512), 1),
                                               (1538, 1, 2368, (256, 256), 3), (3264, 2, 1088, (128, 512), 3)])
def test_matrix_core_large_tiles(n, m, d, tile, splits):
    """The two large tiles with a ragged last row and column tile, bias, and a K range that is no
    multiple of the loop's unrolled units: bf16 rows from the epilogue and partial sums of K
    splits."""
    p = gemm_plan(True, n, d, m * d)
    assert (deep_tile(p), p.splits) == (tile, splits)
    assert n % tile[0] != 0 and d % tile[1] != 0
    _case(n, m, d, "bf16", n + m, True)
