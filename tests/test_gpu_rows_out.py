"""Tiles that leave row by row behind their own main loop, through the LDS that the next tile's loads then fill: several tiles per
workgroup (eight workgroups), k ranges shorter and longer than the load ring, ragged rows and columns; results and every ready flag.
All tiles that can have several rounds, the 32x64 ones, whose waves read one another's rings on the way out, among them."""
import numpy as np
import pytest

from oracle import codec, tp_gemm
from paper_2511_13940_amd import workloads as wl
from tests import harness as hz, test_gpu_ag_gemm_k as agk, test_gpu_bf16_slots as slots16
from tests.test_gpu_gemm_rs import check_rs

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24
GRID = dict(comm_cus=248)


@pytest.mark.parametrize("units", [2, 5])                  # k-tiles of 128 bytes
@pytest.mark.parametrize("dtype,layout,M,N,tile", [
    ("bf16", "kn", 2056, 48, "128x128"), ("fp8", "nk", 2056, 48, "128x128"),
    ("bf16", "kn", 3080, 48, "256x128"), ("bf16", "nk", 3080, 48, "256x128"), ("fp8", "kn", 3080, 48, "256x128"),
    ("bf16", "kn", 64, 2064, "128x256"), ("bf16", "nk", 64, 2064, "128x256")])
def test_gemm_rs(dtype, layout, M, N, tile, units):
    P, rank, kl = 2, 1, units * (64 if dtype == "bf16" else 128)
    r = hz.route("gemm_rs", P, rank, M, N, P * kl, dtype, b_layout=layout, **GRID)
    assert r.tile == tile and r.first > 8 and not r.late
    inp = wl.gemm_rs_inputs(P, M, N, P * kl, dtype, rank, seed=M + units)
    B = np.ascontiguousarray(inp["B_local"].T) if layout == "nk" else inp["B_local"]
    res = hz.run_gemm_rs(P, rank, M, N, P * kl, dtype, inp["A_local"], B, inp["partials"], inp["scale_a"], inp["scale_b"], epoch=3,
                         b_layout=layout, **GRID)
    check_rs(P, rank, dtype, inp, res, kl)
    assert np.all(res["flags_in"][rank] == 3) and np.all(res["flags_out"][1 - rank] == 3) and np.all(res["flags_out"][rank] == 0)


@pytest.mark.parametrize("act", ["none", "silu"])
@pytest.mark.parametrize("dtype,layout,M,n,k,tile", [
    ("bf16", "kn", 1032, 48, 128, "128x64"), ("fp8", "nk", 1032, 48, 128, "128x64"), ("bf16", "nk", 2056, 80, 128, "128x128"),
    ("fp8", "kn", 2056, 80, 128, "128x128"), ("bf16", "nk", 64, 2064, 128, "128x256"), ("fp8", "kn", 3080, 80, 128, "256x128"),
    ("bf16", "kn", 16, 528, 512, "32x64"), ("bf16", "kn", 16, 528, 1024, "32x64"), ("bf16", "nk", 32, 528, 128, "32x64"),
    ("fp8", "nk", 16, 2064, 1024, "32x64"), ("bf16", "kn", 64, 2064, 2048, "64x64"), ("bf16", "nk", 64, 2064, 2048, "64x64")])
def test_ag_gemm(dtype, layout, M, n, k, tile, act):
    P, rank, N = 2, 1, 2 * n
    r = hz.route("ag_gemm", P, rank, M, N, k, dtype, b_layout=layout, **GRID)
    assert r.tile == tile and r.first > 8
    inp = wl.ag_gemm_inputs(P, M, N, k, dtype, rank, seed=M + n)
    B = np.ascontiguousarray(inp["B_local"].T) if layout == "nk" else inp["B_local"]
    res = hz.run_ag_gemm(P, rank, M, N, k, dtype, inp["chunks"], B, inp["scale_a"], inp["scale_b"], epoch=3, act=act, b_layout=layout, **GRID)
    A = tp_gemm.gather_chunks(inp["chunks"])
    want = tp_gemm.activation(tp_gemm.local_product(A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"]), act)
    mag = tp_gemm.abs_product(A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"])
    assert res["status"][0] == 0
    # fp32 accumulation in any order times the slope of the activation (1.13 at most), and half a bf16 ulp
    bound = 1.13 * 2 * k * U32 * mag + (2.0 ** -8 + 2.0 ** -20) * np.abs(want) + 2.0 ** -133
    assert np.all(np.abs(codec.bf16_decode(res["C_bits"]) - want) <= bound)


@pytest.mark.parametrize("dtype,M,N,units", [("bf16", 2056, 48, 2), ("bf16", 2056, 80, 5), ("fp8", 2056, 48, 1), ("fp8", 2056, 80, 3)])
def test_gemm_rs_with_bf16_slots(dtype, M, N, units):
    P, rank, kl = 2, 1, units * (64 if dtype == "bf16" else 128)
    r = hz.route("gemm_rs", P, rank, M, N, P * kl, dtype, partial_dtype="bf16", **GRID)
    assert r.tile == "128x128" and r.first > 8 and not r.late
    inp = slots16.inputs(P, M, N, P * kl, dtype, rank, seed=M + units)
    res = hz.run_gemm_rs(P, rank, M, N, P * kl, dtype, inp["A_local"], inp["B_local"], inp["partials16"], inp["scale_a"], inp["scale_b"],
                         epoch=3, partial_dtype="bf16", **GRID)
    slots16.check(P, rank, dtype, inp, res, kl)
    assert np.all(res["flags_in"][rank] == 3) and np.all(res["flags_out"][1 - rank] == 3) and np.all(res["flags_out"][rank] == 0)


# column chunks of A: the own one first, the other waited for or there at the first look
@pytest.mark.parametrize("act", ["none", "silu"])
@pytest.mark.parametrize("dtype,M,n,K,tile", [
    ("bf16", 1032, 48, 256, "128x64"), ("fp8", 1032, 48, 256, "128x64"), ("bf16", 16, 1040, 4096, "64x64"), ("bf16", 2056, 80, 512, "128x128"),
    ("fp8", 2056, 80, 512, "128x128"), ("bf16", 16, 2064, 256, "128x256"), ("fp8", 1032, 272, 256, "256x128")])
def test_ag_gemm_k(dtype, M, n, K, tile, act):
    P, rank, N = 2, 1, 2 * n
    r = hz.route("ag_gemm_k", P, rank, M, N, K, dtype, **GRID)
    assert r.tile == tile and r.first > 8
    inp = agk.inputs(P, M, N, K, dtype, rank, seed=M + n)
    for deliver in ("pre", "dma"):
        res = hz.run_ag_gemm_k(P, rank, M, N, K, dtype, inp["chunks"], inp["B_local"], inp["scale_a"], inp["scale_b"], epoch=3, deliver=deliver,
                               act=act, **GRID)
        agk.check(P, rank, dtype, inp, res, K, act)
