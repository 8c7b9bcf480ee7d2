"""k ranges around the depth of the load ring: fewer k-tiles than stages, as many, one more (where the loads of a k-tile are issued over
several k-steps, the first k-tile that hands loads on is then also the last that takes some), and longer ones; and, for 256x256 tiles of
a reduce-scatter, around twice that depth, from which on a tile's stores are on their way through the first k-tiles of the next."""
import numpy as np
import pytest

from paper_2511_13940_amd import workloads as wl
from tests import harness as hz
from tests.test_gpu_bf16_slots import check as check_rs16
from tests.test_gpu_gemm_rs import check_rs
from tests.test_gpu_tile_shapes import test_ag_gemm as check_ag_gemm

pytestmark = pytest.mark.gpu

SHAPES = [
    # three stages; two groups of waves with one k-step of each k-tile
    ("bf16", "kn", 6640, 1056, "256x128"),
    ("bf16", "nk", 6900, 1056, "256x128"),
    # three stages, the loads of a k-tile issued over its k-steps
    ("fp8", "kn", 6700, 1056, "256x128"),
    ("fp8", "nk", 6854, 1072, "256x128"),
    ("bf16", "nk", 4700, 784, "128x256"),
    ("fp8", "nk", 5640, 656, "128x256"),
    # one k-step per k-tile: pairs of k-tiles, and one more where their number is odd
    ("bf16", "kn", 1104, 1304, "128x64"),                  # four stages
    ("bf16", "kn", 4658, 688, "128x128"),
    ("bf16", "nk", 5890, 536, "128x128"),
    ("bf16", "kn", 2116, 2776, "128x256"),                 # four stages of 64 bytes
    # two stages, several rounds
    ("bf16", "kn", 7704, 5528, "256x256"),
    ("bf16", "nk", 7938, 4072, "256x256"),
]


@pytest.mark.parametrize("ktiles", [2, 3, 4, 5, 7])       # of 128 bytes
@pytest.mark.parametrize("dtype,layout,M,n,tile", SHAPES)
def test_short_k(dtype, layout, M, n, tile, ktiles):
    check_ag_gemm(dtype, 2, 1, M, 2 * n, ktiles * (64 if dtype == "bf16" else 128), layout, "none", tile)


@pytest.mark.parametrize("dtype,layout,M,n,tile", [x for x in SHAPES if x[4] == "256x256"])
def test_one_k_tile(dtype, layout, M, n, tile):            # less than the ring's two stages
    check_ag_gemm(dtype, 2, 1, M, 2 * n, 64, layout, "none", tile)


# units of 128 bytes: with bf16 one k-tile in a ring of two, with fp8 two in a ring of four; twice the ring's depth is four units in both
@pytest.mark.parametrize("units", [3, 4, 5, 7])
@pytest.mark.parametrize("dtype,layout,slots", [("bf16", "kn", "f32"), ("bf16", "nk", "f32"), ("bf16", "kn", "bf16"), ("fp8", "kn", "f32"),
                                                ("fp8", "kn", "bf16")])
def test_stores_under_the_next_main_loop(dtype, layout, slots, units):
    """30 tiles on eight workgroups, rows that start on 128-byte lines: results and every ready flag, inner tiles and edge tiles."""
    P, rank, M, N, kl = 2, 1, 1536, 1056 + 32 * (slots == "bf16"), units * (64 if dtype == "bf16" else 128)
    kw = dict(partial_dtype=slots, b_layout=layout, comm_cus=248)
    r = hz.route("gemm_rs", P, rank, M, N, P * kl, dtype, **kw)
    assert r.tile == "256x256" and r.first == 30 and not r.late and N * (2 if slots == "bf16" else 4) % 128 == 0
    inp = wl.gemm_rs_inputs(P, M, N, P * kl, dtype, rank, seed=units)
    B = np.ascontiguousarray(inp["B_local"].T) if layout == "nk" else inp["B_local"]
    inp["partials16"] = wl.to_bf16_bits(inp["partials"])
    partials = inp["partials16" if slots == "bf16" else "partials"]
    res = hz.run_gemm_rs(P, rank, M, N, P * kl, dtype, inp["A_local"], B, partials, inp["scale_a"], inp["scale_b"], epoch=3, **kw)
    (check_rs16 if slots == "bf16" else check_rs)(P, rank, dtype, inp, res, kl)
    assert np.all(res["flags_in"][rank] == 3) and np.all(res["flags_out"][1 - rank] == 3) and np.all(res["flags_out"][rank] == 0)
