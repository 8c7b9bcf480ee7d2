"""Which way a call goes (tile shape, one or two launches, stream-K tail), decided on the host: checked without a GPU for the cases
that the GPU tests name, so that another choice does not take a test past the path it is there for."""
import random

import pytest

from paper_2511_13940_amd import pk
from tests import harness as hz
from tests import test_gpu_overlap_reduce as ov
from tests import test_gpu_tile_shapes as ts

OVERLAP = pk.PHASE_ALL | pk.PHASE_OVERLAP


@pytest.mark.parametrize("dtype,P,rank,M,N,kl,layout,slots,whole,alone", ts.RS_CASES)
def test_gemm_rs_cases(dtype, P, rank, M, N, kl, layout, slots, whole, alone):
    kw = dict(partial_dtype=slots, b_layout=layout)
    assert ts.tile("gemm_rs", P, rank, M, N, P * kl, dtype, **kw) == whole
    assert ts.tile("gemm_rs", P, rank, M, N, P * kl, dtype, phases=pk.PHASE_GEMM, **kw) == alone


def test_other_cases():
    for P, rank, M, N, kl, dtype, want in ts.COLS_CASES:
        assert ts.tile("gemm_rs_cols", P, rank, M, N, P * kl, dtype) == want
    for dtype, P, rank, M, N, K, layout, _, want in ts.AG_CASES:
        assert ts.tile("ag_gemm", P, rank, M, N, K, dtype, b_layout=layout) == want
    for dtype, P, rank, M, N, K, want in ts.AGK_CASES:
        assert ts.tile("ag_gemm_k", P, rank, M, N, K, dtype) == want


def test_every_tile_shape_is_among_the_cases():
    for dtype in ("bf16", "fp8"):
        seen = {c[8].split()[0] for c in ts.RS_CASES + ts.AG_CASES if c[0] == dtype}
        assert {"256x256", "128x256", "128x128", "128x64", "64x64", "32x32"} <= seen, (dtype, seen)


def test_two_launches_never_take_a_tail_and_their_tiles_add_up():
    rng = random.Random(7)
    two = tails = 0
    for _ in range(4000):
        dtype = rng.choice(["bf16", "fp8"])
        P = rng.choice([1, 2, 3, 4, 5, 8])
        M, N, K = P * rng.randrange(1, 4096), 16 * rng.randrange(1, 1024), P * 128 * rng.randrange(1, 40)
        kw = dict(workspace=True, comm_cus=rng.choice([0, 0, 32, 192]), partial_dtype=rng.choice(["f32", "f32", "bf16"]))
        if kw["partial_dtype"] == "f32":
            kw["b_layout"] = rng.choice(["kn", "kn", "nk"])
        rank = rng.randrange(P)
        over, plain = (hz.route("gemm_rs", P, rank, M, N, K, dtype, phases=ph, **kw) for ph in (OVERLAP, pk.PHASE_ALL))
        assert over.tile == plain.tile and over.late == plain.late and plain.second == 0
        assert over.first + over.second == plain.first
        assert not (over.second and (over.stream_k or over.late))
        assert over.second or over.stream_k == plain.stream_k
        two += over.second > 0
        tails += plain.stream_k
    assert two > 200 and tails > 200


@pytest.mark.parametrize("P,rank,M,N,K,dtype,tile,parts", ov.CASES)
def test_overlap_cases(P, rank, M, N, K, dtype, tile, parts):
    assert pk.pk_gemm_rs_plan(P, M, N, K, dtype).tile_m == tile
    assert ov.launches(P, rank, M, N, K, dtype) == parts


def test_the_reduce_beside_a_gemm_is_the_narrow_one():
    """fp32 slots, P = 2, 4, 8: whatever the tiles and the flags' granularity (bf16 slots and a run-time P have one form each)."""
    rng, seen = random.Random(8), set()
    for _ in range(30000):
        dtype, P = rng.choice(["bf16", "fp8"]), rng.choice([2, 3, 4, 8])
        M, N, K = P * rng.randrange(30, 2400), 16 * rng.randrange(10, 800), P * 128 * rng.choice([1, 2, 4, 16, 24, 32])
        slots = rng.choice(["f32", "f32", "f32", "bf16"])
        r = hz.route("gemm_rs", P, rng.randrange(P), M, N, K, dtype, phases=OVERLAP, partial_dtype=slots)
        if r.second:
            seen.add((dtype, pk.pk_gemm_rs_plan(P, M, N, K, dtype).tile_m, r.tile))
            assert r.narrow_reduce == (slots == "f32" and P != 3), (P, M, N, K, dtype, slots, r)
    assert {("bf16", 128, t) for t in ("256x256", "256x128", "128x256")} | {("bf16", 256, "256x256"), ("fp8", 256, "256x256")} <= seen


@pytest.mark.parametrize("op,P,M,N,K,dtype,layout,tile", [
    ("ag_gemm", 8, 11944, 8 * 280, 6400, "bf16", "nk", "256x128"),           # 59 us; as 128x64 90
    ("ag_gemm", 4, 6524, 4 * 2584, 16256, "bf16", "kn", "256x128"),          # 612 us; as 128x128 741
    ("ag_gemm", 8, 14696, 8 * 584, 14656, "bf16", "kn", "256x256"),          # 327 us; as 128x128 421
    ("ag_gemm", 4, 2356, 4 * 7760, 5376, "bf16", "nk", "128x256"),           # 204 us; as 128x128 259
    ("gemm_rs_cols", 2, 793, 12992, 2 * 5952, "bf16", "kn", "256x256"),      # 134 us; as 128x128 152
    ("ag_gemm", 1, 3098, 6832, 256, "fp8", "kn", "128x256"),                 # 19.3 us; as 256x256 22.4
    ("ag_gemm_k", 8, 4914, 8 * 3984, 15360, "fp8", "kn", "256x128"),         # 277 us; as 128x256 315
    ("ag_gemm_k", 4, 180, 6464, 768, "bf16", "kn", "64x64"),                 # 8.9 us; as 128x64 9.6
    ("ag_gemm_k", 1, 42, 600, 960, "bf16", "kn", "64x64"),                   # 8.7 us; as 128x64 9.6
    ("gemm_ar", 8, 552, 1400, 8 * 704, "bf16", "kn", "64x64"),               # 15.3 us; as 128x64 16.3
    ("ag_gemm", 8, 384, 8 * 2688, 384, "bf16", "kn", "128x64"),              # as 64x64 15% more
])
def test_the_faster_tile(op, P, M, N, K, dtype, layout, tile):
    """Calls that a tile shape measured far slower was estimated below the fastest one for."""
    assert hz.route(op, P, 0, M, N, K, dtype, b_layout=layout).tile == tile
