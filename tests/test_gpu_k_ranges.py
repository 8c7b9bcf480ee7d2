"""k ranges around the depth of the load ring, for the tile shapes whose loads of one k-tile are issued over several k-steps: fewer
k-tiles than stages, as many, one more (the first k-tile that hands loads on is also the last that takes some), and longer ones."""
import pytest

from tests.test_gpu_tile_shapes import test_ag_gemm as check_ag_gemm

pytestmark = pytest.mark.gpu

SHAPES = [
    ("bf16", "kn", 6640, 1056, "256x128"),
    ("bf16", "nk", 6900, 1056, "256x128"),
    ("fp8", "kn", 6700, 1056, "256x128"),
    ("fp8", "nk", 6854, 1072, "256x128"),
    ("bf16", "nk", 4700, 784, "128x256"),
    ("fp8", "nk", 5640, 656, "128x256"),
    # one k-step per k-tile: pairs of k-tiles, and one more where their number is odd
    ("bf16", "kn", 1104, 1304, "128x64"),                  # four stages
    ("bf16", "kn", 4658, 688, "128x128"),
    ("bf16", "nk", 5890, 536, "128x128"),
    ("bf16", "kn", 2116, 2776, "128x256"),                 # four stages of 64 bytes
    ("bf16", "kn", 7704, 5528, "256x256"),                 # the same, several rounds
    ("bf16", "nk", 7938, 4072, "256x256"),                 # two stages
]


@pytest.mark.parametrize("ktiles", [2, 3, 4, 5, 7])       # of 128 bytes, in rings of three stages (if nothing else is said)
@pytest.mark.parametrize("dtype,layout,M,n,tile", SHAPES)
def test_short_k(dtype, layout, M, n, tile, ktiles):
    check_ag_gemm(dtype, 2, 1, M, 2 * n, ktiles * (64 if dtype == "bf16" else 128), layout, "none", tile)
