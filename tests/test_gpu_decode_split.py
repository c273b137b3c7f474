"""The decode attention deals its list of 64-position tiles over 1024 waves (256 CUs), over one
wave per tile when there are fewer, or, where 768 waves or fewer are enough for two or three
tiles each, over as few as it takes.  Tile counts around those limits, with one, two and three KV
heads; and a single tile; against the fp64 oracle at the bf16 tolerance."""
import pytest
import torch

from paper_2608_15943_amd import binding as kb

from gpu_util import small_workload
from test_gpu_parity import _decode_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kb.lib()


@pytest.mark.parametrize("a,g,tiles", [
    (4, 1, [1]),                        # T = 1
    (4, 1, [64] * 15 + [63]),           # T = 1023
    (4, 1, [64] * 16),                  # T = 1024
    (4, 1, [64] * 15 + [65]),           # T = 1025
    (4, 1, [64] * 24),                  # T = 1536: the last on half as many waves as tiles
    (4, 1, [64] * 23 + [65]),           # T = 1537
    (4, 2, [64] * 16),                  # T = 2048
    (4, 2, [64] * 15 + [65]),           # T = 2050
    (4, 2, [64] * 18),                  # T = 2304: the last on a third
    (4, 2, [64] * 17 + [65]),           # T = 2306
    (4, 2, [64] * 23 + [63]),           # T = 3070
    (6, 3, [64] * 16),                  # T = 3072
    (4, 1, [64] * 47 + [65]),           # T = 3073
    (4, 1, [1, 200, 1, 3, 820]),        # T = 1025, ranges that cross several sequences
    # Fewer tiles than waves, so as many pieces as tiles to merge, four waves in turn: up to 1,
    # 3 and 4, 5, 7 and 8, 9, 12, 13 and 16 pieces a wave.
    (4, 1, [4, 15, 17, 31, 33, 48, 49, 63]),
])
def test_tiles_around_the_number_of_waves(a, g, tiles):
    w = small_workload(f"split-a{a}-g{g}-{sum(tiles)}", 2, a * 128, a, g, [0, 0], seed=31)
    lens = [64 * n - 1 - (i % 3) * 20 for i, n in enumerate(tiles)]   # len + 1 positions: n tiles
    _decode_case(w, len(lens), lens, max(lens) // 64 * 64 + 64)
