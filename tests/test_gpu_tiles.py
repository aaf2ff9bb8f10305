"""The compressor's kinds of tile against the oracle, at the sizes where one gives way to the next.
Every output byte is compared.  Quantizer: arXiv 2206.11357 App. A.4, per group (Sec. 5)."""
import numpy as np
import pytest

import synthetic_inputs as syn
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


def as_dtype(x, dtype):
    return syn.f32_to_bf16_bits(x) if dtype == "bf16" else x


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("lanes", [k for k in range(3, 32) if k & (k - 1)])
def test_full_tiles_of_group_sizes_that_are_no_power_of_two(gact, dtype, lanes):
    """`lanes` lanes of 32 elements a group.  A last tile that is exactly full, one element short, one
    element long, one group short; the packed string's pad words after each."""
    G = 32 * lanes
    tile = 64 // lanes * G
    for k, n in enumerate((5 * tile, 5 * tile - 1, 5 * tile + 1, 9 * tile - G, tile)):
        x = as_dtype(syn.draw_numpy(syn.OUTLIER, n, 40 * lanes + k), dtype)
        for bits in (1, 2, 4, 8)[(k + lanes) % 2::2]:
            run_case(gact, x, G, bits, seed=lanes + k)
