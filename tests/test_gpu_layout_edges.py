"""The re-layout kernels at the edges of their rules: row lengths on both sides of the 128-bit loads, a last k tile of every
length, row blocks with one to sixteen rows.  Bytes, against index permutations written out in numpy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2402_10193_amd import binding as bd   # noqa: E402
from gpu_util import to_np                       # noqa: E402
from test_gpu_tiled import tiled_signs_np        # noqa: E402

DEV = "cuda"


@pytest.mark.parametrize("out", [1, 16, 17, 31])
@pytest.mark.parametrize("words", [1, 3, 4, 7, 8, 9, 12, 13, 16, 20, 33])
def test_tile_signs_row_lengths(out, words):
    inn = 32 * words
    packed = torch.randint(-2**31, 2**31, (out, words), dtype=torch.int64, device=DEV).to(torch.int32)
    st = torch.full((bd.tiled_signs_bytes(out, inn) // 4,), 0x5A5A5A5A, dtype=torch.int32, device=DEV)
    bd.tile_signs(packed, out, inn, signs_tiled=st)
    bits = np.unpackbits(to_np(packed).view(np.uint8), axis=1, bitorder="little")
    assert np.array_equal(to_np(st).view(np.uint8), tiled_signs_np(bits))
