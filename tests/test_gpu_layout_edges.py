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


@pytest.mark.parametrize("shift", [0, 8, 1])   # bytes that q is off a 16-byte boundary: 128-bit loads, and the byte form
@pytest.mark.parametrize("out,inn", [(1, 32), (16, 64), (17, 96), (31, 224), (5, 256), (20, 288), (33, 544), (16, 1056)])
def test_tile_base_q8_row_lengths_and_alignment(out, inn, shift):
    from test_gpu_q8 import tiled_q8_np
    store = torch.randint(-127, 128, (out * inn + 16,), dtype=torch.int32, device=DEV).to(torch.int8)
    q = store[shift:shift + out * inn].view(out, inn)
    scale = torch.rand(out, device=DEV)
    assert q.data_ptr() % 16 == shift
    assert np.array_equal(to_np(bd.tile_base_q8(q, scale)), tiled_q8_np(to_np(q), to_np(scale)))


@pytest.mark.parametrize("inn", [8, 24, 100, 2040, 2048, 2056, 4096, 4104, 8200, 11008, 12296, 32768, 32776])
def test_quantiser_chunks_and_special_values(ref, inn):
    """Rows around every number of chunks per thread, lengths without whole chunks, and in the first rows: ties (quotients
    half way between whole numbers), an infinity, a NaN, zeros, subnormal values."""
    g = torch.Generator(device=DEV).manual_seed(inn)
    w = (torch.randn((9, inn), device=DEV, generator=g) * 0.02).half()
    w[0] = (torch.arange(inn, device=DEV) % 255 - 127).half() * 0.5
    w[0, 0] = 127.0                                               # scale 1: quotients n + 1/2
    w[1, inn // 2] = float("inf")
    w[2, inn // 3] = float("nan")
    w[3] = 0
    w[4] = (torch.arange(inn, device=DEV) % 40).half() * 6e-8     # subnormal
    w[5, -1] = float("-inf")
    q, scale = bd.quantize_base_q8(w)
    q_ref, s_ref = ref.quantize_rtn8(to_np(w))
    assert np.array_equal(to_np(scale), s_ref)
    assert np.array_equal(to_np(q), q_ref)
