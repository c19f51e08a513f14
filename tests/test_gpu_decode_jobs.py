"""Decode launches with every number of job slots (distinct tenants per column tile) and every way a launch of 17 to 32 tokens is
cut into its two column tiles, against float64 products of the same tensors (bound: see test_gpu_gemm_edges)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2402_10193_amd import binding as bd   # noqa: E402
from test_gpu_gemm_edges import Tensors, tokens_of   # noqa: E402

DEV = "cuda"

MIXES = [[1] * n for n in range(1, 33)] + [
    [16, 1], [1, 16], [17], [32], [8, 8, 8], [15, 2, 15], [1, 30, 1], [5, 6, 7, 8], [2] * 16, [3] * 10, [13] + [1] * 15, [1] * 15 + [13],
]


@pytest.mark.parametrize("mix", range(len(MIXES)))
def test_decode_launches(mix):
    counts = MIXES[mix]
    out, inn = [(40, 2048), (33, 640), (272, 2176)][mix % 3]     # x resident (one k tile per wavefront); streamed; streamed, ragged
    t = Tensors(out, inn, tokens_of(counts, "shuffled"), len(counts), seed=mix)
    what = f"{out}x{inn} {counts}"
    tiled = bd.TiledTenantTable([bd.tile_signs(p, out, inn) for p in t.packed], t.alpha)
    table = bd.TenantTable(t.packed, t.alpha)
    q, scale = bd.quantize_base_q8(t.w)
    w8 = q.double() * scale.double()[:, None]
    wt = bd.tile_base(t.w)
    # by number: left to itself the library runs many of these small batches in the kernels of 16-column tiles
    y = bd.linear_multitenant_tiled(t.x, wt, out, tiled, t.tok, variant=2)
    t.check(y, what=what + " tiled")
    assert torch.equal(y, bd.linear_multitenant_tiled(t.x, wt, out, tiled, t.tok)), what
    t.check(bd.linear_multitenant(t.x, t.w, table, t.tok, variant=2), what=what + " row-major")
    t.check(bd.linear_multitenant(t.x, t.w, table, t.tok), what=what + " row-major, the library's choice")
    # the 8-bit base: the sum runs over x (1152 + q) and 1152 sum x is taken off again, 2 * 1152 / 127 of the magnitude more per term
    for y in (bd.linear_multitenant_tiled_q8(t.x, bd.tile_base_q8(q, scale), out, tiled, t.tok),   # (always decode launches)
              bd.linear_multitenant_q8(t.x, q, scale, table, t.tok)):
        t.check(y, w8, what + " 8-bit base", extra=(2304.0 * scale.double())[None, :] * t.x.double().abs().sum(dim=1, keepdim=True))


# 25.5 k tiles a row; x of two tiles resident; several row blocks per workgroup; the same with 13.5 and with 20 k tiles; 20.5 k tiles
@pytest.mark.parametrize("out,inn", [(24, 6528), (40, 4096), (4160, 384), (4120, 3456), (4104, 5120), (40, 5248)])
@pytest.mark.parametrize("n", [3, 8, 9, 11, 13, 16, 18, 22, 27, 32])
def test_row_major_rows_of_every_kind(out, inn, n):
    """The ways the row-major kernel fetches base and signs, chosen by the number of job slots and k tiles (the last half tile
    of a row ends the tensor)."""
    t = Tensors(out, inn, tokens_of([1] * n, "shuffled"), n, seed=n)
    table = bd.TenantTable(t.packed, t.alpha)
    q, scale = bd.quantize_base_q8(t.w)
    t.check(bd.linear_multitenant(t.x, t.w, table, t.tok, variant=2), what=f"{out}x{inn} {n}")
    t.check(bd.linear_multitenant_q8(t.x, q, scale, table, t.tok), q.double() * scale.double()[:, None], f"{out}x{inn} {n} 8-bit base",
            extra=(2304.0 * scale.double())[None, :] * t.x.double().abs().sum(dim=1, keepdim=True))


# Streamed x.  More row blocks than compute units, so that workgroups have 2, 3, 4 and 5 of them, odd numbers at the end of a matrix and of the
# launch; `in` whole k tiles, half and ragged ones, one and several per wavefront.
ROW_BLOCKS = [(out, inn, counts) for out, inn in [(4160, 640), (8208, 2176), (12300, 2336), (16400, 2304)]
              for counts in ([1, 2], [1] * 11, [16], [3] * 10, [30, 2])]
# Two row blocks of a matrix at a time where two are left: one column tile of at least 12 k tiles (4 and 6 slots: 30), ...
ROW_BLOCKS += [(4160, 3104, [1] * 11), (4160, 3328, [2] * 7), (8208, 3328, [1] * 11), (12300, 3200, [1] * 16), (16400, 3104, [1] * 9), (4160, 7808, [1] * 3),
               (8208, 7744, [2] * 5)]
# ... two of 12 k tiles, or of 5 with at least 12 slots
ROW_BLOCKS += [(4160, 3328, [5] * 5), (8208, 3104, [9, 9]), (4160, 1280, [1] * 24), (8208, 1184, [1] * 27), (12300, 1408, [1] * 32), (16400, 1280, [1] * 24)]


@pytest.mark.parametrize("out,inn,counts", ROW_BLOCKS)
def test_row_blocks_in_pairs(out, inn, counts):
    t = Tensors(out, inn, tokens_of(counts, "shuffled"), len(counts), seed=len(counts))
    what = f"{out}x{inn} {counts}"
    nan = lambda n=out: torch.full((len(t.tok), n), float("nan"), dtype=torch.float16, device=DEV)
    signs = [bd.tile_signs(p, out, inn) for p in t.packed]
    tiled, wt = bd.TiledTenantTable(signs, t.alpha), bd.tile_base(t.w)
    y = bd.linear_multitenant_tiled(t.x, wt, out, tiled, t.tok, y=nan(), variant=2)
    t.check(y, what=what + " tiled")
    # matrices that end inside a workgroup's row blocks: each gives the bits of its own call
    group = bd.TiledGroup([wt, wt, wt], [out, 48, 2000], [tiled] * 3)
    for part, n in zip(bd.linear_multitenant_tiled_group(t.x, group, t.tok, ys=[nan(), nan(48), nan(2000)]), (out, 48, 2000)):
        assert torch.equal(part, y[:, :n]), what + f" group, {n} rows"
    two = bd.TiledPlaneTable([[s, s] for s in signs], t.alpha.repeat_interleave(2) * 0.5)
    t.check(bd.linear_multitenant_tiled_kbit(t.x, wt, out, two, t.tok, y=nan()), what=what + " two planes of half the scale")
    q, scale = bd.quantize_base_q8(t.w)
    w8 = q.double() * scale.double()[:, None]
    extra = t.x.double().abs() @ torch.full_like(w8, 2 * 1152.0 / 127).mul_(w8.abs().amax(dim=1, keepdim=True)).t()
    wq = bd.tile_base_q8(q, scale)
    y = bd.linear_multitenant_tiled_q8(t.x, wq, out, tiled, t.tok, y=nan())
    t.check(y, w8, what + " 8-bit base", extra)
    w48 = bd.tile_base_q8(q[:48].contiguous(), scale[:48].contiguous())       # (the scales are behind a matrix's own tiles)
    group = bd.TiledGroup([wq, w48, wq], [out, 48, out], [tiled] * 3)
    for part, n in zip(bd.linear_multitenant_tiled_group_q8(t.x, group, t.tok, ys=[nan(), nan(48), nan()]), (out, 48, out)):
        assert torch.equal(part, y[:, :n]), what + f" 8-bit group, {n} rows"
    if inn % 128 == 0:
        table = bd.TenantTable(t.packed, t.alpha)
        t.check(bd.linear_multitenant(t.x, t.w, table, t.tok, y=nan(), variant=2), what=what + " row-major")
        t.check(bd.linear_multitenant_q8(t.x, q, scale, table, t.tok, y=nan()), w8, what + " row-major, 8-bit base", extra)
