"""The GEMM and wide-batch kernels at the edges of their tiles and dispatch rules, element by element against float64 products
of the same tensors (torch, on the device).

Bound per element: y is rounded once to binary16 (half an ulp, 2^-11 of the value, 2^-25 below the normal range) and the
products are summed in binary32 -- `in` terms in some order: sqrt(in) * 2^-23 of sum |x| |w| covers the rounding of the
partial sums several times over.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2402_10193_amd import binding as bd   # noqa: E402

DEV = "cuda"


def expand(packed, inn):
    sh = torch.arange(32, dtype=torch.int32, device=packed.device)
    return ((packed[:, :, None] >> sh) & 1).reshape(packed.shape[0], inn).double() * 2 - 1


class Tensors:
    """Random tensors of one linear: fp16 base, one sign plane and scale per tenant, x for `tok`."""

    def __init__(self, out, inn, tok, n_tenants, seed=0):
        g = torch.Generator(device=DEV).manual_seed(7919 * out + 31 * inn + len(tok) + seed)
        self.out, self.inn, self.tok, self.nt = out, inn, tok, n_tenants
        self.w = (torch.randn((out, inn), device=DEV, generator=g) * 0.02).half()
        self.packed = [torch.randint(-2**31, 2**31, (out, inn // 32), dtype=torch.int64, device=DEV, generator=g).to(torch.int32)
                       for _ in range(n_tenants)]
        self.alpha = (0.0016 * (0.5 + torch.rand(n_tenants, device=DEV, generator=g))).half().float()
        self.x = torch.randn((len(tok), inn), device=DEV, generator=g).half()

    def check(self, y, w64=None, what="", extra=0.0):
        """extra: magnitudes that the kernel adds up beside |x| |w| and takes off again"""
        x, w64 = self.x.double(), self.w.double() if w64 is None else w64
        exact, mag = x @ w64.t(), x.abs() @ w64.abs().t()
        for t in set(self.tok):
            rows = torch.tensor([i for i, e in enumerate(self.tok) if e == t], device=DEV)
            a = self.alpha[t].double()
            exact[rows] += a * (x[rows] @ expand(self.packed[t], self.inn).t())
            mag[rows] += a * x[rows].abs().sum(dim=1, keepdim=True)
        bound = 2.0**-11 * exact.abs() + 2.0**-25 + self.inn**0.5 * 2.0**-23 * (mag + extra)
        worst = ((y.double() - exact).abs() / bound).max().item()
        assert worst <= 1.0, (what, worst)


def tokens_of(counts, order="grouped"):
    tok = [t for t, n in enumerate(counts) for _ in range(n)]
    if order == "shuffled":
        p = torch.randperm(len(tok), generator=torch.Generator().manual_seed(len(tok))).tolist()
        tok = [tok[i] for i in p]
    return tok


@pytest.mark.parametrize("out,inn,counts", [
    (256, 64, [1]),                   # one step, one row: half a tile
    (256, 128, [64, 65]),             # a half tile exactly full, and one row more than that
    (257, 192, [128, 0, 129]),        # one output row beyond a tile, an idle tenant, odd number of steps
    (300, 320, [3, 200, 31]),
    (1000, 1024, [97, 33, 64, 5]),
    (255, 128, [40]), (256, 96, [40]),   # just outside the rule: the 128 x 128 tiles
])
def test_gemm_q8_tiles(out, inn, counts):
    t = Tensors(out, inn, tokens_of(counts, "shuffled"), len(counts))
    q, scale = bd.quantize_base_q8(t.w)
    big = out >= 256 and inn % 64 == 0
    for variant in (0, 4) + (5,) * big:      # the library's choice; the GEMM on 128 x 128 tiles; on 128 x 256 tiles
        y = torch.full((len(t.tok), out), float("nan"), dtype=torch.float16, device=DEV)
        bd.linear_multitenant_gemm_q8(t.x, q, scale, bd.TenantTable(t.packed, t.alpha), t.tok, y=y, variant=variant)
        t.check(y, q.double() * scale.double()[:, None], f"q8 {out}x{inn} {counts} variant {variant}")
    if not big:
        with pytest.raises(bd.BitDeltaError):
            bd.linear_multitenant_gemm_q8(t.x, q, scale, bd.TenantTable(t.packed, t.alpha), t.tok, variant=5)


# The same entry points with a few tokens per tenant, which panels of 64 output rows take: `in` of whole and half units of 128, one to
# many per half of the row, the half unit in either half; `out` that ends inside a row block, a panel, not at a multiple of four;
# every number of column tiles per workgroup (by the number of them on some 4096 rows) and several launches' worth.
PANELS = [(16, 128, [17]), (41, 1152, [20, 1, 33, 16, 0, 15, 40]), (373, 2240, [9, 31, 2, 5]), (24, 192, [40, 7]), (64, 704, [9] * 40 + [16] * 30),
          (35, 4480, [12, 18, 30]), (203, 448, [5, 40]), (1, 320, [3]),
          (4090, 192, [3] * 8), (4033, 576, [16] * 11 + [1]), (4096, 320, [5] * 16), (4096, 192, [2] * 20)]


@pytest.mark.parametrize("k", [0, 1, 2, 3, 4])   # 0: the 8-bit base
@pytest.mark.parametrize("case", range(len(PANELS)))
def test_gemm_forms_in_panels(case, k):
    """Panels by their number, in every split, which all give the same bits; the GEMM's tiles by theirs; the library's choice."""
    out, inn, counts = PANELS[case]
    t = Tensors(out, inn, tokens_of(counts, "shuffled"), len(counts), seed=case)
    what = f"{out}x{inn} {counts} k {k}"
    nan = lambda: torch.full((len(t.tok), out), float("nan"), dtype=torch.float16, device=DEV)
    splits = [128 + n for n in range(1, {0: 5, 1: 5, 2: 4, 3: 3, 4: 2}[k] + 1)]
    if k == 0:
        q, scale = bd.quantize_base_q8(t.w)
        table, w8 = bd.TenantTable(t.packed, t.alpha), q.double() * scale.double()[:, None]
        run = lambda variant=0: bd.linear_multitenant_gemm_q8(t.x, q, scale, table, t.tok, y=nan(), variant=variant)
        panels = run(128)
        for y in (panels, run(4), run()):
            t.check(y, w8, what)
    else:
        g = torch.Generator(device=DEV).manual_seed(case)
        planes = [[p] + [torch.randint(-2**31, 2**31, p.shape, dtype=torch.int64, device=DEV, generator=g).to(torch.int32) for _ in range(k - 1)]
                  for p in t.packed]
        alpha = (t.alpha[:, None] * 0.55 ** torch.arange(k, device=DEV)).half().float()
        table = bd.PlaneTable([torch.stack(p) for p in planes], alpha.reshape(-1))
        run = lambda variant=0: bd.linear_multitenant_gemm_kbit(t.x, t.w, table, t.tok, y=nan(), variant=variant)
        panels = run(128)
        x, w64 = t.x.double(), t.w.double()
        exact, mag, delta = x @ w64.t(), x.abs() @ w64.abs().t(), torch.zeros((len(t.tok), 1), dtype=torch.float64, device=DEV)
        for e in set(t.tok):
            rows = torch.tensor([i for i, f in enumerate(t.tok) if f == e], device=DEV)
            for j in range(k):
                exact[rows] += alpha[e, j].double() * (x[rows] @ expand(planes[e][j], inn).t())
                delta[rows] += alpha[e, j].double() * x[rows].abs().sum(dim=1, keepdim=True)
        bound = 2.0**-11 * exact.abs() + 2.0**-25 + inn**0.5 * 2.0**-23 * (mag + delta)      # as in `check`
        # the GEMM's tiles form the planes' sum in fp16: k - 1 additions, each rounded by at most 2^-11 of the scales' sum; over a row these
        # errors meet x of random signs, so their sum is below 6 standard deviations in all of some 10^6 elements
        of_row = alpha.double().sum(dim=1)[torch.tensor(t.tok, device=DEV)][:, None]
        in_fp16 = 6 * (k - 1) * 2.0**-11 * of_row * x.norm(dim=1, keepdim=True)
        for y, b in ((panels, bound), (run(4), bound + in_fp16), (run(), bound + in_fp16)):
            worst = ((y.double() - exact).abs() / b).max().item()
            assert worst <= 1.0, (what, worst)
    for variant in splits:
        assert torch.equal(run(variant), panels), (what, variant)
    assert torch.equal(run(), run()), what
    with pytest.raises(bd.BitDeltaError):
        run(splits[-1] + 1)


# More than 32 tokens with a few per tenant, as the library chooses to run them (which kernel that is, an estimate says),
# against float64; the kernel of 16-column tiles by its number: test_wide_every_split.
# Rows of `out` around one and two row blocks, one unit of `in` and counts that are no multiple of the eight wavefronts,
# columns of 1, 15, 16, 17 and 33 tokens, one and several chunks of column tiles, more than one launch's worth of tiles.
WIDE = [
    (1, 128, [33]),
    (16, 256, [16, 17]),
    (17, 384, [1, 15, 16, 17, 33, 0, 2]),
    (33, 1152, [40]),
    (47, 1024, [3] * 12),
    (300, 2176, [7, 9, 20, 1, 30, 12, 5, 8]),
    (4112, 512, [12] * 9),
    (64, 640, [9] * 40 + [16] * 30),         # 70 column tiles: two launches
    (2064, 1024, [15] * 3),                  # 129 row blocks
    (4096, 256, [16] * 5),
]


@pytest.mark.parametrize("order", ["grouped", "shuffled"])
@pytest.mark.parametrize("case", range(len(WIDE)))
def test_wide_batches(case, order):
    out, inn, counts = WIDE[case]
    t = Tensors(out, inn, tokens_of(counts, order), len(counts), seed=case)
    what = f"wide {out}x{inn} {counts} {order}"
    nan = lambda: torch.full((len(t.tok), out), float("nan"), dtype=torch.float16, device=DEV)
    table = bd.TenantTable(t.packed, t.alpha)
    for ws in ("auto", None):
        y = bd.linear_multitenant(t.x, t.w, table, t.tok, y=nan(), workspace=ws)
        t.check(y, what=what + f" row-major, workspace {ws}")
        assert torch.equal(bd.linear_multitenant(t.x, t.w, table, t.tok, workspace=ws), y)      # bitwise reproducible
    t.check(bd.linear_multitenant(t.x, t.w, table, t.tok, variant=2), what=what + " decode launches")
    tiled = bd.TiledTenantTable([bd.tile_signs(p, out, inn) if n else None for p, n in zip(t.packed, counts)], t.alpha)
    wt = bd.tile_base(t.w)
    y = bd.linear_multitenant_tiled(t.x, wt, out, tiled, t.tok, y=nan())
    t.check(y, what=what + " tiled")
    group = bd.TiledGroup([wt, wt], [out, out], [tiled, tiled])
    ya, yb = bd.linear_multitenant_tiled_group(t.x, group, t.tok, ys=[nan(), nan()])
    t.check(ya, what=what + " group")
    assert torch.equal(ya, yb), what + " group"


# The kernel of 16-column tiles, asked for by number, in every split it has: one and two row blocks per workgroup, every number
# of column tiles, the last chunk partly filled; `out` that ends inside a row block and inside a pair of them; units of `in`
# fewer than the eight wavefronts, as many, and an odd number of them; k tiles likewise.
WIDE_SPLITS = [16 + n for n in range(1, 11)] + [32 + n for n in range(1, 7)]


@pytest.mark.parametrize("variant", [10] + WIDE_SPLITS)
@pytest.mark.parametrize("out,inn,counts", [
    (41, 1152, [20, 1, 33, 16, 0, 15, 40]),      # 11 column tiles; 3 row blocks; 9 units
    (16, 128, [17]),                             # 1 row block, 1 unit, 2 column tiles
    (373, 2176, [9, 31, 2, 5]),                  # 24 row blocks, 17 units
    (64, 640, [9] * 40 + [16] * 30),             # 70 column tiles: two launches
    (24, 2048, [40, 7]),                         # eight k tiles: one per wavefront
    (35, 4480, [12, 18, 30]),                    # 17.5 k tiles
])
def test_wide_every_split(out, inn, counts, variant):
    t = Tensors(out, inn, tokens_of(counts, "shuffled"), len(counts), seed=variant)
    what = f"wide {out}x{inn} {counts} variant {variant}"
    nan = lambda: torch.full((len(t.tok), out), float("nan"), dtype=torch.float16, device=DEV)
    y = bd.linear_multitenant(t.x, t.w, bd.TenantTable(t.packed, t.alpha), t.tok, y=nan(), variant=variant)
    t.check(y, what=what + " row-major")
    tiled = bd.TiledTenantTable([bd.tile_signs(p, out, inn) if n else None for p, n in zip(t.packed, counts)], t.alpha)
    wt = bd.tile_base(t.w)
    if variant >= 37 and (inn + 255) // 256 not in (1, 2, 4, 8):   # no room for the sums of three kinds
        with pytest.raises(bd.BitDeltaError):
            bd.linear_multitenant_tiled(t.x, wt, out, tiled, t.tok, variant=variant)
        return
    y = bd.linear_multitenant_tiled(t.x, wt, out, tiled, t.tok, y=nan(), variant=variant)
    t.check(y, what=what + " tiled")
    # on the serving layout: the decode launches' bits, at scales of a fine-tune and where alpha times a part of the row's +-1 sum
    # is much larger than the result
    assert torch.equal(y, bd.linear_multitenant_tiled(t.x, wt, out, tiled, t.tok, variant=2)), what
    large = bd.TiledTenantTable(tiled.tiled, t.alpha * 2e4)
    assert torch.equal(*(bd.linear_multitenant_tiled(t.x, wt, out, large, t.tok, variant=v) for v in (variant, 2))), what


# Hardly more than one token per tenant, where panels were taken although the kernel of 16-column tiles (36: two row blocks, four tiles) or
# decode launches (2) are the quicker ones: the library's choice gives those kernels' bits.
@pytest.mark.parametrize("out,inn,counts,variant", [(460, 9472, [2] * 8 + [1] * 45, 36), (5250, 1280, [2] * 6 + [1] * 52, 2)])
def test_one_token_per_tenant_keeps_its_kernel(out, inn, counts, variant):
    t = Tensors(out, inn, tokens_of(counts, "shuffled"), len(counts), seed=6)
    table = bd.TenantTable(t.packed, t.alpha)
    y = bd.linear_multitenant(t.x, t.w, table, t.tok)
    t.check(y, what=f"{out}x{inn}")
    assert torch.equal(y, bd.linear_multitenant(t.x, t.w, table, t.tok, variant=variant))


# Row-major batches that one decode launch could take: one or two row blocks (18, 34: the same bits) and panels (128) per workgroup, and those
# that stay a decode launch (2), each with the kernel that the library chooses on 256 compute units; one token, full and part-filled column
# tiles, a token per tenant, idle tenants, `out` that ends inside a row block.  (A single unit of `in`: all of them give the same bits.)
@pytest.mark.parametrize("out,inn,counts,chosen", [
    (330, 768, [1, 0, 9, 14], 18), (994, 640, [2] * 15, 18), (467, 2432, [1] * 15, 18), (4501, 512, [16, 0, 15], 18), (2727, 640, [17, 15], 18),
    (953, 4736, [4] * 6, 18), (9217, 640, [5, 6, 5, 16], 128), (1533, 6912, [2] * 16, 2), (11577, 1152, [21, 1], 128), (16, 128, [32], 18),
    (2049, 4096, [1], 2), (4224, 512, [1] * 32, 128),
])
@pytest.mark.parametrize("order", ["grouped", "shuffled"])
def test_few_tokens_rowmajor(out, inn, counts, chosen, order):
    t = Tensors(out, inn, tokens_of(counts, order), len(counts), seed=3)
    table = bd.TenantTable(t.packed, t.alpha)
    y = torch.full((len(t.tok), out), float("nan"), dtype=torch.float16, device=DEV)
    t.check(bd.linear_multitenant(t.x, t.w, table, t.tok, y=y), what=f"{out}x{inn} {counts} {order}")
    forms = {v: bd.linear_multitenant(t.x, t.w, table, t.tok, variant=v) for v in (2, 18, 34, 128)}
    for f in forms.values():
        t.check(f, what=f"{out}x{inn} {counts} {order}")
    assert torch.equal(forms[18], forms[34])
    assert [v for v in (2, 18, 128) if torch.equal(y, forms[v])] == ([chosen] if inn > 128 else [2, 18, 128])
    g = torch.cuda.CUDAGraph()
    captured = torch.empty_like(y)
    with torch.cuda.graph(g):
        bd.linear_multitenant(t.x, t.w, table, t.tok, y=captured)
    for _ in range(2):
        captured.fill_(float("nan"))
        g.replay()
        assert torch.equal(captured, y)


# The same on the serving layout, where the wide kernel gives the bits of a decode launch: `in` of less than a k tile and not a
# multiple of one as well.
@pytest.mark.parametrize("out,inn,counts", [
    (414, 5376, [2] * 14 + [3, 0]), (14008, 512, [11, 17]), (368, 4352, [15, 16]), (1081, 3584, [8] * 4), (15357, 1280, [31]),
    (1150, 512, [1] * 17), (1001, 128, [32]), (742, 2432, [3] * 10), (452, 3072, [1]), (300, 2304, [1, 0, 7]),
])
@pytest.mark.parametrize("order", ["grouped", "shuffled"])
def test_few_tokens_tiled(out, inn, counts, order):
    t = Tensors(out, inn, tokens_of(counts, order), len(counts), seed=4)
    wt = bd.tile_base(t.w)
    table = bd.TiledTenantTable([bd.tile_signs(p, out, inn) for p in t.packed], t.alpha)
    y = torch.full((len(t.tok), out), float("nan"), dtype=torch.float16, device=DEV)
    t.check(bd.linear_multitenant_tiled(t.x, wt, out, table, t.tok, y=y), what=f"{out}x{inn} {counts} {order}")
    for variant in (2, 10):
        assert torch.equal(y, bd.linear_multitenant_tiled(t.x, wt, out, table, t.tok, variant=variant)), variant
    # an infinite scale, also where the +-1 sums of whole parts of the row are zero: what a decode launch and a group of matrices give
    t.x[:, inn // 3:] = 0
    alpha = t.alpha.clone()
    alpha[0], alpha[-1] = float("inf"), float("-inf")
    table = bd.TiledTenantTable(table.tiled, alpha)
    y = bd.linear_multitenant_tiled(t.x, wt, out, table, t.tok).view(torch.int16)
    assert torch.equal(y, bd.linear_multitenant_tiled(t.x, wt, out, table, t.tok, variant=2).view(torch.int16))
    for part in bd.linear_multitenant_tiled_group(t.x, bd.TiledGroup([wt, wt], [out, out], [table, table]), t.tok):
        assert torch.equal(y, part.view(torch.int16))


# Panels of four row blocks (row-major, variants 128 and 128 + n): chunks of 1 to 5 column tiles, the last one partly
# filled; one, two, an odd number and more than four units per half of `in`, the second half a unit shorter or empty; `out` that
# ends inside a row block, a panel, and not at a multiple of four.
@pytest.mark.parametrize("tiles", [8, 11, 16, 19, 20, 66])
@pytest.mark.parametrize("out,inn", [(4096, 128), (4090, 256), (4033, 384), (4050, 1152), (4067, 1280), (2050, 2304)])
def test_wide_panels(out, inn, tiles):
    counts = [[16, 3, 1, 15, 9][i % 5] for i in range(tiles - 2)] + [17]
    t = Tensors(out, inn, tokens_of(counts, "shuffled"), len(counts), seed=tiles)
    table = bd.TenantTable(t.packed, t.alpha)
    what = f"panels {out}x{inn} {tiles} tiles"
    y = torch.full((len(t.tok), out), float("nan"), dtype=torch.float16, device=DEV)
    t.check(bd.linear_multitenant(t.x, t.w, table, t.tok, y=y, variant=128), what=what)
    for variant in range(128, 134):                   # bitwise reproducible, and in every split
        y2 = torch.full_like(y, float("nan"))
        assert torch.equal(bd.linear_multitenant(t.x, t.w, table, t.tok, y=y2, variant=variant), y), (what, variant)
    t.check(bd.linear_multitenant(t.x, t.w, table, t.tok, variant=10), what=what + " the library's split")
    # infinities and NaN stay in their token and their row; an infinite scale gives the sign of the +-1 sum
    t.x[5, inn - 1], t.x[9, 0], t.w[out - 1, 3] = float("inf"), float("nan"), float("nan")
    alpha = t.alpha.clone()
    alpha[t.tok[0]] = float("inf")
    bad = bd.linear_multitenant(t.x, t.w, bd.TenantTable(t.packed, alpha), t.tok, variant=128)
    keep = [i for i, e in enumerate(t.tok) if i not in (5, 9) and e != t.tok[0]]
    assert torch.equal(bad[keep][:, :-1], y[keep][:, :-1]) and torch.isnan(bad[9]).all() and torch.isnan(bad[:, -1]).all()
    assert not torch.isfinite(bad[5]).any()
    s = t.x[0].double() @ expand(t.packed[t.tok[0]], inn).t()
    sure = (s.abs() > 1e-3) & (torch.arange(out, device=DEV) < out - 1)
    assert torch.equal(bad[0][sure], torch.where(s > 0, float("inf"), float("-inf")).half()[sure])


def test_a_token_on_the_serving_layout_does_not_depend_on_its_batch():
    """Batches of 1, 2, 31, 90 and 200 tokens and a group of two matrices: the same bits for the same token."""
    out, inn, counts = 528, 1536, [3, 40, 9, 1, 17, 0, 60, 20, 50]
    t = Tensors(out, inn, tokens_of(counts, "shuffled"), len(counts), seed=5)
    tiled = bd.TiledTenantTable([bd.tile_signs(p, out, inn) for p in t.packed], t.alpha)
    wt = bd.tile_base(t.w)
    y = bd.linear_multitenant_tiled(t.x, wt, out, tiled, t.tok)
    for first, n in ((0, 1), (7, 2), (100, 31), (60, 90)):
        part = bd.linear_multitenant_tiled(t.x[first:first + n].contiguous(), wt, out, tiled, t.tok[first:first + n])
        assert torch.equal(part, y[first:first + n]), (first, n)
    group = bd.TiledGroup([wt, wt], [out, out], [tiled, tiled])
    for part in bd.linear_multitenant_tiled_group(t.x, group, t.tok):
        assert torch.equal(part, y), "group"


@pytest.mark.parametrize("inn", [2048, 640, 256])
@pytest.mark.parametrize("variant", [10, 18, 24, 26, 34, 36])
def test_wide_sums_that_cancel(variant, inn):
    """Whole numbers in x, so that +-1 sums are exact, and about one in fifty of them zero although no part of the row is.  A large
    scale must not leave the rounding of its products with the parts (bound of `check`: rounding of the base product and
    one of alpha times the finished sum); an infinite one gives the sign of the sum, and NaN where it is zero or the base
    product is the opposite infinity."""
    out, counts = 200, [9, 20, 33]
    t = Tensors(out, inn, tokens_of(counts), 3, seed=41)
    t.x = torch.randint(-1, 2, t.x.shape, device=DEV, generator=torch.Generator(device=DEV).manual_seed(3)).half()
    t.alpha = torch.tensor([65504.0, 0.25, 60000.0], device=DEV)
    s = torch.empty((len(t.tok), out), dtype=torch.float64, device=DEV)
    for e in set(t.tok):
        rows = torch.tensor([i for i, k in enumerate(t.tok) if k == e], device=DEV)
        s[rows] = t.x[rows].double() @ expand(t.packed[e], inn).t()
    assert (s == 0).sum() > 100
    base, a = t.x.double() @ t.w.double().t(), t.alpha[torch.tensor(t.tok, device=DEV)].double()[:, None]
    y = bd.linear_multitenant(t.x, t.w, bd.TenantTable(t.packed, t.alpha), t.tok, variant=variant)
    exact = base + a * s
    bound = 2.0**-11 * exact.abs() + 2.0**-25 + inn**0.5 * 2.0**-23 * (t.x.double().abs() @ t.w.double().abs().t()) + 2.0**-23 * (a * s).abs()
    small = exact.abs() < 65000                                  # beyond: fp16 infinity
    assert ((y.double() - exact).abs() <= bound)[small].all()

    alpha = torch.tensor([float("inf"), 0.002, float("-inf")], device=DEV)
    t.w[7, 30], t.w[9, inn - 50] = float("inf"), float("-inf")
    base = t.x.double() @ t.w.double().t()
    want = base + alpha[torch.tensor(t.tok, device=DEV)].double()[:, None] * s
    rows = torch.tensor([i for i, k in enumerate(t.tok) if k != 1], device=DEV)
    tiled = bd.TiledTenantTable([bd.tile_signs(p, out, inn) for p in t.packed], alpha)
    for y in (bd.linear_multitenant(t.x, t.w, bd.TenantTable(t.packed, alpha), t.tok, variant=variant),
              bd.linear_multitenant_tiled(t.x, bd.tile_base(t.w), out, tiled, t.tok, variant=variant)):
        got, exp = y[rows].double(), want[rows]
        assert torch.equal(torch.isnan(got), torch.isnan(exp))
        assert torch.equal(torch.nan_to_num(got, nan=0.0), torch.nan_to_num(exp, nan=0.0))


def test_wide_non_finite_values():
    """Infinities and NaN in x, W and the scales stay in their token, their output row, their tenant; an infinite scale gives
    the sign of the +-1 sum, or NaN where that sum is zero, also where x is zero over whole parts of the row."""
    out, inn, counts = 40, 1024, [20, 9, 131]
    t = Tensors(out, inn, tokens_of(counts), 3, seed=99)
    clean_x, clean_w = t.x.clone(), t.w.clone()
    t.x[3, 5] = float("inf")
    t.x[7, 900] = float("nan")
    t.w[11, 130] = float("nan")
    t.x[20:29, 128:] = 0                       # tenant 1: seven of eight units are zero
    t.x[21] = 0
    alpha = t.alpha.clone()
    alpha[1] = float("inf")
    table = bd.TenantTable(t.packed, alpha)
    s1 = t.x[20:29].double() @ expand(t.packed[1], inn).t()
    tiled = [bd.tile_signs(p, out, inn) for p in t.packed]
    for y, clean in ((bd.linear_multitenant(t.x, t.w, table, t.tok),
                      bd.linear_multitenant(clean_x, clean_w, bd.TenantTable(t.packed, t.alpha), t.tok)),
                     (bd.linear_multitenant_tiled(t.x, bd.tile_base(t.w), out, bd.TiledTenantTable(tiled, alpha), t.tok),
                      bd.linear_multitenant_tiled(clean_x, bd.tile_base(clean_w), out, bd.TiledTenantTable(tiled, t.alpha), t.tok))):
        keep_rows = [i for i in range(len(t.tok)) if i not in (3, 7) and not 20 <= i < 29]
        keep_cols = [n for n in range(out) if n != 11]
        assert torch.equal(y[keep_rows][:, keep_cols], clean[keep_rows][:, keep_cols])
        assert torch.isnan(y[7]).all() and torch.isnan(y[:, 11]).all()
        assert not torch.isfinite(y[3]).any()
        got = y[20:29][:, keep_cols]
        want = s1[:, keep_cols]
        assert torch.equal(torch.isnan(got), want == 0)
        assert torch.equal(got[want != 0], torch.where(want[want != 0] > 0, float("inf"), float("-inf")).half())


@pytest.mark.parametrize("n_tenants", [7, 8 * 40, 8 * 40 + 1, 3000])
def test_tokens_grouped_whatever_the_tenant_ids(n_tenants):
    """Ids close together and far apart (grouped through a table of counts, or by sorting where that would be larger than the
    batch): the bits of the same batch with the ids 0..6."""
    out, inn, ids = 48, 640, sorted({0, 1, 2, n_tenants // 2, n_tenants - 3, n_tenants - 2, n_tenants - 1})
    close = tokens_of([9, 3, 11, 1, 5, 8, 3][:len(ids)], "shuffled")
    t = Tensors(out, inn, close, len(ids))
    packed = [t.packed[0]] * n_tenants
    alpha = torch.zeros(n_tenants, device=DEV)
    for i, e in enumerate(ids):
        packed[e], alpha[e] = t.packed[i], t.alpha[i]
    far = [ids[e] for e in close]
    a, b = bd.TenantTable(t.packed, t.alpha), bd.TenantTable(packed, alpha)
    for variant in (0, 2, 4, 5, 10):
        assert torch.equal(*(bd.linear_multitenant(t.x, t.w, table, tok, variant=variant) for table, tok in ((a, close), (b, far)))), variant
    st = [bd.tile_signs(p, out, inn) for p in t.packed]
    a = bd.TiledTenantTable(st, t.alpha)
    b = bd.TiledTenantTable([st[ids.index(e)] if e in ids else None for e in range(n_tenants)], alpha)
    wt = bd.tile_base(t.w)
    assert torch.equal(*(bd.linear_multitenant_tiled(t.x, wt, out, table, tok) for table, tok in ((a, close), (b, far))))
    assert torch.equal(*(bd.linear_multitenant_tiled_gemm(t.x, wt, out, table, tok) for table, tok in ((a, close), (b, far))))


def test_gemm_more_tiles_than_compute_units():
    """Over 256 tiles of all heights (32, 64, 128 rows; 64, 128, 256 of the one-product form), long ones first, an eighth of either
    kind per XCD: every output element is written, by its own tile."""
    out, inn, counts = 8456, 64, [130, 5, 64, 65, 33, 0, 300, 1, 90, 260]
    t = Tensors(out, inn, tokens_of(counts, "shuffled"), len(counts))
    tiled = bd.TiledTenantTable([bd.tile_signs(p, out, inn) for p in t.packed], t.alpha)
    wt = bd.tile_base(t.w)
    nan = lambda: torch.full((len(t.tok), out), float("nan"), dtype=torch.float16, device=DEV)
    t.check(bd.linear_multitenant_tiled_gemm(t.x, wt, out, tiled, t.tok, y=nan()), what="two products")
    t.check(bd.linear_multitenant(t.x, t.w, bd.TenantTable(t.packed, t.alpha), t.tok, y=nan(), variant=5), what="row-major")
    q, scale = bd.quantize_base_q8(t.w)
    for variant in (4, 5):
        y = bd.linear_multitenant_gemm_q8(t.x, q, scale, bd.TenantTable(t.packed, t.alpha), t.tok, y=nan(), variant=variant)
        t.check(y, q.double() * scale.double()[:, None], f"8-bit base, variant {variant}")
    y = bd.linear_multitenant_tiled_gemm(t.x, wt, out, tiled, t.tok, one_product=True, y=nan())
    for e in set(t.tok):   # one product: the fine-tuned weight rounded to binary16
        rows = torch.tensor([i for i, k in enumerate(t.tok) if k == e], device=DEV)
        w = (t.w.double() + t.alpha[e].double() * expand(t.packed[e], inn)).half().double()
        exact, mag = t.x[rows].double() @ w.t(), t.x[rows].double().abs() @ w.abs().t()
        bound = 2.0**-11 * exact.abs() + 2.0**-25 + inn**0.5 * 2.0**-23 * mag
        assert ((y[rows].double() - exact).abs() <= bound).all(), e
