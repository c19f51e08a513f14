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

    def check(self, y, w64=None, what=""):
        x, w64 = self.x.double(), self.w.double() if w64 is None else w64
        exact, mag = x @ w64.t(), x.abs() @ w64.abs().t()
        for t in set(self.tok):
            rows = torch.tensor([i for i, e in enumerate(self.tok) if e == t], device=DEV)
            a = self.alpha[t].double()
            exact[rows] += a * (x[rows] @ expand(self.packed[t], self.inn).t())
            mag[rows] += a * x[rows].abs().sum(dim=1, keepdim=True)
        bound = 2.0**-11 * exact.abs() + 2.0**-25 + self.inn**0.5 * 2.0**-23 * mag
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
    y = torch.full((len(t.tok), out), float("nan"), dtype=torch.float16, device=DEV)
    bd.linear_multitenant_gemm_q8(t.x, q, scale, bd.TenantTable(t.packed, t.alpha), t.tok, y=y)
    t.check(y, q.double() * scale.double()[:, None], f"q8 {out}x{inn} {counts}")
