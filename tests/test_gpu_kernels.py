"""Kernels and dispatch branches at the sizes where they change: edges of tiles, remainders, the smallest and
largest of a branch's range, each against a plain torch evaluation of the same step."""
import pytest
import torch

from paper_2502_16927_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


def ragged_offsets(rows):
    return torch.tensor([0] + torch.tensor(rows).cumsum(0).tolist(), dtype=torch.int32, device=DEV)


def ffn_reference(xp, rows, w1, w2):
    """Pre-activation and output of the experts in fp64."""
    a, o, at = [], [], 0
    for e, n in enumerate(rows):
        pre = xp[at:at + n].double() @ w1[e].double()
        a.append(pre)
        o.append(torch.nn.functional.gelu(pre) @ w2[e].double())
        at += n
    return torch.cat(a), torch.cat(o)


# fp32 products: one wavefront per 32 x 32 tile from 2048 tiles on, four wavefronts on a quarter of K each below
@pytest.mark.parametrize("rows,r,h", [((1, 0, 31, 32), 64, 64),           # fewer rows than a tile, an empty expert
                                      ((33, 5), 64, 192),                 # a row past a tile
                                      ((97, 1000, 3), 128, 1984),         # either side of the line: 2170 tiles up, 140 down
                                      ((2100, 2100), 64, 1024)])
def test_f32_expert_products(rows, r, h):
    g = torch.Generator(device=DEV).manual_seed(sum(rows) + r)
    n, total = len(rows), sum(rows)
    xp = torch.randn((total, r), generator=g, device=DEV)
    w1 = torch.randn((n, r, h), generator=g, device=DEV) * r ** -0.5
    w2 = torch.randn((n, h, r), generator=g, device=DEV) * h ** -0.5
    dims = B.make_dims(total, 256, r, n, 1, h, B.F32)
    act, o = torch.empty((total, h), device=DEV), torch.empty((total, r), device=DEV)
    B.bigmac_grouped_ffn(dims, xp, ragged_offsets(rows), w1, w2, act, o, B.alloc_bytes(B.workspace_bytes(dims, B.WS_GROUPED_FFN)))
    ref_a, ref_o = ffn_reference(xp, rows, w1, w2)
    # a sum of K fp32 products is off by about sqrt(K) 2^-24 of its norm (2.7e-6 at K = 2048); the activation adds 4e-7
    assert rel(act, ref_a) < 5e-6
    assert rel(o, ref_o) < 1e-5
