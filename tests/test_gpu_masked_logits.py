"""Residuals of rows with masked columns (-inf, or the type's lowest value), over every route of the residual: threads, waves
and parts of a row that hold masked columns alone."""
import pytest
import torch

from paper_2609_36738_amd import bom
from tests.gpu_util import dev, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

BF16 = [(64, 10), (300, 1000), (300, 1001), (5000, 1000), (5000, 3001),   # one launch, register rows, one wave per row
        (64, 4104), (64, 4099), (2500, 4099), (4000, 9001), (64, 20000), (64, 20001), (64, 32003), (64, 50257), (64, 50304),
        (64, 70000), (600, 128256),                                       # split rows
        (64, 70001)]                                                      # two passes
F32 = [(64, 10), (300, 1000), (5000, 2000), (64, 4100), (64, 4097), (64, 20000), (64, 20001), (64, 32000)]


@pytest.mark.parametrize("mask", ["inf", "lowest"])
@pytest.mark.parametrize("N,V,dtype", [(*c, torch.bfloat16) for c in BF16] + [(*c, torch.float32) for c in F32])
def test_masked_columns(N, V, dtype, mask):
    log(f"[masked residual] N={N} V={V} {dtype} {mask}")
    g = torch.Generator(device=dev()).manual_seed(V)
    Z = torch.randn((N, V), generator=g, device=dev()).to(dtype)
    x = float("-inf") if mask == "inf" else torch.finfo(dtype).min
    c = V // 2
    Z[1, :c] = x
    Z[2, c + 1:] = x
    Z[3, torch.arange(V, device=dev()) != c] = x          # one column left
    Z[4, ::2] = x
    Z[5, min(c + 1, V - 1):] = x
    Z[5, :max(c - 8, 0)] = x
    Z[6, torch.arange(V, device=dev()) != V - 1] = x      # the last column alone
    y = torch.full((N,), c | 1, dtype=torch.int32, device=dev())
    y[3], y[5], y[6] = c, c, V - 1
    y[8] = -100
    out = bom.bom_residual(Z, y)
    ok = y != -100
    p = torch.softmax(Z.double(), 1)
    p[torch.arange(N, device=dev())[ok], y[ok].long()] -= 1
    p *= ok[:, None]
    lse = torch.logsumexp(Z.double(), 1)
    zf = Z.float()
    assert torch.equal(out["row_argmax"].long(), (zf == zf.max(1, keepdim=True).values).int().argmax(1))
    # fp32 of values below 16; one rounding of R, fp32: the error of lse in the exponent
    assert float((out["row_lse"] - lse).abs().max()) <= 4e-6
    step = 2.0 ** -8 if dtype == torch.bfloat16 else 1e-5
    assert bool(((out["R"].double() - p).abs() <= p.abs() * step + 2e-7).all())
    assert float((out["s"] - p.sum(0) / int(ok.sum())).abs().max()) <= 1e-6


# A row with every column masked has no distribution; its argmax still is a column
@pytest.mark.parametrize("N,V,dtype", [(64, 20001, torch.bfloat16), (64, 70001, torch.bfloat16), (64, 70000, torch.bfloat16),
                                       (64, 32000, torch.float32)])
def test_all_masked_row(N, V, dtype):
    Z = torch.randn((N, V), device=dev()).to(dtype)
    Z[1] = float("-inf")
    out = bom.bom_residual(Z, torch.zeros(N, dtype=torch.int32, device=dev()))
    assert out["row_argmax"][1] == 0 and not torch.isfinite(out["row_lse"][1])
    rest = torch.arange(N, device=dev()) != 1
    assert torch.isfinite(out["row_lse"][rest]).all() and torch.isfinite(out["R"][rest]).all()
