"""The one-workgroup residual of small batches of short rows, at the ends of its range and past them (one wave per row)."""
import pytest
import torch

from paper_2609_36738_amd import bom
from tests.gpu_util import dev, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


@pytest.mark.parametrize("N", [1, 63, 65, 256, 257, 5000])
@pytest.mark.parametrize("V,dtype", [(1000, "f32"), (1023, "f32"), (2, "f32"), (10, "f32"), (16, "f32"), (17, "f32"), (64, "f32"), (3, "bf16"),
                                     (8, "bf16"), (63, "bf16"), (64, "bf16"), (127, "bf16"), (128, "bf16")])
def test_small_residual(N, V, dtype):
    log(f"[small residual] N={N} V={V} {dtype}")
    g = torch.Generator(device=dev()).manual_seed(N + V)
    Z = (torch.randn((N, V), generator=g, device=dev()) * 2).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    if N > 3:
        y[1::5] = -100
        y[2] = -7
    ok = (y >= 0) & (y < V)
    R = torch.full((N, V + 1), 7.0, dtype=Z.dtype, device=dev())
    out = bom.bom_residual(Z, y, R=R[:, :V])
    p = torch.softmax(Z.double(), 1)
    p[torch.arange(N, device=dev())[ok], y[ok].long()] -= 1
    p *= ok[:, None]
    n = int(ok.sum())
    lse = torch.logsumexp(Z.double(), 1)
    zf = Z.float()
    first = (zf == zf.max(1, keepdim=True).values).int().argmax(1)
    tgt = torch.where(ok, zf.gather(1, y.clamp(0, V - 1).long()[:, None])[:, 0], torch.zeros(N, device=dev()))
    assert out["n_valid"].item() == n and out["flags"].item() == (bom.BOM_FLAG_LABEL_RANGE if N > 3 else 0)
    assert torch.equal(out["row_argmax"].long(), first) and torch.equal(out["row_target"], tgt)
    assert float((out["row_lse"] - lse).abs().max()) <= 2e-6            # fp32 of values below 16
    step = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -21                 # one rounding; fp32: a few of exp and 1 / sum
    assert bool(((R[:, :V].double() - p).abs() <= p.abs() * step + 2e-7).all()) and (R[:, V] == 7.0).all()
    assert float((out["s"] - p.sum(0) / n).abs().max()) <= 3e-7         # means of values below 1
    ce = float(((lse - tgt) * ok).sum() / n)
    assert abs(float(out["loss"]) - ce) <= 1e-6 * max(1.0, ce)


def test_small_residual_all_ignored():
    Z = torch.randn((70, 9), device=dev())
    out = bom.bom_residual(Z, torch.full((70,), -100, dtype=torch.int32, device=dev()))
    assert out["flags"].item() == bom.BOM_FLAG_EMPTY and out["n_valid"].item() == 0 and out["loss"].item() == 0
    assert (out["s"] == 0).all() and (out["R"] == 0).all() and (out["row_target"] == 0).all()


# one wave per row with up to 32 fp32 columns per lane, any number of waves per workgroup; wider rows take the other kernels
@pytest.mark.parametrize("N,V", [(1024, 1028), (1100, 2000), (2561, 2048), (2100, 1672), (9000, 2052)])
def test_fp32_rows_per_wave(N, V):
    test_small_residual(N, V, "f32")


@pytest.mark.parametrize("N,V", [(3072, 2400), (3100, 4096), (3071, 2400), (3300, 3999), (700, 1000)])
def test_bf16_rows_per_wave(N, V):
    test_small_residual(N, V, "bf16")


# Nearly 2^31 rows: a wave's next row number passes the largest int
def test_rows_up_to_the_largest_int():
    N, V = 2 ** 31 - 300, 2
    if torch.cuda.mem_get_info()[0] < 80e9:
        pytest.skip("needs 80 GB of free memory")
    log(f"[small residual] N={N} V={V}")
    Z = torch.zeros((N, V), dtype=torch.bfloat16, device=dev())
    Z[N - 1, 1] = 3.0
    out = bom.bom_residual(Z, torch.zeros(N, dtype=torch.int32, device=dev()), write_R=False)
    assert out["n_valid"].item() == N and out["flags"].item() == 0
    assert out["s"].tolist() == [-0.5, 0.5]                             # exact sums; the last row is below half a rounding
    lse, am = out["row_lse"], out["row_argmax"]
    assert abs(float(lse[N - 1]) - 3.0485874) < 1e-6 and int(am[N - 1]) == 1
    assert float(lse[:N - 1].min()) == float(lse[:N - 1].max()) and abs(float(lse[0]) - 0.6931472) < 1e-7
    assert int(am[:N - 1].max()) == 0
