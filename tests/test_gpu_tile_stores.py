"""Outputs of the 256 x 256 tiles at their edges: rows and columns left over, rows at any alignment, values beside the output."""
import pytest
import torch

from paper_2609_36738_amd import bom
from tests.gpu_util import dev, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


# last row tile of one row, of all but one and whole; last column tile of eight columns, of nine (the eighth and ninth
# moved), of one and whole; the output's row pitch beyond its columns
@pytest.mark.parametrize("N,d,V,pad", [(2049, 776, 8200, 0), (511, 264, 8201, 1), (512, 504, 8449, 3), (1535, 1032, 8192, 3),
                                       (2049, 520, 16641, 1)])
@pytest.mark.parametrize("out", [torch.float32, torch.bfloat16])
def test_tile_edges(N, d, V, pad, out):
    log(f"[tile stores] N={N} d={d} V={V} pad={pad} {out}")
    g = torch.Generator(device=dev()).manual_seed(13)

    def rand(shape, std, t=torch.bfloat16):
        return (torch.randn(shape, generator=g, device=dev()) * std).to(t)

    H, W = rand((N, d), 1.0), rand((d, V), 0.02)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    R = rand((N, V), 0.1)
    q = rand((V,), 0.05, torch.float32)
    nv = torch.full((1,), N, dtype=torch.int32, device=dev())
    dW = torch.full((d, V + pad + 1), 7.0, dtype=out, device=dev())
    dH = torch.full((N, d + pad + 1), 7.0, dtype=out, device=dev())
    bom.bom_head_vjp(H, W, R, y, q, nv, lam=0.5, dW=dW[:, :V], dH=dH[:, :d])
    G = (0.5 * R.double() + 0.5 * q.double()) / N
    for got, ref, k in ((dW[:, :V], H.double().t() @ G, N), (dH[:, :d], G @ W.double().t(), V)):
        # fp32 sums of k exact products (error below sqrt(k) 2^-23 of the typical value), then one rounding to bf16
        lim = ref.norm() / ref.numel() ** 0.5 * k ** 0.5 * 2.0 ** -20 + (ref.abs() * 2.0 ** -8 if out == torch.bfloat16 else 0.0)
        assert bool(((got.double() - ref).abs() <= lim).all())
    assert (dW[:, V:] == 7.0).all() and (dH[:, d:] == 7.0).all()
    Z = torch.full((N, V + pad + 1), 7.0, dtype=torch.bfloat16, device=dev())
    bom.bom_head_forward(H, W, Z=Z[:, :V])
    ref = H.double() @ W.double()
    assert bool(((Z[:, :V].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-5).all()) and (Z[:, V:] == 7.0).all()


# forward tiles streamed one after another by a workgroup: one k tile and less, a part of a second, several, both orders of
# the tiles and a row pitch of Z past the streamed stores' range (single tiles)
@pytest.mark.parametrize("N,d,V,ldz", [(4099, 40, 20000, 0), (4099, 72, 20003, 0), (4400, 64, 16648, 3), (9000, 136, 2568, 0),
                                       (2300, 200, 33288, 1), (257, 64, 20008, 1 << 21)])
@pytest.mark.parametrize("bias", [False, True])
def test_streamed_forward(N, d, V, ldz, bias):
    log(f"[streamed forward] N={N} d={d} V={V} ldz={ldz} bias={bias}")
    g = torch.Generator(device=dev()).manual_seed(14)

    def rand(shape, std):
        return (torch.randn(shape, generator=g, device=dev()) * std).to(torch.bfloat16)

    H, W = rand((N, d), 1.0), rand((d, V), 0.02)
    b = rand((V,), 0.1) if bias else None
    Z = torch.full((N, ldz if ldz > V else V + ldz), 7.0, dtype=torch.bfloat16, device=dev())
    bom.bom_head_forward(H, W, b=b, Z=Z[:, :V])
    ref = H.double() @ W.double() + (b.double() if bias else 0.0)
    assert bool(((Z[:, :V].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-5).all()) and (Z[:, V:] == 7.0).all()


# dW alone where the plan of dH has whole rounds and leftover rows that split k, aligned and ragged
@pytest.mark.parametrize("N,d,V", [(4100, 3848, 4096), (4100, 3848, 4097)])
def test_no_dH(N, d, V):
    log(f"[no dH] N={N} d={d} V={V}")
    g = torch.Generator(device=dev()).manual_seed(15)

    def rand(shape, std, t=torch.bfloat16):
        return (torch.randn(shape, generator=g, device=dev()) * std).to(t)

    H, W, R = rand((N, d), 1.0), rand((d, V), 0.02), rand((N, V), 0.1)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    q = rand((V,), 0.05, torch.float32)
    nv = torch.full((1,), N, dtype=torch.int32, device=dev())
    a = bom.bom_head_vjp(H, W, R, y, q, nv, lam=0.5, want_dH=False)
    ref = H.double().t() @ ((0.5 * R.double() + 0.5 * q.double()) / N)
    # fp32 sums of N exact products
    assert a["dH"] is None and float((a["dW"] - ref).norm() / ref.norm()) <= 1e-5


# rows of Z that are whole cache lines and not, and widths and sizes on both sides of where stores bypass the L2
@pytest.mark.parametrize("N,d,V,ldz", [(3000, 32, 26520, 0), (3000, 504, 8200, 8201), (3000, 512, 8200, 0), (1000, 8, 30001, 0),
                                       (2050, 64, 32000, 0), (2050, 64, 32000, 32064), (8200, 512, 17904, 0), (2050, 2048, 4104, 0)])
def test_forward_stores(N, d, V, ldz):
    test_streamed_forward(N, d, V, ldz, True)


# dW alone over few rows: SIMT below a number of rows, the matrix kernels from it on, from R and from the logits
@pytest.mark.parametrize("N", [1, 19, 20, 43, 44, 51, 52, 63, 64])
@pytest.mark.parametrize("d,V", [(264, 1000), (72, 5001), (136, 9000)])
@pytest.mark.parametrize("logits", [False, True])
def test_no_dH_few_rows(N, d, V, logits):
    log(f"[no dH] N={N} d={d} V={V} logits={logits}")
    g = torch.Generator(device=dev()).manual_seed(17)

    def rand(shape, std, t=torch.bfloat16):
        return (torch.randn(shape, generator=g, device=dev()) * std).to(t)

    H, W, Z = rand((N, d), 1.0), rand((d, V), 0.02), rand((N, V), 1.0)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    y[1::5] = 3
    res = bom.bom_residual(Z, y, ignore_index=3)
    q, s = rand((V,), 0.05, torch.float32), rand((V,), 0.05, torch.float32)
    a = bom.bom_head_vjp(H, W, Z if logits else res["R"], y, q, res["n_valid"], s=s, lam=0.5, ignore_index=3, want_dH=False,
                         want_db=True, row_lse=res["row_lse"] if logits else None)
    ok = y != 3
    G = (0.5 * res["R"].double() + 0.5 * q.double()) * ok[:, None] / int(ok.sum())
    ref = H.double().t() @ G
    # fp32 sums of N exact products; on the 128-tile kernel G is rounded to bf16, from the logits R a second time in some places
    assert float((a["dW"] - ref).norm() / ref.norm()) <= 2.0 ** -8
    assert float((a["db"] - 0.5 * (s + q)).abs().max()) <= 1e-7
