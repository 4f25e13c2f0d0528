"""The fp32 head products on the matrix cores: ragged tiles, split k ranges of either product, the logits route."""
import pytest
import torch

from paper_2609_36738_amd import bom
from tests.gpu_util import dev, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

LAM = 0.25


def _rand(g, shape, std):
    return torch.randn(shape, generator=g, device=dev()) * std


# name, N, d, V: tiles of both edges, k shorter than one tile, dW's or dH's k range split, both unsplit
CASES = [("ragged", 601, 301, 707), ("split_dh", 70, 300, 20011), ("split_dw", 8200, 66, 130), ("one_row", 1, 65, 9001),
         ("two_columns", 9000, 130, 2), ("unsplit", 1500, 520, 1111)]


@pytest.mark.parametrize("logits", [False, True], ids=["residual", "logits"])
@pytest.mark.parametrize("name,N,d,V", CASES, ids=[c[0] for c in CASES])
def test_head_vjp_f32(name, N, d, V, logits):
    log(f"[f32 vjp] {name} N={N} d={d} V={V} logits={logits}")
    g = torch.Generator(device=dev()).manual_seed(3)
    H, W, Z = _rand(g, (N, d), 1.0), _rand(g, (d, V), 0.02), _rand(g, (N, V), 1.0)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    if N > 3:
        y[1::7] = -100
        y[2] = V
    ok = (y >= 0) & (y < V)
    lse = torch.logsumexp(Z.double(), 1)
    R = torch.softmax(Z.double(), 1)
    R[torch.arange(N, device=dev())[ok], y[ok].long()] -= 1
    R *= ok[:, None]
    nv = ok.sum().to(torch.int32).reshape(1)
    q, s = _rand(g, (V,), 0.05), _rand(g, (V,), 0.05)
    dW = torch.full((d, V + 1), 7.0, device=dev())
    dW0 = _rand(g, (d, V), 0.01)
    dW[:, :V] = dW0
    third = Z if logits else R.float()
    for dt in (torch.float32, torch.bfloat16):
        dW[:, :V] = dW0
        out = bom.bom_head_vjp(H, W, third, y, q, nv, s=s, lam=LAM, dW=dW[:, :V], dW_beta=0.5, want_db=True,
                               dh_dtype=dt, row_lse=lse.float() if logits else None)
        G = ((1 - LAM) * R + LAM * q.double()) * ok[:, None] / nv
        rW, rH = H.double().t() @ G + 0.5 * dW0.double(), G @ W.double().t()
        eW = float((dW[:, :V] - rW).norm() / rW.norm())
        eH = float((out["dH"].double() - rH).norm() / rH.norm())
        log(f"    {dt} rel err dW={eW:.2e} dH={eH:.2e}")
        # fp32 sums of up to 20011 terms: sqrt(k) 2^-24 stays below 1e-5; bf16 dH: one rounding, at most 2^-9
        assert eW <= 1e-5 and eH <= (1e-5 if dt == torch.float32 else 2.0 ** -8)
        assert (dW[:, V] == 7.0).all()
    assert float((out["db"] - ((1 - LAM) * s + LAM * q)).abs().max()) <= 1e-6


# dW alone over few rows: SIMT up to a number of rows that grows with the gradient, the matrix kernel past it; 32 rows of more
# than 128 features (a whole k tile) on the matrix kernel, of fewer on SIMT; wide heads of few features
@pytest.mark.parametrize("logits", [False, True], ids=["residual", "logits"])
@pytest.mark.parametrize("N,d,V", [(1, 1001, 4003), (16, 1001, 4003), (17, 1001, 4003), (28, 130, 100003), (29, 130, 100003),
                                   (32, 128, 100003), (33, 128, 100003), (32, 1024, 36001), (48, 1024, 36001),
                                   (49, 1024, 36001), (48, 65, 130001), (16, 3, 125001), (60, 33, 200003), (61, 33, 200003),
                                   (64, 64, 300001)])
def test_head_vjp_f32_dw_alone(N, d, V, logits):
    log(f"[f32 dW alone] N={N} d={d} V={V} logits={logits}")
    g = torch.Generator(device=dev()).manual_seed(5)
    H, Z = _rand(g, (N, d + 3), 1.0)[:, :d], _rand(g, (N, V + 1), 1.0)[:, :V]
    W = _rand(g, (d, V), 0.02)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    if N > 3:
        y[1::7] = -100
        y[2] = V
    ok = (y >= 0) & (y < V)
    lse = torch.logsumexp(Z.double(), 1)
    R = torch.softmax(Z.double(), 1)
    R[torch.arange(N, device=dev())[ok], y[ok].long()] -= 1
    R *= ok[:, None]
    third = Z if logits else R.float()
    third[~ok] = float("nan")                    # a row outside the supervised ones adds nothing, whatever it holds
    nv = ok.sum().to(torch.int32).reshape(1)
    q, s = _rand(g, (V,), 0.05), _rand(g, (V,), 0.05)
    dW = torch.full((d, V + 1), 7.0, device=dev())
    dW0 = _rand(g, (d, V), 0.01)
    dW[:, :V] = dW0
    out = bom.bom_head_vjp(H, W, third, y, q, nv, s=s, lam=LAM, dW=dW[:, :V], dW_beta=0.5, want_db=True, want_dH=False,
                           row_lse=lse.float() if logits else None)
    G = ((1 - LAM) * R + LAM * q.double()) * ok[:, None] / nv
    rW = H.double().t() @ G + 0.5 * dW0.double()
    # at most 64 fp32 products and sums; from the logits p = 2^(z log2 e - lse log2 e) on arguments below 32: 32 2^-24 at most
    eW = float((dW[:, :V] - rW).norm() / rW.norm())
    log(f"    rel err dW={eW:.2e}")
    assert eW <= 1e-5 and (dW[:, V] == 7.0).all()
    assert float((out["db"] - ((1 - LAM) * s + LAM * q)).abs().max()) <= 1e-6


@pytest.mark.parametrize("N,d,V", [(1, 1, 2), (65, 33, 129), (600, 301, 1001)])
def test_head_forward_f32(N, d, V):
    log(f"[f32 forward] N={N} d={d} V={V}")
    g = torch.Generator(device=dev()).manual_seed(4)
    H, W, b = _rand(g, (N, d), 1.0), _rand(g, (d, V), 0.02), _rand(g, (V,), 0.1)
    Z = torch.full((N, V + 3), 7.0, device=dev())
    bom.bom_head_forward(H, W, b=b, Z=Z[:, :V])
    ref = H.double() @ W.double() + b.double()
    assert float((Z[:, :V] - ref).norm() / ref.norm()) <= 1e-6 and (Z[:, V:] == 7.0).all()


# fewer than four features: a small Z and a large one (SIMT), and four
@pytest.mark.parametrize("N,d,V", [(100, 1, 9000), (301, 1, 9001), (1000, 3, 9000), (65, 2, 40000), (301, 4, 9001)])
def test_head_forward_f32_few_features(N, d, V):
    test_head_forward_f32(N, d, V)
