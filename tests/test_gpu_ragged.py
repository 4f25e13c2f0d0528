"""Rows at any alignment: vocabularies that are not a multiple of eight, odd leading dimensions, odd bases. Each
operand lies inside a buffer of NaNs, so a word read past a row's end that reaches a result shows."""
import pytest
import torch

from paper_2609_36738_amd import bom
from tests.gpu_util import dev, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

LAM = 0.5


def _embed(t, pad=0, offset=0):
    """t as a view with leading dimension V + pad and a base `offset` elements past an aligned one, NaNs around."""
    n, v = t.shape
    buf = torch.full((n * (v + pad) + offset + 64,), float("nan"), dtype=t.dtype, device=dev())
    view = buf.as_strided((n, v), (v + pad, 1), offset)
    view.copy_(t)
    return view


def _rand(g, shape, std, dtype):
    return (torch.randn(shape, generator=g, device=dev()) * std).to(dtype)


# name, N, d, V, row padding of R and W, base offset of R and W
CASES = [
    ("fused_v9", 37, 40, 9, 0, 0),
    ("fused_v8_odd_ld", 64, 64, 8, 1, 0),
    ("fused_one_row", 1, 72, 263, 0, 1),
    ("fused_v65", 130, 200, 65, 0, 0),
    ("fused_v333", 200, 64, 333, 0, 3),
    ("fused_v8185", 70, 32, 8185, 0, 0),
    ("wide_short_k", 5, 32, 9001, 0, 0),
    ("wide_odd_base", 300, 264, 8200, 0, 1),
    ("wide_odd_ld", 300, 264, 8192, 3, 0),
    ("wide_n_tail_tile", 520, 776, 12289, 0, 0),   # the last column alone in its tile
    ("wide_pair", 1031, 768, 32003, 0, 0),
] + [(f"wide_k_tail{r}", 257, 520, 8192 + r, 0, r & 1) for r in range(1, 8)]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_head_vjp_any_alignment(case):
    name, N, d, V, pad, off = case
    log(f"[ragged vjp] {name} N={N} d={d} V={V} pad={pad} offset={off}")
    g = torch.Generator(device=dev()).manual_seed(5)
    H = _rand(g, (N, d), 1.0, torch.bfloat16)
    W = _embed(_rand(g, (d, V), 0.02, torch.bfloat16), pad, off)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    if N > 3:
        y[1::7] = -100
        y[2] = V          # out of range: not supervised
    ok = (y >= 0) & (y < V)
    R = _embed(_rand(g, (N, V), 0.1, torch.bfloat16) * ok[:, None], pad, off)
    q = _rand(g, (V,), 0.05, torch.float32)
    s = _rand(g, (V,), 0.05, torch.float32)
    nv = ok.sum().to(torch.int32).reshape(1)
    dW0 = _rand(g, (d, V), 0.01, torch.float32)
    dW = torch.full((d, V + 1), 7.0, device=dev())   # an odd leading dimension; the extra column stays
    dW[:, :V] = dW0
    out = bom.bom_head_vjp(H, W, R, y, q, nv, s=s, lam=LAM, dW=dW[:, :V], dW_beta=0.5, want_db=True,
                           dh_dtype=torch.float32)
    G = (((1 - LAM) * R.double() + LAM * q.double()) * ok[:, None]) / nv
    rW, rH = H.double().t() @ G + 0.5 * dW0.double(), G @ W.double().t()
    eW = float((dW[:, :V] - rW).norm() / rW.norm())
    eH = float((out["dH"] - rH).norm() / rH.norm())
    log(f"    rel err dW={eW:.2e} dH={eH:.2e}")
    # fp32 sums of exact bf16 products: the rounding of k terms grows like sqrt(k) 2^-24, below 1e-5 at k = 32003
    assert eW <= 1e-5 and eH <= 1e-5
    assert (dW[:, V] == 7.0).all()
    ref = (1 - LAM) * s + LAM * q
    assert float((out["db"] - ref).abs().max()) <= 1e-6


# dW's whole rounds run over the full k range and the column tile left over splits it: a last tile of one to nine columns,
# whose chunk across the end of the row is read from columns of the tile before it. From R, and from the logits, where the
# last of two panels has such a tile.
@pytest.mark.parametrize("N,d,V,logits", [(2048, 1024, 16384 + r, False) for r in (1, 3, 7, 9)] +
                         [(4099, 3848, 4097, False), (16300, 3848, 20481, True), (16300, 3848, 20487, True)])
@pytest.mark.parametrize("beta", [0.0, 0.5])
def test_split_tile_of_few_columns(N, d, V, logits, beta):
    log(f"[ragged split tile] N={N} d={d} V={V} logits={logits} beta={beta}")
    g = torch.Generator(device=dev()).manual_seed(8)
    H, W = _rand(g, (N, d), 1.0, torch.bfloat16), _rand(g, (d, V), 0.02, torch.bfloat16)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    y[1::7] = -100
    y[::5] = V - 1                     # weight on the last column
    ok = y >= 0
    Z = _rand(g, (N, V), 1.0, torch.bfloat16)
    res = bom.bom_residual(Z, y)
    q = _rand(g, (V,), 1e-3, torch.float32)
    dW0 = _rand(g, (d, V), 1e-3, torch.float32)
    kw = dict(lam=LAM, dW_beta=beta, row_lse=res["row_lse"] if logits else None)
    out = bom.bom_head_vjp(H, W, Z if logits else res["R"], y, q, res["n_valid"], dW=dW0.clone(), **kw)
    c0 = V - 300                       # the last columns, the tile before them among them
    G = (((1 - LAM) * res["R"][:, c0:].double() + LAM * q[c0:].double()) * ok[:, None]) / int(ok.sum())
    ref = H.double().t() @ G + beta * dW0[:, c0:].double()
    # per column: fp32 sums of N exact products; with the logits one more rounding of R to bf16 in some elements
    err = (out["dW"][:, c0:] - ref).norm(dim=0) / ref.norm(dim=0)
    log(f"    column error {float(err.max()):.2e}")
    assert float(err.max()) <= (2.0 ** -8 if logits else 1e-5)
    ws = out["workspace"].fill_(0xFF)  # NaN in every word: a partial sum that is not written shows
    again = bom.bom_head_vjp(H, W, Z if logits else res["R"], y, q, res["n_valid"], dW=dW0.clone(), workspace=ws, **kw)
    assert torch.equal(again["dW"], out["dW"])


# 64 x 64 tiles (k in one to nine steps, both operands ragged), 256 x 256 tiles, and those dealt tile by tile (the last two:
# fewer than eight column tiles under more than 32 row tiles)
@pytest.mark.parametrize("N,d,V,pad,off", [(33, 40, 9, 0, 0), (1, 64, 8, 1, 0), (65, 520, 130, 0, 3), (200, 328, 1000, 0, 0),
                                            (300, 264, 8201, 0, 1), (257, 520, 12289, 3, 0), (1031, 768, 32003, 0, 0),
                                            (16384, 512, 1000, 0, 0), (9000, 520, 1027, 0, 0)])
def test_head_forward_any_alignment(N, d, V, pad, off):
    log(f"[ragged forward] N={N} d={d} V={V} pad={pad} offset={off}")
    g = torch.Generator(device=dev()).manual_seed(6)
    H = _rand(g, (N, d), 1.0, torch.bfloat16)
    W = _embed(_rand(g, (d, V), 0.02, torch.bfloat16), pad, off)
    b = _rand(g, (V,), 0.1, torch.bfloat16)
    Z = torch.full((N, V + 1), 7.0, dtype=torch.bfloat16, device=dev())
    bom.bom_head_forward(H, W, b=b, Z=Z[:, :V])
    ref = H.double() @ W.double() + b.double()
    err = (Z[:, :V].double() - ref).abs()
    # one rounding to bf16 (2^-9 of the value) and fp32 sums of d products of size 0.02
    assert bool((err <= ref.abs() * 2.0 ** -8 + 1e-5).all())
    assert (Z[:, V] == 7.0).all()


# Rows of W so far apart that 32 of them span 4 GB: none past the last one is read in place of a row that is there, whose
# infinity would turn the sums to NaN
def test_head_forward_rows_far_apart():
    N, d, V, ld = 300, 8, 1001, 1 << 26
    log(f"[ragged forward] rows {ld} apart")
    g = torch.Generator(device=dev()).manual_seed(16)
    H = _rand(g, (N, d), 1.0, torch.bfloat16).abs() + 0.5
    W = torch.empty(((d - 1) * ld + V,), dtype=torch.bfloat16, device=dev()).as_strided((d, V), (ld, 1))
    W.copy_(_rand(g, (d, V), 0.02, torch.bfloat16))
    W[0, 3] = float("inf")
    Z = bom.bom_head_forward(H, W)
    assert (Z[:, 3] == float("inf")).all()
    Z[:, 3] = 0
    W[0, 3] = 0
    ref = H.double() @ W.double()
    ref[:, 3] = 0
    assert bool(((Z.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-5).all())


# One chunk per thread (64 to 512 threads), rows parked in LDS (1024 and 512 threads, the tail chunk in the first, a
# middle and the last position), and rows past one workgroup's LDS (two passes).
# The first ones: one wave per row, with one to eight chunks per lane, aligned and ragged, rows in one and several turns.
RES_CASES = [(9000, 8, 0, 0), (700, 511, 0, 0), (5000, 1000, 0, 0), (3000, 1025, 0, 1), (4200, 2049, 1, 0), (2100, 4096, 0, 0),
             (37, 8, 1, 0), (300, 9, 0, 0), (5, 511, 0, 1), (260, 1001, 0, 0), (33, 4095, 2, 3), (40, 4096, 1, 0),
             (700, 4097, 0, 0), (20, 8199, 0, 1), (300, 12345, 0, 0), (9, 32773, 1, 0), (600, 50257, 0, 0),
             (3, 57343, 0, 1), (70, 57345, 0, 0), (21, 65541, 3, 0), (1, 128257, 0, 1)]


# Several workgroups per CU (two and three chunks per thread, from 3500 rows on), and the two passes element by element
RES_CASES += [(3500, 8191, 0, 0), (3501, 8192, 1, 0), (3600, 12281, 0, 0), (3499, 8191, 0, 0), (9000, 6001, 0, 1), (3600, 12290, 0, 0),
              (1536, 4097, 0, 0), (2100, 8201, 0, 0), (1536, 16000, 0, 1)]


@pytest.mark.parametrize("N,V,pad,off", RES_CASES)
def test_residual_any_alignment(N, V, pad, off):
    log(f"[ragged residual] N={N} V={V} pad={pad} offset={off}")
    g = torch.Generator(device=dev()).manual_seed(7)
    Z = _embed(_rand(g, (N, V), 2.0, torch.bfloat16), pad, off)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    y[0] = V - 1                        # a label in the columns past the last whole chunk
    if N > 4:
        y[1::9] = -100
        y[3] = V
    ok = (y >= 0) & (y < V)
    Rbuf = torch.full((N, V + pad), 7.0, dtype=torch.bfloat16, device=dev())
    out = bom.bom_residual(Z, y, R=Rbuf[:, :V])
    p = torch.softmax(Z.double(), 1)
    p[torch.arange(N, device=dev())[ok], y[ok].long()] -= 1
    p *= ok[:, None]
    n = int(ok.sum())
    lse = torch.logsumexp(Z.double(), 1)
    assert out["n_valid"].item() == n and out["flags"].item() == (bom.BOM_FLAG_LABEL_RANGE if N > 4 else 0)
    assert float((out["row_lse"] - lse).abs().max()) <= 4e-6          # fp32 of values up to about 14
    zf = Z.float()
    first = (zf == zf.max(1, keepdim=True).values).int().argmax(1)    # the lowest column holding the maximum
    assert torch.equal(out["row_argmax"].long(), first)
    tgt = torch.where(ok, zf.gather(1, y.clamp(0, V - 1).long()[:, None])[:, 0], torch.zeros(N, device=dev()))
    assert torch.equal(out["row_target"], tgt)
    # R: one rounding to bf16 of an fp32 value good to 1e-6
    assert bool(((Rbuf[:, :V].double() - p).abs() <= p.abs() * 2.0 ** -8 + 1e-9).all())
    assert (Rbuf[:, V:] == 7.0).all()
    assert float((out["s"] - p.sum(0) / n).norm() / (p.sum(0) / n).norm()) <= 2e-6
    again = bom.bom_residual(Z, y)
    assert torch.equal(again["R"], Rbuf[:, :V]) and torch.equal(again["s"], out["s"])


# A number of rows that is not a multiple of eight, past the fused launch and with few output tiles of either product: the
# history term is much larger than R, and R is multiplied as stored all the same
@pytest.mark.parametrize("N,d,V", [(8201, 32, 4504), (9001, 264, 64), (33, 264, 9000), (257, 64, 20000), (8193, 8, 16)])
@pytest.mark.parametrize("want_dH", [True, False])
def test_any_number_of_rows(N, d, V, want_dH):
    log(f"[any rows] N={N} d={d} V={V} dH={want_dH}")
    g = torch.Generator(device=dev()).manual_seed(19)
    H, W = _rand(g, (N, d), 1.0, torch.bfloat16), _rand(g, (d, V), 0.05, torch.bfloat16)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    y[1::7] = -100
    ok = y >= 0
    res = bom.bom_residual((H.float() @ W.float()).bfloat16(), y)
    q = _rand(g, (V,), 0.05, torch.float32)
    out = bom.bom_head_vjp(H, W, res["R"], y, q, res["n_valid"], lam=LAM, want_dH=want_dH, dh_dtype=torch.float32)
    G = ((1 - LAM) * res["R"].double() + LAM * q.double()) * ok[:, None] / int(ok.sum())
    rW, rH = H.double().t() @ G, G @ W.double().t()
    # fp32 sums of exact products and the rank-1 term's fp32 vectors
    assert float((out["dW"] - rW).norm() / rW.norm()) <= 1e-5
    assert not want_dH or float((out["dH"] - rH).norm() / rH.norm()) <= 1e-5
