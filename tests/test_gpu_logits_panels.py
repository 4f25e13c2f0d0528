"""Large bf16 head VJPs from the logits: R formed in one panel of columns or in several, aligned and ragged, or in the
products' copies where the workspace holds no panel."""
import math

import pytest
import torch

from paper_2609_36738_amd import bom
from tests.gpu_util import dev, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


# name, N, d, V, lambda, want dH, ignore_index (one of them a class)
CASES = [("one_panel_ragged", 2056, 264, 6001, 0.5, True, -100),
         ("two_panels", 20000, 64, 16392, 0.5, True, -100),
         ("two_panels_ragged", 20000, 72, 16395, 0.25, True, 0),
         ("two_panels_no_history", 20000, 72, 16395, 0.0, True, -100),
         # the small products (one launch, and 128-tile kernels), an ignored label inside [0, V)
         ("fused_ignored_class", 200, 64, 264, 0.5, True, 3), ("fused_ignored_class_ragged", 200, 64, 333, 0.5, True, 3),
         ("tiles128_ignored_class", 64, 128, 8200, 0.5, True, 3),
         ("narrow_panels_no_dH", 70000, 32, 8257, 0.5, False, -100),
         # one tile along d and many rows: no panel, above and below the line in N and in V
         ("one_d_tile", 6200, 256, 8008, 0.5, True, 5), ("one_d_tile_few_rows", 6136, 256, 8008, 0.5, True, -100),
         ("one_d_tile_few_columns", 6200, 256, 7992, 0.5, True, -100), ("one_d_tile_no_dH", 6149, 40, 8000, 0.25, False, -100)]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_head_vjp_logits_panels(case):
    name, N, d, V, lam, want_dH, ig = case
    log(f"[logits panels] {name} N={N} d={d} V={V}")
    g = torch.Generator(device=dev()).manual_seed(9)

    def rand(shape, std, dtype=torch.bfloat16):
        return (torch.randn(shape, generator=g, device=dev()) * std).to(dtype)

    H, W, Z = rand((N, d), 1.0), rand((d, V), 0.02), rand((N, V), 1.0)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    y[1::7] = ig
    y[2] = V
    y[3] = V - 1
    q, s = rand((V,), 0.01, torch.float32), rand((V,), 0.01, torch.float32)
    res = bom.bom_residual(Z, y, ignore_index=ig)
    kw = dict(s=s, lam=lam, ignore_index=ig, want_db=True, want_dH=want_dH, dh_dtype=torch.float32)
    dW0 = rand((d, V), 1e-3, torch.float32)
    a = bom.bom_head_vjp(H, W, Z, y, q, res["n_valid"], row_lse=res["row_lse"], dW=dW0.clone(), dW_beta=0.5, **kw)
    b = bom.bom_head_vjp(H, W, res["R"], y, q, res["n_valid"], dW=dW0.clone(), dW_beta=0.5, **kw)
    ok = (y >= 0) & (y < V) & (y != ig)
    R = res["R"].double()
    G = ((1 - lam) * R + lam * q.double()) * ok[:, None] / int(ok.sum())
    ref = dict(dW=H.double().t() @ G + 0.5 * dW0.double(), dH=G @ W.double().t())
    for k in ("dW", "dH") if want_dH else ("dW",):
        # the stored R and the R formed from Z differ by at most one rounding of bf16 in some elements
        ez = float((a[k] - ref[k]).norm() / ref[k].norm())
        er = float((b[k] - ref[k]).norm() / ref[k].norm())
        log(f"    {k}: rel err {ez:.2e} (stored R {er:.2e})")
        # (the 128-tile kernels round G to bf16 as well: 2^-9 at most)
        assert er <= (2.0 ** -9 if name.startswith("tiles128") else 1e-5) and ez <= 2.0 ** -8
    assert torch.equal(a["db"], b["db"])
    assert math.isfinite(float(a["dW"].sum()))


# The workspace that a stored R needs holds no panel: the 256-tile products (whole rounds, split leftovers on either side,
# both products in one grid, k ranges and rows that no tile divides) form R as they copy it, ragged rows go to the SIMT
# kernels, and the result is that of the panels. One label is an ignore_index inside [0, V).
SMALL_WS = [("leftovers", 2048, 1024, 16392, 0.5, True, "f32"), ("rows_left", 4100, 3848, 4096, 0.5, True, "f32"),
            ("pair", 1032, 768, 32000, 0.25, True, "f32"), ("pair_bf16_dW", 1032, 768, 32000, 0.5, True, "bf16"),
            ("odd_rows", 2049, 520, 6008, 0.5, True, "f32"), ("no_history", 2056, 264, 6000, 0.0, True, "f32"),
            ("no_dH", 4100, 3848, 4096, 0.5, False, "bf16"), ("several_panels", 20000, 264, 16392, 0.5, True, "f32"),
            ("ragged", 520, 264, 6001, 0.5, True, "f32"), ("ragged_bf16_dW", 520, 264, 6001, 0.5, True, "bf16")]


@pytest.mark.parametrize("case", SMALL_WS, ids=[c[0] for c in SMALL_WS])
def test_logits_workspace_without_panel(case):
    name, N, d, V, lam, want_dH, dw = case
    log(f"[logits, no panel] {name} N={N} d={d} V={V}")
    g = torch.Generator(device=dev()).manual_seed(10)

    def rand(shape, std, dtype=torch.bfloat16):
        return (torch.randn(shape, generator=g, device=dev()) * std).to(dtype)

    H, W, Z = rand((N, d), 1.0), rand((d, V), 0.02), rand((N, V), 1.0)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    ig = 3
    y[1::7] = ig
    y[2] = V
    y[4] = V - 1
    q, s = rand((V,), 0.01, torch.float32), rand((V,), 0.01, torch.float32)
    res = bom.bom_residual(Z, y, ignore_index=ig)
    dW_dt = torch.bfloat16 if dw == "bf16" else torch.float32
    code = bom.BOM_BF16 if dw == "bf16" else bom.BOM_F32
    small = bom.bom_head_vjp_workspace_bytes(N, d, V, bom.BOM_BF16, code)
    assert bom.bom_head_vjp_logits_workspace_bytes(N, d, V, bom.BOM_BF16, code) >= small + 2 * N * min(V, 4096)
    out = {}
    for key, nb in (("panels", bom.bom_head_vjp_logits_workspace_bytes(N, d, V, bom.BOM_BF16, code)), ("copies", small)):
        ws = torch.full((nb + 4096,), 0xFF, dtype=torch.uint8, device=dev())
        dW = torch.full((d, V), 7.0, dtype=dW_dt, device=dev())
        db = torch.empty(V, dtype=dW_dt, device=dev())
        dH = torch.full((N, d), 7.0, device=dev()) if want_dH else None
        bom._check(bom.load().bom_head_vjp(
            H.data_ptr(), d, W.data_ptr(), V, Z.data_ptr(), 0, V, bom.BOM_BF16, N, d, V, y.data_ptr(), ig,
            res["row_lse"].data_ptr(), q.data_ptr(), s.data_ptr(), res["n_valid"].data_ptr(), lam, dW.data_ptr(), code, V, 0.0,
            db.data_ptr(), dH.data_ptr() if want_dH else None, bom.BOM_F32, d, ws.data_ptr(), nb,
            torch.cuda.current_stream().cuda_stream))
        assert bool((ws[nb:] == 0xFF).all())
        out[key] = dict(dW=dW, db=db, dH=dH)
    ok = (y >= 0) & (y < V) & (y != ig)
    R = torch.exp(Z.double() - res["row_lse"].double()[:, None])
    R[torch.arange(N, device=dev())[ok], y[ok].long()] -= 1
    G = ((1 - lam) * R + lam * q.double()) * ok[:, None] / int(ok.sum())
    ref = dict(dW=H.double().t() @ G, dH=G @ W.double().t())
    for k in ("dW", "dH") if want_dH else ("dW",):
        e = {x: float((out[x][k].double() - ref[k]).norm() / ref[k].norm()) for x in out}
        log(f"    {k}: rel err panels {e['panels']:.2e} copies {e['copies']:.2e}")
        # R (and dW in bf16) rounded to bf16: 2^-9 at most each
        assert max(e.values()) <= 2.0 ** -8
    assert torch.equal(out["panels"]["db"], out["copies"]["db"])


# More rows than one grid of the panel kernel has workgroups for
def test_panel_of_many_rows():
    N, d, V = 2 ** 24 + 1000, 64, 256
    if torch.cuda.mem_get_info()[0] < 100e9:
        pytest.skip("needs 100 GB of free memory")
    log(f"[logits panels] N={N} d={d} V={V}")
    g = torch.Generator(device=dev()).manual_seed(18)
    H = torch.empty((N, d), dtype=torch.bfloat16, device=dev()).normal_(generator=g)
    W = (torch.randn((d, V), generator=g, device=dev()) * 0.02).to(torch.bfloat16)
    Z = torch.empty((N, V), dtype=torch.bfloat16, device=dev()).normal_(generator=g)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    q = torch.randn(V, generator=g, device=dev()) * 0.01
    res = bom.bom_residual(Z, y, write_R=False)
    out = bom.bom_head_vjp(H, W, Z, y, q, res["n_valid"], lam=0.5, row_lse=res["row_lse"], dh_dtype=torch.float32)
    rW = torch.zeros((d, V), dtype=torch.float64, device=dev())
    for i in range(0, N, 1 << 21):
        j = min(N, i + (1 << 21))
        G = torch.softmax(Z[i:j].double(), 1)
        G[torch.arange(j - i, device=dev()), y[i:j].long()] -= 1
        G = (0.5 * G + 0.5 * q.double()) / N
        rW += H[i:j].double().t() @ G
        rH = G @ W.double().t()
        # R rounded to bf16
        assert float((out["dH"][i:j] - rH).norm() / rH.norm()) <= 2.0 ** -8
    # R rounded to bf16, and fp32 sums of 2^24 products
    assert float((out["dW"] - rW).norm() / rW.norm()) <= 2.0 ** -8
