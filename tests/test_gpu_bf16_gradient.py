"""bf16 dW and db: rounded where the fp32 product is stored, on every route, against the fp32 dW of the same call."""
import pytest
import torch

from paper_2609_36738_amd import bom
from tests.gpu_util import dev, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]


# name, N, d, V, operand dtype, logits input: one launch of small tiles, 256-tile launches (whole rounds, split leftovers, both
# products in one grid), panels of R, 128-tile and SIMT kernels and fp32 operands (rounded in a pass)
CASES = [("fused", 200, 136, 264, "bf16", False), ("fused_ragged", 70, 64, 333, "bf16", False),
         ("wide_split", 512, 256, 4096, "bf16", False), ("wide_rounds", 300, 1032, 70000, "bf16", False),
         ("pair", 1031, 768, 32003, "bf16", False), ("panels", 20000, 72, 16395, "bf16", True),
         ("tiles128", 64, 128, 8200, "bf16", False), ("simt", 60, 65, 500, "bf16", False), ("f32", 600, 72, 300, "f32", False)]


@pytest.mark.parametrize("beta", [0.0, 0.5])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_bf16_gradient(case, beta):
    name, N, d, V, dtype, logits = case
    log(f"[bf16 gradient] {name} N={N} d={d} V={V} beta={beta}")
    g = torch.Generator(device=dev()).manual_seed(12)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16

    def rand(shape, std, t=dt):
        return (torch.randn(shape, generator=g, device=dev()) * std).to(t)

    H, W, Z = rand((N, d), 1.0), rand((d, V), 0.02), rand((N, V), 1.0)
    y = torch.randint(0, V, (N,), generator=g, device=dev(), dtype=torch.int32)
    y[1::7] = -100
    res = bom.bom_residual(Z, y)
    q = rand((V,), 0.01, torch.float32)
    dW0 = rand((d, V + 1), 1e-3, torch.bfloat16)
    kw = dict(s=res["s"], lam=0.5, want_db=True, dW_beta=beta, row_lse=res["row_lse"] if logits else None)
    third = Z if logits else res["R"]
    a = dW0.float()
    f = bom.bom_head_vjp(H, W, third, y, q, res["n_valid"], dW=a[:, :V], **kw)
    b = dW0.clone()
    h = bom.bom_head_vjp(H, W, third, y, q, res["n_valid"], dW=b[:, :V], **kw)
    # the same fp32 sums, rounded once: equal to the rounded fp32 result
    assert torch.equal(b[:, :V], a[:, :V].to(torch.bfloat16)) and torch.equal(b[:, V], dW0[:, V])
    assert torch.equal(h["db"], f["db"].to(torch.bfloat16)) and torch.equal(h["dH"], f["dH"])
