"""Steps that read the numerator twice, around the sizes at which its last part stays in the memory-side cache."""
import pytest
import torch

from paper_2609_36738_amd import bom
from tests.gpu_util import dev, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs an MI355X")]

KEEP = 1 << 26   # fp32 elements of the numerator that stay cached (256 MB)


# name, P, state, layout, split numerator
CASES = [("all_kept", KEEP - 3, "f32", "dense", False), ("some_streamed", KEEP + 8 * 2048 * 256 * 4 + 5, "f32", "dense", False),
         ("split", KEEP // 2 + 4099, "f32", "dense", True), ("bf16", 2 * KEEP + 8 * 2048 * 256 + 9, "bf16", "dense", False),
         ("rows_kept", KEEP - 4, "f32", "factored", False), ("rows_streamed", KEEP + 4096 * 70 + 4, "f32", "factored", False),
         ("rows_split", KEEP // 2 + 4096 * 65 + 8, "f32", "factored", True)]

# the step's buffers all cached (up to 200 MB) and just past it
ALL = 200 << 20
CASES += [("cached", ALL // 12, "f32", "dense", False), ("past_cached", ALL // 12 + 1, "f32", "dense", False),
          ("cached_split", ALL // 16, "f32", "dense", True), ("past_cached_split", ALL // 16 + 4, "f32", "dense", True),
          ("cached_bf16", ALL // 6, "bf16", "dense", False), ("past_cached_bf16", ALL // 6 + 8, "bf16", "dense", False),
          ("rows_cached", ALL // 8, "f32", "factored", False), ("rows_past_cached", ALL // 8 + 4, "f32", "factored", False)]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_numerator_read_twice(case):
    name, P, state, layout, split = case
    log(f"[update order] {name} P={P}")
    g = torch.Generator(device=dev()).manual_seed(15)
    dt = torch.float32 if state == "f32" else torch.bfloat16
    theta = torch.randn(P, generator=g, device=dev()).to(dt)
    u = (torch.randn(P, generator=g, device=dev()) * 1e-3).to(dt)
    h = (torch.randn(P, generator=g, device=dev()) * 1e-3).to(dt) if split else None
    fac = layout == "factored"
    rows, C = -(-P // 4096), 4096
    blocks = -(-rows // 4096)
    v = torch.zeros(rows if fac else P, device=dev(), dtype=dt)
    v_col = torch.zeros(blocks * C, device=dev()) if fac else None
    cfg = bom.make_update_cfg(lr=1e-3, beta2=0.999, eps=1e-8, t=1, lam=0.5, factored=fac, clip_norm=1.0, state_dtype=dt)
    want = theta.double()
    bom.bom_update(theta, v, u, cfg, v_col=v_col, h=h, weight_decay=0.1)
    up = (0.5 * u.double() + 0.5 * h.double()) if split else u.double()
    up *= min(1.0, 1.0 / (float(up.norm()) + 1e-6))
    want *= 1 - 1e-4
    w2 = 1 - float(torch.tensor(0.999))   # 1 - beta2 for beta2 held in fp32: 1.3e-5 of it off 0.001
    rnd = 2.0 ** -8 if state == "bf16" else 2.0 ** -22   # rounding of the stored value
    if not fac:
        ref_v = w2 * up * up
        assert bool(((v.double() - ref_v).abs() <= ref_v * 1e-5 + ref_v * rnd + 1e-30).all())
        want -= 1e-3 * up / (up.abs() + 1e-8)
    else:
        sq = torch.zeros(rows * C, dtype=torch.float64, device=dev())
        sq[:P] = up * up
        for b in range(blocks):
            s = sq[b * C * C:(b + 1) * C * C].view(-1, C)
            r, c = s.sum(1), s.sum(0)
            # fp32 sums of up to 4096 non-negative squares in groups: below 64 roundings each way
            assert bool(((v[b * 4096:b * 4096 + len(r)].double() - w2 * r).abs() <= w2 * r * 1e-5).all())
            assert bool(((v_col[b * C:(b + 1) * C].double() - w2 * c).abs() <= w2 * c * 1e-5).all())
            lo, hi = b * C * C, min((b + 1) * C * C, P)
            want[lo:hi] -= 1e-3 * up[lo:hi] / ((torch.outer(r, c) / r.sum()).view(-1)[:hi - lo].sqrt() + 1e-8)
    # the step is at most a few lr in size; its own error (eps beside |u'| ~ 1e-7 in fp32) is below 1e-5 of it
    assert bool(((theta.double() - want).abs() <= want.abs() * rnd + 1e-3 * 1e-4).all())
