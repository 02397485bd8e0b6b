"""Sizes at which the rules that choose a kernel, and the kernels' tiles, have their edges."""
import numpy as np
import pytest
import torch

from paper_2503_05066_amd import capmoe

pytestmark = pytest.mark.gpu


# ------------------------------------------------------------------------------------------------
# combine: rows of less than a wave's pieces, a piece more, two pieces a lane; none, all and more than 64 slots taken
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("n,d,slots,dtype", [
    (1, 8, 1, "bf16"), (3, 512, 8, "bf16"), (5, 520, 9, "bf16"), (16384, 64, 2, "bf16"), (16385, 64, 2, "bf16"),
    (16385, 504, 3, "bf16"), (16384, 1024, 5, "bf16"), (16383, 1032, 5, "bf16"), (700, 1024, 130, "bf16"),
    (2, 4, 2, "f32"), (129, 260, 17, "f32"), (16385, 252, 3, "f32"), (16384, 512, 2, "f32"), (40, 256, 70, "f32")])
def test_combine(n, d, slots, dtype):
    if slots <= 64:
        desc = capmoe.make_desc(n, d, 64, slots, 128, 1, capmoe.MODE_NONE, capmoe.SCOPE_LOCAL, 1.0,
                                capmoe.DTYPE_BF16 if dtype == "bf16" else capmoe.DTYPE_F32)
    else:  # more slots than one wave has lanes: a device's experts beside the listed ones
        desc = capmoe.make_desc(n, d, 2 * (slots - 4), 4, 128, 2, capmoe.MODE_EXPANDED_DROP, capmoe.SCOPE_LOCAL, 1.0,
                                capmoe.DTYPE_BF16 if dtype == "bf16" else capmoe.DTYPE_F32)
    assert capmoe.moe_query(desc)[1] == slots
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    rows = 3 * n + 1
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    yp = torch.randn((rows, d), generator=gen, device="cuda").to(act)
    weight = torch.rand(rows, generator=gen, device="cuda")
    pair_row = torch.randint(0, rows, (n, slots), generator=gen, device="cuda", dtype=torch.int32)
    share = torch.rand((n, 1), generator=gen, device="cuda")
    share[: n // 4], share[n - n // 4:] = 0.0, 1.0        # tokens without a row, tokens whose slots all hold one
    pair_row[torch.rand((n, slots), generator=gen, device="cuda") >= share] = -1
    y = torch.full((n, d), 7.0, dtype=act, device="cuda")
    capmoe.moe_combine(desc, yp, weight, pair_row, y)
    torch.cuda.synchronize()
    ref = torch.zeros((n, d), dtype=torch.float64, device="cuda")
    mass = torch.zeros((n, d), dtype=torch.float64, device="cuda")
    for s in range(slots):
        r = pair_row[:, s].long()
        w = torch.where(r >= 0, weight[r.clamp(min=0)], 0.0).double()[:, None]
        v = w * yp[r.clamp(min=0)].double()
        ref += v
        mass += v.abs()
    # one fp32 rounding per slot (half a unit of the running sum, which the mass bounds), one rounding to bf16
    bound = slots * 2.0 ** -24 * mass + (2.0 ** -8 * ref.abs() if dtype == "bf16" else 0.0)
    assert bool(((y.double() - ref).abs() <= bound).all())
    assert bool((y[(pair_row < 0).all(dim=1)] == 0).all())
