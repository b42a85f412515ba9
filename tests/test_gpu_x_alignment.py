"""x at addresses that are not multiples of 16 bytes: the kernels whose loads go straight to LDS take it through registers, with
the same bits."""
import numpy as np
import pytest

from helpers import lists_from_mask
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("skip", [1, 2, 4])  # elements: 2, 4 and 8 bytes
@pytest.mark.parametrize("d,E,m,d_h,T", [(768, 24, 128, 128, 3200), (768, 128, 24, 128, 1000), (512, 40, 100, 128, 16500), (256, 70, 90, 64, 130),
                                         (2048, 600, 2, 512, 1600),
                                         # 32 and 64 tokens a workgroup, a last chunk of four K blocks; hidden rows in slices of 128
                                         (1280, 100, 8, 128, 7000), (1024, 60, 8, 128, 12300), (2048, 600, 2, 512, 4100)])
def test_unaligned_x(d, E, m, d_h, T, skip):
    import torch
    from paper_2310_04361_amd import binding as B
    print(f"x alignment d={d} E={E} m={m} T={T} skip={skip}", flush=True)
    cfg = wl.Config("align", T, d, E, m, d_h, False, "gelu_erf", "bf16", (0.5,), ffn_bias=True)
    layer, x = wl.make_layer(cfg, m), wl.make_input(cfg, T)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    buf = torch.zeros(T * d + 16, dtype=xd.dtype, device="cuda")
    away = buf[skip:skip + T * d].view(T, d)
    away.copy_(xd)
    assert away.data_ptr() % 16 != 0
    tau = float(np.float32(0.5))
    for lists in (False, True):
        want, _ = B.dmoe_forward(L, xd, tau, want_lists=lists)
        got, _ = B.dmoe_forward(L, away, tau, want_lists=lists)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    mask = wl.bernoulli_mask(T, E, 0.2, seed=3)
    offsets, token_lists = lists_from_mask(mask)
    od, ld = torch.from_numpy(offsets).cuda(), torch.from_numpy(token_lists).cuda()
    want, got = B.dmoe_expert_ffn(L, xd, od, ld), B.dmoe_expert_ffn(L, away, od, ld)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
