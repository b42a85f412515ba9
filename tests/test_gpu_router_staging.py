"""Staging of x in the router: rows of 64, 32 and 16 tokens per workgroup, one chunk, whole chunks and a shorter last one,
and both sides of the rules between large chunks and four workgroups per CU (256 groups of 64 tokens, 512 of the router alone) and
between loads to LDS and to registers (256 workgroups of 32 tokens; the router alone)."""
import numpy as np
import pytest

from helpers import TOL, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,E,d_h,T", [(256, 128, 128, 33), (768, 128, 128, 1000), (1280, 100, 64, 9000), (768, 512, 128, 1300), (2304, 40, 128, 3000),
                                       (768, 128, 128, 16384), (768, 128, 128, 16385), (256, 128, 64, 16449), (768, 300, 128, 16500),
                                       (512, 200, 256, 17000), (256, 130, 512, 7000),
                                       (768, 128, 128, 8192), (768, 128, 128, 8193), (1280, 100, 64, 11001),
                                       # the router alone: chunks of four blocks of d_h = 64 and 128, 257 workgroups of 64 tokens at d_h = 256
                                       (256, 70, 64, 32801), (256, 70, 128, 32801), (512, 40, 256, 16400)])
def test_scores_and_decisions(oracle, d, E, d_h, T):
    import torch
    from paper_2310_04361_amd import binding as B
    print(f"router staging d={d} E={E} d_h={d_h} T={T}", flush=True)
    cfg = wl.Config("staging", T, d, E, 8, d_h, False, "relu", "bf16", (0.5,), router_bias=True)
    layer, x = wl.make_layer(cfg, d_h), wl.make_input(cfg, T)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    tau = float(np.float32(0.5))
    _, ex = B.dmoe_forward(L, xd, tau, want_scores=True, want_mask=True)
    alone = B.dmoe_router(L, xd)
    torch.cuda.synchronize()
    assert torch.equal(ex["scores"], alone)
    s = alone.cpu().numpy()
    mask, _ = oracle.select(s.astype(np.float64), tau)
    assert np.array_equal(B.mask_bits_to_bool(ex["mask_bits"], E), mask)
    idx = np.unique(np.concatenate([np.arange(min(T, 70)), np.random.default_rng(T).choice(T, 200), np.arange(max(0, T - 70), T)]))
    ref = oracle.router(x[idx], layer["r_w1"], layer["r_b1"], layer["r_w2"], layer["r_b2"])
    assert tokenwise_rel_err(s[idx], ref) <= TOL[cfg.dtype]
