"""The one-launch fp32 layer at the edges of its variants: rows that end inside, at and just beyond a
register column, more experts than one mask word, neuron counts that leave part of a wavefront's rows
empty, a single expert, and the last widths that fit (16 d + 2 E + d_h <= 16384, 16 d + E without the gate) with the
first that take the kernels for wide layers instead, for the whole layer and for its experts alone."""
import numpy as np
import pytest

from helpers import TOL, lists_from_mask, oracle_ffn, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,m,d_h,gated,tau", [
    (1, 1, 1, 1, 1, False, 0.5), (5, 63, 16, 16, 33, True, 0.5), (128, 64, 16, 16, 32, False, 0.5),
    (17, 65, 65, 3, 64, False, 0.7), (9, 128, 64, 7, 65, True, 0.3), (9, 129, 63, 7, 130, False, 0.0),
    (4, 256, 130, 5, 16, True, 1.0), (4, 257, 20, 33, 32, False, 0.3), (3, 512, 9, 70, 40, True, 0.2),
    (3, 513, 300, 2, 24, False, 0.6), (2, 960, 12, 9, 48, False, 0.0), (2, 1025, 6, 11, 20, True, 0.4),
    (2, 1020, 16, 9, 32, False, 0.4), (2, 1021, 16, 9, 32, True, 0.4), (2, 1023, 16, 5, 32, False, 0.4), (2, 1024, 1, 5, 32, False, 0.4),
])
def test_fp32_layer_edges(oracle, T, d, E, m, d_h, gated, tau):
    import torch
    from paper_2310_04361_amd import binding as B
    cfg = wl.Config("f32", T, d, E, m, d_h, gated, "gelu_tanh" if gated else "gelu_erf", "f32", (tau,),
                    ffn_bias=not gated, router_bias=True)
    layer, x = wl.make_layer(cfg, 5), wl.make_input(cfg, 5)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    tau32 = float(np.float32(tau))
    y, ex = B.dmoe_forward(L, xd, tau32, want_scores=True, want_mask=True, want_lists=True)
    plain, _ = B.dmoe_forward(L, xd, tau32)
    scores = B.dmoe_router(L, xd)
    torch.cuda.synchronize()
    assert torch.equal(ex["scores"], scores)  # the bits of the stand-alone router
    assert torch.equal(plain, y)              # whatever else the caller asks for
    mask, _ = oracle.select(scores.cpu().numpy().astype(np.float64), tau32)
    assert np.array_equal(B.mask_bits_to_bool(ex["mask_bits"], E), mask)
    offsets, lists = lists_from_mask(mask)
    assert np.array_equal(ex["offsets"].cpu().numpy(), offsets)
    assert np.array_equal(ex["token_lists"].cpu().numpy()[:offsets[-1]], lists)
    ref = oracle_ffn(oracle, layer, x, mask)
    # fp32 sums of up to E * m products: the bar of every fp32 test here
    assert tokenwise_rel_err(B.from_device(y, cfg.dtype), ref) <= TOL["f32"]
    keep = np.arange(T)[:, None] % 2 == np.arange(E)[None, :] % 2  # some tokens without any expert if E == 1
    offsets, lists = lists_from_mask(mask * keep, 3)
    y2 = B.dmoe_expert_ffn(L, xd, torch.from_numpy(offsets).cuda(), torch.from_numpy(np.resize(lists, max(len(lists), 1))).cuda())
    ref = oracle_ffn(oracle, layer, x, (mask * keep).astype(mask.dtype))
    assert tokenwise_rel_err(B.from_device(y2, cfg.dtype), ref) <= TOL["f32"]


def test_fp32_layer_of_more_tokens_than_one_launch_holds(oracle):
    """A workgroup of 1024 threads per token: 2^22 tokens are 2^32 threads, more than a launch can have."""
    import torch
    from paper_2310_04361_amd import binding as B
    T, d, E, m, d_h = (1 << 22) + 70, 4, 2, 1, 4
    cfg = wl.Config("f32_many", 64, d, E, m, d_h, False, "relu", "f32", (0.5,), ffn_bias=True, router_bias=True)
    layer = wl.make_layer(cfg, 3)
    L = B.Layer(layer, cfg.dtype)
    x = torch.randn((T, d), device="cuda", generator=torch.Generator(device="cuda").manual_seed(5))
    bad = torch.full_like(x, float("nan"))
    y, ex = B.dmoe_forward(L, x, 0.5, want_scores=True, want_mask=True, y=bad.clone())
    y1, _ = B.dmoe_forward(L, x, 0.5, y=bad.clone())
    yk, _ = B.dmoe_forward_topk(L, x, 1, y=bad.clone())
    assert torch.equal(y, y1)
    assert torch.equal(ex["scores"], B.dmoe_router(L, x))
    for t0 in (0, 1 << 21, 1 << 22, T - 64):  # ends of launches
        rows = slice(max(t0 - 32, 0), min(t0 + 64, T))
        xs, scores = x[rows].cpu().numpy().astype(np.float64), ex["scores"][rows].cpu().numpy().astype(np.float64)
        mask, _ = oracle.select(scores, 0.5)
        assert np.array_equal(B.mask_bits_to_bool(ex["mask_bits"][rows], E), mask)
        assert tokenwise_rel_err(B.from_device(y[rows], cfg.dtype), oracle_ffn(oracle, layer, xs, mask)) <= TOL["f32"]
        top = oracle.select_topk(scores, 1)
        assert tokenwise_rel_err(B.from_device(yk[rows], cfg.dtype), oracle_ffn(oracle, layer, xs, top)) <= TOL["f32"]
    assert torch.isfinite(y).all() and torch.isfinite(yk).all()
