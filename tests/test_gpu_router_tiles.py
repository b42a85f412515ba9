"""The router of small and medium batches in two launches (hidden rows tile by tile, then scores and gate) at the
edges of its tiles: token counts around 16, 32 and 64, both tile sizes and the first batch beyond them, expert
counts off a 16-expert tile, a mask word and the kernels' register variants, one to eight K blocks per wavefront."""
import numpy as np
import pytest

from helpers import TOL, lists_from_mask, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,d_h,bias", [
    (65, 2048, 256, 256, False), (79, 2048, 65, 128, True), (81, 1024, 129, 256, True), (127, 2048, 7, 128, False),
    (129, 512, 300, 512, True), (1023, 2048, 120, 256, True), (1025, 1024, 257, 256, False), (2049, 2048, 33, 256, False),
    (513, 2048, 512, 512, True), (97, 4096, 16, 128, False),
    (70, 2048, 1, 512, True),  # fewer H rows than hidden rows: one launch
    # tiles of 32 x 64 and tiles of tokens off a multiple of eight; the tiles of 64 x 128; the last and first batch beyond
    (2535, 2048, 40, 128, True), (1311, 1024, 70, 256, False), (4032, 512, 33, 512, True), (4033, 512, 33, 512, True),
    (6080, 1024, 20, 256, True), (6081, 1024, 20, 256, False), (1025, 2048, 600, 512, True), (4100, 1024, 1025, 512, False),
])
def test_router_tiles(oracle, T, d, E, d_h, bias):
    import torch
    from paper_2310_04361_amd import binding as B
    cfg = wl.Config("router_tiles", T, d, E, 8, d_h, True, "gelu_tanh", "bf16", (0.5,), router_bias=bias)
    print(f"router tiles T={T} d={d} E={E} d_h={d_h}", flush=True)
    layer, x = wl.make_layer(cfg, 8), wl.make_input(cfg, 8)
    L = B.Layer(layer, cfg.dtype)
    xd, tau = B.to_device(x, cfg.dtype), float(np.float32(0.6))
    y, ex = B.dmoe_forward(L, xd, tau, want_scores=True, want_mask=True, want_lists=True)
    y2, ex2 = B.dmoe_forward(L, xd, tau, want_mask=True)
    torch.cuda.synchronize()
    scores = ex["scores"].cpu().numpy().astype(np.float64)
    ref = oracle.router(x, layer["r_w1"], layer["r_b1"], layer["r_w2"], layer["r_b2"])
    assert tokenwise_rel_err(scores, ref) <= TOL["bf16"]  # the bar of every bf16 router test
    mask, _ = oracle.select(scores, tau)                  # the gate on the library's own scores: bit for bit
    assert np.array_equal(B.mask_bits_to_bool(ex["mask_bits"], E), mask)
    offsets, lists = lists_from_mask(mask)
    assert np.array_equal(ex["offsets"].cpu().numpy(), offsets)
    assert np.array_equal(ex["token_lists"].cpu().numpy()[:offsets[-1]], lists)
    assert torch.equal(ex["mask_bits"], ex2["mask_bits"]) and torch.equal(y, y2)


@pytest.mark.parametrize("T,d,E,d_h,top_k", [
    # small batches, one launch, and every tile of the hidden rows on either side of its rule (2048 wide: 32 x 32 below 160 tiles
    # of 32 x 64, 32 x 128 from 320 to 512 of them), the first batch in one launch again
    (1, 2048, 256, 256, None), (16, 2048, 256, 256, None), (64, 2048, 256, 256, None), (65, 2048, 256, 256, None),
    (333, 2048, 256, 256, None), (1248, 2048, 256, 256, None), (1249, 2048, 256, 256, None), (2528, 2048, 256, 256, None),
    (2529, 2048, 256, 256, None), (4096, 2048, 256, 256, None), (4097, 2048, 256, 256, None), (6081, 2048, 256, 256, None),
    # part of a trip of 16 K blocks: 8, 12, 20 and 36 of them
    (300, 512, 120, 512, None), (1500, 768, 120, 512, None), (2600, 1280, 65, 256, None), (700, 2304, 64, 128, None),
    # the top-k gate, and more experts than the fused gate takes
    (333, 2048, 256, 512, 9), (2000, 2048, 256, 256, 9), (1023, 2048, 600, 512, None), (2049, 2048, 1100, 512, None),
    (9, 512, 1100, 128, 5), (12, 256, 30, 64, 3), (40, 256, 1030, 32, None), (50, 768, 128, 128, None), (700, 768, 128, 128, None),
])
def test_forward_decides_by_the_scores_of_the_router(oracle, T, d, E, d_h, top_k):
    """One order of the sums in all forms of the router: the same bits from dmoe_router and dmoe_forward."""
    import torch
    from paper_2310_04361_amd import binding as B
    cfg = wl.Config("router_bits", T, d, E, 8, d_h, True, "gelu_tanh", "bf16", (0.5,), router_bias=True)
    print(f"router bits T={T} d={d} E={E} d_h={d_h} top_k={top_k}", flush=True)
    layer, x = wl.make_layer(cfg, 4), wl.make_input(cfg, 4)
    L, xd, tau = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype), float(np.float32(0.5))
    _, ex = B.dmoe_forward(L, xd, tau, want_scores=True, want_mask=True, top_k=top_k)
    scores = B.dmoe_router(L, xd)
    sel = B.dmoe_select(scores, tau, top_k=top_k)
    torch.cuda.synchronize()
    assert torch.equal(ex["scores"], scores)
    assert torch.equal(ex["mask_bits"], sel["mask_bits"])
