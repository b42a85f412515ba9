"""Whole forwards at the token counts between a decode batch and a full prefill, where the launch
shapes change: the walk of the down-projection divided into more or fewer parts, the scan over the
token groups inside the list fill or in a kernel of its own, one to a few token groups, one to eight
windows of the up-projection.  Lists and
masks bit-exact, outputs against the oracle on every token."""
import numpy as np
import pytest

from helpers import TOL, check_fully_8bit, oracle_ffn, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2310_04361_amd import binding
    binding.lib()
    return binding


# (d, E, m, d_h, gated, weight format)
WIDE_GATED = (512, 130, 64, 128, True, "native")
NARROW = (768, 100, 24, 128, False, "native")
TINY = (256, 700, 6, 64, False, "native")
CASES = [(shape, T) for shape in (WIDE_GATED, NARROW) for T in (17, 33, 64, 65, 129, 500, 513, 1100)] + \
        [(NARROW, 2364)] + [((256, E, m, 64, g, "native"), 2950) for m, g in ((6, False), (8, True), (24, False))
                            for E in (10, 40, 80)] + \
        [(TINY, T) for T in (64, 200, 1030)] + \
        [((512, 260, 64, 64, True, "a8"), T) for T in (17, 65, 520)] + \
        [((512, E, 64, 64, True, "a8"), 300) for E in (33, 97)] + \
        [((256, 40, 128, 64, False, "a8"), 100), ((512, 130, 64, 128, True, "e4m3"), 48)]


@pytest.mark.parametrize("shape,T", CASES)
def test_small_batches(B, oracle, shape, T):
    import torch
    d, E, m, dh, gated, fmt = shape
    print(f"small batch {shape} T={T}", flush=True)
    cfg = wl.Config("small", T, d, E, m, dh, gated, "gelu_tanh" if gated else "gelu_erf", "bf16", (0.4,),
                    ffn_bias=not gated, router_bias=True)
    layer, x = wl.make_layer(cfg, T), wl.make_input(cfg, T)
    if fmt != "native":
        layer = wl.quantize_experts_e4m3(layer)
        layer["x8"] = layer["a8"] = fmt == "a8"
    L = B.Layer(layer, cfg.dtype)
    tau = float(np.float32(0.4))
    xd = B.to_device(x, cfg.dtype)
    y, ex = B.dmoe_forward(L, xd, tau, want_scores=True, want_mask=True, want_lists=True)
    y2, _ = B.dmoe_forward(L, xd, tau)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    mask, _ = oracle.select(ex["scores"].cpu().numpy().astype(np.float64), tau)
    assert np.array_equal(B.mask_bits_to_bool(ex["mask_bits"], E), mask)
    _, offsets, lists = oracle.bucket(mask)
    assert np.array_equal(ex["offsets"].cpu().numpy(), offsets)
    assert np.array_equal(ex["token_lists"].cpu().numpy()[: offsets[-1]], lists)
    got = B.from_device(y, cfg.dtype)
    if fmt == "a8":
        xq, _ = oracle.quantize_rows_e4m3(x)
        check_fully_8bit(oracle, layer, xq, mask, got, oracle_ffn(oracle, layer, xq, mask, quantize_h=True), TOL["bf16"])
    else:
        err = tokenwise_rel_err(got, oracle_ffn(oracle, layer, x, mask))
        print(f"  err={err:.3e}", flush=True)
        assert err <= TOL["bf16"]


# (d, E, m, d_h, gated, weight format), tokens: where a divided walk takes the most shares for its size, and
# the last batch that is divided
@pytest.mark.parametrize("shape,T", [((256, 17, 128, 64, False, "native"), 4781), ((256, 2016, 16, 64, False, "native"), 40),
                                     ((768, 97, 48, 64, False, "a8"), 2439), ((256, 700, 64, 64, True, "a8"), 128),
                                     ((512, 130, 64, 128, True, "native"), 8192), ((512, 130, 64, 128, True, "native"), 65)])
def test_nothing_behind_the_workspace(B, shape, T):
    import torch
    d, E, m, dh, gated, fmt = shape
    print(f"workspace {shape} T={T}", flush=True)
    cfg = wl.Config("small", T, d, E, m, dh, gated, "gelu_tanh" if gated else "gelu_erf", "bf16", (0.4,),
                    ffn_bias=not gated, router_bias=True)
    layer = wl.make_layer(cfg, T)
    if fmt != "native":
        layer = wl.quantize_experts_e4m3(layer)
        layer["x8"] = layer["a8"] = True
    L, tau = B.Layer(layer, cfg.dtype), float(np.float32(0.4))
    xd = B.to_device(wl.make_input(cfg, T), cfg.dtype)
    y = B.dmoe_forward(L, xd, tau)[0]
    need = L.workspace(T).numel()
    room = torch.full((need + (64 << 20),), 255, dtype=torch.uint8, device="cuda")
    L._ws = room[:need]
    y2 = B.dmoe_forward(L, xd, tau)[0]
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    assert bool((room[need:] == 255).all())
