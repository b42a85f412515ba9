"""Small batches whose up-projections work from the gate's token sets: the same bits as with lists (which a caller gets by
asking for them), at the edges of rows of 16 tokens, groups of 64, work items of 64, 128 and 256 rows and of the rows that a
lane holds."""
import numpy as np
import pytest

from helpers import TOL, lists_from_mask, oracle_ffn, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2310_04361_amd import binding
    binding.lib()
    return binding


# one of each up-projection: one weight tile (plain, gated; more items than the chip holds at once), 32-neuron rows (plain, gated),
# 64-neuron rows, 256-row items (gated, plain)
SHAPES = {
    "tile": dict(d=256, E=70, m=6, gated=False), "tile_gated": dict(d=256, E=1100, m=8, gated=True),
    "rows32": dict(d=512, E=33, m=24, gated=False), "rows32_gated": dict(d=256, E=17, m=30, gated=True),
    "rows64": dict(d=256, E=20, m=40, gated=False), "wide_gated": dict(d=512, E=40, m=60, gated=True),
    "wide": dict(d=768, E=12, m=128, gated=False),
}
TOKENS = [17, 63, 64, 65, 127, 129, 255, 257, 1023, 1024, 1025, 1039, 2047, 2049, 3072]


def layer_of(B, name, T, fmt="native"):
    s = SHAPES[name]
    cfg = wl.Config("sets", T, s["d"], s["E"], s["m"], 64, s["gated"], "gelu_tanh" if s["gated"] else "gelu_erf", "bf16", (0.4,),
                    ffn_bias=not s["gated"], router_bias=True)
    layer, x = wl.make_layer(cfg, T), wl.make_input(cfg, T + 1)
    if fmt != "native":
        layer = wl.quantize_experts_e4m3(layer)
        layer[fmt] = True
    return cfg, layer, x


CASES = [(name, "native", T) for name in sorted(SHAPES) for T in TOKENS]
CASES += [(name, fmt, T) for name in ("wide", "wide_gated") for fmt in ("x8", "a8") for T in (17, 128, 129, 257, 1024, 1040)]


@pytest.mark.parametrize("name,fmt,T", CASES)
def test_sets_and_lists(B, name, fmt, T):
    import torch
    print(f"token sets {name} {fmt} T={T}", flush=True)
    cfg, layer, x = layer_of(B, name, T, fmt)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    for tau in (0.0, 0.4, 1.0):  # every expert, some, one or two
        tau = float(np.float32(tau))
        want, _ = B.dmoe_forward(L, xd, tau, want_lists=True)
        L._ws.fill_(0xff)  # (nothing may rest on what an earlier call left)
        got, _ = B.dmoe_forward(L, xd, tau)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), tau
    want, _ = B.dmoe_forward(L, xd, 0.0, top_k=3, want_lists=True)
    got, _ = B.dmoe_forward(L, xd, 0.0, top_k=3)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("name", ["tile", "tile_gated", "rows32", "rows64", "wide_gated", "wide"])
@pytest.mark.parametrize("T", [17, 130, 1030])
def test_given_lists(B, oracle, name, T):
    """Decisions from outside: an expert that nobody selects, one that all do, one with the last token only."""
    import torch
    print(f"token sets of given lists {name} T={T}", flush=True)
    cfg, layer, x = layer_of(B, name, T)
    L = B.Layer(layer, cfg.dtype)
    mask = (np.random.default_rng(T).random((T, cfg.E)) < 0.3).astype(np.uint8)
    mask[:, 0], mask[:, 1], mask[:, 2] = 0, 1, 0
    mask[T - 1, 2] = 1
    offsets, lists = lists_from_mask(mask, shuffle_seed=1)
    y = B.dmoe_expert_ffn(L, B.to_device(x, cfg.dtype), torch.from_numpy(offsets).cuda(), torch.from_numpy(lists).cuda())
    torch.cuda.synchronize()
    assert tokenwise_rel_err(B.from_device(y, cfg.dtype), oracle_ffn(oracle, layer, x, mask)) <= TOL["bf16"]
