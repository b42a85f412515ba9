"""Down-projection of small batches: the column and wavefront splits at the edges of their ranges (few experts for
many wavefronts, one expert group or several, narrow and wide experts, weights below and above the sizes
from which they take 64 columns)."""
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


# (d, E, m, gated, weight format, tokens)
CASES = [(256, 15, 24, False, "native", (17, 64)), (256, 16, 64, True, "native", (33, 49)),
         (768, 47, 128, False, "native", (32, 48, 50, 64)), (1024, 300, 32, False, "native", (18, 47, 64)),
         (256, 31, 128, False, "e4m3", (20, 40, 64)), (2048, 64, 24, True, "e4m3", (31, 63)),
         (2048, 192, 64, True, "e4m3", (17, 33, 64)), (2048, 193, 64, True, "e4m3", (17, 33, 64)),
         # column counts that do not divide the workgroups of a chip; bf16 weights above the size for 64 columns
         (1280, 140, 48, False, "native", (20, 40, 60)), (3072, 50, 24, True, "native", (17, 33, 49)),
         (2048, 1220, 24, False, "native", (18, 47, 64))]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c[:5]))
def test_small_down_splits(B, oracle, case):
    import torch
    d, E, m, gated, fmt, tokens = case
    for T in tokens:
        print(f"small down {case[:5]} T={T}", flush=True)
        cfg = wl.Config("down", T, d, E, m, 64, gated, "gelu_tanh" if gated else "gelu_erf", "bf16", (0.4,),
                        ffn_bias=not gated, router_bias=False)
        layer = wl.make_layer(cfg, T)
        if fmt == "e4m3":
            layer = wl.quantize_experts_e4m3(layer)
        L, x = B.Layer(layer, cfg.dtype), wl.make_input(cfg, T)
        xd = B.to_device(x, cfg.dtype)
        y, ex = B.dmoe_forward(L, xd, 0.4, want_mask=True)
        torch.cuda.synchronize()
        mask = B.mask_bits_to_bool(ex["mask_bits"], E)
        assert tokenwise_rel_err(B.from_device(y, cfg.dtype), oracle_ffn(oracle, layer, x, mask)) <= TOL["bf16"]
        # experts that nobody selected at either end and between, and a token without any
        mask = wl.bernoulli_mask(T, E, 0.2, seed=T)
        mask[:, : E // 4] = mask[:, -1:] = mask[T // 2] = 0
        offs, lst = lists_from_mask(mask, shuffle_seed=1)
        y = B.dmoe_expert_ffn(L, xd, torch.from_numpy(offs).cuda(),
                              torch.from_numpy(np.concatenate([lst, np.zeros(1, np.int32)])).cuda())
        torch.cuda.synchronize()
        assert tokenwise_rel_err(B.from_device(y, cfg.dtype), oracle_ffn(oracle, layer, x, mask)) <= TOL["bf16"]
