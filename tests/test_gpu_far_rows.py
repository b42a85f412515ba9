"""Gathers of x beyond 2 GiB: the narrow up-projections switch from 32-bit row offsets to 64-bit addresses.  Tokens on
both sides of the 2 GiB mark and a batch just below it, for the kernels of tiles of 32 neurons, of one-tile
experts and of wide ones, plain and gated."""
import numpy as np
import pytest

from helpers import TOL, lists_from_mask, oracle_ffn, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,gated,T", [(24, False, 524288 + 70), (8, True, 524288 + 70), (6, False, 524288 + 70),
                                       (20, True, 524288 + 70), (24, False, 524287), (60, True, 524288 + 70),
                                       (128, False, 524288 + 70), (64, True, 524287)])
def test_far_rows(oracle, m, gated, T):
    import torch
    from paper_2310_04361_amd import binding as B
    d, E = 2048, 2
    cfg = wl.Config("far", 8, d, E, m, 64, gated, "gelu_tanh" if gated else "gelu_erf", "bf16", (0.5,), ffn_bias=not gated)
    print(f"far rows m={m} gated={gated} T={T}", flush=True)
    layer = wl.make_layer(cfg, 2)
    L = B.Layer(layer, cfg.dtype)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((T, d), device="cuda", generator=gen, dtype=torch.bfloat16)
    # expert 0: every third token; expert 1: the last 200
    lists = torch.cat([torch.arange(0, T, 3), torch.arange(T - 200, T)]).to(torch.int32)
    n0 = (T + 2) // 3
    offsets = torch.tensor([0, n0, n0 + 200], dtype=torch.int32)
    y = B.dmoe_expert_ffn(L, x, offsets.cuda(), lists.cuda())
    torch.cuda.synchronize()
    idx = np.array([0, 1, 3, 262143, 524283, 524286, T - 200, T - 3, T - 2, T - 1])
    mask = np.zeros((len(idx), E), np.uint8)
    mask[:, 0], mask[:, 1] = idx % 3 == 0, idx >= T - 200
    at = torch.from_numpy(idx).cuda()
    ref = oracle_ffn(oracle, layer, B.from_device(x[at], "bf16"), mask)
    got = B.from_device(y[at], "bf16")
    keep = np.abs(ref).max(axis=1) > 0
    assert (got[~keep] == 0).all()
    assert tokenwise_rel_err(got[keep], ref[keep]) <= TOL["bf16"]


@pytest.mark.parametrize("T,E,m", [(131, 840, 32), (70, 840, 27), (131, 840, 24), (131, 780, 32)])
def test_narrow_gated_experts_with_a_large_item_table(oracle, T, E, m):
    """More than about 820 gated experts of 25 to 32 leave LDS for one workgroup per CU and take the weights by address;
    fewer and narrower ones by a buffer that skips padding rows."""
    import torch
    from paper_2310_04361_amd import binding as B
    cfg = wl.Config("items", T, 256, E, m, 64, True, "gelu_tanh", "bf16", (0.5,))
    print(f"item table T={T} E={E} m={m}", flush=True)
    layer, x = wl.make_layer(cfg, 3), wl.make_input(cfg, 3)
    mask = wl.bernoulli_mask(T, E, 0.3, seed=5)
    mask[:, 7] = 0
    mask[:, E - 1] = 1
    offsets, lists = lists_from_mask(mask)
    y = B.dmoe_expert_ffn(B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype), torch.from_numpy(offsets).cuda(), torch.from_numpy(lists).cuda())
    assert tokenwise_rel_err(B.from_device(y, cfg.dtype), oracle_ffn(oracle, layer, x, mask)) <= TOL["bf16"]
