"""Wide up-projection from lists: experts whose rows end at the edges of wavefronts (64 rows) and items (256), an expert that
nobody selects, the shortest walk over K (d = 256), and the same bits from a cold start and a warm one."""
import numpy as np
import pytest

from helpers import TOL, lists_from_mask, oracle_ffn, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu

COUNTS = [1, 0, 63, 64, 65, 128, 192, 255, 256, 257, 512, 513, 1025, 3137]


@pytest.mark.parametrize("d,m,gated", [(256, 64, True), (256, 128, False), (768, 57, True), (768, 100, False), (1024, 64, True)])
def test_rows_of_experts(oracle, d, m, gated):
    import torch
    from paper_2310_04361_amd import binding as B
    T, E = 3137, len(COUNTS)  # (more tokens than the kernels without lists take)
    print(f"wide up d={d} m={m} gated={gated}", flush=True)
    cfg = wl.Config("wide", T, d, E, m, 64, gated, "gelu_tanh" if gated else "gelu_erf", "bf16", (0.5,), ffn_bias=not gated)
    layer, x = wl.make_layer(cfg, d), wl.make_input(cfg, m)
    rng = np.random.default_rng(d + m)
    mask = np.zeros((T, E), np.uint8)
    for e, n in enumerate(COUNTS):
        mask[rng.choice(T, n, replace=False), e] = 1
    offsets, lists = lists_from_mask(mask)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    od, ld = torch.from_numpy(offsets).cuda(), torch.from_numpy(lists).cuda()
    L.workspace(T).fill_(0xff)
    flush = torch.empty(512 << 20, dtype=torch.uint8, device="cuda")  # more than the caches hold
    flush.fill_(1)
    y = B.dmoe_expert_ffn(L, xd, od, ld)
    again = B.dmoe_expert_ffn(L, xd, od, ld)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), again.view(torch.int16))
    assert tokenwise_rel_err(B.from_device(y, cfg.dtype), oracle_ffn(oracle, layer, x, mask)) <= TOL["bf16"]
