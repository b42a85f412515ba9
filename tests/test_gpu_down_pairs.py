"""The pair-proportional down-projection at sizes whose H is beyond the 32-bit offsets of the other kernels, for every
length of an H row (one piece, two, 32, 64 and 128 neurons): densities on both sides of a tile of 32 rows, a ragged
last chunk, and an expert whose hidden row holds an infinity, which reaches the tokens that selected it and no other."""
import numpy as np
import pytest

from helpers import TOL, oracle_ffn, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,m,p", [(8193, 4096, 7, 0.004), (8193, 4096, 8, 0.3), (33000, 1024, 16, 0.01), (33000, 1024, 13, 0.3),
                                     (8193, 4096, 24, 0.02), (33000, 512, 50, 0.1), (33000, 256, 128, 0.05)])
def test_pair_kernel_rows(oracle, T, E, m, p):
    import torch
    from paper_2310_04361_amd import binding as B
    cfg = wl.Config("pairs", T, 256, E, m, 32, False, "gelu_erf", "bf16", (0.5,), ffn_bias=True)
    print(f"pair kernel T={T} E={E} m={m} p={p}", flush=True)
    layer, x = wl.make_layer(cfg, 7), wl.make_input(cfg, 7)
    layer["b_up"][5, 0] = np.inf
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    gen = torch.Generator(device="cuda").manual_seed(9)
    keep = torch.rand((E, T), device="cuda", generator=gen) < p
    keep[5], keep[:, 11] = False, False
    keep[5, 100:T:1000] = True
    lists = keep.nonzero()[:, 1].to(torch.int32).contiguous()
    offsets = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), keep.sum(dim=1).cumsum(0)]).to(torch.int32)
    B.timing(True)
    y = B.dmoe_expert_ffn(L, xd, offsets, lists)
    torch.cuda.synchronize()
    launched = {k: n for k, (n, _) in B.timing_read().items() if n}
    B.timing(False)
    assert launched.get("expert_down_sparse") == 1 and "expert_down" not in launched
    idx = np.unique(np.concatenate([np.arange(0, T, T // 60), [0, 11, 100, 127, 128, 1100, T - 2, T - 1]]))
    at = torch.from_numpy(idx).cuda()
    mask = keep[:, at].T.cpu().numpy().astype(np.uint8)
    got, ref = B.from_device(y[at], cfg.dtype), oracle_ffn(oracle, layer, x[idx], mask)
    inf = mask[:, 5] == 1
    assert inf.any() and np.array_equal(np.isinf(ref).any(axis=1), inf)
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    assert tokenwise_rel_err(got[~inf], ref[~inf]) <= TOL["bf16"]
    assert np.array_equal(got[idx == 11][0], layer["b_down"])
    assert torch.isfinite(y[~keep[5]]).all()
