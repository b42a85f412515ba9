"""The waits inside the small-batch forward: workgroups that give up on what others compute
(dmoe_small_give_up) leave the same results, bit for bit, as those that see it, also where only some of
them give up and on a workspace that holds NaN everywhere; and calls on several streams, each with a
workspace of its own, do not see each other's exchange."""
import numpy as np
import pytest

from helpers import TOL, oracle_ffn, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2310_04361_amd import binding
    binding.lib()
    return binding


def make(B, shape, T, fmt, n=1):
    d, E, m, dh, gated = shape
    cfg = wl.Config("small", T, d, E, m, dh, gated, "gelu_tanh" if gated else "gelu_erf", "bf16", (0.4,),
                    ffn_bias=not gated, router_bias=True)
    layers = [wl.make_layer(cfg, T + i) for i in range(n)]
    if fmt == "e4m3":
        layers = [wl.quantize_experts_e4m3(l) for l in layers]
    return cfg, layers, [B.Layer(l, cfg.dtype) for l in layers], wl.make_input(cfg, T)


# (d, E, m, d_h, gated), weight format, tokens, tau: few touched experts (the up-projection waits for the
# gate), the widest router with the most experts of the fused gate, several items per workgroup; and a
# layer so small that nobody waits for the gate
CASES = [((512, 512, 64, 256, True), "native", 1, 0.6), ((512, 512, 64, 256, True), "native", 16, 0.95),
         ((512, 512, 64, 256, True), "e4m3", 33, 0.95), ((768, 1024, 24, 512, False), "native", 2, 0.7),
         ((768, 1024, 24, 512, False), "native", 50, 0.95), ((1024, 130, 128, 128, False), "native", 3, 0.8),
         ((256, 33, 24, 64, False), "native", 16, 0.5)]


@pytest.mark.parametrize("shape,fmt,T,tau", CASES)
def test_give_up(B, oracle, shape, fmt, T, tau):
    import torch
    print(f"give up {shape} {fmt} T={T} tau={tau}", flush=True)
    cfg, (layer,), (L,), x = make(B, shape, T, fmt)
    xd, tau = B.to_device(x, cfg.dtype), float(np.float32(tau))
    forward = lambda: B.dmoe_forward(L, xd, tau, want_scores=True, want_mask=True)
    y, ex = forward()
    mask, _ = oracle.select(ex["scores"].cpu().numpy().astype(np.float64), tau)
    assert np.array_equal(B.mask_bits_to_bool(ex["mask_bits"], L.E), mask)
    assert tokenwise_rel_err(B.from_device(y, cfg.dtype), oracle_ffn(oracle, layer, x, mask)) <= TOL["bf16"]
    try:
        for every in (1, 2, 3, 8):
            print(f"  every {every}", flush=True)
            L.workspace(T).fill_(255)
            B.check(B.lib().dmoe_small_give_up(every))
            y2, ex2 = forward()
            torch.cuda.synchronize()
            assert torch.equal(ex2["scores"], ex["scores"]) and torch.equal(ex2["mask_bits"], ex["mask_bits"])
            assert torch.equal(y2, y)
    finally:
        B.check(B.lib().dmoe_small_give_up(0))
    L.workspace(T).fill_(255)
    assert torch.equal(forward()[0], y)


def test_give_up_in_a_group(B):
    import torch
    cfg, _, Ls, x = make(B, (768, 512, 24, 128, False), 16, "native", 3)
    xd, taus = B.to_device(x, cfg.dtype), [float(np.float32(t)) for t in (0.95, 0.0, 0.9)]
    ys = B.dmoe_forward_group(Ls, xd, taus)
    try:
        for every in (1, 3, 8):
            for ws in B._group_ws.values():
                ws.fill_(255)
            B.check(B.lib().dmoe_small_give_up(every))
            ys2 = B.dmoe_forward_group(Ls, xd, taus)
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(ys, ys2))
    finally:
        B.check(B.lib().dmoe_small_give_up(0))


@pytest.mark.parametrize("shape,T,tau", [((512, 130, 64, 256, True), 16, 0.5), ((768, 512, 24, 128, False), 1, 0.7),
                                         ((768, 512, 24, 128, False), 40, 0.95)])
def test_streams(B, shape, T, tau):
    import torch
    print(f"streams {shape} T={T} tau={tau}", flush=True)
    cfg, _, Ls, x = make(B, shape, T, "native", 3)
    rng, tau = np.random.default_rng(T), float(np.float32(tau))
    xs = [B.to_device(x[rng.permutation(T)] * np.float32(2.0 ** (i % 3)), cfg.dtype) for i in range(12)]
    want = [[B.dmoe_forward(L, xd, tau)[0] for xd in xs] for L in Ls]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in Ls]
    got = [[torch.empty_like(xd) for xd in xs] for _ in Ls]
    for L in Ls:
        L.workspace(T)                      # (one per layer, so one per stream)
    torch.cuda.synchronize()
    for i, xd in enumerate(xs):
        for L, s, ys in zip(Ls, streams, got):
            with torch.cuda.stream(s):
                B.dmoe_forward(L, xd, tau, y=ys[i])
    torch.cuda.synchronize()
    for ys, ws in zip(got, want):
        assert all(torch.equal(a, b) for a, b in zip(ys, ws))
