"""Routers of 513 to 2048 experts with scores, gate and counts in one launch: the scores are those of the stand-alone router, the
decisions the oracle's on them, and what follows from the counts (lists, outputs) is right, at the edges of tiles of 16
experts, words of 64, workgroups of 16 tokens and of the rule (2300, 2600 and 1500 tokens for up to 1024, 1792 and 2048 experts, at most 191
groups of 64 tokens)."""
import numpy as np
import pytest

from helpers import TOL, oracle_ffn, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,E,d_h,T,one", [
    (1536, 513, 512, 2300, True), (1536, 527, 512, 2309, True), (3328, 800, 256, 2320, True), (1280, 1024, 512, 2335, True), (1280, 1024, 512, 2299, False),
    (1280, 1025, 512, 2647, True), (1280, 1025, 512, 2599, False), (512, 1792, 512, 2600, True), (512, 1793, 512, 1501, True), (512, 1999, 512, 1501, True),
    (256, 2048, 512, 2100, True), (256, 2048, 512, 1500, True), (256, 2048, 512, 1499, False), (2048, 2048, 256, 3100, True),
    (1536, 530, 512, 12224, True), (1536, 530, 512, 12225, False), (256, 2049, 512, 2600, False)])
def test_decisions(oracle, d, E, d_h, T, one):
    import torch
    from paper_2310_04361_amd import binding as B
    print(f"scores and gate d={d} E={E} d_h={d_h} T={T}", flush=True)
    cfg = wl.Config("gate", T, d, E, 1, d_h, False, "gelu_erf", "bf16", (0.5,), ffn_bias=True, router_bias=E % 2 == 1)
    layer, x = wl.make_layer(cfg, E), wl.make_input(cfg, T)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    alone = B.dmoe_router(L, xd)
    for tau in (0.0, 0.6, 1.0):
        tau = float(np.float32(tau))
        y, ex = B.dmoe_forward(L, xd, tau, want_scores=True, want_mask=True, want_lists=True)
        L._ws.fill_(0xff)
        B.timing(True)
        bare, _ = B.dmoe_forward(L, xd, tau)
        launches = B.timing_read()
        B.timing(False)
        assert launches["router"][0] == 1 and launches["mask_count"][0] == (0 if one else 1), launches  # the gate with the scores or after them
        assert torch.equal(ex["scores"], alone)
        mask, _ = oracle.select(ex["scores"].cpu().numpy().astype(np.float64), tau)
        assert np.array_equal(B.mask_bits_to_bool(ex["mask_bits"], E), mask)
        offsets, lists = ex["offsets"].cpu().numpy(), ex["token_lists"].cpu().numpy()
        assert np.array_equal(offsets, np.concatenate([[0], mask.sum(axis=0).cumsum()]))
        assert np.array_equal(lists[:offsets[-1]], np.nonzero(mask.T)[1])
        assert torch.equal(y.view(torch.int16), bare.view(torch.int16))
        idx = np.unique([0, 15, T // 2, T - 1])
        assert tokenwise_rel_err(B.from_device(y, cfg.dtype)[idx], oracle_ffn(oracle, layer, x[idx], mask[idx])) <= TOL["bf16"]
