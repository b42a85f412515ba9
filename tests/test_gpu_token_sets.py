"""Small batches whose up-projections work from the gate's token sets: the same bits as with lists (which a caller gets by
asking for them), at the edges of rows of 16 tokens, groups of 64, work items of 64, 128 and 256 rows and of the rows that a
lane holds.  Whether a call takes that way is seen from the launches that fill lists."""
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
# 64-neuron rows, wide experts in items of 128 rows and, where there are more than 256 of those, of 256 (gated, plain)
SHAPES = {
    "tile": dict(d=256, E=70, m=6, gated=False), "tile_gated": dict(d=256, E=1100, m=8, gated=True),
    "rows32": dict(d=512, E=33, m=24, gated=False), "rows32_gated": dict(d=256, E=17, m=30, gated=True),
    "rows64": dict(d=256, E=60, m=40, gated=False), "wide_gated": dict(d=512, E=40, m=60, gated=True),
    "wide": dict(d=512, E=24, m=128, gated=False), "wide_24": dict(d=768, E=24, m=128, gated=False), "wide_130": dict(d=256, E=130, m=100, gated=False),
    "wide_gated_210": dict(d=256, E=210, m=60, gated=True), "tile_gated_2048": dict(d=512, E=2048, m=2, gated=True),
}
TOKENS = [63, 64, 65, 127, 129, 255, 257, 1023, 1024, 1025, 1039, 2047, 2049, 3072]
# items of 256 rows: 24 experts from 1281 tokens on, 130 from 129 on, 40 from 769 on
TOKENS_OF = {"wide_24": [1280, 1281, 1379, 2561], "wide_130": [128, 129, 200, 257, 300, 1025], "wide_gated_210": [704, 705, 720], "tile_gated_2048": [1792, 1793]}
# up to here: no lists (2048 tokens of one weight tile; where only small batches of plain wide experts do without the merge by pairs of experts)
LAST = {"tile": 2048, "tile_gated": 2048, "tile_gated_2048": 2048, "wide_130": 2016}
# the same of gates that keep many (a threshold below 0.45, more than a fifth of the experts) or all
LAST_MANY, LAST_ALL = {"tile_gated_2048": 1792, "wide_gated_210": 704}, {"wide_gated_210": 704}
SMALL = {"tile": 16, "tile_gated": 16, "tile_gated_2048": 16, "rows64": 16}  # up to here, otherwise up to 64, the kernels for a few tokens


def has_sets(name, T, fmt="native", last={}):
    return (16 if fmt == "a8" else SMALL.get(name, 64)) < T <= min(LAST.get(name, 3072), last.get(name, 3072))


def layer_of(B, name, T, fmt="native"):
    s = SHAPES[name]
    cfg = wl.Config("sets", T, s["d"], s["E"], s["m"], 64, s["gated"], "gelu_tanh" if s["gated"] else "gelu_erf", "bf16", (0.4,),
                    ffn_bias=not s["gated"], router_bias=True)
    layer, x = wl.make_layer(cfg, T), wl.make_input(cfg, T + 1)
    if fmt != "native":
        layer = wl.quantize_experts_e4m3(layer)
        layer[fmt] = True
    return cfg, layer, x


def forward_without_lists(B, L, xd, tau, **kw):
    """y and whether the call did without lists."""
    L._ws.fill_(0xff)  # (nothing may rest on what an earlier call left)
    B.timing(True)
    y, _ = B.dmoe_forward(L, xd, tau, **kw)
    launches = B.timing_read()
    B.timing(False)
    assert launches["small_up"][0] + launches["expert_up"][0] == 1, launches
    return y, launches["expert_up"][0] == 1 and launches["fill_lists"][0] == 0 and launches["scan_groups"][0] == 0


CASES = [(name, "native", T) for name in sorted(SHAPES) for T in [17] * (name in SMALL and name not in TOKENS_OF) + TOKENS_OF.get(name, TOKENS)]
CASES += [(name, fmt, T) for name in ("wide", "wide_gated") for fmt in ("x8", "a8") for T in [17] * (fmt == "a8") + [128, 129, 257, 1024, 1040]]


@pytest.mark.parametrize("name,fmt,T", CASES)
def test_sets_and_lists(B, name, fmt, T):
    import torch
    print(f"token sets {name} {fmt} T={T}", flush=True)
    cfg, layer, x = layer_of(B, name, T, fmt)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    for tau in (0.0, 0.4, 0.45, 1.0):  # every expert, some, on the other side of the line, one or two
        tau = float(np.float32(tau))
        want, _ = B.dmoe_forward(L, xd, tau, want_lists=True)
        got, sets = forward_without_lists(B, L, xd, tau)
        assert sets == has_sets(name, T, fmt, LAST_ALL if tau == 0 else LAST_MANY if tau < float(np.float32(0.45)) else {})
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), tau
    for k, last in ((cfg.E // 5, {}), (cfg.E // 5 + 1, LAST_MANY), (cfg.E, LAST_ALL)):
        want, _ = B.dmoe_forward(L, xd, 0.0, top_k=k, want_lists=True)
        got, sets = forward_without_lists(B, L, xd, 0.0, top_k=k)
        assert sets == has_sets(name, T, fmt, last)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))


GIVEN = [(name, T) for name in ("tile", "tile_gated", "rows32", "rows64", "wide_gated", "wide") for T in (65, 130, 1030)]
GIVEN += [("wide_24", 1379), ("wide_24", 2561), ("wide_130", 130), ("wide_130", 300)]


@pytest.mark.parametrize("name,T", GIVEN)
def test_given_lists(B, oracle, name, T):
    """Decisions from outside: an expert that nobody selects, one that all do, one with the last token only, and items that
    are just full, one row short and one row over."""
    import torch
    print(f"token sets of given lists {name} T={T}", flush=True)
    cfg, layer, x = layer_of(B, name, T)
    L = B.Layer(layer, cfg.dtype)
    rng = np.random.default_rng(T)
    mask = (rng.random((T, cfg.E)) < 0.3).astype(np.uint8)
    mask[:, 0], mask[:, 1], mask[:, 2] = 0, 1, 0
    mask[T - 1, 2] = 1
    for e, rows in enumerate((63, 64, 65, 127, 128, 129, 255, 256, 257), start=3):
        mask[:, e] = 0
        mask[rng.permutation(T)[:rows], e] = 1
    offsets, lists = lists_from_mask(mask, shuffle_seed=1)
    off_d, list_d, xd = torch.from_numpy(offsets).cuda(), torch.from_numpy(lists).cuda(), B.to_device(x, cfg.dtype)
    L.workspace(T).fill_(0xff)
    B.timing(True)
    y = B.dmoe_expert_ffn(L, xd, off_d, list_d)
    launches = B.timing_read()
    B.timing(False)
    assert has_sets(name, T) and launches["fill_lists"][0] == launches["scan_groups"][0] == 0, launches
    assert tokenwise_rel_err(B.from_device(y, cfg.dtype), oracle_ffn(oracle, layer, x, mask)) <= TOL["bf16"]
