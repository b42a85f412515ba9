"""The down-projection of sparse selections (two of four experts per structured-sparse instruction) at the
edges of its walk: expert counts around a quad, a mask word and a loop trip, every packing of pieces, divided
walks, a last chunk of few tokens, and selections in which tokens keep three and four of a quad (level 2 of
the tiles), next to tokens without any expert.  All tokens are checked for finiteness, sampled ones against
the oracle."""
import numpy as np
import pytest

from helpers import TOL, lists_from_mask, oracle_ffn, tokenwise_rel_err
from paper_2310_04361_amd import workloads as wl

pytestmark = pytest.mark.gpu


def selection(T, E, p, dense_every, seed):
    """Bernoulli(p), and every dense_every-th token keeps all experts but a random few."""
    rng = np.random.default_rng(seed)
    mask = rng.random((T, E)) < p
    if dense_every:
        rows = np.arange(3, T, dense_every)
        mask[rows] = rng.random((len(rows), E)) < 0.8
        mask[rows[::4]] = True
    mask[5::97] = False
    return mask.astype(np.uint8)


def working_kernel(B, call):
    """Both kernels are launched and the pair count on the device decides which one works: the one that takes the time
    (the other ends at once, 4 us against 9 and more; medians of five calls)."""
    us = {"expert_down": [], "expert_down_sparse": []}
    for _ in range(5):
        B.timing(True)
        call()
        read = B.timing_read()
        B.timing(False)
        for k in us:
            assert read[k][0] == 1
            us[k].append(read[k][1])
    med = {k: float(np.median(v)) for k, v in us.items()}
    first, second = sorted(med, key=med.get, reverse=True)
    assert med[first] > 1.5 * med[second], med
    return first


def densities(T, d, E, m):
    """(most pairs, most quads) as shares of T E for up to 256 workgroups of 128 tokens x 256 columns and no walk or shape
    in which the dense kernel is the only other one; above them the dense kernel."""
    assert -(-T // 128) * (d // 256) <= 256
    most, a, b = (0.14, 0.165, 33.0) if m <= 8 else (0.11, 0.105, 1.8) if m <= 48 else (0.11, 0.125, 1.6) if m <= 64 else (0.075, 0.105, 0.45)
    quads = min(most, a - b / E)
    pairs = 0.0 if m <= 8 else 0.03
    if m > 8 and E < 32 and quads < 0.03:
        pairs = 0.007 if m <= 64 else 0.01
    return pairs, max(pairs, quads)


@pytest.mark.parametrize("T,d,E,m,gated,p,dense_every", [
    # undivided walks (65 chunks x 2 slices of 256 columns), H rows of 64: one expert to three mask words
    (8300, 512, 1, 64, True, 0.09, 0), (8300, 512, 3, 57, True, 0.05, 40), (8300, 512, 5, 64, True, 0.05, 40),
    (8257, 512, 64, 63, True, 0.08, 0), (8300, 512, 66, 64, True, 0.05, 32), (8300, 512, 130, 60, False, 0.09, 0),
    # the other packings: six pieces (three k-steps a stage), sixteen
    (8300, 512, 18, 48, True, 0.05, 32), (8300, 512, 67, 41, False, 0.09, 0),
    (8300, 512, 68, 41, False, 0.07, 0), (8300, 512, 27, 48, True, 0.03, 32), (8300, 512, 18, 64, True, 0.03, 0),
    (8300, 512, 24, 128, False, 0.03, 32), (8300, 512, 21, 100, False, 0.06, 0),
    # one piece: four quads per stage
    (8300, 512, 2048, 8, True, 0.05, 32), (8300, 512, 1990, 5, False, 0.1, 0), (8300, 512, 2011, 1, True, 0.12, 0),
    # divided walks
    (1200, 2048, 256, 64, True, 0.05, 32), (1190, 2048, 253, 64, True, 0.1, 0),
    # so sparse that the work goes by pairs
    (8300, 512, 70, 64, True, 0.01, 0), (8300, 512, 24, 128, False, 0.004, 0), (8300, 512, 66, 40, False, 0.0, 0),
])
def test_sparse_selections(oracle, T, d, E, m, gated, p, dense_every):
    import torch
    from paper_2310_04361_amd import binding as B
    cfg = wl.Config("quad", T, d, E, m, 64, gated, "gelu_tanh" if gated else "gelu_erf", "bf16", (0.5,),
                    ffn_bias=not gated)
    print(f"T={T} d={d} E={E} m={m} gated={gated} p={p} dense_every={dense_every}", flush=True)
    layer, x = wl.make_layer(cfg, 11), wl.make_input(cfg, 11)
    mask = selection(T, E, p, dense_every, 12)
    offsets, lists = lists_from_mask(mask)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    off_d, list_d = torch.from_numpy(offsets).cuda(), torch.from_numpy(np.resize(lists, max(len(lists), 1))).cuda()
    y = B.dmoe_expert_ffn(L, xd, off_d, list_d)
    sparse = mask.mean() <= densities(T, d, E, m)[1]
    assert working_kernel(B, lambda: B.dmoe_expert_ffn(L, xd, off_d, list_d)) == ("expert_down_sparse" if sparse else "expert_down")
    assert torch.equal(B.dmoe_expert_ffn(L, xd, off_d, list_d), y)  # run-to-run reproducible
    got = B.from_device(y, cfg.dtype)
    assert np.isfinite(got).all()
    # ends of chunks and groups, dense and empty tokens, some others
    idx = np.unique(np.concatenate([[0, 3, 5, 63, 64, 127, 128, T - 1], np.arange(3, T, max(dense_every, 1) * 16)[:12],
                                    np.random.default_rng(1).integers(0, T, 30)]))
    ref = oracle_ffn(oracle, layer, x[idx], mask[idx])
    if not gated:
        assert np.allclose(got[5], np.broadcast_to(layer["b_down"], got[5].shape), atol=1e-2)
    zero = np.abs(ref).max(axis=1) == 0
    assert (np.abs(got[idx][zero]) == 0).all()
    assert tokenwise_rel_err(got[idx][~zero], ref[~zero]) <= TOL["bf16"]


@pytest.mark.parametrize("T,d,E,m,gated,limits", [
    (8300, 512, 256, 64, True, None), (8300, 512, 64, 48, True, None), (8300, 512, 20, 64, True, None), (8300, 512, 10, 64, True, None),
    (8300, 512, 96, 128, False, None), (8300, 512, 5, 128, False, None), (8300, 512, 1200, 8, True, (0.1375,)),
    (1200, 2048, 256, 64, True, (0.11,)),  # a divided walk
    # more than one workgroup per CU: 0.125 - 3.4 / E, 0.1 - 5 / E, 0.105 - 1.1 / E, 0.165 - 75 / E
    (17000, 512, 60, 64, True, (0.03, 0.125 - 3.4 / 60)), (17000, 512, 130, 41, True, (0.03, 0.1 - 5.0 / 130)),
    (17000, 512, 40, 64, True, (0.125 - 3.4 / 40,)),
    (17000, 512, 20, 100, False, (0.03, 0.105 - 1.1 / 20)), (17000, 512, 900, 8, True, (0.165 - 75.0 / 900,)),
    # 384-column workgroups of the dense kernel: pairs up to 3 %, the dense kernel above
    (11000, 768, 24, 64, False, (0.03,)), (11000, 768, 24, 128, False, (0.03,)),
])
def test_limits_of_the_pair_count(oracle, T, d, E, m, gated, limits):
    """The last number of pairs that a way of working takes and the first that it leaves to the next: pairs, then quads
    (one kernel), then the dense kernel."""
    import torch
    from paper_2310_04361_amd import binding as B
    cfg = wl.Config("limits", T, d, E, m, 64, gated, "gelu_tanh" if gated else "gelu_erf", "bf16", (0.5,), ffn_bias=not gated)
    layer, x = wl.make_layer(cfg, 13), wl.make_input(cfg, 13)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    if limits is None:
        limits = sorted(set(densities(T, d, E, m)))
    order = np.random.default_rng(14).permutation(T * E)
    idx = np.unique(np.concatenate([[0, 63, 64, 127, 128, T - 1], np.random.default_rng(1).integers(0, T, 60)]))
    for i, limit in enumerate(limits):
        for more in (0, 1):
            n = int(limit * float(T) * float(E)) + more
            print(f"limits T={T} d={d} E={E} m={m} pairs={n}", flush=True)
            mask = np.zeros(T * E, np.uint8)
            mask[order[:n]] = 1
            mask = mask.reshape(T, E)
            offsets, lists = lists_from_mask(mask)
            off_d, list_d = torch.from_numpy(offsets).cuda(), torch.from_numpy(lists).cuda()
            y = B.dmoe_expert_ffn(L, xd, off_d, list_d)
            dense = i == len(limits) - 1 and more
            assert working_kernel(B, lambda: B.dmoe_expert_ffn(L, xd, off_d, list_d)) == ("expert_down" if dense else "expert_down_sparse")
            got, ref = B.from_device(y, cfg.dtype)[idx], oracle_ffn(oracle, layer, x[idx], mask[idx])
            some = np.abs(ref).max(axis=1) > 0
            assert (got[~some] == 0).all()
            assert tokenwise_rel_err(got[some], ref[some]) <= TOL["bf16"]


@pytest.mark.parametrize("T,d,E,m,gated", [
    (8300, 512, 96, 64, True), (8300, 512, 300, 48, True), (8300, 512, 96, 128, False), (4300, 1280, 699, 64, True),
    (50432, 768, 24, 100, False),
])
def test_even_and_uneven_selections_of_the_same_size(oracle, T, d, E, m, gated):
    """Up to 3 % the tiles that the pairs make decide between pairs and quads: as many pairs spread evenly (a tile for
    nearly every expert and chunk), on a few experts only, and in a part of the batch only."""
    import torch
    from paper_2310_04361_amd import binding as B
    cfg = wl.Config("even", T, d, E, m, 64, gated, "gelu_tanh" if gated else "gelu_erf", "bf16", (0.5,), ffn_bias=not gated)
    layer, x = wl.make_layer(cfg, 13), wl.make_input(cfg, 13)
    L, xd = B.Layer(layer, cfg.dtype), B.to_device(x, cfg.dtype)
    rng = np.random.default_rng(14)
    idx = np.unique(np.concatenate([[0, 63, 64, 127, 128, T - 1], rng.integers(0, T, 60)]))
    few, part = max(E // 20, 1), T // 8
    for name, share in (("even", np.full((1, E), 0.028)), ("few", np.where(np.arange(E) % (E // few) == 1, 0.5, 0.001)[None]),
                        ("part", np.where(np.arange(T) // part == 3, 0.2, 0.001)[:, None])):
        mask = (rng.random((T, E)) < share).astype(np.uint8)
        assert mask.mean() <= 0.03
        print(f"{name} T={T} d={d} E={E} m={m} pairs={mask.sum()}", flush=True)
        offsets, lists = lists_from_mask(mask)
        off_d, list_d = torch.from_numpy(offsets).cuda(), torch.from_numpy(lists).cuda()
        y = B.dmoe_expert_ffn(L, xd, off_d, list_d)
        assert torch.equal(B.dmoe_expert_ffn(L, xd, off_d, list_d), y)
        assert working_kernel(B, lambda: B.dmoe_expert_ffn(L, xd, off_d, list_d)) == "expert_down_sparse"
        got, ref = B.from_device(y, cfg.dtype)[idx], oracle_ffn(oracle, layer, x[idx], mask[idx])
        some = np.abs(ref).max(axis=1) > 0
        assert (got[~some] == 0).all()
        assert tokenwise_rel_err(got[some], ref[some]) <= TOL["bf16"]
