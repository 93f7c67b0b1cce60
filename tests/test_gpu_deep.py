"""GPU parity of the eviction path against the CPU oracle (through the C ABI)."""
import numpy as np
import pytest

from paper_2507_06517_amd import workloads as wl

import parity

pytestmark = pytest.mark.gpu


def test_config1_fp32(oracle):
    rep = parity.check_deep_layer(oracle, wl.config1(0))
    print("config1 deep", rep)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("l,lw,hn,pool,budget", [(300, 16, 4, 7, 64), (1000, 8, 2, 1, 200), (777, 64, 4, 15, 100),
                                                 (130, 32, 8, 3, 33), (65, 64, 1, 7, 64)])
def test_small_ragged(oracle, dtype, l, lw, hn, pool, budget):
    L = wl.small_random(3, dtype, B=2, H=2, l=l, hn=hn, lw=lw, pool=pool, budget=budget)
    parity.check_deep_layer(oracle, L)


@pytest.mark.parametrize("seed", range(12))
def test_shape_sweep(oracle, seed):
    # sequence lengths around the block and stage sizes of the kernels (128-key stages, 1024 keys
    # per block), every window x group size up to the limit of 256 rows, odd pooling widths
    rng = np.random.default_rng(2000 + seed)
    hn = int(rng.choice([1, 2, 4, 8]))
    lw = int(rng.choice([w for w in (1, 3, 16, 32, 64, 128, 256) if w * hn <= 256]))
    l = lw + int(rng.choice([0, 1, 127, 128, 129, 1023, 1024, 1025, 2047, 3000, 5000]))
    pool = int(rng.choice([1, 3, 7, 15, 31]))
    budget = int(rng.integers(lw, l + 2))
    dtype = ("f16", "bf16", "f32")[seed % 3]
    L = wl.small_random(200 + seed, dtype, B=1, H=2, l=l, hn=hn, lw=lw, pool=pool, budget=budget)
    rep = parity.check_deep_layer(oracle, L, norm=seed & 1)
    print("sweep", seed, dtype, l, lw, hn, pool, budget, rep, flush=True)


def test_norm_none_and_budget_edges(oracle):
    L = wl.small_random(4, "f16", B=1, H=2, l=600, hn=4, lw=32, pool=7, budget=100)
    parity.check_deep_layer(oracle, L, norm=1)
    for budget in (32, 33, 599, 600, 5000):       # window only, +1, all but one, all, more than all
        parity.check_deep_layer(oracle, L, budget=budget)


def test_zero_queries_closed_form():
    # Q = 0 makes every softmax row uniform: with the paper's divisor the last k context
    # tokens win, without it all tie and the first k win (lowest index).
    L = wl.small_random(5, "f16", B=1, H=1, l=700, hn=4, lw=16, pool=1, budget=116)
    L.Qw = np.zeros_like(L.Qw)
    lc = 700 - 16
    kept, _, _, sc = parity.gpu_deep(L, norm=0)
    assert kept[0, 0].tolist() == list(range(lc - 100, 700))
    h = sum(1.0 / (lc + b + 1) for b in range(16))
    np.testing.assert_allclose(sc[0, 0, :lc], h / (700 - np.arange(lc)), rtol=1e-5)
    kept, _, _, sc = parity.gpu_deep(L, norm=1)
    assert kept[0, 0].tolist() == list(range(100)) + list(range(lc, 700))


def test_per_unit_budgets(oracle):
    L = wl.small_random(6, "f16", B=2, H=2, l=500, hn=4, lw=16, pool=7, budget=64)
    budgets = [16, 64, 200, 500]
    kept, Ko, Vo, sc = parity.gpu_deep(L, budget=16, budgets=budgets, out_stride=500)
    for u, bud in enumerate(budgets):
        b, h = divmod(u, 2)
        one = wl.Layer(L.dtype, L.K[b:b + 1, h:h + 1], L.V[b:b + 1, h:h + 1], L.Qw[b:b + 1, 4 * h:4 * h + 4],
                       4, 16, 7, bud, 64)
        p64, k64 = parity.oracle_deep(oracle, one, bud)
        parity.check_deep_unit(p64[0, 0], k64[0, 0], sc[b, h], kept[b, h], 16, 500, {})


def test_config2(oracle):
    rep = parity.check_deep_layer(oracle, wl.config2(0))
    print("config2 deep", rep)


def test_deterministic_across_runs():
    L = wl.config2(1)
    a = parity.gpu_deep(L)
    b = parity.gpu_deep(L)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("lc,pool", [(1, 1), (255, 3), (4093, 5), (4096, 9), (4097, 15), (8192, 17), (8190, 19), (16384, 7), (16383, 11),
                                     (16385, 7)])
def test_selection_by_unit_and_over_several_workgroups(oracle, lc, pool):
    # the workgroup per unit takes up to 16384 context positions in steps of 4096, pooled over up to 17; beyond that
    # segments of 2048; around the steps, the last of them ragged, half of the positions kept and few
    L = wl.small_random(7, "f16", B=1, H=2, l=lc + 16, hn=1, lw=16, pool=pool, budget=16 + (lc + 1) // 2)
    parity.check_deep_layer(oracle, L)
    parity.check_deep_layer(oracle, L, budget=16 + (lc + 40) // 41)


@pytest.mark.parametrize("l", [2100, 9000, 17000])
def test_more_ties_than_are_ranked_at_once(l):
    # zero queries without the divisor: all scores equal, thousands of candidates for the threshold; the first win
    L = wl.small_random(8, "f16", B=1, H=1, l=l, hn=4, lw=16, pool=7, budget=1016)
    L.Qw = np.zeros_like(L.Qw)
    kept, _, _, _ = parity.gpu_deep(L, norm=1)
    assert kept[0, 0].tolist() == list(range(1000)) + list(range(l - 16, l))


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("H,l,lw,hn", [(1, 33, 16, 4), (1, 700, 32, 4), (2, 2300, 64, 4), (8, 2065, 32, 4), (8, 3000, 16, 4), (60, 1100, 64, 4),
                                       (130, 600, 16, 1)])
def test_stage_sizes_and_blocks(oracle, dtype, H, l, lw, hn):
    # 32 to 256 keys per stage and one to several stages per block, as the number of units and their length have it,
    # with 64, 128 and 256 query rows; blocks and stages that the sequence does not fill
    L = wl.small_random(9, dtype, B=1, H=H, l=l, hn=hn, lw=lw, pool=3, budget=lw + l // 7)
    units = [(0, h) for h in sorted({0, H // 2, H - 1})]
    p64, k64 = zip(*[[x[0, 0] for x in parity.oracle_deep(oracle, wl.Layer(dtype, L.K[:, h:h + 1], L.V[:, h:h + 1], L.Qw[:, hn * h:hn * (h + 1)],
                                                                           hn, lw, 3, L.budget, 64), L.budget)] for _, h in units])
    kept, _, _, sc = parity.gpu_deep(L)
    for (b, h), p, k in zip(units, p64, k64):
        parity.check_deep_unit(p, k, sc[b, h], kept[b, h], lw, l, {})


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("B,H,l,lw,hn", [(1, 1, 2049, 8, 4), (1, 1, 8200, 64, 4), (1, 2, 8191, 32, 4), (1, 1, 33000, 32, 2)])
def test_few_long_units(oracle, dtype, B, H, l, lw, hn):
    # one or two units cut into up to a hundred chunks whose statistics every block merges
    L = wl.small_random(l, dtype, B=B, H=H, l=l, hn=hn, lw=lw, pool=7, budget=lw + 100, n_centroids=24)
    print("units", dtype, H, l, parity.check_deep_layer(oracle, L), flush=True)


@pytest.mark.parametrize("l,lw,hn", [(8192, 64, 4), (8192, 32, 1)])
def test_one_unit_takes_no_longer_than_eight(l, lw, hn):
    # (one took 22 to 38 % longer where it was cut into as many chunks as the chip has compute units)
    import torch
    from paper_2507_06517_amd import binding as sb
    took = []
    for H in (1, 8):
        g = torch.Generator(device="cuda").manual_seed(H)
        K, Q = (torch.randn((1, h, n, 128), generator=g, device="cuda").half() for h, n in ((H, l), (H * hn, lw)))
        plan = sb.plan_deep(K, hn, "f16", lw, 7, lw + 500, want_scores=False)
        took.append(parity.least_us(lambda: plan.run(K, K, Q), calls=20))
    print("units", l, lw * hn, [round(t, 1) for t in took], flush=True)
    assert took[0] < 1.12 * took[1]


def test_kept_tokens_that_stand_together_take_no_longer():
    # zero queries: the paper's divisor keeps the last 2000 context tokens, which one workgroup copied where the copies
    # went by segments of the context (half as long again); without the divisor random queries keep tokens from everywhere
    import torch
    from paper_2507_06517_amd import binding as sb
    g = torch.Generator(device="cuda").manual_seed(3)
    K, Q = (torch.randn((1, 4, n, 128), generator=g, device="cuda") for n in (20000, 16))
    took = []
    for q, norm in ((torch.zeros_like(Q), 0), (Q, 1)):
        plan = sb.plan_deep(K, 1, "f32", 16, 7, 2016, norm=norm, want_scores=False)
        took.append(parity.least_us(lambda: plan.run(K, K, q), calls=20))
        kept = plan.kept[0, 0].cpu().numpy()
        assert (np.diff(kept) == 1).all() == (norm == 0)
    print("kept together, spread", [round(t, 1) for t in took], flush=True)
    assert took[0] < 1.15 * took[1]


@pytest.mark.parametrize("H", [8, 1])
def test_selection_takes_time_in_proportion_to_the_context(H):
    # eight times the context: 12 times the time where every workgroup of a unit read all of its keys, however many there were
    import torch
    from paper_2507_06517_amd import binding as sb
    took = []
    for l in (65536, 524288):
        g = torch.Generator(device="cuda").manual_seed(l)
        K, Q = (torch.randn((1, H, n, 128), generator=g, device="cuda", dtype=torch.float16) for n in (l, 16))
        plan = sb.plan_deep(K, 1, "f16", 16, 7, 2016, want_scores=False)
        took.append(parity.least_us(lambda: plan.run(K, K, Q)))
    print("units", H, "contexts of 65536, 524288", [round(t, 1) for t in took], flush=True)
    assert took[1] < 9 * took[0]


@pytest.mark.parametrize("dtype,H", [("f16", 5), ("f32", 5), ("bf16", 20), ("f16", 50)])
def test_budgets_and_padding_of_long_contexts(oracle, dtype, H):
    # more than 16384 positions, a ragged last segment; five units are selected by many workgroups each, twenty by six, fifty by one.
    # Only the window, one more, a few, half, all but one, all and more than all; rows behind what is kept
    # are -1 and zeros; with and without V
    l, lw = 20011, 16
    L = wl.small_random(10, dtype, B=1, H=H, l=l, hn=1, lw=lw, pool=7, budget=lw)
    some = [lw, lw + 1, 300, l // 2, l - 1, l, l + 5]
    budgets = [some[u % len(some)] for u in range(H)]
    if H == 5:
        budgets = [lw, 300, l // 2, l - 1, l + 5]
    kept, Ko, Vo, sc = parity.gpu_deep(L, budget=lw, budgets=budgets, out_stride=l + 3)
    for u, bud in enumerate(budgets[:len(some)]):
        one = wl.Layer(dtype, L.K[:, u:u + 1], L.V[:, u:u + 1], L.Qw[:, u:u + 1], 1, lw, 7, min(bud, l), 64)
        p64, k64 = parity.oracle_deep(oracle, one, min(bud, l))
        parity.check_deep_unit(p64[0, 0], k64[0, 0], sc[0, u], kept[0, u], lw, l, {})
        n = min(bud, l)
        assert np.array_equal(Ko[0, u, :n], L.K[0, u][kept[0, u, :n]]) and not Ko[0, u, n:].any()
        assert np.array_equal(Vo[0, u, :n], L.V[0, u][kept[0, u, :n]]) and not Vo[0, u, n:].any()
    import torch
    from paper_2507_06517_amd import binding as sb
    K, Q = (sb.to_device(x, dtype) for x in (L.K, L.Qw))
    alone = sb.compress_deep(K, None, Q, 1, dtype, lw, 7, lw, scale=parity.scale_of(128), out_stride=l + 3,
                             budgets=torch.tensor(budgets, dtype=torch.int32, device="cuda"))
    assert np.array_equal(alone[0].cpu().numpy(), kept) and np.array_equal(sb.to_host_bits(alone[1], dtype), Ko) and alone[2] is None


@pytest.mark.parametrize("H,l", [(30, 17000), (60, 17000), (2, 70000), (8, 70000), (20, 70000)])
def test_ties_and_no_ties_over_several_trips(H, l):
    # one workgroup per unit and several, keys of one trip and of more.  Zero queries: without the divisor all scores tie and the
    # first win, with it the last ones; units of different budgets
    import torch
    from paper_2507_06517_amd import binding as sb
    lw = 16
    K = torch.randn((1, H, l, 128), device="cuda", dtype=torch.float16)
    Q = torch.zeros((1, H, lw, 128), device="cuda", dtype=torch.float16)
    k = [1 + (u * 9973) % (l - lw) for u in range(H)]
    budgets = torch.tensor([lw + x for x in k], dtype=torch.int32, device="cuda")
    for norm in (0, 1):
        kept, Ko, _, _ = sb.compress_deep(K, None, Q, 1, "f16", lw, 7, lw, norm=norm, budgets=budgets, out_stride=l, want_scores=False)
        for u in range(H):
            # (a score is the largest of the seven around it: with the divisor the last four tie, the first of them wins)
            first = 0 if norm else l - lw - k[u]
            got = kept[0, u]
            assert (got[k[u]:k[u] + lw] == torch.arange(l - lw, l, device="cuda")).all() and (got[k[u] + lw:] == -1).all()
            if norm or k[u] > 3:
                assert (got[:k[u]] == torch.arange(first, first + k[u], device="cuda")).all()
            assert torch.equal(Ko[0, u, :k[u] + lw], K[0, u][got[:k[u] + lw].long()]) and not Ko[0, u, k[u] + lw:].any()


@pytest.mark.parametrize("few_rows", [False, True])
@pytest.mark.parametrize("H,lc", [(2, 32768), (2, 32769), (60, 20000), (3, 70000), (1, 2200000)])
def test_selection_in_runs(H, lc, few_rows):
    # keys that stay in registers and one more, one workgroup per unit, runs of several trips (above 2097152 positions); few distinct rows:
    # more scores share the threshold's bin than fit in LDS, and many of all runs tie with the threshold
    import torch
    from paper_2507_06517_amd import binding as sb
    lw, l = 16, lc + 16
    g = torch.Generator(device="cuda").manual_seed(lc + few_rows)
    Q = torch.randn((1, H, lw, 128), generator=g, device="cuda", dtype=torch.float16)
    K = torch.randn((1, H, 8 if few_rows else l, 128), generator=g, device="cuda", dtype=torch.float16)
    if few_rows:
        K = K[:, :, torch.randint(0, 8, (l,), generator=g, device="cuda")].contiguous()
    k = [1 + (u * 9973 + lc // 3) % (lc - 1) for u in range(H)]
    budgets = torch.tensor([lw + x for x in k], dtype=torch.int32, device="cuda")
    kept, Ko, _, sc = sb.compress_deep(K, None, Q, 1, "f16", lw, 1 if few_rows else 7, lw, norm=1, budgets=budgets, out_stride=max(k) + lw)
    for u in range(H):
        own = kept[0, u, :k[u]].cpu().numpy()
        assert np.array_equal(own, parity.lowest_index_topk(sc[0, u, :lc].cpu().numpy(), k[u]))
        assert (kept[0, u, k[u]:k[u] + lw] == torch.arange(lc, l, device="cuda")).all() and (kept[0, u, k[u] + lw:] == -1).all()
        assert torch.equal(Ko[0, u, :k[u] + lw], K[0, u][kept[0, u, :k[u] + lw].long()]) and not Ko[0, u, k[u] + lw:].any()


@pytest.mark.parametrize("l", [2000, 9000])
def test_ranking_of_few_and_of_many_keys_of_a_bin(l):
    # scores that tie by the hundred: from a few to thousands of keys share the bin in which the selection ends, whichever it is
    import torch
    from paper_2507_06517_amd import binding as sb
    lw = 16
    lc = l - lw
    rows = [1, 2, 3, 5, 8, 16, 60, 120, 125, 126, 127, 128, 129, 130, 140, 260]
    g = torch.Generator(device="cuda").manual_seed(l)
    Q = torch.randn((1, len(rows), lw, 128), generator=g, device="cuda", dtype=torch.float16)
    K = torch.randn((1, len(rows), l, 128), generator=g, device="cuda", dtype=torch.float16)
    for u, n in enumerate(rows):                       # every n-th token is one and the same
        K[0, u, ::n] = K[0, u, :1]
    for k in (1, lc // 130, lc // 16, lc // 2, lc - 1):
        kept, _, _, sc = sb.compress_deep(K, None, Q, 1, "f16", lw, 1, lw + k, norm=1)
        for u in range(len(rows)):
            assert np.array_equal(kept[0, u, :k].cpu().numpy(), parity.lowest_index_topk(sc[0, u, :lc].cpu().numpy(), k))
