"""GPU parity of the codebook path against the CPU oracle (through the C ABI)."""
import numpy as np
import pytest

from paper_2507_06517_amd import workloads as wl

import parity

pytestmark = pytest.mark.gpu


def test_config1_fp32_with_cap(oracle):
    L = wl.config1(0)
    res, g = parity.check_shallow_layer(oracle, L)
    assert any(o["n_codes_uncapped"] > L.max_codes for o in res)      # the cap path is exercised
    parity.check_shallow_layer(oracle, L, cap=512)                      # and the uncapped one


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("l", [1, 31, 33, 257, 300, 1100, 2500])
def test_small_ragged(oracle, dtype, l):
    L = wl.small_random(7, dtype, B=1, H=2, l=l, lw=1, cap=max(1, l // 5), n_centroids=6, noise_frac=0.3)
    parity.check_shallow_layer(oracle, L)
    parity.check_shallow_layer(oracle, L, cap=l)


@pytest.mark.parametrize("l,n_centroids", [(1100, 6), (2500, 6), (2500, 40), (3300, 64)])
def test_without_adjacency_export(oracle, l, n_centroids):
    # no adjacency output requested, graphs whose rows are kept as bits (few centroids) and as words
    # (many centroids)
    L = wl.small_random(12, "f16", B=1, H=2, l=l, lw=1, cap=l, n_centroids=n_centroids, noise_frac=0.3)
    parity.check_shallow_layer(oracle, L, debug=False)


@pytest.mark.parametrize("l", [255, 256, 257, 511, 513, 769, 1023, 1024, 1025, 1281, 2049])
def test_panel_boundaries_without_adjacency_export(oracle, l):
    # lengths around multiples of the 32-token tiles, of the 1024 tokens that fill a batch of the list kernel's
    # steps, and where a second batch begins
    L = wl.small_random(31, "f16", B=1, H=2, l=l, lw=1, cap=l, n_centroids=max(4, l // 24), noise_frac=0.2,
                        drift_sigma=0.002)
    parity.check_shallow_layer(oracle, L, debug=False)


@pytest.mark.parametrize("seed", range(12))
def test_graph_sweep(oracle, seed):
    # graphs of many shapes (sparse to nearly complete, with and without drift and isolated
    # tokens, sizes that are not tile multiples), each compared with the oracle's loop in full
    rng = np.random.default_rng(1000 + seed)
    l = int(rng.integers(40, 3000))
    dtype = ("f16", "bf16", "f32")[seed % 3]
    L = wl.small_random(100 + seed, dtype, B=1, H=2, l=l, lw=1, cap=l,
                        n_centroids=int(rng.integers(1, 60)), noise_frac=float(rng.uniform(0.0, 0.6)),
                        drift_sigma=float(rng.choice([0.0, 0.002, 0.006])))
    L.theta_k = float(rng.choice([0.5, 0.8, 0.9, 0.95, 0.98, 0.995]))
    L.theta_v = float(rng.choice([0.3, 0.7, 0.9, 0.97, 0.99]))
    res, g = parity.check_shallow_layer(oracle, L, debug=bool(seed & 1))
    parity.check_shallow_layer(oracle, L, cap=max(1, l // int(rng.integers(2, 40))), debug=False)
    print("sweep", seed, dtype, l, L.theta_k, L.theta_v, [o["n_codes_uncapped"] for o in res], flush=True)


def test_threshold_extremes_and_single_tensor(oracle):
    L = wl.small_random(8, "f16", B=1, H=1, l=200, lw=1, cap=200)
    L.theta_k, L.theta_v = 1.0, -1.5
    res, g = parity.check_shallow_layer(oracle, L)
    assert g["n_codes_k"][0, 0] == 200 and g["n_codes_v"][0, 0] == 1
    L.theta_k = 0.98
    parity.check_shallow_layer(oracle, L, tensors=("k",))
    parity.check_shallow_layer(oracle, L, tensors=("v",))


def test_knife_edge_pairs_are_decided_exactly(oracle):
    # a random-walk drift gives a continuum of similarities around theta: many pairs fall
    # inside the fp16 guard band and must still match the double-precision decision
    L = wl.small_random(9, "f16", B=1, H=2, l=1500, lw=1, cap=1500, n_centroids=3, noise_frac=0.0,
                        drift_sigma=0.004)
    res, g = parity.check_shallow_layer(oracle, L)
    X = wl.to_f64(L.K[0, 0], "f16")
    Xn = X / np.linalg.norm(X, axis=1, keepdims=True)
    S = Xn @ Xn.T
    assert (np.abs(S - L.theta_k) < 1e-3).sum() > 1000                # the band is well populated


def test_more_close_pairs_than_the_pair_list_holds(oracle):
    # every pair of tokens has a cosine within a few 1e-3 of theta: a step of the list kernel finds more pairs
    # too close to decide in fp32 than a wave's list of waiting pairs holds (192), so the list is emptied in
    # the middle of steps as well as at the end of a batch
    rng = np.random.default_rng(77)
    n, d, theta = 1200, 128, 0.98
    c = rng.standard_normal(d)
    c /= np.linalg.norm(c)
    u = rng.standard_normal((n, d))
    u -= np.outer(u @ c, c)
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    x = np.sqrt(theta) * c + np.sqrt(1 - theta) * u           # cos(x_a, x_b) = theta + (1 - theta) u_a.u_b
    x *= rng.uniform(0.5, 2.0, (n, 1))
    K = wl.cast(x[None, None], "f16")
    S = wl.to_f64(K[0, 0], "f16")
    S /= np.linalg.norm(S, axis=1, keepdims=True)
    close = (np.abs(S @ S.T - theta) < 2e-4).sum() // 2
    assert close > 32 * n, "the input must hold many close pairs"
    L = wl.Layer("f16", K, K.copy(), np.zeros((1, 1, 1, d), np.float16), 1, 1, 1, n, n, theta_k=theta, theta_v=theta)
    parity.check_shallow_layer(oracle, L, tensors=("k",))
    parity.check_shallow_layer(oracle, L, tensors=("k",), cap=100, debug=False)
    # the library's own count of decisions in double precision: more than 30 per row and step
    import torch
    from paper_2507_06517_amd import binding as sb
    Kd = sb.to_device(L.K, "f16")
    plan = sb.plan_shallow(Kd, "f16", theta, theta, n, tensors=("k",))
    plan.run(Kd, None)
    torch.cuda.synchronize()
    assert plan.stats()[0, 2] > 32 * n


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_counts_of_double_precision_decisions_by_problem(dtype):
    # the waves of a problem count for themselves, one or four of them per row tile (40 problems of 29 row tiles, one
    # problem); the same pairs are close to theta either way
    import torch
    from paper_2507_06517_amd import binding as sb
    rng = np.random.default_rng(12)
    theta = float(np.float32(0.98))
    c, u = rng.standard_normal((40, 1, 128)), rng.standard_normal((40, 900, 128))
    c /= np.linalg.norm(c, axis=2, keepdims=True)
    u -= (u * c).sum(axis=2, keepdims=True) * c
    u /= np.linalg.norm(u, axis=2, keepdims=True)
    X = wl.cast((np.sqrt(theta) * c + np.sqrt(1 - theta) * u)[None], dtype)   # cos(x_a, x_b) = theta + (1 - theta) u_a.u_b
    X[0, 3] = X[0, 4]                                    # (two alike, one with nothing but zeros)
    X[0, 7] = 0
    K, V = sb.to_device(np.ascontiguousarray(X[:, :20]), dtype), sb.to_device(np.ascontiguousarray(X[:, 20:]), dtype)
    plan = sb.plan_shallow(K, dtype, theta, theta, 900)
    counts = []
    for _ in range(2):
        plan.run(K, V)
        torch.cuda.synchronize()
        counts.append(plan.stats()[:, 2].copy())
    alone = []
    one = sb.plan_shallow(K[:, :1].contiguous(), dtype, theta, theta, 900, tensors=("k",))
    for i in range(40):
        one.run(sb.to_device(np.ascontiguousarray(X[:, i:i + 1]), dtype), None)
        torch.cuda.synchronize()
        alone.append(int(one.stats()[0, 2]))
    assert counts[0].tolist() == counts[1].tolist() == alone
    assert alone[3] == alone[4] and alone[7] == 0 and min(alone[:7]) > 900


def test_duplicates_and_zero_vectors(oracle):
    L = wl.small_random(10, "f16", B=1, H=1, l=400, lw=1, cap=400)
    L.K[0, 0, 100:150] = L.K[0, 0, 7]            # exact duplicates
    L.K[0, 0, 200:203] = 0                        # zero vectors
    L.V[0, 0, 5] = 0
    res, g = parity.check_shallow_layer(oracle, L)
    assert len(set(g["ref_k"][0, 0, 100:150].tolist() + [g["ref_k"][0, 0, 7]])) == 1


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_cosine_exactly_at_the_threshold(oracle, dtype):
    # cos(e_0 + e_1 + e_2 + e_3, e_0) = 1 / 2 and cos(e_4 + e_5, e_4 + e_6) = 1 / 2 with every
    # intermediate exact in any precision: Eq. 9 is strict, so at theta = 1/2 these pairs are not
    # adjacent, and one float below they are (the approximate cosine sits inside the guard band,
    # the double-precision decision has to get the equality right)
    L = wl.small_random(14, dtype, B=1, H=1, l=300, lw=1, cap=300)
    rows = np.zeros((8, L.K.shape[-1]))
    rows[0, 0] = 1
    rows[1, :4] = 1
    rows[2, [4, 5]] = 1
    rows[3, [4, 6]] = 1
    rows[4:] = 4 * rows[:4]                            # the same again, scaled: magnitudes drop out
    L.K[0, 0, 40:48] = wl.cast(rows, dtype)
    L.V[0, 0, 40:48] = wl.cast(rows, dtype)
    L.theta_k = L.theta_v = 0.5
    res, g = parity.check_shallow_layer(oracle, L)
    adj = lambda a, b: (g["adj_k"][0, 0, a, b >> 5] >> (b & 31)) & 1
    assert adj(40, 41) == 0 and adj(42, 43) == 0 and adj(40, 45) == 0 and adj(40, 44) == 1 and adj(41, 45) == 1
    L.theta_k = L.theta_v = float(np.nextafter(np.float32(0.5), np.float32(0)))
    res, g = parity.check_shallow_layer(oracle, L)
    assert adj(40, 41) == 1 and adj(42, 43) == 1 and adj(40, 45) == 1


@pytest.mark.parametrize("dtype,l,cap", [("f16", 1500, 80), ("bf16", 2100, 2100), ("f32", 700, 30)])
def test_two_halves_with_the_eviction_call_beside_the_second(oracle, dtype, l, cap):
    # spindle_shallow_graph, an event, spindle_shallow_codebook, and spindle_compress_deep on a side
    # stream that waits for the event (what bench.py times): both results against the oracle
    L = wl.small_random(31, dtype, B=1, H=3, l=l, lw=16, budget=l // 5, cap=cap, n_centroids=60, noise_frac=0.2)
    got, g = parity.gpu_layer_two_streams(L)
    parity.check_deep_layer(oracle, L, got=got)
    parity.check_shallow_layer(oracle, L, g=g)


@pytest.mark.parametrize("dtype,l,cap", [("f16", 1500, 80), ("bf16", 2100, 2100)])
def test_consecutive_layers_pipelined(oracle, dtype, l, cap):
    # five runs over two sets of buffers, the similarity phase of a run beside the codebook phase and the
    # eviction call of the run before: what both sets hold at the end against the oracle
    L = wl.small_random(32, dtype, B=1, H=3, l=l, lw=16, budget=l // 5, cap=cap, n_centroids=60, noise_frac=0.2)
    for got, g in parity.gpu_layers_pipelined(L):
        parity.check_deep_layer(oracle, L, got=got)
        parity.check_shallow_layer(oracle, L, g=g)


def test_cut_tokens_with_many_equidistant_entries(oracle):
    # zero vectors have cosine 0 with every entry: when their own entry is cut, every stored entry
    # ties, the candidate lists of the matrix-core search run full and the exhaustive search must
    # give entry 0; near-duplicates of one token, cut as well, must all land on the same entry
    L = wl.small_random(13, "f16", B=1, H=1, l=700, lw=1, cap=40, n_centroids=60, noise_frac=0.5)
    L.K[0, 0, 300:310] = 0
    L.V[0, 0, 5] = 0
    res, g = parity.check_shallow_layer(oracle, L)
    assert res[0]["n_codes_uncapped"] > 40
    assert (g["ref_k"][0, 0, 300:310] == 0).all()


def test_config2(oracle):
    res, g = parity.check_shallow_layer(oracle, wl.config2(0))
    print("config2 codes", [o["n_codes_uncapped"] for o in res])


@pytest.mark.parametrize("dtype,l,cap", [("f16", 500, 500), ("f16", 777, 60), ("bf16", 1301, 2000), ("bf16", 333, 25),
                                         ("f32", 513, 600), ("f32", 1000, 48)])
def test_reconstruct(oracle, dtype, l, cap):
    # Eq. 14 on the library's own codebook, references and magnitudes against the oracle's
    # reconstruction from its own: ragged lengths, with and without references moved by the cap.
    # Tolerance: max(1e-3, one unit in the last place of the storage type) relative per element
    # (two roundings to the storage type, each half a unit: the stored entry and the product),
    # plus the spacing of the type's subnormals times the magnitude for components near zero.
    import torch
    from paper_2507_06517_amd import binding as sb
    L = wl.small_random(11 + l, dtype, B=1, H=2, l=l, lw=1, cap=cap, n_centroids=40, noise_frac=0.2)
    K, V = sb.to_device(L.K, dtype), sb.to_device(L.V, dtype)
    out = sb.compress_shallow(K, V, dtype, L.theta_k, L.theta_v, cap)
    Rk = sb.reconstruct(out["C_k"], out["ref_k"], out["mag_k"], dtype)
    Rv = sb.reconstruct(out["C_v"], out["ref_v"], out["mag_v"], dtype)
    torch.cuda.synchronize()
    rel = max(parity.RTOL, parity.ULP[dtype])
    tiny = {"f16": 2.0 ** -24, "bf16": 2.0 ** -126, "f32": 2.0 ** -126}[dtype]
    capped = 0
    for R, src, theta in ((Rk, L.K, L.theta_k), (Rv, L.V, L.theta_v)):
        Rh = wl.to_f64(sb.to_host_bits(R, dtype), dtype)
        for h in range(2):
            X = wl.to_f64(src[0, h], dtype)
            o = oracle.shallow_unit(X, float(np.float32(theta)), cap)
            capped += o["n_codes_uncapped"] > cap
            want = oracle.reconstruct(o["C"], o["ref"], o["mag"])
            err = np.abs(Rh[0, h] - want)
            assert np.all(err <= np.abs(want) * rel + tiny * np.maximum(o["mag"], 1.0)[:, None]), err.max()
            # every row has its token's magnitude, and its direction is that of the token's entry
            nr = np.linalg.norm(Rh[0, h], axis=1)
            assert np.allclose(nr, o["mag"], rtol=2 * rel, atol=1e-30)
            if o["n_codes_uncapped"] <= cap:          # Alg. 1's guarantee holds when nothing was cut
                c = np.einsum("ad,ad->a", Rh[0, h], X) / np.maximum(nr * o["mag"], 1e-300)
                assert np.all(c[o["mag"] > 0] > theta - 2 * rel)
    assert (capped > 0) == (cap < 100), "the small caps are meant to cut entries, the large ones not"


def test_reconstruct_ignores_rows_without_an_entry():
    # references outside [0, max_codes) (what a full table leaves at decode time: -1) give zero rows
    import torch
    from paper_2507_06517_amd import binding as sb
    Cb = torch.randn((1, 1, 4, 128), device="cuda").half()
    ref = torch.tensor([[[0, -1, 3, 4, 2]]], dtype=torch.int32, device="cuda")
    mag = torch.tensor([[[2.0, 3.0, 0.5, 1.0, 0.0]]], dtype=torch.float32, device="cuda")
    R = sb.reconstruct(Cb, ref, mag, "f16")
    torch.cuda.synchronize()
    assert torch.equal(R[0, 0, 0], (Cb[0, 0, 0].float() * 2.0).half()) and torch.equal(R[0, 0, 2], (Cb[0, 0, 3].float() * 0.5).half())
    assert not R[0, 0, 1].any() and not R[0, 0, 3].any() and not R[0, 0, 4].any()


def test_deterministic_across_runs():
    L = wl.config2(2)
    a = parity.gpu_shallow(L)
    b = parity.gpu_shallow(L)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


def test_measurement_aids_run_and_leave_results_alone():
    # the two calibration calls compute nothing the method needs; they must run, report sane
    # figures and not disturb a later call on the same workspace
    import torch
    from paper_2507_06517_amd import binding as sb
    L = wl.config2(3)
    K, V = sb.to_device(L.K, L.dtype), sb.to_device(L.V, L.dtype)
    plan = sb.plan_shallow(K, L.dtype, L.theta_k, L.theta_v, L.max_codes)
    a = {k: v.clone() for k, v in plan.run(K, V).items()}
    ms = sb.spindle_calibrate_similarity(plan)
    for mode in (1, 2):
        assert 0.0 < sb.spindle_calibrate_similarity(plan, mode) < 50.0
    tf = sb.spindle_calibrate_mfma(512)
    tf_data = sb.spindle_calibrate_mfma(512, 1)
    assert 0.0 < ms < 50.0 and 50.0 < tf < 2600.0 and 50.0 < tf_data < 2600.0, (ms, tf, tf_data)
    b = plan.run(K, V)
    torch.cuda.synchronize()
    for k in a:
        assert torch.equal(a[k].view(torch.uint8), b[k].view(torch.uint8)), k


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("ncut", [1, 31, 64, 65, 129, 300, 700])
def test_cut_tokens_with_one_several_and_too_many_candidates(oracle, dtype, ncut):
    # 96 stored entries along axes, twice each so that they are picked first; the tokens whose entries are cut are near one
    # of them, or between two (equal cosines, or a little off), or as near to 64 of them (more than a list of candidates
    # holds), or zero, or hold a NaN; blocks of 64 cut tokens where they are few, of 256 where they are more than a
    # quarter, ragged either way
    rng = np.random.default_rng(ncut)
    axes = np.repeat(np.eye(128)[:96], 2, axis=0) * rng.uniform(0.5, 2.0, (192, 1))
    far = rng.standard_normal((ncut, 128))
    far /= np.linalg.norm(far, axis=1, keepdims=True)
    kind = np.arange(ncut) % 5
    for i in range(ncut):
        j, k = rng.choice(96, 2, replace=False)
        if kind[i] == 1:
            far[i] = 0.3 * far[i]
            far[i, j] = 0.9
        elif kind[i] == 2:
            far[i, [j, k]] = 0.5 + (i % 2) * rng.uniform(0.0, 2e-3, 2)
        elif kind[i] == 3:
            far[i] = rng.choice([-1.0, 1.0], 128)
    if ncut > 60:
        far[50], far[55] = 0.0, 1.0
    x = np.concatenate([axes, far])[rng.permutation(192 + ncut)]
    K = wl.cast(x[None, None], dtype)
    if ncut > 60:
        spoilt = int(np.flatnonzero((x == 1.0).all(1))[0])
        K[0, 0, spoilt, 3] = wl.cast(np.array([np.nan]), dtype)[0]
    L = wl.Layer(dtype, K, K.copy(), np.zeros_like(K[:, :, :1]), 1, 1, 1, 192 + ncut, 96, theta_k=0.97, theta_v=0.97)
    if ncut <= 60:
        res, g = parity.check_shallow_layer(oracle, L, tensors=("k",), debug=False)
        assert res[0]["n_codes_uncapped"] > 96
        return
    # (the oracle's cosine of a NaN is not the library's business: that token's own reference only has to exist)
    g = parity.gpu_shallow(L, tensors=("k",), debug=False)
    clean = np.array(L.K)
    clean[0, 0, spoilt] = wl.cast(np.ones(128), dtype)
    o = oracle.shallow_unit(wl.to_f64(clean[0, 0], dtype), float(np.float32(0.97)), 96)
    keep = np.arange(192 + ncut) != spoilt
    assert np.array_equal(g["ref_k"][0, 0][keep], o["ref"][keep]) and 0 <= g["ref_k"][0, 0, spoilt] < 96


@pytest.mark.parametrize("dtype,n,cap", [("f16", 1024, 128), ("bf16", 1024, 128), ("f32", 512, 64), ("f16", 4096, 512)])
def test_padding_by_the_hundred_is_cut(oracle, dtype, n, cap):
    # half of a prompt is padding: its zero rows are entries of their own and hundreds of them are cut.  Their cosine is 0 with
    # every entry, so none of them needs a search: the call takes about as long as one with as many tokens in clusters
    # (four to five times as long where every such row was compared with all entries, one after the other)
    from paper_2507_06517_amd import binding as sb
    L = wl.small_random(n, dtype, B=1, H=1, l=n, lw=1, cap=cap, n_centroids=20, noise_frac=0.0)
    plain_in = sb.to_device(L.K, dtype), sb.to_device(L.V, dtype)
    plan = sb.plan_shallow(plain_in[0], dtype, L.theta_k, L.theta_v, cap)
    plain = parity.least_us(lambda: plan.run(*plain_in))
    L.K[:, :, ::2], L.V[:, :, ::2] = 0, 0
    res, _ = parity.check_shallow_layer(oracle, L, debug=False)
    assert all(o["n_codes_uncapped"] > cap + 200 for o in res)
    padded = sb.to_device(L.K, dtype), sb.to_device(L.V, dtype)
    took = parity.least_us(lambda: plan.run(*padded))
    print("cut padding", dtype, n, cap, round(plain), round(took), flush=True)
    assert took < 2.0 * plain


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_few_tokens_with_a_large_table(oracle, dtype):
    # the rows behind the stored entries are zero whatever the buffers held, for tables from one block's share up; the
    # largest is cleared across the chip, in about the time of the smallest (5 to 8 times that by the tokens' block alone)
    import torch
    from paper_2507_06517_amd import binding as sb
    L = wl.small_random(5, dtype, B=1, H=1, l=64, lw=1, cap=64, n_centroids=6, noise_frac=0.3)
    K, V = sb.to_device(L.K, dtype), sb.to_device(L.V, dtype)
    took = []
    for cap in (64, 127, 129, 1000, 4099, 65536):
        plan = sb.plan_shallow(K, dtype, L.theta_k, L.theta_v, cap)
        for t in "kv":
            plan.out["C_" + t].fill_(7.0)
        out = plan.run(K, V)
        torch.cuda.synchronize()
        g = {k: (sb.to_host_bits(v, dtype) if k.startswith("C_") else v.cpu().numpy()) for k, v in out.items()}
        parity.check_shallow_layer(oracle, L, cap=cap, g=g)
        took.append(parity.least_us(lambda: plan.run(K, V), calls=20))
    print("table sizes", dtype, [round(t) for t in took], flush=True)
    assert took[-1] < 2.5 * took[0]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("units,n,cap", [(1, 1, 1), (3, 63, 7), (2, 65, 300), (5, 129, 64), (1, 70001, 33), (40, 4100, 9)])
def test_reconstruct_blocks_and_large_outputs(dtype, units, n, cap):
    # around the rows a block takes, several units, and outputs above 32 MiB, which are streamed; references out of the
    # table give zero rows.  The product of two floats rounded to the cache type: exact
    import torch
    from paper_2507_06517_amd import binding as sb
    g = torch.Generator(device="cuda").manual_seed(n)
    dt = sb.torch_dtype(dtype)
    Cb = torch.randn((1, units, cap, 128), generator=g, device="cuda").to(dt)
    ref = torch.randint(-1, cap + 1, (1, units, n), generator=g, device="cuda", dtype=torch.int32)
    mag = torch.rand((1, units, n), generator=g, device="cuda") * 20
    R = sb.reconstruct(Cb, ref, mag, dtype)
    ok = (ref >= 0) & (ref < cap)
    at = ref.clamp(0, cap - 1).long().unsqueeze(3).expand(1, units, n, 128)
    want = (torch.gather(Cb.float(), 2, at) * mag.unsqueeze(3)).to(dt)
    want = torch.where(ok.unsqueeze(3), want, torch.zeros_like(want))
    assert torch.equal(R, want)
