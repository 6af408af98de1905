"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_12280_amd import workloads as W

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2511_12280_amd import binding as B
    from parity import (GpuStep, check_assign, check_attend, check_full_sample, check_kept, check_merge,
                        check_scores, attend_form, gpu_attend, gpu_attend_weighted, key_weights)


def _chain(samples, keeps, dtype, mode="mean", assign_rows=None, check=None):
    step = GpuStep(samples, keeps, dtype, B.D3TOM_MERGE_MEAN if mode == "mean" else B.D3TOM_MERGE_SUM)
    S = step.importance()
    kept, slot = step.select_topk()
    mout = step.merge()
    stats = []
    for b in (range(len(samples)) if check is None else check):
        stats.append(check_full_sample(step, b, S, kept, slot, mout, assign_rows=assign_rows, mode=mode))
    return step, S, kept, mout, stats


# ---- the tiny fp32 layer: whole chain including the attention on the merged rows -------------------
def test_tiny_f32_chain_with_attention():
    wl = W.WORKLOADS["tiny_f32"]
    g = W.SampleGen(wl)
    s = g.step(16)
    k = oracle.keep_count(wl.V, 0.25)
    assert k == 36 and B.d3tom_keep_count(wl.V, 0.25) == 36
    step, S, kept, mout, stats = _chain([s], [k], "f32")
    assert stats[0]["kept_excused"] == 0 and stats[0]["assign_excused"] == 0
    y = mout["y"][0]
    assert y.shape == (100, 256)
    q2, k2, v2 = g.proj.qkv(y)                       # projection of the merged rows (host, not on the path)
    o = gpu_attend([(q2, k2, v2)], "f32")[0]
    check_attend(o, q2, k2, v2, "f32")


# ---- bf16 cases spanning several tiles with ragged tails ----------------------------------------------
@pytest.mark.parametrize("P,V,O,H,dh,D,keep,mode", [
    (37, 700, 40, 8, 128, 20, 0.23, "mean"),
    (5, 333, 9, 4, 64, 3, 0.50, "mean"),
    (0, 130, 17, 2, 128, 17, 0.10, "sum"),
    (3, 1000, 70, 4, 128, 70, 0.77, "mean"),
])
def test_bf16_cases(P, V, O, H, dh, D, keep, mode):
    c = W.random_case(100 + V, P + V + O, H * dh, H, P, V, D, dtype="bf16", centres=max(4, V // 6))
    k = oracle.keep_count(V, keep)
    _chain([c], [k], "bf16", mode=mode)


def test_f32_generic_case_and_odd_head_size():
    c = W.random_case(7, 150, 4 * 36, 4, 10, 120, 6, dtype="f32", centres=9)      # dh = 36
    _chain([c], [oracle.keep_count(120, 0.3)], "f32")
    c = W.random_case(8, 90, 2 * 40, 2, 4, 80, 5, dtype="bf16", centres=9)        # bf16 with dh = 40: generic kernels
    _chain([c], [oracle.keep_count(80, 0.25)], "bf16")


@pytest.mark.parametrize("dtype,H,dh,N,k", [
    ("f32", 2, 4, 66, 1), ("f32", 1, 64, 65, 16), ("f32", 3, 68, 64, 17), ("f32", 2, 256, 257, 64), ("f32", 1, 252, 330, 65), ("f32", 4, 64, 577, 143),
    ("bf16", 3, 8, 256, 63), ("bf16", 2, 136, 129, 33), ("bf16", 1, 256, 321, 129),
])
def test_generic_kernels_sixteen_lanes_to_a_row(dtype, H, dh, N, k):
    """Generic kernels: keys around the 64 of a wave and the 256 of a turn, rows of 1 to 128 chunks (a row of lanes takes 16 of them, a
    turn of the cosines 64), kept slots around 16 and 64."""
    V = N - 6
    samples = [W.random_case(830 + N, N, H * dh, H, 2, V, 4, dtype=dtype, centres=max(2, k // 3)), W.random_case(831, 7, H * dh, H, 1, 3, 2, dtype=dtype)]
    _chain(samples, [k, 2], dtype)
    qkv = [W.random_qkv(832 + N, n, H, dh, dtype) for n in (N, 1)]
    qkv[0][1][:, H - 1, :] *= 4.0
    for (q, kk, v), o in zip(qkv, gpu_attend(qkv, dtype)):
        check_attend(o, q, kk, v, dtype)


# ---- tile-edge shapes: counts that sit exactly on, one below and one above the kernels' tile sizes --------
@pytest.mark.parametrize("P,V,O,D,k", [
    (0, 512, 16, 16, 128),       # keys = one 512-key chunk + deciders, kept = one 128-slot column tile, pruned = 6 x 64
    (1, 513, 33, 33, 129),       # one past every boundary
    (0, 511, 256, 256, 127),     # the largest decider set, one below the boundaries
    (3, 257, 17, 17, 256),       # a single pruned token
    (5, 640, 48, 47, 64),        # 9 row tiles x 1 half-filled column tile (split along the contraction)
])
def test_tile_edge_shapes(P, V, O, D, k):
    c = W.random_case(1000 + V + k, P + V + O, 2 * 128, 2, P, V, D, dtype="bf16", centres=max(4, V // 9))
    step, S, kept, mout, stats = _chain([c], [k], "bf16")
    assert mout["y"][0].shape[0] == P + k + O
    n_m = P + k + O
    qkv = W.random_qkv(2000 + n_m, n_m, 2, 128, "bf16")
    check_attend(gpu_attend([qkv], "bf16")[0], *qkv, "bf16")


# ---- ragged batch ----------------------------------------------------------------------------------
def test_ragged_batch_bf16():
    shapes = [(20, 300, 30, 9, 0.2), (64, 513, 64, 33, 0.5), (1, 128, 5, 1, 0.1), (7, 129, 300, 100, 0.33), (0, 64, 2, 2, 1.0)]
    samples, keeps = [], []
    for i, (P, V, O, D, keep) in enumerate(shapes):
        samples.append(W.random_case(200 + i, P + V + O, 4 * 128, 4, P, V, D, dtype="bf16", centres=max(3, V // 5)))
        keeps.append(oracle.keep_count(V, keep))
    step, S, kept, mout, stats = _chain(samples, keeps, "bf16")
    # keep ratio 1: identity
    np.testing.assert_array_equal(mout["y"][4], samples[4]["x"])
    np.testing.assert_array_equal(kept[4], np.arange(64))


@pytest.mark.parametrize("batch", [12, 13, 14])
def test_merge_large_batch_tiles(batch):
    """Batches of several rounds of cosine tiles: samples on pairs of XCDs (as many on each, or not) and on all of them, sizes
    from one row over a tile to the largest."""
    V = [2304, 1, 129, 257, 700, 2303, 64, 1900, 513, 1025, 2048, 300, 1111, 1536][:batch]
    samples = [W.random_case(400 + i, 4 + v + 8, 128, 1, 4, v, 3, dtype="bf16", centres=max(2, v // 6)) for i, v in enumerate(V)]
    keeps = [oracle.keep_count(v, 0.5 if i % 3 == 0 else 0.11) for i, v in enumerate(V)]
    _chain(samples, keeps, "bf16", check=[0, 1, 2, 5, batch - 1])


@pytest.mark.parametrize("batch,V", [(16, 1088), (16, 1089), (15, 1089), (33, 576), (33, 448)])
def test_merge_batches_around_half_a_round(batch, V):
    """Batches of 16 and more samples take 256-row tiles above 128 tiles of 128 rows (bounds of 128, 144, 135, 132 and 99 of them)."""
    rng = np.random.default_rng([batch, V])
    sizes = [V] + [int(v) for v in rng.integers(70, V, batch - 1)]
    samples = [W.random_case(740 + i, v + 5, 64, 1, 5, v, 1, dtype="bf16", centres=max(2, v // 6)) for i, v in enumerate(sizes)]
    kept = [np.sort(rng.choice(v, size=64, replace=False)).astype(np.int32) for v in sizes]
    out = GpuStep(samples, [64] * batch, "bf16").merge(kept)
    for b, s in enumerate(samples):
        check_assign(out["assign"][b], s["x"], s["vis_start"], s["V"], kept[b])
        check_merge({key: out[key][b] for key in out}, s["x"], s["vis_start"], s["V"], kept[b], "bf16")


@pytest.mark.parametrize("big,small", [(1, 15), (2, 14), (4, 12), (7, 9), (1, 69), (3, 66), (0, 130), (0, 31)])
def test_merge_batch_tiles_in_equal_runs(big, small):
    """The tiles of a whole batch cut into one run per XCD, whose rest of the last round is cut into quarter, half or no parts of a
    tile: totals of 7 to 32 tiles a run, samples before and behind the 64 looked at together, pruned counts around a tile and its parts."""
    sizes = [(2304, 1152), (2303, 1279), (2100, 900), (1409, 1153), (2304, 1024), (2047, 1000), (1700, 1100)][:big]
    sizes += [[(400, 144), (1, 1), (129, 64), (321, 64), (90, 90), (577, 320), (65, 1), (256, 255), (513, 256)][i % 9] for i in range(small)]
    sizes = [sizes[i] for i in np.random.default_rng(big).permutation(len(sizes))]
    rng = np.random.default_rng(small)
    samples = [W.random_case(700 + i, V + 5, 64, 1, 5, V, 1, dtype="bf16", centres=max(2, V // 6)) for i, (V, _) in enumerate(sizes)]
    kept = [np.sort(rng.choice(V, size=k, replace=False)).astype(np.int32) for V, k in sizes]
    out = GpuStep(samples, [k for _, k in sizes], "bf16").merge(kept)
    for b, s in enumerate(samples):
        check_assign(out["assign"][b], s["x"], s["vis_start"], s["V"], kept[b],
                     only=None if s["V"] < 700 else np.sort(rng.choice(s["V"], 200, replace=False)))
        check_merge({key: out[key][b] for key in out}, s["x"], s["vis_start"], s["V"], kept[b], "bf16")


@pytest.mark.parametrize("dh,copies", [(64, 128), (128, 128), (64, 4), (128, 4), (64, 1), (128, 1)])
def test_importance_decider_groups_and_chunks(dh, copies):
    """Decider counts around the 128 rows staged at a time and around 16-row blocks, key counts around the key chunks of both
    sweeps: one copy of the batch has chunks of 256 keys, 4 have chunks of 512, 128 stream the keys."""
    shapes = [(383, 127, 33), (384, 256, 128), (385, 257, 129), (520, 255, 256), (170, 1, 144)]      # tokens, visual, deciders
    samples = [W.random_case(600 + i, N, 8 * dh, 8, 3, V, D, dtype="bf16") for i, (N, V, D) in enumerate(shapes)]
    for s, (_, _, D) in zip(samples, shapes):
        s["dec_idx"] = np.resize(s["dec_idx"], D).astype(np.int32)         # (repeats where there are fewer positions)
        s["D"] = D
    batch = samples * copies
    S = GpuStep(batch, [max(1, s["V"] // 4) for s in batch], "bf16").importance()
    for i, s in enumerate(samples):
        ref = oracle.importance(s["q"], s["k"], s["dec_idx"], s["vis_start"], s["V"])
        check_scores(S[i], ref)
        np.testing.assert_array_equal(S[i], S[len(batch) - len(samples) + i])


@pytest.mark.parametrize("dh", [64, 128])
def test_importance_streaming_stages(dh):
    """Large launches: key and visual counts around the 64-key stages, the four stages in flight and the chunks a sample is cut into,
    decider counts that leave waves with none to four blocks of 16."""
    shapes = [(1, 1, 1), (64, 63, 16), (65, 64, 17), (129, 65, 33), (576, 513, 64), (705, 577, 65), (1100, 1024, 256), (1025, 1, 200)]
    samples = [W.random_case(660 + i, N, 8 * dh, 8, 0, V, D, dtype="bf16") for i, (N, V, D) in enumerate(shapes)]
    for s, (_, _, D) in zip(samples, shapes):
        s["dec_idx"] = np.resize(s["dec_idx"], D).astype(np.int32)         # (repeats where there are fewer positions)
        s["D"] = D
    batch = samples * 8                                                     # 64 samples x 8 heads, two chunks each
    S = GpuStep(batch, [max(1, s["V"] // 4) for s in batch], "bf16").importance()
    for i, s in enumerate(samples):
        check_scores(S[i], oracle.importance(s["q"], s["k"], s["dec_idx"], s["vis_start"], s["V"]))
        np.testing.assert_array_equal(S[i], S[len(batch) - len(samples) + i])


@pytest.mark.parametrize("dtype,H,dh,D,N,copies", [
    ("bf16", 2, 128, 9, 1100, 1), ("bf16", 2, 64, 40, 1100, 1),           # chunks of 256 keys, logits kept or not
    ("bf16", 16, 64, 9, 1100, 2), ("bf16", 16, 128, 40, 1100, 2),         # chunks of 512 keys, logits kept or not
    ("bf16", 16, 128, 160, 1200, 16), ("bf16", 16, 64, 145, 1200, 16),    # keys streamed, chunks of 640
    ("f32", 2, 64, 9, 300, 1), ("f32", 2, 64, 40, 300, 1)])               # generic kernels
def test_importance_chunk_of_infinite_logits(dtype, H, dh, D, N, copies):
    """Keys whose logits are all -inf (an infinite key channel) have probability 0, also where they are all the keys of a chunk of the
    first sweep: the first chunk, one in the middle, the ragged last one."""
    samples = []
    for i, (j0, j1) in enumerate([(0, 640), (256, 1088), (512, N), (N - 1, N), (0, N - 1)]):
        s = W.random_case(680 + i, N, H * dh, H, 3, N - 3 - D, D, dtype=dtype)
        s["q"][:, :, 5] = 0.5
        s["k"][j0:min(j1, N - 1 if j0 == 0 else N), :, 5] = -np.inf
        samples.append(s)
    batch = samples * copies
    S = GpuStep(batch, [8] * len(batch), dtype).importance()
    for i, s in enumerate(samples):
        ref = oracle.importance(s["q"], s["k"], s["dec_idx"], s["vis_start"], s["V"])
        assert np.isfinite(ref).all()
        check_scores(S[i], ref)
        np.testing.assert_array_equal(S[i], S[len(batch) - len(samples) + i])


@pytest.mark.parametrize("dtype,H,dh,D", [("bf16", 8, 64, 8), ("bf16", 4, 128, 16), ("bf16", 16, 128, 16), ("bf16", 32, 64, 32), ("bf16", 5, 128, 7),
                                          ("f32", 4, 64, 16), ("f32", 5, 36, 13), ("bf16", 3, 40, 9)])
def test_importance_rows_beyond_float32_add_nothing(dtype, H, dh, D):
    """Small decider sets: a (head, decider) row whose logits overflow leaves no mark on the scores, whether the sample has all of the rows
    that the launch is unrolled for or not (two samples, the second with fewer deciders)."""
    samples = []
    for N, n in ((90, D), (70, max(1, D - 3))):
        s = W.random_case(695 + N, N, H * dh, H, 2, N - 2 - n, n, dtype=dtype)
        s["q"][s["dec_idx"][n // 2], H - 1] = np.float32(2.0 ** 127)
        samples.append(s)
    for batch in (samples, samples[:1]):
        S = GpuStep(batch, [4] * len(batch), dtype).importance()
        for got, s in zip(S, batch):
            dec = s["dec_idx"]
            z = np.einsum("ihc,jhc->hij", s["q"][dec].astype(np.float64), s["k"].astype(np.float64)) / np.sqrt(dh)
            z[H - 1, len(dec) // 2] = 0.0
            e = np.exp(z - z.max(-1, keepdims=True))
            prob = e / e.sum(-1, keepdims=True)
            prob[H - 1, len(dec) // 2] = 0.0
            check_scores(got, prob.sum((0, 1))[s["vis_start"]:s["vis_start"] + s["V"]] / H)


@pytest.mark.parametrize("fill", [np.nan, np.inf])
@pytest.mark.parametrize("dtype,H,dh,D", [("bf16", 8, 64, 8), ("bf16", 16, 128, 16), ("bf16", 5, 128, 7), ("bf16", 3, 64, 40), ("f32", 4, 64, 16),
                                          ("bf16", 3, 40, 9), ("f32", 3, 36, 40)])
def test_importance_row_of_nan_reaches_the_scores(dtype, H, dh, D, fill):
    """A decider whose logits in one head are all NaN (NaN in its query, or infinities that cancel) makes its sample's scores NaN and no other's,
    whether the sample has all rows that the launch is unrolled for or not, with one chunk of keys and with several."""
    samples = []
    for N, n in ((90, D), (70, max(1, D - 3)), (1300, D)):
        s = W.random_case(697 + N, N, H * dh, H, 2, N - 2 - n, n, dtype=dtype)
        s["q"][s["dec_idx"][n // 2], H - 1] = fill
        samples.append(s)
    samples.append(W.random_case(698, 60, H * dh, H, 2, 58 - D, D, dtype=dtype))
    for batch in (samples, samples[:1], samples[2:3]):
        S = GpuStep(batch, [4] * len(batch), dtype).importance()
        for got, s in zip(S, batch):
            assert np.isnan(got).all() if s is not samples[-1] else np.isfinite(got).all()


@pytest.mark.parametrize("dtype,H,dh", [("f32", 4, 64), ("f32", 3, 36), ("bf16", 2, 40), ("f32", 400, 8)])
def test_importance_generic_kept_logits(dtype, H, dh):
    """Generic kernels: decider counts around the largest set whose first sweep leaves its probabilities (larger ones form their logits
    again), key counts around blocks of 16 and 256; with 400 heads more rows than the kept logits of the MFMA path may have."""
    shapes = [(40, 16, 1), (257, 239, 32), (256, 17, 5)]                   # tokens, visual, deciders
    for extra in (0, 1):
        samples = [W.random_case(640 + i, N, H * dh, H, 3, V, D + extra, dtype=dtype) for i, (N, V, D) in enumerate(shapes)]
        for s, (_, _, D) in zip(samples, shapes):
            s["dec_idx"] = np.resize(s["dec_idx"], D + extra).astype(np.int32)
            s["D"] = D + extra
        S = GpuStep(samples, [max(1, s["V"] // 4) for s in samples], dtype).importance()
        for i, s in enumerate(samples):
            check_scores(S[i], oracle.importance(s["q"], s["k"], s["dec_idx"], s["vis_start"], s["V"]))


@pytest.mark.parametrize("D", [3, 32, 33, 100])
@pytest.mark.parametrize("dtype,H,dh", [("f32", 4, 64), ("f32", 2, 256), ("f32", 3, 36), ("f32", 2, 132), ("bf16", 3, 96)])
def test_importance_generic_one_key_has_the_row(dtype, H, dh, D):
    """Every decider row goes to one key, whose logit of some thousands is next to the others' infinity: its probability is 1, however the
    logit was rounded, if the sum of exponentials holds the same logit.  (A logit formed in another order there is off by up to
    2^-11, and so is then the probability.)"""
    V, P = 140, 5
    s = W.random_case(880 + D, P + V + D, H * dh, H, P, V, D, dtype=dtype)
    s["dec_idx"] = np.arange(P + V, P + V + D, dtype=np.int32); s["D"] = D
    target = np.random.default_rng(D).permutation(V)[:D]
    s["q"] = W.round_to(s["q"] * np.float32(30), dtype)
    s["k"] = W.round_to(s["k"] * np.float32(10), dtype)
    s["k"][P + target] = s["q"][s["dec_idx"]]
    ref = np.zeros(V); ref[target] = 1.0
    np.testing.assert_allclose(oracle.importance(s["q"], s["k"], s["dec_idx"], P, V), ref, atol=1e-12)
    S = GpuStep([s], [4], dtype).importance()[0]
    np.testing.assert_allclose(S, ref, rtol=0, atol=2e-6)


@pytest.mark.parametrize("dtype,H,dh,D", [("bf16", 8, 64, 8), ("bf16", 5, 128, 13), ("bf16", 16, 64, 16), ("bf16", 257, 64, 1), ("bf16", 64, 64, 16),
                                          ("bf16", 35, 64, 31), ("bf16", 384, 64, 32), ("bf16", 385, 64, 32), ("bf16", 97, 128, 32),
                                          ("f32", 4, 64, 16), ("f32", 5, 36, 13), ("f32", 8, 32, 32), ("f32", 9, 32, 29)])
def test_importance_rows_per_thread(dtype, H, dh, D):
    """(head, decider) rows around what one, four and sixteen a thread take: 64, 65, 256, 257, 1024 and 1085 of them; 3104 and 12288 in several
    passes, the latter the most whose statistics fit into LDS, and 12320, which take a second sweep over the keys.  In float32 as many
    rows of probabilities for the generic path's sums."""
    samples = [W.random_case(690 + N, N, H * dh, H, 2, N - 2 - n, n, dtype=dtype) for N, n in ((70, D), (49, 1))]
    S = GpuStep(samples, [4, 4], dtype).importance()
    for i, s in enumerate(samples):
        check_scores(S[i], oracle.importance(s["q"], s["k"], s["dec_idx"], s["vis_start"], s["V"]))


@pytest.mark.parametrize("V,k", [(2100, 97), (2200, 96), (2300, 193), (3000, 900), (2801, 768)])
def test_merge_column_tiles_of_96(V, k):
    """Single samples whose cosine tiles fill one round with 96 kept slots per tile: k around multiples of 96 and 128."""
    c = W.random_case(500 + k, 5 + V + 6, 256, 2, 5, V, 3, dtype="bf16", centres=max(3, k // 3))
    _chain([c], [k], "bf16")


# ---- top-k in isolation: exact, ties, extremes ---------------------------------------------------------
def _topk_only(scores_list, ks):
    V = [len(s) for s in scores_list]
    lay = B.Layout(V, [0] * len(V), V, [[0]] * len(V), ks)
    sc = torch.from_numpy(np.concatenate(scores_list).astype(np.float32)).cuda()
    kept = torch.zeros(sum(ks), dtype=torch.int32, device="cuda")
    slot = torch.zeros(sum(V), dtype=torch.int32, device="cuda")
    B.d3tom_select_topk(sc, lay, kept, slot)
    torch.cuda.synchronize()
    return GpuStep.split(kept.cpu().numpy(), ks), GpuStep.split(slot.cpu().numpy(), V)


def test_topk_exact_including_ties_and_extremes():
    rng = np.random.default_rng(0)
    cases = [
        (rng.standard_normal(1).astype(np.float32), 1),
        (rng.standard_normal(1000).astype(np.float32), 1),
        (rng.standard_normal(1000).astype(np.float32), 1000),
        (rng.random(3645).astype(np.float32), 365),
        (np.round(rng.random(5000) * 8).astype(np.float32) / 8, 1234),          # heavy ties
        (np.zeros(777, np.float32), 100),                                      # all equal: lowest indices
        (np.concatenate([-rng.random(500), rng.random(500)]).astype(np.float32), 600),   # negative scores
        (rng.random(B.D3TOM_MAX_VISUAL).astype(np.float32) * 1e-6, 4000),      # largest supported |V|
        (np.float32(1.0) + rng.integers(0, 3, 4097).astype(np.float32) * np.float32(2 ** -23), 2048),  # 1-ulp apart
    ]
    kept, slot = _topk_only([c[0] for c in cases], [c[1] for c in cases])
    for (s, k), kg, sg in zip(cases, kept, slot):
        kr, sr = oracle.select_topk(s, k)
        np.testing.assert_array_equal(kg, kr)
        np.testing.assert_array_equal(sg, sr)


@pytest.mark.parametrize("V,k", [(1, 1), (1023, 77), (1024, 1), (1024, 1023), (1025, 300), (4095, 4095), (4096, 5), (4097, 2000)])
@pytest.mark.parametrize("ties", [False, True])
def test_topk_sizes_around_keys_per_thread(V, k, ties):
    """Largest samples around the numbers of keys that a thread holds, alone and with a sample of other size in front; few distinct values:
    the threshold's bin has more keys than are ranked at once, where there are that many."""
    rng = np.random.default_rng(V + k)
    both = [rng.integers(0, 3, n).astype(np.float32) if ties else rng.random(n).astype(np.float32) for n in (V, (V + 1) // 2)]
    for scores, ks in ((both[:1], [k]), (both[::-1], [(k + 1) // 2, k])):
        kept, slot = _topk_only(scores, ks)
        for s, kk, kg, sg in zip(scores, ks, kept, slot):
            kr, sr = oracle.select_topk(s, kk)
            np.testing.assert_array_equal(kg, kr)
            np.testing.assert_array_equal(sg, sr)


# ---- workspace -------------------------------------------------------------------------------------------
@pytest.mark.parametrize("P,V,O,D,k,d", [(8, 700, 16, 9, 150, 512),      # normal cosine path (several tiles)
                                          (4, 300, 8, 5, 40, 4096)])      # few tiles, long rows: split along k
def test_workspace_contents_do_not_matter(P, V, O, D, k, d):
    """The workspace carries no state: whatever bytes it holds on entry (zeros, all-ones = NaN / -1), the
    outputs are bit-identical."""
    c = W.random_case(11, P + V + O, d, d // 128, P, V, D, dtype="bf16", centres=30)
    runs = []
    for fill in (0, 255):
        step = GpuStep([c], [k], "bf16")
        step.ws_imp.fill_(fill); step.ws_merge.fill_(fill)
        S = step.importance()
        step.ws_imp.fill_(fill)
        kept, slot = step.select_topk()
        mout = step.merge()
        runs.append((S[0], kept[0], mout["y"][0], mout["assign"][0], mout["counts"][0], mout["src_pos"][0]))
    for a, b in zip(*runs):
        np.testing.assert_array_equal(a, b)


# ---- attention in isolation ---------------------------------------------------------------------------
@pytest.mark.parametrize("H,dh,dtype", [(4, 128, "bf16"), (3, 64, "bf16"), (2, 64, "f32"), (2, 40, "bf16")])
def test_attend_varlen(H, dh, dtype):
    lens = [1, 63, 64, 65, 200, 231, 493] if dh in (64, 128) and dtype == "bf16" else [1, 65, 300]
    qkv = [W.random_qkv(300 + n, n, H, dh, dtype) for n in lens]
    outs = gpu_attend(qkv, dtype)
    for (q, k, v), o in zip(qkv, outs):
        check_attend(o, q, k, v, dtype)


@pytest.mark.parametrize("longest", [512, 513])
@pytest.mark.parametrize("H,dh", [(5, 128), (3, 64)])
def test_attend_both_sides_of_the_short_sample_limit(H, dh, longest):
    """Up to 512 keys per sample the keys are split across the waves of a workgroup; one key more and the
    tiled kernel takes the whole batch, short samples included."""
    lens = [1, 31, 32, 33, 97, 129, longest]
    qkv = [W.random_qkv(700 + n, n, H, dh, "bf16") for n in lens]
    outs = gpu_attend(qkv, "bf16")
    for (q, k, v), o in zip(qkv, outs):
        check_attend(o, q, k, v, "bf16")


@pytest.mark.parametrize("rise", [0.0, 9.0])
@pytest.mark.parametrize("H,dh,weighted,lens", [
    (3, 128, False, [513, 640, 641, 1, 128, 129]),                  # few heads: 64-query tiles
    (3, 64, True, [577, 640, 64, 65]),
    (6, 128, False, [513, 640, 641, 1, 128, 129]),                  # 128-query tiles, one round of them
    (20, 64, True, [577, 640, 64, 65]),                             # (heads of 64: always, in a batch)
    (32, 64, True, [700, 513, 257, 64, 192, 193, 33, 128]),
    (32, 128, False, [513, 512, 257, 256, 255, 63, 1, 65]),         # enough heads for 256-query tiles
    (60, 64, True, [705]), (60, 64, False, [641]),
])
def test_attend_tile_widths_and_rising_logits(H, dh, weighted, lens, rise):
    """The query tile widths of the tiled kernel; with `rise` later keys exceed the first tile's largest logit by hundreds, so
    that the running maximum moves with almost every tile."""
    qkv = []
    for n in lens:
        q, k, v = W.random_qkv(800 + n, n, H, dh, "bf16")
        k = W.round_to(k * (1 + rise * np.arange(n, dtype=np.float32) / n)[:, None, None], "bf16")
        qkv.append((q, k, v))
    if weighted:
        vis = [n // 5 for n in lens]
        counts = [(1 + np.arange(n // 2) % 37).astype(np.int32) for n in lens]
        outs = gpu_attend_weighted(qkv, counts, vis, "bf16")
        for (q, k, v), o, vs, c in zip(qkv, outs, vis, counts):
            check_attend(o, q, k, v, "bf16", key_weight=key_weights(len(q), vs, c))
    else:
        for (q, k, v), o in zip(qkv, gpu_attend(qkv, "bf16")):
            check_attend(o, q, k, v, "bf16")


def _attend_rounded_probabilities(q, k, v, weight, tile=64, parts=1):
    """Attention as a kernel computes it whose only loss is the rounding of the probabilities to bf16, relative to the running
    maximum over tiles of keys, which `parts` waves or groups take in turn, each with a maximum of its own: float32 state, float32 row
    sums of the unrounded probabilities, output rounded to bf16."""
    out = torch.zeros(q.shape, dtype=torch.float32)
    qt, kt, vt, lw = torch.from_numpy(q), torch.from_numpy(k), torch.from_numpy(v), torch.from_numpy(np.log2(weight)).float()
    for h in range(q.shape[1]):
        s2 = qt[:, h] @ kt[:, h].T * (np.log2(np.e) / np.sqrt(q.shape[2])) + lw
        states = []
        for part in range(parts):
            m, l, acc = torch.full((len(q), 1), -np.inf), torch.zeros(len(q), 1), torch.zeros(len(q), q.shape[2])
            for j in range(part * tile, len(k), parts * tile):
                m_new = torch.maximum(m, s2[:, j:j + tile].amax(1, keepdim=True))
                p, alpha = torch.exp2(s2[:, j:j + tile] - m_new), torch.exp2(m - m_new)
                l, acc, m = l * alpha + p.sum(1, keepdim=True), acc * alpha + p.bfloat16().float() @ vt[j:j + tile, h], m_new
            states.append((m, l, acc))
        top = torch.stack([m for m, _, _ in states]).amax(0)
        f = [torch.exp2(m - top) for m, _, _ in states]
        out[:, h] = sum(acc * x for (_, _, acc), x in zip(states, f)) / sum(l * x for (_, l, _), x in zip(states, f))
    return out.bfloat16().double().numpy()


@pytest.mark.parametrize("spread", [1.0, 2.0, 4.0])
@pytest.mark.parametrize("H,dh,n,weighted,form", [(2, 128, 1300, False, "tiles 64"), (2, 64, 1300, False, "tiles 64"), (2, 128, 1300, True, "tiles 64"), (13, 128, 1300, False, "tiles 128"),
                                                  (32, 128, 1198, False, "tiles 192"), (32, 128, 1600, False, "tiles 256"), (32, 64, 1300, True, "tiles 256")])
def test_attend_error_is_that_of_rounded_probabilities(H, dh, n, weighted, form, spread):
    """The tiled kernel against float64, in 2-norm: no further off than the rounding of the probabilities against the running
    maximum makes it, with query tiles of 64 (two groups with a maximum each: the first three), 128, 192 and 256.  Both sides round almost the same probabilities, so the two errors agree to a fraction of a percent (the
    bound of 2 % leaves room for ties of the rounding); any fixed reference of the exponents is 4 % off at unit logit spread and
    8 to 15 % at 2 and 4.  `spread` is the standard deviation of the logits."""
    assert attend_form(H, [n], dh) == form
    q, k, v = W.random_qkv(870 + n + dh, n, H, dh, "bf16")
    q, k = (W.round_to(t * np.float32(np.sqrt(spread)), "bf16") for t in (q, k))
    vis, counts = n // 5, (1 + np.arange(n // 2) % 6).astype(np.int32)
    weight = key_weights(n, vis, counts) if weighted else np.ones(n)
    o = (gpu_attend_weighted([(q, k, v)], [counts], [vis], "bf16") if weighted else gpu_attend([(q, k, v)], "bf16"))[0]
    rows = np.arange(0, n, 1 if H == 2 else 9)
    ref = oracle.attend(q, k, v, rows=rows, key_weight=weight)[rows]
    off = lambda a: np.linalg.norm(a - ref) / np.linalg.norm(ref)
    got, bound = off(o.astype(np.float64)[rows]), off(_attend_rounded_probabilities(q[rows], k, v, weight, parts=2 if H == 2 else 1))
    print(f"attention error {got:.4e}, rounded probabilities {bound:.4e}, ratio {got / bound:.4f}")
    assert got <= 1.02 * bound


@pytest.mark.parametrize("spread", [1.0, 2.0, 4.0])
@pytest.mark.parametrize("H,dh,n,weighted,copies", [(8, 128, 100, False, 1), (16, 64, 128, True, 1), (32, 128, 231, True, 1), (32, 64, 256, False, 1),
                                                    (32, 128, 493, False, 1), (32, 128, 300, False, 4), (8, 64, 493, True, 3), (8, 128, 512, False, 16)])
def test_attend_error_of_short_samples(H, dh, n, weighted, copies, spread):
    """Samples of at most 512 keys, alone and in a batch: the error against float64 is that of probabilities rounded relative to four
    running maxima over tiles of 32 keys.  Both sides round almost the same probabilities, and the two errors agree to 1e-4; the bound
    of 1 % leaves room for ties of the rounding, while maxima over tiles of 64 keys are 1.2 to 5 % off, in two groups as well as in one."""
    q, k, v = W.random_qkv(875 + n + dh, n, H, dh, "bf16")
    q, k = (W.round_to(t * np.float32(np.sqrt(spread)), "bf16") for t in (q, k))
    vis, counts = n // 5, (1 + np.arange(n // 2) % 6).astype(np.int32)
    weight = key_weights(n, vis, counts) if weighted else np.ones(n)
    o = (gpu_attend_weighted([(q, k, v)] * copies, [counts] * copies, [vis] * copies, "bf16") if weighted else gpu_attend([(q, k, v)] * copies, "bf16"))[-1]
    q64, k64, v64 = (torch.from_numpy(t).double().transpose(0, 1).contiguous() for t in (q, k, v))
    s64 = torch.matmul(q64, k64.transpose(1, 2).contiguous()) / np.sqrt(dh) + torch.from_numpy(np.log(weight))
    ref = torch.matmul(torch.softmax(s64, -1), v64).transpose(0, 1).numpy()
    off = lambda a: np.linalg.norm(a - ref) / np.linalg.norm(ref)
    got, bound = off(o.astype(np.float64)), off(_attend_rounded_probabilities(q, k, v, weight, tile=32, parts=4))
    print(f"attention error {got:.4e}, rounded probabilities {bound:.4e}, ratio {got / bound:.4f}")
    assert got <= 1.01 * bound


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("H,dh,lens,queries", [
    (32, 128, [256], 32), (32, 128, [257], 32),                             # 256 tiles of 32 queries, and more
    (32, 128, [450], 64), (32, 128, [480], 64), (40, 128, [350], 64), (48, 128, [300], 64), (64, 128, [500], 64), (96, 64, [300], 64), (64, 64, [449], 64),
    (16, 64, [512], 32), (16, 64, [512, 300], 32), (17, 64, [512, 40], 32),                         # 512 tiles with heads of 64, and more
    (5, 128, [2], 32), (5, 128, [33], 32), (5, 64, [129], 32), (5, 128, [385], 32),         # one to four steps of four tiles, the last one with a single tile
    (9, 128, [1, 31, 32, 33, 63, 64, 65, 97, 127, 128, 129, 255, 384, 511], 32), (12, 64, [64, 1, 95, 96, 97, 130, 257, 512], 32),     # steps without tiles
])
def test_attend_short_samples_by_halves_of_64_queries(H, dh, lens, queries, weighted):
    """The short-sample kernel with 32 and with 64 queries to a workgroup, at the edges of tiles, halves and steps."""
    assert attend_form(H, lens, dh) == f"short {queries}"
    qkv = [W.random_qkv(1010 + n, n, H, dh, "bf16") for n in lens]
    vis, counts = [n // 5 for n in lens], [(1 + np.arange(n // 2) % 37).astype(np.int32) for n in lens]
    outs = gpu_attend_weighted(qkv, counts, vis, "bf16") if weighted else gpu_attend(qkv, "bf16")
    for (q, k, v), o, vs, c in zip(qkv, outs, vis, counts):
        n = len(q)
        rows = np.union1d(np.arange(0, n, 1 if n < 66 else 13), np.arange(max(n - 9, 0), n))
        check_attend(o, q, k, v, "bf16", rows=rows, key_weight=key_weights(n, vs, c) if weighted else None)


@pytest.mark.parametrize("H,dh,longest,batch,weighted", [
    (5, 128, 300, 40, False),            # several rounds of 128-query tiles, heads that do not divide among the XCDs
    (5, 128, 600, 32, True),             # ... of 256-query tiles
    (9, 128, 1030, 16, False), (9, 128, 1030, 16, True),
    (44, 64, 2550, 1, False), (44, 64, 2550, 1, True),          # heads of 64: only one sample has 256-query tiles
    (44, 64, 2813, 1, True),                                    # ... where they save rounds
    (9, 64, 1030, 16, False), (9, 64, 1030, 16, True),          # ... and a batch one workgroup per 128-query tile
    (12, 128, 520, 64, False), (12, 128, 520, 65, False),       # as many samples as a wave has lanes, one more
    (12, 128, 100, 65, False), (12, 128, 100, 66, True),        # one workgroup per 128-query tile, several rounds
    (9, 64, 100, 65, False), (9, 64, 130, 65, True),
])
def test_attend_tiles_in_turn(H, dh, longest, batch, weighted):
    """Ragged batches of several rounds, from samples of one key to the longest: a workgroup takes one tile after the other, or (more than
    64 samples; 128-query tiles with heads of 64) has one, and waves without a query skip their products."""
    edge = [longest, 1, 2, 63, 64, 65, 127, 128, 129, 192, 193, 255, 256, 257]
    lens = [min(longest, n) for n in (edge + [17 + 37 * i % longest for i in range(batch)])[:batch]]
    lens = lens[batch // 2:] + lens[:batch // 2]
    base = W.random_qkv(880 + dh, longest, H, dh, "bf16")
    qkv = [tuple(np.roll(t, i, axis=0)[:n] for t in base) for i, n in enumerate(lens)]
    vis, counts = [n // 5 for n in lens], [(1 + np.arange(n // 2) % 37).astype(np.int32) for n in lens]
    outs = gpu_attend_weighted(qkv, counts, vis, "bf16") if weighted else gpu_attend(qkv, "bf16")
    for i, ((q, k, v), o, vs, c) in enumerate(zip(qkv, outs, vis, counts)):
        rows = np.arange(0, len(q), 1 if len(q) < 130 else 7)
        check_attend(o, q, k, v, "bf16", rows=np.union1d(rows, [len(q) - 1]), key_weight=key_weights(len(q), vs, c) if weighted else None)


def _drawn_lengths(seed, choices=(1, 64, 65, 128, 129, 192, 193, 256, 257, 320, 384, 385, 520, 300)):
    import random
    r = random.Random(seed)
    r.choice([31, 32, 30])
    return [r.choice(choices) for _ in range(32)]


def _last_tiles_apart(H, lens, width):
    """The kernel's estimate: whether last tiles with at most half of their queries are items of their own behind all others."""
    P = sum(-(-n // width) for n in lens) * H // 8
    S = sum(0 < n % width <= width // 2 for n in lens) * H // 8
    among, full = -(-P // 32), -(-(P - S) // 32)
    free = full * 32 - (P - S)
    return len(lens) <= 32 and S > 0 and full + 0.72 * (-(-(S - free) // 32) if S > free else 0) <= 0.99 * among * (P - 0.28 * S) / P


@pytest.mark.parametrize("H,dh,lens,weighted,form", [
    (40, 128, [1540], False, "tiles 128 in turn"), (40, 128, [1566], True, "tiles 128 in turn"), (32, 128, [650] * 3, False, "tiles 128 in turn"),
    (64, 128, [4098], False, "tiles 256 in turn"), (128, 128, [2050], True, "tiles 256 in turn"),
    (20, 128, [1025, 1030, 260, 300, 513], True, "tiles 256 in turn"),
    (9, 128, _drawn_lengths(9), True, "tiles 256 in turn"), (13, 128, _drawn_lengths(393), False, "tiles 256 in turn"), (12, 128, _drawn_lengths(352), False, "tiles 256 in turn"),     # as many samples as have two places
    (20, 64, [1025, 1030, 260, 300, 513], True, "tiles 128"), (12, 64, _drawn_lengths(352), False, "tiles 128"),      # (heads of 64 in a batch: every tile for itself)
])
def test_attend_short_last_tiles_behind_the_others(H, dh, lens, weighted, form):
    """Lengths at which the last tiles with at most half of their queries are items of their own behind all others (the estimate of the
    passes over an XCD's 32 units says so), heads that do not divide among the XCDs too: every row has to be there."""
    assert attend_form(H, lens, dh) == form and ("turn" not in form or _last_tiles_apart(H, lens, int(form.split()[1])))
    base = W.random_qkv(930 + H, max(lens), H, dh, "bf16")
    qkv = [tuple(np.roll(t, i, axis=0)[:n] for t in base) for i, n in enumerate(lens)]
    vis, counts = [n // 5 for n in lens], [(1 + np.arange(n // 2) % 37).astype(np.int32) for n in lens]
    outs = gpu_attend_weighted(qkv, counts, vis, "bf16") if weighted else gpu_attend(qkv, "bf16")
    for (q, k, v), o, vs, c in zip(qkv, outs, vis, counts):
        n = len(q)
        rows = np.union1d(np.arange(0, n, 1 if n < 66 else 41), np.arange(max(n - 12, 0), n))
        check_attend(o, q, k, v, "bf16", rows=rows, key_weight=key_weights(n, vs, c) if weighted else None)


@pytest.mark.parametrize("H,dh,n,weighted,form", [
    (60, 128, 770, False, "tiles 256"), (60, 128, 896, True, "tiles 256"), (60, 128, 897, False, "tiles 256"), (60, 64, 705, True, "tiles 256"), (60, 64, 737, False, "tiles 256"),
    (60, 128, 520, False, "tiles 192"), (60, 128, 640, True, "tiles 192"), (60, 128, 641, False, "tiles 192"),
    (32, 128, 520, False, "tiles 128"), (32, 128, 560, True, "tiles 128"),
    (2, 128, 513, False, "tiles 64"), (2, 128, 560, True, "tiles 64"), (2, 64, 656, False, "tiles 64")])
def test_attend_last_tile_with_few_queries(H, dh, n, weighted, form):
    """One round of tiles whose last one leaves waves without a query: with 256 queries those only load and keep step, with fewer they compute
    with rows that are zero and store nothing."""
    assert attend_form(H, [n], dh) == form
    q, k, v = W.random_qkv(910 + n, n, H, dh, "bf16")
    vs, c = n // 5, (1 + np.arange(n // 2) % 37).astype(np.int32)
    o = (gpu_attend_weighted([(q, k, v)], [c], [vs], "bf16") if weighted else gpu_attend([(q, k, v)], "bf16"))[0]
    rows = np.union1d(np.arange(0, n, 31), np.arange(max(n - 9, 0), n))
    check_attend(o, q, k, v, "bf16", rows=rows, key_weight=key_weights(n, vs, c) if weighted else None)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("rise", [0.0, 9.0])
@pytest.mark.parametrize("H,dh,lens", [
    (3, 128, [65]), (2, 128, [127]), (2, 128, [128]), (2, 64, [129]), (2, 128, [191]), (2, 64, [192]), (2, 128, [193]),     # (for the short-sample kernel)
    (3, 128, [513]), (2, 128, [575]), (2, 64, [576]), (2, 128, [577]), (2, 64, [639]), (2, 128, [640]), (2, 64, [641]),      # odd and even numbers of tiles
    (2, 64, [513, 1, 64, 65, 66, 127, 128]), (2, 128, [520, 129, 191, 192, 193, 256]),      # one and two tiles of keys a group
    (2, 128, [520, 577, 641, 1, 63, 64, 65, 129]),      # samples without a tile for group 1, a last tile of it past the end
    (5, 64, [700, 130, 2, 66, 127, 320]),
    (1, 128, [2050]), (9, 64, [1030]),
    (32, 128, [520]), (36, 64, [520, 300]), (130, 64, [128]), (2, 128, [64]), (3, 64, [33]),      # 128-query tiles, one round of them
])
def test_attend_groups_that_share_queries(H, dh, lens, rise, weighted):
    """64-query tiles whose two groups of waves take the tiles of keys in turn, at the edges of tiles and of pairs of tiles, and the one
    round of 128-query tiles that is left beside them.  With `rise` later keys exceed earlier ones by far, so that one group's part of a row
    outweighs the other's; reversed rows the other way round."""
    qkv = []
    for i, n in enumerate(lens):
        q, k, v = W.random_qkv(990 + n, n, H, dh, "bf16")
        up = np.arange(n, dtype=np.float32) / n
        k = W.round_to(k * (1 + rise * (up if i % 2 == 0 else up[::-1]))[:, None, None], "bf16")
        qkv.append((q, k, v))
    vis, counts = [n // 5 for n in lens], [(1 + np.arange(n // 2) % 37).astype(np.int32) for n in lens]
    outs = gpu_attend_weighted(qkv, counts, vis, "bf16") if weighted else gpu_attend(qkv, "bf16")
    for (q, k, v), o, vs, c in zip(qkv, outs, vis, counts):
        n = len(q)
        rows = np.union1d(np.arange(0, n, 1 if n < 66 else 13), np.arange(max(n - 9, 0), n))
        check_attend(o, q, k, v, "bf16", rows=rows, key_weight=key_weights(n, vs, c) if weighted else None)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("rise", [0.0, 9.0])
@pytest.mark.parametrize("H,lens,form", [
    (32, [1025], "tiles 192"), (32, [1152], "tiles 192"), (32, [1153], "tiles 192"), (32, [1281], "tiles 192"), (32, [1536], "tiles 192"), (40, [1040], "tiles 192"),   # last tiles of 65 to 192 queries, one round
    (32, [700, 129], "tiles 192"), (32, [1, 700], "tiles 192"), (16, [768, 193, 64, 1], "tiles 192"), (16, [129, 700, 1, 128], "tiles 192"), (3, [700, 193] * 8, "tiles 192"),      # ragged, samples of one tile
    (32, [2049], "tiles 192 in turn"), (32, [2113], "tiles 192 in turn"), (36, [1631], "tiles 192 in turn"), (64, [1409], "tiles 192 in turn"),
    (32, [700, 1, 128, 129], "tiles 128 in turn"), (64, [513, 144], "tiles 128 in turn"),       # beside them: a batch of more than one round,
    (60, [769], "tiles 256"), (32, [1537], "tiles 256"), (33, [3072], "tiles 256 in turn"),     # one sample that takes a round more
])
def test_attend_tiles_of_192_queries(H, lens, form, rise, weighted):
    """Two query blocks to a wave of one group of waves, one to a wave of the other: every row around the borders between waves, groups and tiles.  With `rise` later
    keys exceed earlier ones by far, and the running maximum of every block moves with almost every tile."""
    dh = 128
    assert attend_form(H, lens, dh) == form
    base = W.random_qkv(960 + H, max(lens), H, dh, "bf16")
    qkv = [tuple(np.roll(t, i, axis=0)[:n] for t in base) for i, n in enumerate(lens)]
    qkv = [(q, W.round_to(k * (1 + rise * np.arange(len(k), dtype=np.float32) / len(k))[:, None, None], "bf16"), v) for q, k, v in qkv]
    vis, counts = [n // 5 for n in lens], [(1 + np.arange(n // 2) % 37).astype(np.int32) for n in lens]
    outs = gpu_attend_weighted(qkv, counts, vis, "bf16") if weighted else gpu_attend(qkv, "bf16")
    for (q, k, v), o, vs, c in zip(qkv, outs, vis, counts):
        n = len(q)
        edges = [r for t in range(0, n, 192) for r in (t, t + 31, t + 32, t + 127, t + 128, t + 143, t + 144, t + 191)]
        rows = np.array(sorted({r for r in edges if r < n} | set(range(max(n - 9, 0), n))))
        check_attend(o, q, k, v, "bf16", rows=rows, key_weight=key_weights(n, vs, c) if weighted else None)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("rise", [0.0, 9.0])
@pytest.mark.parametrize("H,dh,n,batches", [
    (32, 128, 1100, [(1, "tiles 192"), (2, "tiles 128 in turn"), (3, "tiles 256 in turn")]),
    (20, 128, 1300, [(1, "tiles 192"), (2, "tiles 256"), (3, "tiles 128 in turn"), (4, "tiles 256 in turn")]),
    (60, 64, 705, [(1, "tiles 256"), (2, "tiles 128")]),
    (32, 128, 493, [(1, "short 64"), (2, "short 32")]), (64, 64, 500, [(1, "short 64"), (2, "short 32")]),
])
def test_attend_bits_do_not_depend_on_the_width_of_the_tiles(H, dh, n, batches, rise, weighted):
    """Tiles of 128, 192 and 256 queries add a row's products alike, and so do the short-sample kernel's of 32 and 64: a sample has the same bits alone and beside others.
    (A stack relies on it in front of its merge.)"""
    q, k, v = W.random_qkv(1100 + n, n, H, dh, "bf16")
    k = W.round_to(k * (1 + rise * np.arange(n, dtype=np.float32) / n)[:, None, None], "bf16")
    vis, counts = n // 5, (1 + np.arange(n // 2) % 37).astype(np.int32)
    outs = []
    for copies, form in batches:
        assert attend_form(H, [n] * copies, dh) == form
        qkv = [(q, k, v)] * copies
        outs += gpu_attend_weighted(qkv, [counts] * copies, [vis] * copies, "bf16") if weighted else gpu_attend(qkv, "bf16")
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])


def test_attend_special_cases_bf16():
    q, k, v = W.random_qkv(5, 150, 2, 128, "bf16", spread=2.0)
    v1 = np.broadcast_to(v[:1], v.shape).copy()
    o = gpu_attend([(q, k, v1)], "bf16")[0]
    np.testing.assert_allclose(o, v1, atol=1e-2)            # identical value rows come back (rows sum to one)
    perm = np.random.default_rng(1).permutation(150)
    o1 = gpu_attend([(q, k, v)], "bf16")[0]
    o2 = gpu_attend([(q, k[perm], v[perm])], "bf16")[0]
    np.testing.assert_allclose(o1, o2, atol=2e-2)           # no mask: key order is irrelevant


# ---- size-weighted attention (member counts of the merge as key weights) -------------------------------
@pytest.mark.parametrize("H,dh,dtype,lens", [
    (4, 128, "bf16", [700, 65, 1300]),          # tiled kernel, ragged
    (3, 64, "bf16", [300, 1, 512, 33]),         # short-sample kernel
    (2, 64, "f32", [90, 17]),                   # generic kernel, float32
    (2, 40, "bf16", [70]),                      # generic kernel, odd head size
])
def test_attend_weighted_varlen(H, dh, dtype, lens):
    rng = np.random.default_rng(len(lens) * 100 + dh)
    qkv = [W.random_qkv(900 + n, n, H, dh, dtype) for n in lens]
    vis, counts = [], []
    for n in lens:
        vs = int(rng.integers(0, max(1, n // 3)))
        kn = int(rng.integers(0, n - vs + 1))          # merged rows: anything from none to the rest of the sample
        vis.append(vs)
        counts.append(rng.integers(1, 40, size=kn).astype(np.int32))
    outs = gpu_attend_weighted(qkv, counts, vis, dtype)
    plain = gpu_attend(qkv, dtype)
    for (q, k, v), o, o1, vs, c, n in zip(qkv, outs, plain, vis, counts, lens):
        check_attend(o, q, k, v, dtype, key_weight=key_weights(n, vs, c))
        if len(c) and c.max() > 1 and n > 1:
            assert np.abs(o - o1).max() > 1e-3          # the weights do change the result
    # all counts 1: the plain attention, bit for bit (same kernel arithmetic up to the added zero)
    ones = [np.ones(len(c), np.int32) for c in counts]
    for o, o1 in zip(gpu_attend_weighted(qkv, ones, vis, dtype), plain):
        np.testing.assert_allclose(o, o1, atol=TOL_SAME[dtype])


TOL_SAME = {"bf16": 2.0 ** -7, "f32": 1e-5}


@pytest.mark.parametrize("H,dh,lens", [
    (4, 64, [192]),                 # one query a workgroup: the last size of a single round
    (4, 64, [193]),                 # two: the last workgroup holds one query
    (4, 64, [256]), (4, 64, [257]),             # two, one; one and two chunks of keys
    (4, 64, [511, 1, 300]),         # two: ragged, a sample of one query
    (2, 36, [601, 90]), (3, 256, [300]),        # two: chunks of the channels that do not divide the threads, the widest head
])
def test_generic_queries_per_workgroup(H, dh, lens):
    rng = np.random.default_rng(sum(lens) + dh)
    qkv = [W.random_qkv(70 + n, n, H, dh, "f32") for n in lens]
    counts = [rng.integers(1, 40, size=n // 2).astype(np.int32) for n in lens]
    vis = [n // 4 for n in lens]
    for (q, k, v), o, w, vs, c, n in zip(qkv, gpu_attend(qkv, "f32"), gpu_attend_weighted(qkv, counts, vis, "f32"), vis, counts, lens):
        check_attend(o, q, k, v, "f32")
        check_attend(w, q, k, v, "f32", key_weight=key_weights(n, vs, c))


def test_merge_counts_feed_weighted_attention():
    """The counts d3tom_merge writes are what d3tom_attend_weighted reads: merge a sample, project the merged rows
    (host, not on the path), attend with the counts as key weights, compare with the oracle given the same weights."""
    wl = W.WORKLOADS["tiny_f32"]
    g = W.SampleGen(wl)
    s = g.step(16)
    k = oracle.keep_count(wl.V, 0.25)
    step, S, kept, mout, stats = _chain([s], [k], "f32")
    q2, k2, v2 = g.proj.qkv(mout["y"][0])
    n_m = q2.shape[0]
    cu = torch.tensor([0, n_m], dtype=torch.int32, device="cuda")
    o = torch.zeros((n_m,) + q2.shape[1:], dtype=torch.float32, device="cuda")
    B.d3tom_attend_weighted(B.to_device(q2, "f32"), B.to_device(k2, "f32"), B.to_device(v2, "f32"), cu, n_m,
                            1.0 / np.sqrt(q2.shape[2]), step.counts, step.lay.kept_off, step.lay.vis_start, o)
    torch.cuda.synchronize()
    assert mout["counts"][0].sum() == wl.V
    check_attend(B.to_host(o), q2, k2, v2, "f32", key_weight=key_weights(n_m, s["vis_start"], mout["counts"][0]))


# ---- the merge layer in one call, kept counts computed on the device --------------------------------------
@pytest.mark.parametrize("tight", [True, False])
def test_merge_layer_one_call_with_device_side_keep_counts(tight):
    """d3tom_merge_layer against the three separate calls on a ragged batch: the kept counts it computes on the
    device from the ratios are those of d3tom_keep_count (and of the oracle), and with tight bounds on them every
    output is bit-identical to the separate calls; with the loosest bounds (1 .. |V|) the launches are shaped
    differently, so the outputs are checked against the oracle instead."""
    shapes = [(20, 300, 30, 9, 0.2), (64, 513, 64, 33, 0.5), (1, 128, 5, 1, 0.1), (7, 129, 300, 20, 1.0 / 3.0), (0, 64, 2, 2, 1.0),
              (3, 700, 9, 4, 0.25)]
    samples, ratios = [], []
    for i, (P, V, O, D, keep) in enumerate(shapes):
        samples.append(W.random_case(300 + i, P + V + O, 4 * 128, 4, P, V, D, dtype="bf16", centres=max(3, V // 5)))
        ratios.append(keep)
    keeps = [oracle.keep_count(s["V"], r) for s, r in zip(samples, ratios)]
    assert keeps == [B.d3tom_keep_count(s["V"], r) for s, r in zip(samples, ratios)]
    ref = GpuStep(samples, keeps, "bf16")
    S = ref.importance(); kept, slot = ref.select_topk(); mout = ref.merge()
    lay = ref.lay
    nb = lay.B
    dev_i32 = lambda n: torch.full((n,), -7, dtype=torch.int32, device="cuda")
    scores = torch.zeros(lay.sum_V, dtype=torch.float32, device="cuda")
    keep_k, kept_off, out_off = dev_i32(nb), dev_i32(nb + 1), dev_i32(nb + 1)
    kept_idx = dev_i32(nb * lay.max_V)
    y = torch.zeros((lay.sum_N, ref.d), dtype=torch.bfloat16, device="cuda")
    assign, counts, src_pos = dev_i32(lay.sum_V), dev_i32(nb * lay.max_V), dev_i32(lay.sum_N)
    ws = B.workspace(B.d3tom_merge_layer_workspace_bytes(nb, lay.max_N, lay.max_V, ref.H, ref.dh, lay.max_D))
    ws.fill_(255)
    lo, hi = (min(keeps), max(keeps)) if tight else (1, lay.max_V)
    B.d3tom_merge_layer(ref.q, ref.k, ref.x, None, lay, ref.scale, torch.tensor(ratios, dtype=torch.float64, device="cuda"),
                        lo, hi, B.D3TOM_MERGE_MEAN, scores, keep_k, kept_off, kept_idx, out_off, y, assign, counts, src_pos, ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(keep_k.cpu().numpy(), keeps)
    np.testing.assert_array_equal(kept_off.cpu().numpy(), np.concatenate([[0], np.cumsum(keeps)]))
    np.testing.assert_array_equal(out_off.cpu().numpy(), np.concatenate([[0], np.cumsum(lay.Nm)]))
    np.testing.assert_array_equal(scores.cpu().numpy(), np.concatenate(S))
    np.testing.assert_array_equal(kept_idx[:lay.sum_keep].cpu().numpy(), np.concatenate(kept))
    got = dict(y=GpuStep.split(B.to_host(y[:lay.sum_Nm]), lay.Nm), assign=GpuStep.split(assign.cpu().numpy(), lay.V),
               counts=GpuStep.split(counts[:lay.sum_keep].cpu().numpy(), lay.keep),
               src_pos=GpuStep.split(src_pos[:lay.sum_Nm].cpu().numpy(), lay.Nm))
    for b in range(nb):
        if tight:
            for key in got:
                np.testing.assert_array_equal(got[key][b], mout[key][b])
        else:
            check_full_sample(ref, b, S, kept, slot, got)


@pytest.mark.parametrize("dtype,d,H,shapes", [
    ("f32", 96, 2, [(5, 90, 7, 3, 0.3), (0, 33, 4, 2, 0.5), (9, 200, 1, 6, 0.12)]),       # float32: the generic kernels
    ("bf16", 4096, 32, [(8, 260, 6, 3, 0.15)]),                                           # one short sample: cosine GEMM cut along the contraction
    ("bf16", 200, 5, [(3, 150, 5, 4, 0.4), (6, 61, 2, 1, 0.7)]),                          # bf16 rows of 400 bytes, head size 40: generic kernels
])
def test_merge_layer_one_call_on_every_kernel_path(dtype, d, H, shapes):
    """The one-call merge layer prepares the merge inside its selection launch (row norms by token, pruned list,
    token table); every cosine kernel reads that form (a split contraction its list and table only).  Each path against the
    separate calls, bit for bit, and the separate calls against the oracle."""
    samples, ratios = [], []
    for i, (P, V, O, D, keep) in enumerate(shapes):
        samples.append(W.random_case(500 + i, P + V + O, d, H, P, V, D, dtype=dtype, centres=max(3, V // 6)))
        ratios.append(keep)
    keeps = [oracle.keep_count(s["V"], r) for s, r in zip(samples, ratios)]
    ref = GpuStep(samples, keeps, dtype)
    S = ref.importance(); kept, slot = ref.select_topk(); mout = ref.merge()
    for b in range(len(samples)):
        check_full_sample(ref, b, S, kept, slot, mout)
    S1, kept1, m1 = ref.merge_layer(ratios)
    for b in range(len(samples)):
        np.testing.assert_array_equal(S1[b], S[b])
        np.testing.assert_array_equal(kept1[b], kept[b])
        for key in m1:
            np.testing.assert_array_equal(m1[key][b], mout[key][b])


@pytest.mark.parametrize("shapes", [
    [(3, 300, 5, 2, 128.4 / 300), (2, 301, 4, 3, 129 / 301), (4, 260, 4, 1, 258 / 260)],       # one, two and three column tiles
    [(6, 700, 9, 4, 640 / 700), (5, 640, 3, 2, 513 / 640)],                                    # five: a second turn for one wave
])
def test_merge_split_contraction_waves_per_row(shapes):
    """Cosines cut along the contraction: kept counts around multiples of the 128-slot tiles and of four tiles (one per wave of a
    pruned row), both through the one call and through the separate ones."""
    samples = [W.random_case(520 + i, P + V + O, 2048, 16, P, V, D, dtype="bf16", centres=max(3, V // 6)) for i, (P, V, O, D, _) in enumerate(shapes)]
    ratios = [r for *_, r in shapes]
    ref = GpuStep(samples, [oracle.keep_count(s["V"], r) for s, r in zip(samples, ratios)], "bf16")
    S = ref.importance(); kept, slot = ref.select_topk(); mout = ref.merge()
    S1, kept1, m1 = ref.merge_layer(ratios)
    for b in range(len(samples)):
        check_full_sample(ref, b, S, kept, slot, mout)
        check_full_sample(ref, b, S1, kept1, slot, m1)


@pytest.mark.parametrize("d,shapes", [
    (4096, [(130, 20)]), (4096, [(400, 50)]), (4096, [(640, 200), (90, 30)]),            # 16, 8 and 4 slices, one and two column tiles
    (2048, [(200, 30)]), (2048, [(900, 200)]), (2048, [(900, 300), (64, 63)]),           # 8, 4 and 2
    (1024, [(300, 90), (129, 1)]), (1024, [(1300, 500)]), (512, [(300, 129)]),           # 4, 2 and 2
])
def test_merge_slices_of_the_contraction(d, shapes):
    """Every number of slices that short samples have their contraction cut into, with one, two and more column tiles: assignments and rows
    against the oracle."""
    samples = [W.random_case(760 + V + k, V + 5, d, d // 128, 5, V, 1, dtype="bf16", centres=max(2, V // 6)) for V, k in shapes]
    rng = np.random.default_rng(d)
    kept = [np.sort(rng.choice(V, size=k, replace=False)).astype(np.int32) for V, k in shapes]
    out = GpuStep(samples, [k for _, k in shapes], "bf16").merge(kept)
    for b, s in enumerate(samples):
        check_assign(out["assign"][b], s["x"], s["vis_start"], s["V"], kept[b])
        check_merge({key: out[key][b] for key in out}, s["x"], s["vis_start"], s["V"], kept[b], "bf16")


def test_merge_bounds_that_split_the_contraction_differently():
    """A ragged batch whose tight bounds on kept and pruned counts (separate calls) cut the contraction into slices while the looser ones of the one
    call do not: the sums' last bits may differ then, and both are held to the oracle's rule for near-ties."""
    shapes = [(4, 1000, 6, 3, 0.9), (9, 300, 5, 2, 0.1)]
    samples = [W.random_case(860 + i, P + V + O, 2048, 16, P, V, D, dtype="bf16", centres=V // 6) for i, (P, V, O, D, _) in enumerate(shapes)]
    ratios = [r for *_, r in shapes]
    ref = GpuStep(samples, [oracle.keep_count(s["V"], r) for s, r in zip(samples, ratios)], "bf16")
    assert ref.lay.max_pruned == 270 and ref.lay.max_V - min(ref.lay.keep) == 970
    S = ref.importance(); kept, slot = ref.select_topk(); mout = ref.merge()
    S1, kept1, m1 = ref.merge_layer(ratios)
    for b in range(len(samples)):
        check_full_sample(ref, b, S, kept, slot, mout)
        check_full_sample(ref, b, S1, kept1, slot, m1)


@pytest.mark.parametrize("dtype,H,dh,V,D", [
    ("f32", 4, 32, 255, 32), ("f32", 4, 64, 256, 16), ("f32", 4, 32, 257, 16), ("f32", 1, 64, 1, 1), ("f32", 3, 36, 200, 30), ("f32", 43, 4, 100, 3),
    ("f32", 3, 32, 90, 33), ("f32", 1, 64, 1030, 3), ("f32", 2, 32, 520, 20), ("bf16", 5, 40, 130, 24), ("bf16", 2, 136, 700, 9),
])
def test_importance_generic_scores_from_probabilities(dtype, H, dh, V, D):
    """Generic kernels: (head, decider) rows around 16, 64 and 128, decider counts around 32, visual tokens around 64 and the 256 whose scores the
    one call's selection forms, tokens around the 256, 512 and 1024 of a workgroup.  A second sample has fewer deciders and tokens.  Against
    the oracle, and the one call against the separate calls bit for bit."""
    samples = [W.random_case(850 + V, V + D + 3, H * dh, H, 1, V, D, dtype=dtype, centres=max(2, V // 8)),
               W.random_case(851, 12, H * dh, H, 3, 6, 2 if D > 1 else 1, dtype=dtype)]
    keeps = [oracle.keep_count(s["V"], 0.3) for s in samples]
    step, S, kept, mout, _ = _chain(samples, keeps, dtype)
    S1, kept1, m1 = step.merge_layer([0.3, 0.3])
    for b in range(2):
        np.testing.assert_array_equal(S1[b], S[b])
        np.testing.assert_array_equal(kept1[b], kept[b])
        for key in m1:
            np.testing.assert_array_equal(m1[key][b], mout[key][b])


@pytest.mark.parametrize("dtype,d,H", [("bf16", 512, 4), ("bf16", 4096, 32), ("f32", 96, 2), ("f32", 2048, 16)])
def test_merge_layer_one_call_with_more_rows_than_expected(dtype, d, H):
    """Samples with more output rows than the longest one without the longest visual part has: their workgroups take several rows (a merged one,
    then copied ones, or another merged one; one or two workgroups a row).  Against the separate calls, bit for bit."""
    shapes = [(2, 300, 3, 2, 0.02), (40, 20, 90, 3, 0.5), (0, 31, 250, 1, 1.0), (1, 100, 2, 2, 0.9)]
    samples = [W.random_case(810 + i, P + V + O, d, H, P, V, D, dtype=dtype) for i, (P, V, O, D, _) in enumerate(shapes)]
    ratios = [r for *_, r in shapes]
    ref = GpuStep(samples, [oracle.keep_count(s["V"], r) for s, r in zip(samples, ratios)], dtype)
    ref.importance(); kept, _ = ref.select_topk(); mout = ref.merge()
    _, kept1, m1 = ref.merge_layer(ratios)
    for b in range(len(samples)):
        np.testing.assert_array_equal(kept1[b], kept[b])
        for key in m1:
            np.testing.assert_array_equal(m1[key][b], mout[key][b])


@pytest.mark.parametrize("kv", [False, True])
@pytest.mark.parametrize("d", [256, 4096])               # one workgroup a row, two half rows
def test_merge_writes_no_more_rows_than_max_out(d, kv):
    """A sample whose visual count on the device exceeds the stated max_V is clamped: its other visual tokens are then not
    merged away and would be rows of the output, but the outputs have max_out rows.  The rows behind those are as they were (the
    buffers of this test have room for every token, so that nothing outside them is ever at stake)."""
    P, V, O, D = 9, 400, 7, 2
    c = W.random_case(905, P + V + O, d, d // 64, P, V, D, dtype="bf16")
    lay = B.Layout([c["N"]], [P], [V], [c["dec_idx"]], [40])
    max_V, max_out = 100, P + 40 + O
    kept = torch.arange(40, dtype=torch.int32, device="cuda")
    x = B.to_device(c["x"], "bf16")
    full = lambda *shape, dtype=torch.int32: torch.full(shape, -7, dtype=dtype, device="cuda")
    y, v_out = (full(c["N"], d, dtype=torch.bfloat16) for _ in range(2))
    assign, counts, src = full(V), full(40), full(c["N"])
    lay.max_V, lay.max_pruned, lay.max_Nm = max_V, max_V - 40, max_out
    ws = B.workspace(B.d3tom_workspace_bytes(B.D3TOM_OP_MERGE, 1, lay.max_N, max_V, 1, d, D))
    if kv:
        B.d3tom_merge_kv(x, x.flip(0), lay, kept, B.D3TOM_MERGE_MEAN, y, v_out, assign, counts, src, ws)
    else:
        B.d3tom_merge(x, None, lay, kept, B.D3TOM_MERGE_MEAN, y, assign, counts, src, ws)
    torch.cuda.synchronize()
    assert torch.equal(y[:P], x[:P])
    assert bool((y[max_out:] == -7).all()) and bool((v_out[max_out:] == -7).all()) and bool((src[max_out:] == -7).all())
    assert bool((assign[max_V:] == -7).all())


@pytest.mark.parametrize("dtype,d,H,V,k", [
    ("bf16", 4096, 32, 300, 100),         # contraction cut in 16
    ("bf16", 2048, 16, 700, 513),         # cut in 2, five column tiles
    ("bf16", 512, 4, 2400, 1000),         # not cut
    ("bf16", 200, 5, 300, 100),           # generic kernels
    ("f32", 256, 4, 300, 100),
])
def test_merge_layer_one_call_breaks_ties_like_the_separate_calls(dtype, d, H, V, k):
    """Kept rows that are the same up to the order of the elements inside blocks, pruned rows constant on such blocks: all
    cosines of a pruned row are equal, and which slot wins goes by the last bit of dot products and norms (elements of very
    different size, so that sums in another order round otherwise).  The one call has to decide every one of them as the
    separate calls do."""
    P, blk = 5, 40 if d == 200 else 128
    c = W.random_case(540 + d, P + V + 6, d, H, P, V, 3, dtype=dtype)
    ref = GpuStep([c], [k], dtype)
    ref.importance(); kept, slot = ref.select_topk()
    rng = np.random.default_rng(541)
    x = c["x"].copy()
    base = ((1 + rng.random((d // blk, blk))) * 2.0 ** rng.integers(-8, 3, (d // blk, blk))).astype(np.float32)
    x[P:P + V] = np.repeat(rng.standard_normal((V, d // blk)).astype(np.float32), blk, axis=1)
    x[P + kept[0]] = np.stack([rng.permuted(base, axis=1).reshape(d) for _ in range(k)])
    ref.x.copy_(B.to_device(W.round_to(x, dtype), dtype))
    mout = ref.merge()
    S1, kept1, m1 = ref.merge_layer([k / V])
    np.testing.assert_array_equal(kept1[0], kept[0])
    assert len(np.unique(np.delete(mout["assign"][0], kept[0]))) > 3           # the last bits do decide
    for key in m1:
        np.testing.assert_array_equal(m1[key][0], mout[key][0])


@pytest.mark.parametrize("pruned", [1, 4, 64])
def test_merge_largest_kept_set_with_split_contraction(pruned):
    """Almost all of the largest supported number of visual tokens kept: few rows against 16320 to 16383 slots are cut along the
    contraction, and the step behind it holds the norms of all slots in LDS (above 16376 of them more than 64 KB)."""
    V = B.D3TOM_MAX_VISUAL
    c = W.random_case(530 + pruned, 3 + V + 2, 512, 4, 3, V, 2, dtype="bf16", centres=V // 3)
    kept = np.delete(np.arange(V), np.linspace(0, V - 1, pruned).astype(int)).astype(np.int32)
    out = GpuStep([c], [V - pruned], "bf16").merge([kept])
    check_assign(out["assign"][0], c["x"], 3, V, kept)
    check_merge({key: out[key][0] for key in out}, c["x"], 3, V, kept, "bf16")


@pytest.mark.parametrize("d_sim", [128, 72])          # MFMA cosine path (a multiple of 64) and the generic one
def test_merge_layer_one_call_with_separate_similarity_features(d_sim):
    """`sim` != x in the one-call merge layer: the selection launch takes its row norms from `sim` (other row length
    than the payload), the payload rows come from x.  Against d3tom_merge with the same `sim`, bit for bit, and that
    against the oracle's assignment on the `sim` rows."""
    shapes = [(4, 210, 6, 3, 0.2), (0, 77, 3, 2, 0.6)]
    samples, ratios = [], []
    for i, (P, V, O, D, keep) in enumerate(shapes):
        samples.append(W.random_case(600 + i, P + V + O, 256, 4, P, V, D, dtype="bf16", centres=9))
        ratios.append(keep)
    keeps = [oracle.keep_count(s["V"], r) for s, r in zip(samples, ratios)]
    rng = np.random.default_rng(601)
    sim_rows = W.round_to(rng.standard_normal((sum(s["N"] for s in samples), d_sim)).astype(np.float32), "bf16")
    ref = GpuStep(samples, keeps, "bf16")
    S = ref.importance(); kept, slot = ref.select_topk(); mout = ref.merge(sim_rows=sim_rows)
    off = 0
    for b, s in enumerate(samples):
        check_assign(mout["assign"][b], sim_rows[off:off + s["N"]], s["vis_start"], s["V"], kept[b])
        off += s["N"]
    S1, kept1, m1 = ref.merge_layer(ratios, sim_rows=sim_rows)
    for b in range(len(samples)):
        np.testing.assert_array_equal(S1[b], S[b])
        np.testing.assert_array_equal(kept1[b], kept[b])
        for key in m1:
            np.testing.assert_array_equal(m1[key][b], mout[key][b])


# ---- degenerate inputs the oracle defines ------------------------------------------------------------------
@pytest.mark.parametrize("dtype,d,H", [("bf16", 512, 4), ("bf16", 4096, 32), ("f32", 96, 2)])
def test_zero_rows_in_the_similarity_features(dtype, d, H):
    """A zero row has cosine 0 with everything: a zero PRUNED row ties on all slots and goes to slot 0; a zero KEPT
    row scores 0 against every pruned row, so it wins exactly the pruned rows whose other cosines are all negative.
    MFMA path (bf16, d a multiple of 64, tiled and split along the contraction) and generic path (float32)."""
    P, V, O = 6, 330, 10
    c = W.random_case(71, P + V + O, d, H, P, V, 4, dtype=dtype, centres=3, noise=1.0)
    x = c["x"].copy()
    rng = np.random.default_rng(72)
    kept = np.sort(rng.choice(V, size=9, replace=False)).astype(np.int32)
    pruned = np.setdiff1d(np.arange(V), kept)
    zero_pruned, zero_kept = pruned[[3, 100, 250]], kept[[0, 5]]
    x[P + zero_pruned] = 0.0
    x[P + zero_kept] = 0.0
    # make a few pruned rows point away from every non-zero kept row, so that the zero kept rows get members
    x[P + pruned[[7, 8]]] = -x[P + kept[2]]
    c["x"] = x
    step = GpuStep([c], [len(kept)], dtype)
    out = step.merge([kept])
    a = out["assign"][0]
    ref, bc = oracle.assign(x, P, V, kept, return_cos=True)
    assert np.all(a[zero_pruned] == 0) and np.all(ref[zero_pruned] == 0) and np.all(bc[zero_pruned] == 0.0)
    check_assign(a, x, P, V, kept)
    check_merge({key: out[key][0] for key in out}, x, P, V, kept, dtype)
    assert np.isfinite(out["y"][0]).all()


def test_deciders_anywhere_with_a_repeat_on_the_mfma_path():
    """Decider positions inside and in front of the visual block, one of them listed twice (its row counts twice):
    the score is defined for any list of rows."""
    P, V, O, H, dh = 40, 600, 30, 4, 128
    c = W.random_case(73, P + V + O, H * dh, H, P, V, 3, dtype="bf16", centres=50)
    c["dec_idx"] = np.array([5, P + 10, P + V - 1, P + 10, P + V + 7, 0, 39], dtype=np.int32)
    c["D"] = len(c["dec_idx"])
    k = oracle.keep_count(V, 0.2)
    step = GpuStep([c], [k], "bf16")
    S = step.importance()
    S_ref = oracle.importance(c["q"], c["k"], c["dec_idx"], P, V)
    check_scores(S[0], S_ref)
    kept, slot = step.select_topk()
    check_kept(kept[0], slot[0], S_ref, k)
    # and a long list (above the size whose logits are kept) with the same properties
    c["dec_idx"] = np.concatenate([np.arange(P + 100, P + 140), np.arange(0, 8), [P + 100, P + 100]]).astype(np.int32)
    c["D"] = len(c["dec_idx"])
    step = GpuStep([c], [k], "bf16")
    check_scores(step.importance()[0], oracle.importance(c["q"], c["k"], c["dec_idx"], P, V))


def test_one_token_merged_away_at_full_width():
    """keep_k = V - 1 at d = 4096: a single pruned row against V - 1 kept rows on the MFMA path."""
    P, V, O, H, dh = 4, 300, 6, 32, 128
    c = W.random_case(74, P + V + O, H * dh, H, P, V, 2, dtype="bf16", centres=20)
    step, S, kept, mout, stats = _chain([c], [V - 1], "bf16")
    assert mout["counts"][0].sum() == V and mout["counts"][0].max() == 2 and mout["y"][0].shape[0] == P + V - 1 + O


# ---- full-size workloads ---------------------------------------------------------------------------------
def test_llada_v_1024_full_chain():
    wl = W.WORKLOADS["llada_v_1024"]
    g = W.SampleGen(wl)
    s = g.step(32)
    k = oracle.keep_count(wl.V, 0.10)
    assert k == 103
    step, S, kept, mout, stats = _chain([s], [k], "bf16")
    assert mout["y"][0].shape[0] == 231
    q2, k2, v2 = g.proj.qkv(mout["y"][0])
    o = gpu_attend([(q2, k2, v2)], "bf16")[0]
    check_attend(o, q2, k2, v2, "bf16")
    # also the 263-token length quoted for this workload
    qkv = g.attention_inputs(263, 32)
    check_attend(gpu_attend([qkv], "bf16")[0], *qkv, "bf16")


@pytest.mark.parametrize("s_idx", [0, 5, 6, 16, 31])        # 5 | 6: the cosine tile height changes between them
def test_lavida_3645_sweep_steps_sampled(s_idx):
    wl = W.WORKLOADS["lavida_3645_sweep"]
    g = W.SampleGen(wl)
    sch = W.sweep_schedule(wl)[s_idx]
    s = g.step(sch["D"])
    k = oracle.keep_count(wl.V, sch["keep_ratio"])
    rng = np.random.default_rng(s_idx)
    step = GpuStep([s], [k], "bf16")
    S = step.importance(); kept, slot = step.select_topk(); mout = step.merge()
    pruned = np.setdiff1d(np.arange(wl.V), kept[0])
    rows = rng.choice(pruned, size=192, replace=False)
    st = check_full_sample(step, 0, S, kept, slot, mout, assign_rows=rows)
    n_m = wl.N - (wl.V - k)
    assert mout["y"][0].shape[0] == n_m
    # the benchmark's step calls the merge layer in one piece, with the keep ratio on the device: same kernels,
    # same launch shapes, so every output is that of the separate calls bit for bit
    S1, kept1, m1 = step.merge_layer([sch["keep_ratio"]])
    np.testing.assert_array_equal(S1[0], S[0])
    np.testing.assert_array_equal(kept1[0], kept[0])
    for key in m1:
        np.testing.assert_array_equal(m1[key][0], mout[key][0])
    qkv = g.attention_inputs(n_m, sch["D"])
    o = gpu_attend([qkv], "bf16")[0]
    check_attend(o, *qkv, "bf16", rows=rng.choice(n_m, size=48, replace=False))


def test_serving_shape_ragged_subset():
    wl = W.WORKLOADS["serving_b16"]
    proj = W.Projections(wl)
    draws = W.serving_draws(wl)[:3]
    samples = [W.SampleGen(wl, proj, seed=dr["seed"]).step(dr["D"]) for dr in draws]
    keeps = [oracle.keep_count(wl.V, dr["keep_ratio"]) for dr in draws]
    rng = np.random.default_rng(3)
    step = GpuStep(samples, keeps, "bf16")
    S = step.importance(); kept, slot = step.select_topk(); mout = step.merge()
    for b in range(len(samples)):
        pruned = np.setdiff1d(np.arange(wl.V), kept[b])
        check_full_sample(step, b, S, kept, slot, mout, assign_rows=rng.choice(pruned, size=96, replace=False))


def test_serving_shape_full_batch_of_16():
    """The whole ragged serving batch in one launch set (the configuration the kernels' batch mapping and
    the XCD-aware grids see in production): every sample's index outputs are checked for consistency, four
    samples (first, last, fewest kept, most deciders) are checked against the oracle stage by stage, and
    the attention over the 16 merged lengths is checked on sampled query rows."""
    wl = W.WORKLOADS["serving_b16"]
    proj = W.Projections(wl)
    draws = W.serving_draws(wl)
    gens = [W.SampleGen(wl, proj, seed=dr["seed"]) for dr in draws]
    samples = [g.step(dr["D"]) for g, dr in zip(gens, draws)]
    keeps = [oracle.keep_count(wl.V, dr["keep_ratio"]) for dr in draws]
    rng = np.random.default_rng(5)
    step = GpuStep(samples, keeps, "bf16")
    S = step.importance(); kept, slot = step.select_topk(); mout = step.merge()
    for b in range(wl.B):
        assert len(kept[b]) == keeps[b] and (np.diff(kept[b]) > 0).all()
        np.testing.assert_array_equal(np.where(slot[b] >= 0)[0], kept[b])
        assert mout["counts"][b].sum() == wl.V and mout["counts"][b].min() >= 1
        np.testing.assert_array_equal(mout["assign"][b][kept[b]], np.arange(keeps[b]))
        np.testing.assert_array_equal(np.bincount(mout["assign"][b], minlength=keeps[b]), mout["counts"][b])
        assert mout["y"][b].shape == (wl.N - (wl.V - keeps[b]), wl.d)
    detail = sorted({0, wl.B - 1, int(np.argmin(keeps)), int(np.argmax([dr["D"] for dr in draws]))})
    for b in detail:
        pruned = np.setdiff1d(np.arange(wl.V), kept[b])
        check_full_sample(step, b, S, kept, slot, mout, assign_rows=rng.choice(pruned, size=64, replace=False))
    qkv = [g.attention_inputs(wl.N - (wl.V - k), dr["D"]) for g, dr, k in zip(gens, draws, keeps)]
    outs = gpu_attend(qkv, "bf16")
    for b in detail[:3]:
        rows = rng.choice(qkv[b][0].shape[0], size=24, replace=False)
        check_attend(outs[b], *qkv[b], "bf16", rows=rows)


# ---- edge cases, determinism, error paths ---------------------------------------------------------------
def test_edge_counts():
    # k = 1 (everything merges into one token), D = 1, visual block at the very end
    c = W.random_case(31, 80, 2 * 128, 2, 10, 70, 1, dtype="bf16", centres=3)
    step, S, kept, mout, stats = _chain([c], [1], "bf16")
    assert mout["counts"][0][0] == 70 and mout["y"][0].shape[0] == 11
    # identical visual rows: every pruned token ties on all slots -> lowest slot takes all
    c2 = W.random_case(32, 60, 128, 1, 5, 50, 2, dtype="bf16", centres=1, noise=0.0)
    step, S, kept, mout, stats = _chain([c2], [5], "bf16")
    np.testing.assert_array_equal(mout["counts"][0], [46, 1, 1, 1, 1])
    # one slot with far more members than one staging pass of the scatter kernel holds (several windows,
    # windows that straddle the parts of the table scanned by different waves), in both merge modes
    c3 = W.random_case(33, 1530, 2 * 128, 2, 12, 1500, 4, dtype="bf16", centres=7)
    for mode in ("mean", "sum"):
        step, S, kept, mout, stats = _chain([c3], [1], "bf16", mode=mode)
        assert mout["counts"][0][0] == 1500 and mout["y"][0].shape[0] == 31
    c4 = W.random_case(34, 1210, 128, 1, 5, 1200, 2, dtype="bf16", centres=1, noise=0.0)
    step, S, kept, mout, stats = _chain([c4], [5], "bf16")
    np.testing.assert_array_equal(mout["counts"][0], [1196, 1, 1, 1, 1])


# ---- cosine taken on separate features (Section 4.4 compares keys while other rows are merged) --------
@pytest.mark.parametrize("dtype,d_sim", [("bf16", 256), ("bf16", 4 * 128 + 8), ("f32", 96)])
def test_merge_with_separate_similarity_features(dtype, d_sim):
    # d_sim = 256: MFMA path (split along the contraction, short sequence); 520: not a multiple of 64 -> generic path
    shapes = [(12, 500, 20, 0.3), (0, 260, 5, 0.6)]
    samples, keeps, sims = [], [], []
    for i, (P, V, O, keep) in enumerate(shapes):
        c = W.random_case(800 + i, P + V + O, 4 * 128, 4, P, V, 4, dtype=dtype, centres=max(4, V // 7))
        f = W.random_case(900 + i, P + V + O, d_sim, 1, P, V, 4, dtype=dtype, centres=max(4, V // 9))["x"]
        samples.append(c); keeps.append(oracle.keep_count(V, keep)); sims.append(f)
    rng = np.random.default_rng(9)
    kept = [np.sort(rng.choice(s["V"], size=k, replace=False)).astype(np.int32) for s, k in zip(samples, keeps)]
    out = GpuStep(samples, keeps, dtype).merge(kept, sim_rows=np.concatenate(sims))
    for b, s in enumerate(samples):
        check_assign(out["assign"][b], sims[b], s["vis_start"], s["V"], kept[b])          # routing follows `sim`
        check_merge({key: out[key][b] for key in out}, s["x"], s["vis_start"], s["V"], kept[b], dtype)   # payload is `x`


# ---- KV-cache variant (Section 4.4): one routing from the key cache, both caches aggregated ------------
@pytest.mark.parametrize("mode", ["mean", "sum"])
def test_merge_kv_ragged_batch(mode):
    shapes = [(64, 900, 0, 0.2), (20, 411, 0, 0.5), (0, 1300, 0, 0.1)]          # (prompt, visual, response, keep)
    samples, keeps, vrows = [], [], []
    for i, (P, V, O, keep) in enumerate(shapes):
        c = W.random_case(500 + i, P + V + O, 4 * 128, 4, P, V, 3, dtype="bf16", centres=max(4, V // 8))
        samples.append(c); keeps.append(oracle.keep_count(V, keep))
        vrows.append(W.round_to(np.random.default_rng(600 + i).standard_normal(c["x"].shape).astype(np.float32), "bf16"))
    step = GpuStep(samples, keeps, "bf16", B.D3TOM_MERGE_MEAN if mode == "mean" else B.D3TOM_MERGE_SUM)
    rng = np.random.default_rng(7)
    kept = [np.sort(rng.choice(s["V"], size=k, replace=False)).astype(np.int32) for s, k in zip(samples, keeps)]
    out = step.merge_kv(np.concatenate(vrows), kept)
    for b, s in enumerate(samples):
        check_assign(out["assign"][b], s["x"], s["vis_start"], s["V"], kept[b])
        # both caches against the oracle's aggregation run on the GPU's own routing
        check_merge({"y": out["y"][b], "assign": out["assign"][b], "counts": out["counts"][b], "src_pos": out["src_pos"][b]},
                    s["x"], s["vis_start"], s["V"], kept[b], "bf16", mode)
        check_merge({"y": out["v"][b], "assign": out["assign"][b], "counts": out["counts"][b], "src_pos": out["src_pos"][b]},
                    vrows[b], s["vis_start"], s["V"], kept[b], "bf16", mode)
    # the key half equals what d3tom_merge gives for the same rows and kept set (same kernels, same routing)
    ref = GpuStep(samples, keeps, "bf16", step.mode).merge(kept)
    for b in range(len(samples)):
        np.testing.assert_array_equal(ref["y"][b], out["y"][b])
        np.testing.assert_array_equal(ref["assign"][b], out["assign"][b])


@pytest.mark.parametrize("d,shapes", [(64, [(150, 7)]), (192, [(300, 40)]), (320, [(500, 60), (90, 90), (257, 256), (31, 1)]),
                                      (256, [(3000, 700)]), (1024, [(3645, 912)])])
def test_merge_kv_with_helping_workgroups(d, shapes):
    # sizes at which the cosine launch carries workgroups that only request rows (unsplit, one round, CUs to spare): row bytes that
    # are no multiple of a helper's 512, samples with nothing pruned and with one kept row.  They compute nothing, so caches and routing
    # have to be the same whether or not the rows are cached (helpers stop early where they are), and those of the merge of one payload
    g = torch.Generator(device="cuda"); g.manual_seed(d)
    P = 5
    lay = B.Layout([P + V for V, _ in shapes], [P] * len(shapes), [V for V, _ in shapes], [[0]] * len(shapes), [k for _, k in shapes])
    kc, vc = (torch.randn(lay.sum_N, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    kept = torch.cat([torch.sort(torch.randperm(V, generator=g, device="cuda")[:k])[0] for V, k in shapes]).to(torch.int32)
    ws = B.workspace(B.d3tom_workspace_bytes(B.D3TOM_OP_MERGE, lay.B, lay.max_N, lay.max_V, 1, d, 1))

    def outputs():
        return [torch.full((lay.sum_Nm, d), -1.0, dtype=torch.bfloat16, device="cuda")] + \
               [torch.full((n,), -1, dtype=torch.int32, device="cuda") for n in (lay.sum_V, lay.sum_keep, lay.sum_Nm)]
    got, got_v = outputs(), outputs()[0]
    torch.zeros(1 << 29, dtype=torch.uint8, device="cuda")                  # evicts the rows
    B.d3tom_merge_kv(kc, vc, lay, kept, 0, got[0], got_v, *got[1:], ws)
    check_assign(got[1].cpu().numpy()[:shapes[0][0]], kc[P:P + shapes[0][0]].float().cpu().numpy(), 0, shapes[0][0],
                 kept[:shapes[0][1]].cpu().numpy())
    for x, y in ((kc, got[0]), (vc, got_v)):
        ref = outputs()
        B.d3tom_merge(x, kc, lay, kept, 0, ref[0], *ref[1:], ws)
        for a, r in zip([y] + got[1:], ref):
            assert torch.equal(a, r)


# ---- decider bookkeeping on the device (Section 3.2) ----------------------------------------------------
def test_update_deciders_batch_and_chain_into_importance():
    M = 126336
    specs = [(300, 64, 9), (1152 - 64, 64, 5), (0, 1500, 4), (2688 - 256, 256, 2), (10, 1, 1)]     # (prefix, response, steps)
    trajs = [W.mask_trajectory(70 + i, p, r, t, mask_id=M) for i, (p, r, t) in enumerate(specs)]
    lens = [p + r for p, r, _ in specs]
    seq_off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    nb = len(specs)
    for max_D, pick in ((256, 1), (16, 1), (256, 0)):       # pick: which transition of each trajectory (0 = the first)
        prev = np.concatenate([t[min(pick, len(t) - 2)] for t in trajs])
        cur = np.concatenate([t[min(pick, len(t) - 2) + 1] for t in trajs])
        dec_idx = torch.full((nb * max_D,), -7, dtype=torch.int32, device="cuda")
        dec_off = torch.full((nb + 1,), -7, dtype=torch.int32, device="cuda")
        dec_cnt = torch.full((nb,), -7, dtype=torch.int32, device="cuda")
        B.d3tom_update_deciders(torch.from_numpy(prev).cuda(), torch.from_numpy(cur).cuda(), M, seq_off, max_D,
                                dec_idx, dec_off, dec_cnt)
        torch.cuda.synchronize()
        off, cnt, idx = dec_off.cpu().numpy(), dec_cnt.cpu().numpy(), dec_idx.cpu().numpy()
        o = 0
        for b in range(nb):
            a0 = sum(lens[:b])
            ref = oracle.deciders(prev[a0:a0 + lens[b]], cur[a0:a0 + lens[b]], M)
            assert cnt[b] == len(ref) and off[b] == o
            np.testing.assert_array_equal(idx[o:o + min(len(ref), max_D)], ref[:max_D])
            o += min(len(ref), max_D)
        assert off[nb] == o
    # the device-built list feeds d3tom_importance directly and gives the scores of the host-built one
    c = W.random_case(90, 700, 4 * 128, 4, 30, 600, 12, dtype="bf16", centres=40)
    c["dec_idx"] = np.sort(c["dec_idx"])
    step = GpuStep([c], [60], "bf16")
    S_ref = step.importance()[0].copy()
    prev = np.full(700, 7, np.int32); cur = prev.copy()
    prev[c["dec_idx"]] = M
    so = torch.tensor([0, 700], dtype=torch.int32, device="cuda")
    step.lay.dec_idx.zero_()
    B.d3tom_update_deciders(torch.from_numpy(prev).cuda(), torch.from_numpy(cur).cuda(), M, so, 12,
                            step.lay.dec_idx, step.lay.dec_off, None)
    np.testing.assert_array_equal(step.importance()[0], S_ref)


@pytest.mark.parametrize("nb", [1, 2, 17, 64, 65, 130])            # one sample a workgroup up to 64 samples, runs of two and three above
@pytest.mark.parametrize("share", [0.01, 0.5, 1.0])                # of the positions that were decided last
def test_update_deciders_sizes(nb, share):
    rng = np.random.default_rng(1000 * nb + int(100 * share))
    edge = [4097, 1, 1024, 0, 64, 65, 1025, 4096, 63, 8193, 1023, 2688, 4095]
    lens = [edge[b % len(edge)] if b < 2 * len(edge) else int(rng.integers(0, 300)) for b in range(nb)]
    _check_update_deciders(lens, share, rng)


def _check_update_deciders(lens, share, rng):
    nb = len(lens)
    M, max_D, total = 126336, 200, sum(lens)
    prev, cur = rng.integers(0, 32000, total).astype(np.int32), rng.integers(0, 32000, total).astype(np.int32)
    prev[rng.random(total) < 0.5] = M
    cur[(prev == M) & (rng.random(total) >= share)] = M
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    idx = torch.full((nb * max_D + 1,), -7, dtype=torch.int32, device="cuda")
    off, cnt = torch.full((nb + 1,), -7, dtype=torch.int32, device="cuda"), torch.full((nb,), -7, dtype=torch.int32, device="cuda")
    pad = torch.full((3,), M, dtype=torch.int32)               # ids that lie on 4 bytes only, and a decider on either side of them
    p = torch.cat([pad, torch.from_numpy(prev), pad]).cuda()[3:3 + total]
    c = torch.cat([pad * 0, torch.from_numpy(cur), pad * 0]).cuda()[3:3 + total]
    B.d3tom_update_deciders(p, c, M, torch.from_numpy(offs).cuda(), max_D, idx, off, cnt)
    want, ends, counts = [], [0], []
    for b in range(nb):
        ref = oracle.deciders(prev[offs[b]:offs[b + 1]], cur[offs[b]:offs[b + 1]], M)
        want += list(ref[:max_D])
        ends.append(len(want))
        counts.append(len(ref))
    np.testing.assert_array_equal(off.cpu().numpy(), ends)
    np.testing.assert_array_equal(cnt.cpu().numpy(), counts)
    np.testing.assert_array_equal(idx.cpu().numpy()[:len(want)], want)
    assert (idx.cpu().numpy()[len(want):] == -7).all()


@pytest.mark.parametrize("share", [0.02, 1.0])
@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 1280, 1281, 2049, 4096, 4097, 5120, 8193])
def test_update_deciders_of_one_sample_and_behind_it(n, share):
    """A sample alone, and as the one that the next samples' workgroups count: at the edges of a wave's 64 positions, of the count's turns of 256 and 1024, of
    the own turns of 1024 positions a part and 4096 together."""
    rng = np.random.default_rng(10 * n + int(share))
    for lens in ([n], [n, 70], [70, n, 1], [n] * 18):
        if sum(lens):
            _check_update_deciders(lens, share, rng)


def test_bitwise_determinism():
    c = W.random_case(41, 900, 4 * 128, 4, 30, 800, 12, dtype="bf16", centres=60)
    k = oracle.keep_count(800, 0.2)
    outs = []
    for _ in range(2):
        step = GpuStep([c], [k], "bf16")
        S = step.importance(); kept, slot = step.select_topk(); m = step.merge()
        outs.append((S[0].copy(), kept[0].copy(), m["y"][0].copy(), m["assign"][0].copy()))
    for a, b in zip(outs[0], outs[1]):
        np.testing.assert_array_equal(a, b)
    qkv = W.random_qkv(42, 333, 4, 128, "bf16")
    np.testing.assert_array_equal(gpu_attend([qkv], "bf16")[0], gpu_attend([qkv], "bf16")[0])


def test_error_statuses():
    c = W.random_case(51, 40, 128, 1, 4, 30, 2, dtype="bf16")
    step = GpuStep([c], [5], "bf16")
    lay0 = B.Layout([40], [4], [30], [[]], [5])                                # empty decider set
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_importance(step.q, step.k, lay0, 0.1, step.scores, step.ws_imp)
    assert e.value.status == B.D3TOM_ERR_NO_DECIDERS
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_importance(step.q, step.k, step.lay, 0.1, step.scores, B.workspace(256))
    assert e.value.status == B.D3TOM_ERR_WORKSPACE_TOO_SMALL
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_merge(step.x, None, step.lay, step.kept_idx, 7, step.y, None, None, None, step.ws_merge)
    assert e.value.status == B.D3TOM_ERR_INVALID_ARG
    q = torch.zeros((8, 1, 300), dtype=torch.float32, device="cuda")           # head size above the limit
    cu = torch.tensor([0, 8], dtype=torch.int32, device="cuda")
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_attend(q, q, q, cu, 8, 1.0, torch.zeros_like(q))
    assert e.value.status == B.D3TOM_ERR_UNSUPPORTED
    q2 = torch.zeros((8, 1, 64), dtype=torch.bfloat16, device="cuda")
    for bad_scale in (0.0, -0.125, float("inf"), float("nan")):                # the logit scale must be finite and > 0
        with pytest.raises(B.D3tomError) as e:
            B.d3tom_attend(q2, q2, q2, cu, 8, bad_scale, torch.zeros_like(q2))
        assert e.value.status == B.D3TOM_ERR_INVALID_ARG
        with pytest.raises(B.D3tomError) as e:
            B.d3tom_importance(step.q, step.k, step.lay, bad_scale, step.scores, step.ws_imp)
        assert e.value.status == B.D3TOM_ERR_INVALID_ARG
    torch.cuda.synchronize()
