"""Whole steps at the sizes where the split of the work changes: the edges of the chunks, tiles and groups that the
kernels cut a unit into.  Checked like every step (scores and masses within relative 1e-5 of the oracle, every later
stage exact on the GPU's own floats)."""
import numpy as np
import pytest
import torch

from paper_2605_23200_amd import binding as B
from paper_2605_23200_amd import inputs
from paper_2605_23200_amd.harness import Job
from gpu_util import DEV, assert_close_terms, to_dev, to_host, workspace
from test_gpu_step import check_properties_all_units, check_units

pytestmark = pytest.mark.gpu


def _run(oracle, w, lens=None, scorer=B.SCORER_MEAN_WINDOW, units=None, **kw):
    host = inputs.dense_cache(w, n_threads=4)
    if lens is not None:
        host["seq_lens"][:] = lens
    job = Job(w, host, scorer=scorer, **kw)
    job.step()
    check_properties_all_units(job)
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32),
                list(range(w.units)) if units is None else units, scorer=scorer)
    return job


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype,G,W,T,paged", [("bf16", 4, 32, 127, False), ("bf16", 4, 32, 129, False),
                                                ("f32", 1, 8, 257, False), ("f32", 2, 20, 4097, False),
                                                ("bf16", 7, 32, 385, True), ("bf16", 2, 16, 8193, False),
                                                ("f32", 4, 32, 1000, True), ("f32", 3, 32, 385, False)])   # eight waves, 128 keys
def test_few_units_are_cut_into_short_chunks(oracle, dtype, G, W, T, paged, causal):
    """Few units: chunks of 128 keys (one block per wave), up to one workgroup per CU; a ragged second sequence ends
    inside, on and before a chunk's edge."""
    w = inputs.CONFIGS[1].scaled(L=1, B=2, H=2, G=G, W=W, T=T, T_min=T, dtype=dtype, budget=min(64, T), S=4, n_spans=2,
                                 span_len=(4, 40), paged=paged, causal=causal)
    _run(oracle, w, lens=[T, max(1, T - 1 - (T % 128))])


def _stage_params(units, T, S, **kw):
    return B.make_params(n_layers=1, batch=1, n_kv_heads=units, group=1, window=8, t_max=T, budget=min(64, T),
                         n_segments=S, **kw)


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("T,S", [(63, 4), (64, 4), (65, 4), (1023, 33), (1025, 34), (65536, 8), (65537, 8), (262144, 40),
                                 (262209, 40)])
def test_cuts_at_the_edges_of_pieces_and_groups(oracle, T, S, signed):
    """Pieces of 64 positions, the 65536 / 262144 positions whose pieces the two workgroup sizes hold at once, 33 / 34
    thresholds.  signed: the prefix falls in between, the first position that reaches a threshold still counts."""
    rng = np.random.default_rng(T + S)
    m = (rng.random((3, T)) ** 4).astype(np.float32)
    m[1] *= np.arange(T) % 97 == 0                                     # most pieces hold one or two entries
    if signed:
        m[0] -= (rng.random(T) * 0.15).astype(np.float32)
        m[2] = np.where(np.arange(T) < T // 2, m[2], -m[2] / 2)
    m /= np.abs(m.astype(np.float64)).sum(1, keepdims=True)
    m = np.ascontiguousarray(m.astype(np.float32))
    p = _stage_params(3, T, S)
    bounds, seg_mass = torch.full((3, S + 1), -3, dtype=torch.int32, device=DEV), torch.full((3, S), -3.0, device=DEV)
    B.ams_mass_segment(p, to_dev(np.array([T], np.int32)), to_dev(m), bounds, seg_mass, workspace(p))
    bounds, seg_mass = to_host(bounds), to_host(seg_mass)
    for i in range(3):
        b_o, s_o = oracle.segment(m[i], S)
        np.testing.assert_array_equal(bounds[i], b_o, err_msg=f"unit {i}")
        # a mass is a difference of two prefixes of at most 1 in magnitude, in double
        np.testing.assert_allclose(seg_mass[i], s_o, rtol=1e-6, atol=1e-12)


@pytest.mark.parametrize("T,S,pool", [(1023, 64, 5), (1025, 65, 0), (4097, 16, 63), (65600, 256, 3), (9000, 257, 0)])
def test_mass_step_at_the_edges_of_its_runs(oracle, T, S, pool):
    """Runs of 1024 positions, 64 / 65 and 256 / 257 segments (registers per lane of the quota wave), the widest pool."""
    w = inputs.CONFIGS[0].scaled(H=2, T=T, S=S, budget=min(700, T), n_spans=3, span_len=(8, 60), pool_kernel=pool)
    _run(oracle, w)


def test_many_chunks_take_four_runs_per_workgroup(oracle):
    """512 chunks of 4096 positions: four runs per workgroup, the last chunk ragged, pooled and not."""
    for pool in (0, 5):
        w = inputs.CONFIGS[0].scaled(L=16, H=8, T=12289 + 17, W=4, D=64, dtype="bf16", budget=100, n_spans=3,
                                     span_len=(8, 60), pool_kernel=pool)
        _run(oracle, w, units=[0, 63, 127])


def test_a_peak_on_the_threshold_is_the_cut(oracle):
    """The prefix rises to a threshold within its last bit, at the peak of a piece of 64, and falls from there: the cut is
    at the peak also where only one of two orders of additions reaches the threshold (found by a search over seeds)."""
    T, S, rows = 2560, 4, []
    for seed in (16, 68, 146, 152):
        rng = np.random.default_rng(seed)
        m = (rng.random(T) ** 12 * 1e-3).astype(np.float32)
        pos = int(rng.integers(1, 10)) * 256 + int(rng.integers(4, 40))
        left = 0.25 - m[:pos - 3].astype(np.float64).sum()
        for q in range(pos - 3, pos + 1):
            m[q] = np.float32(left)
            left -= float(m[q])
        m[pos + 1:] = -m[pos + 1:]
        rows.append(m)
    p = _stage_params(4, T, S)
    bounds, seg_mass = torch.full((4, S + 1), -3, dtype=torch.int32, device=DEV), torch.full((4, S), -3.0, device=DEV)
    B.ams_mass_segment(p, to_dev(np.array([T], np.int32)), to_dev(np.stack(rows)), bounds, seg_mass, workspace(p))
    for i in range(4):
        np.testing.assert_array_equal(to_host(bounds)[i], oracle.segment(rows[i], S)[0], err_msg=f"unit {i}")


@pytest.mark.parametrize("T,delta,l_min,l_max", [(70001, 0.01, 8, 200), (270000, 0.05, 16, 1024)])
def test_split_and_merge_on_long_caches(oracle, T, delta, l_min, l_max):
    """Prefixes held whole (up to 262144 positions) and in groups (beyond), segments that the length rules have moved."""
    cap = int(np.ceil(1 / delta)) + 1 + T // l_max
    rng = np.random.default_rng(T)
    m = np.stack([oracle.mass((rng.random(T) ** e).astype(np.float32)) for e in (1, 8)])
    p = _stage_params(2, T, cap, seg_delta=delta, l_min=l_min, l_max=l_max)
    bounds, seg_mass = torch.full((2, cap + 1), -3, dtype=torch.int32, device=DEV), torch.full((2, cap), -3.0, device=DEV)
    B.ams_mass_segment(p, to_dev(np.array([T], np.int32)), to_dev(m), bounds, seg_mass, workspace(p))
    for i in range(2):
        b_o, s_o, _ = oracle.segment_adaptive(m[i], delta, l_min, l_max, cap)
        np.testing.assert_array_equal(to_host(bounds)[i], b_o)
        np.testing.assert_allclose(to_host(seg_mass)[i], s_o, rtol=1e-5, atol=1e-12)


@pytest.mark.parametrize("S", [64, 65, 128, 256, 257, 1024])
def test_quota_ties_at_every_register_count(oracle, S):
    """Equal fractions, empty and full segments: the leftovers go to the lower segments, the sum is the budget."""
    rng = np.random.default_rng(S)
    for budget, levels in ((S // 3 + 1, 2), (2 * S + 1, 3), (7 * S // 2, 1), (20 * S, 1000)):
        lens = rng.integers(0, 30, size=S)
        lens[S // 2] += 9
        bounds = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)[None]
        mass = np.where(lens > 0, (1 + rng.integers(0, levels, size=S)) / 8, 0).astype(np.float32)[None]
        T = int(bounds[0, -1])
        p = _stage_params(1, T, S)
        p.budget = budget
        quota = torch.zeros((1, S), dtype=torch.int32, device=DEV)
        idx, n_kept = torch.zeros((1, budget), dtype=torch.int32, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
        B.ams_select(p, to_dev(np.array([T], np.int32)), torch.zeros((1, T), device=DEV), to_dev(bounds), to_dev(mass),
                     quota, idx, n_kept)
        np.testing.assert_array_equal(to_host(quota)[0], oracle.quota(bounds[0], mass[0], budget, 1), err_msg=f"{budget}")


@pytest.mark.parametrize("must", [False, True])
@pytest.mark.parametrize("threads,lens", [(64, [1024, 1025, 63, 64, 65, 1, 0, 130, 200, 2, 40, 7, 250, 90]),   # 1024 keys
                                          (256, [4096, 4097, 1000, 255, 256, 257]),
                                          (512, [8192, 8193, 100, 2000, 1000]),
                                          (1024, [32768]), (1024, [32769])])
def test_select_at_the_edges_of_its_shapes(oracle, threads, lens, must):
    """Segments that just fit a shape's registers and that do not; scores that fill one bin over several passes (an
    outlier and neighbouring floats), ties by the hundred, signed zeros, infinities and NaN."""
    S, T = len(lens), sum(lens)
    # the rule that picks the shape: the expected length, T / S, against 256, 2560 and 5120
    assert threads == (64 if T <= 256 * S else 256 if T <= 2560 * S else 512 if T <= 5120 * S else 1024)
    cap = 32 * threads if threads == 1024 else 16 * threads
    assert cap in lens or cap + 1 in lens
    bounds = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rng = np.random.default_rng(T + S)
    g = rng.standard_normal((6, T)).astype(np.float32)
    g[1] = (1 + rng.integers(0, 70, T) * 2.0 ** -23).astype(np.float32)
    g[1, ::501] = 3e38
    g[1, 3::701] = -3e38
    g[2] = np.round(g[2])
    g[3] = -1.5
    g[4] = np.float32(1e-40) * rng.integers(0, 3, T).astype(np.float32)
    g[5, ::3], g[5, 1::5], g[5, 2::7], g[5, 4::11] = np.nan, -np.inf, np.inf, -0.0
    for budget in (max(1, T // 16), T // 2, T - 1):
        p = _stage_params(6, T, S)
        p.budget = budget
        if must:
            p.n_sink, p.n_last = 3, 33
        mass = np.tile(np.array(lens, np.float32) / T, (6, 1))
        quota = torch.zeros((6, S), dtype=torch.int32, device=DEV)
        idx, n_kept = torch.zeros((6, budget), dtype=torch.int32, device=DEV), torch.zeros(6, dtype=torch.int32, device=DEV)
        B.ams_select(p, to_dev(np.array([T], np.int32)), to_dev(g), to_dev(np.tile(bounds, (6, 1))), to_dev(mass), quota,
                     idx, n_kept, workspace(p))
        sinks, last, seg_budget = oracle.must_keep(T, budget, p.n_sink, p.n_last)
        for i in range(6):
            q = oracle.quota(bounds, mass[i], seg_budget, 1)
            np.testing.assert_array_equal(to_host(quota)[i], q)
            want = oracle.finalize(g[i], oracle.select(g[i], bounds, q), sinks, last, budget)
            np.testing.assert_array_equal(to_host(idx)[i], want, err_msg=f"row {i} budget {budget}")


@pytest.mark.parametrize("must", [False, True])
@pytest.mark.parametrize("pad", [0, 4])
@pytest.mark.parametrize("lens", [[70001], [131072], [33001, 2, 90001], [32769, 40000],           # 1024 threads
                                  [9, 12001, 8193, 1], [4100, 4097, 3, 300],                       # 512, 256
                                  [5003, 17, 1030, 40] + [9] * 60])                                # one wave
def test_segments_longer_than_the_registers(oracle, lens, pad, must):
    """Selected from memory, by stretches of 256 positions per wave: segments that start and end anywhere, rows whose 16-byte reads
    are aligned (pad) and not; thousands of keys in one bin, bins that hold what is wanted, equal keys in order."""
    S, T = len(lens), sum(lens)
    bounds = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    stride = -(-T // 4) * 4 + pad if pad else T + 1 - T % 2   # odd: no row but the first is aligned
    rng = np.random.default_rng(T + S + pad)
    g = rng.standard_normal((7, T)).astype(np.float32)
    g[1] = (1 + rng.integers(0, 70, T) * 2.0 ** -23).astype(np.float32)
    g[1, ::501] = 3e38
    g[2] = np.round(g[2] * 4)
    g[3] = -1.5
    g[4] = np.exp(6 * g[4])
    g[4, T // 3:2 * T // 3] = 1 + rng.random(2 * T // 3 - T // 3).astype(np.float32) * 1e-4
    g[5, ::3], g[5, 1::5], g[5, 2::7], g[5, 4::11] = np.nan, -np.inf, np.inf, -0.0
    g[6] = np.where(rng.random(T) < 0.01, 1.0, 0.5)
    rows = np.full((7, stride), 9e9, np.float32)                       # past the end: would win
    rows[:, :T] = g
    for budget in (max(1, T // 16), T // 2, T - 1):
        p = _stage_params(7, T, S)
        p.t_stride, p.budget = stride, budget
        if must:
            p.n_sink, p.n_last = 3, 33
        mass = np.tile(np.array(lens, np.float32) / T, (7, 1))
        quota = torch.zeros((7, S), dtype=torch.int32, device=DEV)
        idx, n_kept = torch.zeros((7, budget), dtype=torch.int32, device=DEV), torch.zeros(7, dtype=torch.int32, device=DEV)
        B.ams_select(p, to_dev(np.array([T], np.int32)), to_dev(rows), to_dev(np.tile(bounds, (7, 1))), to_dev(mass), quota,
                     idx, n_kept, workspace(p))
        sinks, last, seg_budget = oracle.must_keep(T, budget, p.n_sink, p.n_last)
        for i in range(7):
            q = oracle.quota(bounds, mass[i], seg_budget, 1)
            np.testing.assert_array_equal(to_host(quota)[i], q)
            want = oracle.finalize(g[i], oracle.select(g[i], bounds, q), sinks, last, budget)
            np.testing.assert_array_equal(to_host(idx)[i], want, err_msg=f"row {i} budget {budget}")


@pytest.mark.parametrize("H", [1, 2, 3, 8])
def test_paged_heads_move_over_the_workgroups(oracle, H):
    """Paged sweeps give the heads of a chunk to workgroups in an order that moves on: every (unit, chunk) once, for head
    counts that do and do not divide the period; ragged lengths end chunks early."""
    w = inputs.CONFIGS[2].scaled(L=2, B=5, H=H, T=2100, T_min=900, D=64, W=4, budget=100, S=4, n_spans=2, span_len=(8, 90))
    _run(oracle, w)


@pytest.mark.parametrize("scorer", [B.SCORER_MEAN_WINDOW, B.SCORER_KEYDIFF, B.SCORER_REDUNDANCY])
@pytest.mark.parametrize("G,W", [(5, 32), (7, 32), (8, 32)])
def test_one_dominant_key_in_any_block(oracle, G, W, scorer):
    """Five or more column blocks.  One key of each unit, in a wave's first, second, middle or last (ragged) block, lies 6 to
    100 units above the others: the running maximum rises late or early, and the key sums see every key once."""
    w = inputs.CONFIGS[1].scaled(L=8, H=8, G=G, W=W, T=4200, budget=300, S=4, n_spans=3, span_len=(8, 90))
    host = inputs.dense_cache(w, n_threads=8)
    units, where = list(range(0, 64, 7)), (0, 40, 128, 150, 700, 1023, 1024, 3000, 4199)
    for n, i in enumerate(units):
        l, h = i // 8, i % 8
        q = inputs.bf16_bits_to_f32(host["Q"][l, 0, h * G + n % G, n % W])
        host["K"][l, 0, h, where[n % len(where)]] = inputs.to_bf16_bits(((0.5, 1.5, 4.0, 8.0)[n % 4] * q).astype(np.float32))
    job = Job(w, host, scorer=scorer)
    job.step()
    check_properties_all_units(job)
    check_units(oracle, job, host, np.zeros((w.units, w.T), np.float32), units + [1, 2], scorer=scorer)


@pytest.mark.parametrize("scorer", [B.SCORER_KEYDIFF, B.SCORER_REDUNDANCY])
@pytest.mark.parametrize("D,G,W,T,paged", [(128, 4, 32, 2049, False), (128, 1, 32, 4100, False), (64, 2, 32, 127, False),
                                            (64, 7, 32, 2048, True), (128, 8, 32, 2500, True), (128, 7, 32, 3333, False),
                                            (64, 4, 32, 31, False), (128, 4, 32, 1, False)])
def test_key_scores_ride_along_with_the_sweeps(oracle, scorer, D, G, W, T, paged):
    """Every number of column blocks, chunk edges, ragged last blocks, single keys; a sequence with zero keys among the
    others.  (The sum of a shorter second sequence must not see the rows past its end.)"""
    w = inputs.CONFIGS[1].scaled(L=1, B=2, H=2, D=D, G=G, W=W, T=T, T_min=T, budget=min(128, T), S=4, n_spans=2,
                                 span_len=(1, 60), paged=paged)
    host = inputs.dense_cache(w, n_threads=4)
    host["seq_lens"][:] = [T, max(1, T - 5)]
    host["K"][0, 0, 1, ::3] = 0
    host["K"][0, 1, :, max(1, T - 5):] = inputs.to_bf16_bits(np.full(1, 1e4, np.float32))[0]
    job = Job(w, host, scorer=scorer)
    job.step()
    check_properties_all_units(job)
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), list(range(w.units)), scorer=scorer)


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("budget", [1, 15, 16, 17, 31, 33, 65])
def test_compaction_at_the_edges_of_its_row_groups(oracle, dtype, D, budget):
    """16, 32 or 64 rows per workgroup: kept counts around them, rows of 128 to 512 bytes."""
    w = inputs.CONFIGS[1].scaled(L=1, H=2, G=1, W=8, D=D, dtype=dtype, T=300, budget=budget, S=2, n_spans=1, span_len=(8, 40))
    _run(oracle, w)


def _labels(job):
    B.ams_profile_begin()
    job.step()
    return [k for k, _ in B.ams_profile_end()]


@pytest.mark.parametrize("scorer", [B.SCORER_MEAN_WINDOW, B.SCORER_LAST_QUERY, B.SCORER_KEYDIFF, B.SCORER_REDUNDANCY,
                                    B.SCORER_EXPECTED_VNORM])
@pytest.mark.parametrize("T,dtype,G,W,D,folded", [(8192, "bf16", 2, 32, 128, True), (8193, "bf16", 2, 32, 64, False),
                                                  (2304, "bf16", 7, 32, 128, True), (4097, "bf16", 4, 32, 128, False),
                                                  (5000, "f32", 2, 20, 128, True), (130, "bf16", 1, 8, 128, True),
                                                  (1, "bf16", 4, 8, 128, True)])
def test_second_sweep_merges_the_statistics_of_small_launches(oracle, T, dtype, G, W, D, folded, scorer):
    """64 chunks of 64 columns and one more, 18 of 224, 33 of 128 (32 KB of statistics is the limit); the empty first sequence has no workgroup that gets as far as its merge, and the scratch
    holds garbage (a status word that nobody cleared would void the event)."""
    w = inputs.CONFIGS[1].scaled(L=1, B=2, H=1, G=G, W=W, D=D, T=T, T_min=T, dtype=dtype, budget=max(1, min(96, T // 3)), S=4,
                                 n_spans=2, span_len=(1, 40))
    host = inputs.dense_cache(w, n_threads=4)
    if T > 1:
        host["seq_lens"][:] = [0, T]
    job = Job(w, host, scorer=scorer)
    job.ws.fill_(255)
    assert ("score_reduce" not in _labels(job)) == folded
    assert to_host(job.n_kept).tolist() == [min(w.budget, int(t)) for t in host["seq_lens"]]
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), [1] if T > 1 else [0, 1], scorer=scorer)


@pytest.mark.parametrize("scorer", [B.SCORER_MEAN_WINDOW, B.SCORER_LAST_QUERY, B.SCORER_REDUNDANCY, B.SCORER_EXPECTED_VNORM])
@pytest.mark.parametrize("H,T,dtype,G,W,D,folded", [(7, 300, "bf16", 4, 32, 128, True),      # 3 chunks: rows of 3, 3 and 1 tails
                                                    (300, 130, "bf16", 1, 8, 64, True),      # 1 chunk: a tail in every row
                                                    (2, 8192, "bf16", 2, 32, 128, True), (1, 8193, "bf16", 2, 32, 64, False),
                                                    (3, 2304, "bf16", 7, 32, 128, True), (2, 1000, "f32", 3, 32, 128, True),
                                                    (5, 5, "bf16", 4, 32, 128, True), (2, 160, "bf16", 1, 256, 128, True),
                                                    (2, 700, "f32", 1, 100, 64, True)])
def test_tails_of_a_causal_window_run_beside_the_sweeps(oracle, H, T, dtype, G, W, D, folded, scorer):
    """The tails are the last workgroups of the sweeps' launches, a row of the grid for as many as a unit has chunks; their
    statistics are one more entry, merged by the second sweep or by the reduction; caches shorter than the window; tails of
    several blocks per wave."""
    w = inputs.CONFIGS[1].scaled(L=1, B=1, H=H, G=G, W=W, D=D, T=T, T_min=T, dtype=dtype, budget=max(1, min(96, T // 3)), S=4,
                                 n_spans=2, span_len=(1, max(1, min(40, T // 2))), causal=True)
    host = inputs.dense_cache(w, n_threads=4)
    job = Job(w, host, scorer=scorer)
    job.ws.fill_(255)
    labels = _labels(job)
    assert ("score_reduce" not in labels) == folded and not any("tail" in x for x in labels)
    assert to_host(job.n_kept).tolist() == [min(w.budget, T)] * H
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), sorted({0, H // 2, H - 1}), scorer=scorer)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("units,T", [(2, 700), (130, 200), (40, 1500)])          # merged by the second sweep, one launch, both
@pytest.mark.parametrize("dtype,G,W", [("bf16", 4, 32), ("bf16", 128, 1), ("bf16", 5, 2), ("bf16", 7, 16), ("bf16", 2, 64), ("bf16", 3, 24),
                                       ("bf16", 7, 32), ("f32", 3, 8), ("f32", 2, 40)])
def test_last_query_in_windows_of_any_length(oracle, dtype, G, W, units, T, causal):
    """Windows of 1, 2, 8, 16 and 32 queries, whose newest ones share lanes, and windows that need a sum of their own; padded
    query columns in those lanes."""
    w = inputs.CONFIGS[1].scaled(L=1, B=1, H=units, G=G, W=W, T=T, T_min=T, dtype=dtype, budget=40, S=4, n_spans=2,
                                 span_len=(4, 30), causal=causal)
    _run(oracle, w, scorer=B.SCORER_LAST_QUERY, units=sorted({0, units // 2, units - 1}))


@pytest.mark.parametrize("path,T,G,W,causal", [(B.SCORE_PATH_TWO_SWEEPS, 4000, 1, 32, False), (B.SCORE_PATH_TWO_SWEEPS, 4000, 2, 32, True),
                                               (B.SCORE_PATH_TWO_SWEEPS, 8193, 4, 32, False), (B.SCORE_PATH_TWO_SWEEPS, 8193, 14, 16, True),
                                               (B.SCORE_PATH_ONE_LAUNCH, 4000, 1, 32, False), (B.SCORE_PATH_ONE_LAUNCH, 4000, 4, 16, False)])
def test_last_query_shares_below_the_smallest_normal_number(path, T, G, W, causal):
    """Exact products (two channels of queries and keys are not zero), Z = T - 32 to a relative 1e-30: a share of the newest query is
    2^x / ((T - 32) G) with x the logit in base 2, formed in fp32 from |x| <= 126 (relative 126 * 2^-23) and rounded once below
    2^-126 (2^-150), by one multiply-add per group's query: the zeros that it is added to change nothing."""
    D = 64
    Q, K = np.zeros((G, W, D), np.float32), np.zeros((T, D), np.float32)
    Q[:, -1, :2] = 8.0
    at = np.arange(32) * (T // 32) + np.arange(32) % 5
    at[-8:] = T - 1 - np.arange(8)                                      # (within a causal window)
    K[at, 0], K[at, 1] = -86.0, -np.arange(32) / 64                     # logits of -86 .. -86.5
    bits = lambda x: (np.ascontiguousarray(x).view(np.uint32) >> 16).astype(np.uint16)
    p = B.make_params(n_layers=1, batch=1, n_kv_heads=1, group=G, window=W, head_dim=D, kv_dtype=B.BF16, t_max=T, t_stride=T, budget=64,
                      n_segments=4, scorer=B.SCORER_LAST_QUERY, causal=causal, score_path=path)
    k, q = to_dev(bits(K)).view(torch.bfloat16).reshape(1, 1, 1, T, D), to_dev(bits(Q)).view(torch.bfloat16).reshape(1, 1, G, W, D)
    u, g = torch.zeros((1, T), device=DEV), torch.zeros((1, T), device=DEV)
    B.ams_score(p, B.dense_view(k, k), to_dev(np.array([T], np.int32)), q, u, g, workspace(p))
    want = np.exp(K[at].astype(np.float64).sum(1)) / (T - 32)            # G equal shares of 1 / G
    got = to_host(g)[0, at].astype(np.float64)
    assert (want < 2.0 ** -126).all()
    err = np.abs(got - want)
    assert (err <= G * 2.0 ** -150 + 127 * 2.0 ** -23 * want).all(), (err / 2.0 ** -149).max()


@pytest.mark.parametrize("vec", [True, False])
@pytest.mark.parametrize("T,S,delta,l_min,l_max,pool,causal,must,one", [
    (2048, 24, 0.1, 16, 256, 5, True, True, True), (2049, 24, 0.1, 16, 256, 5, True, True, True),
    (4096, 30, 0.1, 16, 256, 63, False, False, True), (4097, 32, 0.1, 0, 256, 3, True, False, True),
    (8192, 60, 0.1, 16, 200, 5, True, True, True), (8193, 60, 0.1, 16, 200, 5, True, True, False),
    (3000, 70, 0.0, 0, 0, 0, True, False, True), (1000, 8, 0.0, 0, 0, 31, False, True, True),
    (63, 12, 0.1, 4, 0, 63, False, False, True), (1, 12, 0.1, 0, 0, 3, True, False, True), (700, 1000, 0.001, 0, 0, 5, False, False, True)])
def test_short_caches_form_everything_after_the_scores_in_one_launch(oracle, T, S, delta, l_min, l_max, pool, causal, must, one, vec):
    """Pooled usage or a causal window: pooling, normalisers, masses, cuts and quotas in one workgroup per unit; its three sizes
    and their edges, the widest pool, ragged and empty sequences, 1000 segments, rows of odd stride."""
    w = inputs.CONFIGS[1].scaled(L=1, B=3, H=2, G=1, W=8, T=T, T_min=T, budget=max(1, T // 5), S=S, n_spans=3, span_len=(1, max(1, min(30, T))),
                                 causal=causal, pool_kernel=pool, seg_delta=delta, l_min=l_min, l_max=l_max,
                                 n_sink=4 * must, n_last=32 * must)
    host = inputs.dense_cache(w, n_threads=4)
    host["seq_lens"][:] = [T, 0, max(1, T // 2 - 1)]
    credit = np.abs(np.random.default_rng(T + S).standard_normal((6, T))).astype(np.float32)
    credit /= credit.sum(1, keepdims=True)
    for i, n in enumerate(n for n in host["seq_lens"] for _ in range(2)):
        credit[i, n:] = 0
    job = Job(w, host, credit=credit)
    if not vec:
        job.t_stride = job.p.t_stride = T | 1
        job.credit = torch.zeros((job.units, job.t_stride), device=DEV)
        job.credit[:, :T] = to_dev(credit)
        job.ws = torch.zeros(B.ams_workspace_bytes(job.p), dtype=torch.uint8, device=DEV)
    labels = _labels(job)
    assert ("unit_mass_cuts" in labels) == one and ("mass_ema" in labels) != one and ("vc_sums" in labels) != one
    assert to_host(job.n_kept).tolist() == [min(w.budget, int(t)) for t in host["seq_lens"] for _ in range(2)]
    before = np.zeros((6, job.t_max), np.float32)
    before[:, :T] = credit
    check_units(oracle, job, host, before, [0, 1, 4, 5])


@pytest.mark.parametrize("vec", [True, False])
@pytest.mark.parametrize("T,S,dtype,G,W,D,scorer,must,one", [
    (4096, 64, "bf16", 4, 32, 128, B.SCORER_MEAN_WINDOW, False, True), (4095, 65, "bf16", 4, 32, 128, B.SCORER_MEAN_WINDOW, False, False),
    (2049, 7, "bf16", 1, 8, 64, B.SCORER_LAST_QUERY, True, True), (2048, 16, "f32", 2, 20, 128, B.SCORER_MEAN_WINDOW, True, True),
    (65, 3, "bf16", 2, 32, 128, B.SCORER_LAST_QUERY, False, True), (64, 1, "f32", 1, 8, 64, B.SCORER_MEAN_WINDOW, False, True),
    (1, 4, "bf16", 1, 8, 128, B.SCORER_MEAN_WINDOW, False, True)])
def test_one_launch_scorer_goes_on_to_the_quotas(oracle, T, S, dtype, G, W, D, scorer, must, one, vec):
    """Masses, cuts and quotas in the scorer's workgroups: full and ragged last pieces, an empty sequence, 64 and 65 segments, a
    must-keep set (whose bitmap they clear), rows of odd stride, scratch that holds garbage."""
    w = inputs.CONFIGS[1].scaled(L=1, B=3, H=2, G=G, W=W, D=D, T=T, T_min=T, dtype=dtype, budget=max(1, T // 5), S=S, n_spans=3,
                                 span_len=(1, max(1, min(30, T))), n_sink=3 * must, n_last=20 * must)
    host = inputs.dense_cache(w, n_threads=4)
    host["seq_lens"][:] = [T, 0, max(1, T // 2 - 1)]
    credit = np.abs(np.random.default_rng(T + S).standard_normal((6, T))).astype(np.float32)
    credit /= credit.sum(1, keepdims=True)
    for i, n in enumerate(n for n in host["seq_lens"] for _ in range(2)):
        credit[i, n:] = 0
    job = Job(w, host, scorer=scorer, credit=credit, score_path=B.SCORE_PATH_ONE_LAUNCH)
    if not vec:
        job.t_stride = job.p.t_stride = T | 1
        job.credit = torch.zeros((job.units, job.t_stride), device=DEV)
        job.credit[:, :T] = to_dev(credit)
        job.ws = torch.zeros(B.ams_workspace_bytes(job.p), dtype=torch.uint8, device=DEV)
    job.ws.fill_(255)
    labels = _labels(job)
    assert "score_unit" in labels and any("cuts" in x for x in labels) != one
    assert to_host(job.n_kept).tolist() == [min(w.budget, int(t)) for t in host["seq_lens"] for _ in range(2)]
    assert (to_host(job.idx)[2:4] == -1).all() and (to_host(job.intermediates().bounds)[2:4] == 0).all()
    before = np.zeros((6, job.t_max), np.float32)
    before[:, :T] = credit
    check_units(oracle, job, host, before, [0, 1, 4, 5], scorer=scorer)


@pytest.mark.parametrize("units,T,dtype,G,W,D,scorer,follows", [
    (256, 300, "f32", 1, 8, 64, B.SCORER_MEAN_WINDOW, None), (257, 300, "f32", 1, 8, 64, B.SCORER_MEAN_WINDOW, "unit_mass_cuts"),
    (256, 200, "bf16", 4, 32, 128, B.SCORER_LAST_QUERY, None), (257, 200, "bf16", 4, 32, 128, B.SCORER_LAST_QUERY, "unit_mass_cuts"),
    (512, 200, "bf16", 4, 32, 64, B.SCORER_LAST_QUERY, "unit_mass_cuts"), (258, 2049, "bf16", 4, 32, 64, B.SCORER_MEAN_WINDOW, None),
    (257, 2049, "bf16", 3, 32, 128, B.SCORER_MEAN_WINDOW, "unit_mass_cuts"), (513, 200, "bf16", 4, 32, 128, B.SCORER_LAST_QUERY, "mass_ema"),
    (1536, 130, "bf16", 1, 8, 64, B.SCORER_MEAN_WINDOW, None), (1537, 130, "bf16", 1, 8, 64, B.SCORER_MEAN_WINDOW, "mass_ema"),
    (1536, 97, "bf16", 1, 24, 128, B.SCORER_LAST_QUERY, None), (130, 555, "f32", 3, 32, 128, B.SCORER_MEAN_WINDOW, None)])
def test_units_up_to_which_the_scorer_goes_on_to_the_quotas(oracle, units, T, dtype, G, W, D, scorer, follows):
    """One round of fp32 and of large bf16 tiles (two of most of the latter past 2048 positions), three of small ones; past them the
    scorer hands its sums of usage and credit to the kernel that forms masses and cuts (up to 512 units) or to the position-wise one.
    Short and empty sequences would only repeat the pinned path's test."""
    w = inputs.CONFIGS[1].scaled(L=1, B=1, H=units, G=G, W=W, D=D, T=T, T_min=T, dtype=dtype, budget=T // 4, S=5, n_spans=2,
                                 span_len=(4, 30))
    host = inputs.dense_cache(w, n_threads=4)
    credit = np.random.default_rng(units).random((units, T)).astype(np.float32)
    credit /= credit.sum(1, keepdims=True)
    job = Job(w, host, scorer=scorer, credit=credit)
    labels = _labels(job)
    assert "score_unit" in labels
    assert (follows in labels) if follows else not any("mass" in x or "cuts" in x for x in labels)
    check_properties_all_units(job)
    before = np.zeros((units, job.t_max), np.float32)
    before[:, :T] = credit
    check_units(oracle, job, host, before, [0, 1, units // 2, units - 1], scorer=scorer)


@pytest.mark.parametrize("vec", [True, False])
@pytest.mark.parametrize("T,S,fused", [(2048, 64, True), (2049, 5, True), (4096, 64, True), (4097, 7, True), (8192, 64, True),
                                       (8193, 16, False), (3000, 65, False), (63, 3, True)])
def test_short_caches_form_masses_and_cuts_in_one_launch(oracle, T, S, fused, vec):
    """The three workgroup sizes and their edges, ragged and empty sequences, 64 / 65 segments, rows of odd stride."""
    w = inputs.CONFIGS[1].scaled(L=1, B=3, H=2, G=1, W=8, T=T, T_min=T, budget=max(1, T // 5), S=S, n_spans=3,
                                 span_len=(1, 30))
    host = inputs.dense_cache(w, n_threads=4)
    host["seq_lens"][:] = [T, 0, max(1, T // 2 - 1)]
    job = Job(w, host)
    if not vec:
        job.t_stride = job.p.t_stride = T | 1
        job.credit = torch.zeros((job.units, job.t_stride), device=DEV)
        job.ws = torch.zeros(B.ams_workspace_bytes(job.p), dtype=torch.uint8, device=DEV)
    labels = _labels(job)
    assert ("unit_mass_cuts" in labels) == fused and ("mass_ema" in labels) != fused
    assert to_host(job.n_kept).tolist() == [min(w.budget, int(t)) for t in host["seq_lens"] for _ in range(2)]
    assert (to_host(job.idx)[2:4] == -1).all() and (to_host(job.intermediates().bounds)[2:4] == 0).all()
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), [0, 1, 4, 5])


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 128)])
@pytest.mark.parametrize("T,S,budget,gathers", [(9000, 4, 3000, True), (10240, 4, 4000, True), (10241, 4, 1000, False),
                                                (5000, 16, 128, True), (5000, 16, 127, False), (700, 4, 349, True),
                                                (700, 4, 350, False), (2000, 1, 900, True)])
def test_selection_gathers_its_rows(oracle, T, S, budget, gathers, dtype, D, paged):
    """Shares of a segment's picks over one to sixteen workgroups; picks beyond the list in LDS; a segment longer than the
    registers hold (half of the mass lies in a few positions in front of it); segments kept whole; both layouts."""
    w = inputs.CONFIGS[1].scaled(L=1, B=2, H=2, G=1, W=8, D=D, T=T, T_min=T, dtype=dtype, budget=budget, S=S, n_spans=0,
                                 paged=paged)
    host = inputs.dense_cache(w, n_threads=4)
    host["seq_lens"][:] = [T, T - 3]
    k, q = inputs.as_f32(host["K"]).copy(), inputs.as_f32(host["Q"])
    for h in range(2):
        qbar = q[0, 0, h].mean(0)
        k[0, 0, h, 5:9] += 9 * qbar / np.linalg.norm(qbar)     # the first sequence: most thresholds fall on four positions
    host["K"] = inputs._store(k, dtype)
    job = Job(w, host)
    labels = _labels(job)
    assert ("select_gather" in labels) == gathers and ("compact" in labels) != gathers
    check_properties_all_units(job)
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), list(range(w.units)))


def _chunks_of_first_unit(job):
    """Runs a step over a workspace of ones and counts the chunks of which the first sweep has left statistics: the rows at the
    head of the workspace, up to the first that nothing has written."""
    job.ws.fill_(255)
    job.step()
    n_pad = next(32 * n for n in (1, 2, 4, 7, 8) if 32 * n >= job.w.G * job.w.W)
    rows = job.ws[:min(job.ws.numel(), 600 * n_pad * 8) // (n_pad * 8) * n_pad * 8].view(torch.int32).reshape(-1, n_pad * 2)
    blank = to_host((rows == -1).all(1))
    return int(np.argmax(blank))


@pytest.mark.parametrize("scorer,causal", [(B.SCORER_MEAN_WINDOW, False), (B.SCORER_LAST_QUERY, True), (B.SCORER_KEYDIFF, False),
                                           (B.SCORER_REDUNDANCY, False), (B.SCORER_EXPECTED_VNORM, True),
                                           (B.SCORER_EXPECTED_VNORM, False)])
@pytest.mark.parametrize("units,T,dtype,G,W,D,chunk", [(5, 30000, "bf16", 7, 32, 128, 640),    # one workgroup per CU
                                                       (64, 6000, "bf16", 4, 32, 128, 768),    # two
                                                       (64, 7001, "bf16", 2, 8, 128, 640),     # three
                                                       (20, 15999, "f32", 1, 8, 128, 640),     # two
                                                       (12, 26001, "bf16", 4, 32, 64, 640)])   # three: 512 is too short; two
def test_chunks_that_fill_one_round(oracle, units, T, dtype, G, W, D, chunk, scorer, causal):
    """Chunks that are no power of two: every part of a step that counts in chunks, ragged last chunks."""
    w = inputs.CONFIGS[1].scaled(L=units // 4 if units % 4 == 0 else 1, H=4 if units % 4 == 0 else units, D=D, G=G, W=W, T=T,
                                 T_min=T, dtype=dtype, budget=200, S=8, n_spans=4, span_len=(8, 200), causal=causal)
    host = inputs.dense_cache(w, n_threads=4)
    job = Job(w, host, scorer=scorer)
    if not causal:
        assert _chunks_of_first_unit(job) == -(-T // chunk)
        job.credit.zero_()
        job.ws.zero_()
    job.step()
    check_properties_all_units(job)
    i = units - 1
    if scorer != B.SCORER_REDUNDANCY or T <= 7000:
        units = [i] if scorer == B.SCORER_REDUNDANCY else [0, units // 2, i]
        check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), units, scorer=scorer)
    else:           # the oracle evaluates the T^2 definition, minutes at these lengths: the sum of the unit vectors in double
        u, g = to_host(job.intermediates().u)[i, :T], to_host(job.intermediates().g)[i, :T]
        k = inputs.as_f32(host["K"]).reshape(-1, T, D)[i].astype(np.float64)
        k /= np.linalg.norm(k, axis=1, keepdims=True)
        p = np.exp((k @ k.sum(0) - 1) / (T - 1))
        p /= p.sum()
        imp = job.p.mix_lambda * oracle.pool(u, job.p.score_kernel).astype(np.float64)
        p *= 1 - job.p.mix_lambda
        assert_close_terms(g, imp - p, imp + p, what="g")


@pytest.mark.parametrize("common", [0.0, 30.0])
@pytest.mark.parametrize("D,G,W,L", [(128, 1, 1, 1), (128, 1, 8, 1), (128, 2, 16, 1), (128, 3, 11, 1), (128, 8, 8, 1), (128, 5, 13, 1),
                                     (128, 7, 16, 1), (128, 4, 32, 1), (128, 5, 13, 128), (128, 7, 16, 128), (128, 4, 32, 128),
                                     (128, 4, 32, 127), (64, 1, 3, 1), (64, 4, 32, 1), (64, 3, 43, 1), (64, 7, 32, 1), (64, 9, 25, 1),
                                     (64, 8, 32, 1)])
def test_centred_moments_at_every_number_of_columns(oracle, D, G, W, L, common):
    """Padded columns of every tile shape take no part in the variance; queries with a common part far above their
    differences (the variance must not be a difference of two large numbers).  With 128 channels and 65 to 128 queries the
    centred form starts at 512 workgroups (128 layers here)."""
    w = inputs.CONFIGS[1].scaled(L=L, B=2, H=2, D=D, G=G, W=W, T=700, T_min=700, budget=64, S=4, n_spans=2, span_len=(8, 60))
    host = inputs.dense_cache(w, n_threads=4)
    host["seq_lens"][:] = [700, 681]
    rng = np.random.default_rng(D + G * W)
    q = inputs.as_f32(host["Q"]) + common * rng.standard_normal((L, 2, 2, 1, 1, D)).repeat(G, 3).reshape(L, 2, 2 * G, 1, D)
    k = inputs.as_f32(host["K"]) * (0.05 if common else 1.0)      # logits stay in the supported range
    host["Q"], host["K"] = inputs._store(q.astype(np.float32), "bf16"), inputs._store(k.astype(np.float32), "bf16")
    job = Job(w, host, scorer=B.SCORER_EXPECTED)
    job.step()
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), [0, 1, 2, w.units - 1], scorer=B.SCORER_EXPECTED)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("L,N,H", [(16, 33, 2), (5, 64, 3), (18, 2, 16), (4, 65, 3), (23, 3, 8)])
def test_ragged_batches_count_the_chunks_that_exist(oracle, L, N, H, paged, causal):
    """Launches of more than 1536 workgroups, up to 64 sequences and one more: empty sequences first, in the middle and last,
    lengths around the chunk's edges; every (unit, chunk) once in both sweeps."""
    T = 2100
    w = inputs.CONFIGS[1].scaled(L=L, B=N, H=H, G=1, W=4, D=64, T=T, T_min=T, budget=40, S=2, n_spans=2, span_len=(8, 90),
                                 paged=paged, causal=causal)
    host = inputs.dense_cache(w, n_threads=8)
    lens = np.random.default_rng(N).choice([0, 1, 31, 1023, 1024, 1025, 1030, 2048, 2049, T], size=N)
    lens[0], lens[-1] = 0, 0
    lens[N // 2] = T
    host["seq_lens"][:] = lens
    job = Job(w, host, score_path=B.SCORE_PATH_TWO_SWEEPS)
    assert w.units * ((T + 1023) // 1024) >= 1536
    job.intermediates().u.fill_(-1.0)
    job.step()
    u = job.intermediates().u.double()
    seen = torch.arange(job.t_stride, device=DEV)[None, :] < job.lens.long().repeat_interleave(H).repeat(L)[:, None]
    total = (u * seen).sum(1)
    assert bool(((u >= 0) | ~seen).all()) and bool((u[~seen] == -1).all())
    if not causal:
        assert float((total[seen[:, 0]] - 1).abs().max()) < 1e-4
    live = [i for i in range(w.units) if lens[i // H % N] > 0]
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), live[::max(1, len(live) // 12)])


@pytest.mark.parametrize("n_sink,n_last", [(40, 900), (1, 0), (0, 64)])
@pytest.mark.parametrize("T", [1023, 1025, 6007, 32768, 32769])
def test_gap_of_a_must_keep_set_is_filled(oracle, T, n_sink, n_last):
    """More than 64 positions to fill, and few; keys that share a bin over several passes, ties by the hundred, infinities
    and NaN; the last length whose keys stay in registers and the first that does not."""
    S, rng = 5, np.random.default_rng(T + n_last)
    bounds = np.array([0, 7, T // 5, T // 2, T - 100, T], np.int32)
    g = rng.standard_normal((5, T)).astype(np.float32)
    g[1] = (1 + rng.integers(0, 70, T) * 2.0 ** -23).astype(np.float32)
    g[1, ::501] = 3e38
    g[2] = -1.5
    g[3] = np.round(g[3] * 2)
    g[4, ::3], g[4, 1::5], g[4, 2::7], g[4, 4::11] = np.nan, -np.inf, np.inf, -0.0
    g[:, :40] += 2.0                                                # the segments pick must-keep positions
    g[:, -900:] += 2.0
    mass = np.tile(np.diff(bounds).astype(np.float32) / T, (5, 1))
    for budget in (n_sink + n_last + 3, T // 2 + 500):
        p = _stage_params(5, T, S)
        p.budget, p.n_sink, p.n_last = budget, n_sink, n_last
        quota = torch.zeros((5, S), dtype=torch.int32, device=DEV)
        idx, n_kept = torch.zeros((5, budget), dtype=torch.int32, device=DEV), torch.zeros(5, dtype=torch.int32, device=DEV)
        B.ams_select(p, to_dev(np.array([T], np.int32)), to_dev(g), to_dev(np.tile(bounds, (5, 1))), to_dev(mass), quota,
                     idx, n_kept, workspace(p))
        sinks, last, seg_budget = oracle.must_keep(T, budget, n_sink, n_last)
        n = min(budget, T)
        for i in range(5):
            q = oracle.quota(bounds, mass[i], seg_budget, 1)
            want = oracle.finalize(g[i], oracle.select(g[i], bounds, q), sinks, last, n)
            np.testing.assert_array_equal(to_host(idx)[i, :n], want, err_msg=f"row {i} budget {budget}")


@pytest.mark.parametrize("scorer,units,T,G,one_launch", [
    (B.SCORER_MEAN_WINDOW, 128, 2816, 2, True), (B.SCORER_MEAN_WINDOW, 128, 2817, 2, False), (B.SCORER_LAST_QUERY, 178, 4096, 2, True),
    (B.SCORER_LAST_QUERY, 160, 3500, 2, False), (B.SCORER_LAST_QUERY, 162, 3500, 2, True),
    (B.SCORER_MEAN_WINDOW, 136, 3073, 32, False),      # 680 workgroups, three to a CU
    (B.SCORER_MEAN_WINDOW, 136, 3328, 32, True),       # 544 workgroups: a second round
    (B.SCORER_MEAN_WINDOW, 160, 3072, 32, False), (B.SCORER_MEAN_WINDOW, 160, 3073, 32, True),     # 480 and 640
    (B.SCORER_KEYDIFF, 128, 900, 2, False), (B.SCORER_REDUNDANCY, 130, 300, 2, False)])
def test_short_caches_choose_their_scorer(oracle, scorer, units, T, G, one_launch):
    """Where the one-launch scorer ends: beyond 2816 positions, with up to 160 units, where the sweeps run in one round; scores
    that need the keys."""
    w = inputs.CONFIGS[1].scaled(L=units // 2, H=2, G=G, W=4, D=64, T=T, T_min=T, budget=60, S=4, n_spans=2, span_len=(8, 90))
    host = inputs.dense_cache(w, n_threads=8)
    job = Job(w, host, scorer=scorer)
    assert ("score_unit" in _labels(job)) == one_launch
    check_properties_all_units(job)
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), [0, units // 2, units - 1], scorer=scorer)


@pytest.mark.parametrize("scorer,causal", [(B.SCORER_MEAN_WINDOW, False), (B.SCORER_KEYDIFF, False), (B.SCORER_REDUNDANCY, False),
                                           (B.SCORER_EXPECTED_VNORM, False), (B.SCORER_LAST_QUERY, True), (B.SCORER_KEYDIFF, True)])
@pytest.mark.parametrize("units,t_max,dtype,G,W,D", [(5, 30000, "bf16", 7, 32, 128), (64, 7001, "bf16", 2, 8, 128),
                                                     (20, 15999, "f32", 1, 8, 128)])
@pytest.mark.parametrize("T", [6000, 3201, 129, 1, 0])
def test_a_short_cache_is_shared_by_all_workgroups(oracle, units, t_max, dtype, G, W, D, scorer, causal, T):
    """t_max is a capacity: chunks that would fill one round of workgroups at t_max get shorter with the cache, in steps of 128
    positions, so that as many workgroups share it."""
    w = inputs.CONFIGS[1].scaled(L=units // 4 if units % 4 == 0 else 1, H=4 if units % 4 == 0 else units, D=D, G=G, W=W, T=t_max,
                                 T_min=t_max, dtype=dtype, budget=200, S=8, n_spans=9, span_len=(8, 200), causal=causal)
    host = inputs.dense_cache(w, n_threads=4)
    job = Job(w, host, scorer=scorer)
    at_t_max = _chunks_of_first_unit(job) if not causal else 0
    host["seq_lens"][:] = T
    job.lens.fill_(T)
    if not causal and T > 0:
        assert _chunks_of_first_unit(job) == -(-T // (-(-T // (at_t_max * 128)) * 128))      # multiples of 128
    job.ws.fill_(255)
    job.credit.zero_()
    job.step()
    assert to_host(job.n_kept).tolist() == [min(w.budget, T)] * units
    if T > 0:
        check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), [units // 2] if T > 2000 else [0, units - 1], scorer=scorer)


@pytest.mark.parametrize("path", [B.SCORE_PATH_ONE_READ, B.SCORE_PATH_TWO_SWEEPS])
@pytest.mark.parametrize("T", [16384, 10001, 700])
def test_sums_of_a_short_cache_by_either_scorer(oracle, path, T):
    """8 units with t_max 16384: the one-read scorer leaves a sum per 512 positions, and the sweeps' chunks have 512 at t_max but
    less in a shorter cache."""
    w = inputs.CONFIGS[1].scaled(L=2, H=4, G=2, W=8, T=16384, T_min=16384, budget=300, S=8, n_spans=4, span_len=(8, 200))
    host = inputs.dense_cache(w, n_threads=4)
    job = Job(w, host, score_path=path)
    host["seq_lens"][:] = T
    job.lens.fill_(T)
    job.ws.fill_(255)                                       # entries that nobody writes are no numbers
    job.step()
    assert to_host(job.n_kept).tolist() == [300] * 8
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), [0, 7])


@pytest.mark.parametrize("units", [32767, 32769])             # 65534 rows of the sweeps; 65538 of them, two to a row of the grid
def test_causal_window_over_more_units_than_half_the_grids_rows(oracle, units):
    """One chunk and one tail per unit."""
    w = inputs.CONFIGS[1].scaled(L=1, B=1, H=units, G=1, W=8, D=64, T=40, T_min=40, budget=12, S=2, causal=True)
    rng = np.random.default_rng(units)
    bits = lambda *shape: (rng.standard_normal(shape, np.float32).view(np.uint32) >> 16).astype(np.uint16)
    host = {"K": bits(1, 1, units, 40, 64), "V": bits(1, 1, units, 40, 64), "Q": bits(1, 1, units, 8, 64),
            "seq_lens": np.array([40], np.int32)}
    job = Job(w, host)
    job.step()
    check_properties_all_units(job)
    check_units(oracle, job, host, np.zeros((w.units, job.t_max), np.float32), [0, 1, units // 2, units - 2, units - 1])
