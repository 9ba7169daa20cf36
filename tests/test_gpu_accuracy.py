"""Inputs on which a result hangs on the precision of its intermediate sums: dominant keys, keys that nearly cancel,
segments whose mass is a tiny part of the prefix.  Each bound is derived from the roundings that a result may carry."""
import numpy as np
import pytest
import torch

from paper_2605_23200_amd import binding as B
from paper_2605_23200_amd import inputs
from paper_2605_23200_amd.harness import Job
from gpu_util import DEV, assert_close_rel, assert_close_terms, score_term_magnitudes, to_dev, to_host, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [4, 5, 7, 8])
def test_two_dominant_keys_share_the_mass(oracle, G):
    """Two keys with the same logit, 20 to 23 powers of two above the first keys their waves see, in blocks of different
    waves.  All queries are ones and every key is one repeated number, so the logits are exact and the two keys hold nearly
    half of the mass each.  What is left: the exponential of each key's own maximum and its rounded argument, the weight, at
    most eight column sums (of equal terms: the inexact ones are 3, 5, 6 and 7) and the store, 6 roundings of 2^-24 = 3.6e-7.
    An exponent of 20 carried in fp32 adds up to 1.3e-6 of the share on its own."""
    w = inputs.CONFIGS[1].scaled(L=8, H=8, G=G, W=32, T=4200, budget=300, S=4, n_spans=0)
    host = inputs.dense_cache(w, n_threads=8)
    rng = np.random.default_rng(G)
    one = lambda x: inputs.to_bf16_bits(np.float32(x))
    host["Q"][:] = one(1.0)
    host["K"][:] = one(-1.0)
    t1, t2 = 130, 200                         # second blocks of waves 0 and 2 (blocks of 32 keys, four waves)
    for l in range(8):
        for h in range(8):
            k = host["K"][l, 0, h]
            r1, r2 = rng.integers(1, 128, 2) / 1024.0      # raw logits -16 .. 0 of the waves' first blocks
            k[0:32], k[64:96] = one(-r1), one(-r2)
            k[t1], k[t2] = one(1.25), one(1.25)            # raw logit 160
    job = Job(w, host)
    job.step()
    u = to_host(job.intermediates().u)
    worst = 0.0
    for i in range(0, 64, 3):
        l, h = i // 8, i % 8
        want, _ = oracle.score(host["Q"][l, 0, h * G:(h + 1) * G].reshape(-1, w.D), host["K"][l, 0, h], G, 32)
        assert_close_rel(u[i, :w.T], want, what=f"u unit {i}")
        worst = max(worst, np.abs(u[i, [t1, t2]].astype(np.float64) / want[[t1, t2]] - 1).max())
    assert worst < 3.6e-7, f"{worst:.2e}"


@pytest.mark.parametrize("dtype,D,G,W", [("bf16", 128, 4, 32), ("bf16", 128, 1, 8), ("bf16", 64, 7, 32), ("bf16", 128, 8, 32),
                                         ("f32", 128, 2, 16)])
def test_mean_key_of_keys_that_cancel(oracle, dtype, D, G, W):
    """Two of every four keys cancel and leave a mean key 2^-22 of their size, which only sums in double keep (the oracle
    sums in double; the products with the mean key are fp32, 1e-5 of their terms as everywhere)."""
    T = 1500
    w = inputs.CONFIGS[1].scaled(L=1, H=2, D=D, G=G, W=W, T=T, dtype=dtype, budget=100, S=4, n_spans=0)
    host = inputs.dense_cache(w, n_threads=4)
    k = inputs.as_f32(host["K"]).copy()
    k[..., 1::2, :] *= np.float32(2.0 ** -22)
    k[..., 2::4, :] = -k[..., 0::4, :][..., :k[..., 2::4, :].shape[-2], :]
    k[..., T // 4 * 4:, :] *= np.float32(2.0 ** -22)
    host["K"] = inputs._store(k, dtype)
    job = Job(w, host, scorer=B.SCORER_KEYDIFF)
    job.step()
    g = to_host(job.intermediates().g)
    for h in range(2):
        q = host["Q"][0, 0, h * G:(h + 1) * G].reshape(-1, D)
        _, want = oracle.score(q, host["K"][0, 0, h], G, W, B.SCORER_KEYDIFF)
        assert_close_terms(g[h, :T], want, score_term_magnitudes(B.SCORER_KEYDIFF, q, host["K"][0, 0, h]), what=f"g unit {h}")


@pytest.mark.parametrize("scorer", [B.SCORER_KEYDIFF, B.SCORER_REDUNDANCY])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_a_key_that_is_no_number(scorer, bad):
    """One entry of one key is infinite or NaN: the scores that a bf16 cache gets from the sweeps are numbers, zeros and NaN
    where those of an fp32 cache with the same values are, which come from the streaming kernels."""
    got = []
    for dtype in ("f32", "bf16"):
        w = inputs.CONFIGS[1].scaled(L=1, H=3, G=2, W=8, T=700, dtype=dtype, budget=100, S=4, n_spans=0)
        host = inputs.dense_cache(w, n_threads=2)
        if dtype == "f32":      # the values of the bf16 cache
            host["K"] = inputs.bf16_bits_to_f32(inputs.to_bf16_bits(host["K"])).reshape(host["K"].shape)
        host["K"][0, 0, 1, 300, 77] = bad if dtype == "f32" else np.array([bad], np.float32).view(np.uint32)[0] >> 16
        host["K"][0, 0, 2, 40] = 0
        job = Job(w, host, scorer=scorer)
        job.step()
        got.append(to_host(job.intermediates().g)[:, :700])
    for i in range(3):
        np.testing.assert_array_equal(np.isnan(got[1][i]), np.isnan(got[0][i]), err_msg=f"unit {i}")
        np.testing.assert_array_equal(got[1][i] == 0, got[0][i] == 0, err_msg=f"unit {i}")


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("T,l_max", [(9000, 256), (70001, 1024), (300000, 2048)])
def test_segment_masses_far_below_the_prefix(oracle, T, l_max, static):
    """Final segments with 1e-12 of the mass and less, behind positions that hold nearly all of it: a mass is a sum of its
    own positions (double, stored as fp32: 1e-6), not a difference of prefixes near one."""
    delta, l_min, cap = 0.1, 16, 12 + T // l_max
    rng = np.random.default_rng(T)
    m = rng.random((2, T)) * 1e-17
    m[:, : T // 8] = rng.random((2, T // 8))
    m[1, -40:] = rng.random(40)
    m = (m / m.sum(1, keepdims=True)).astype(np.float32)
    p = B.make_params(n_layers=1, batch=1, n_kv_heads=2, group=1, window=8, t_max=T, budget=64, n_segments=cap,
                      seg_delta=delta, l_min=l_min, l_max=l_max)
    bounds, mass = torch.full((2, cap + 1), -3, dtype=torch.int32, device=DEV), torch.full((2, cap), -3.0, device=DEV)
    args = (p, to_dev(np.array([T], np.int32)), to_dev(m), bounds, mass)
    if static:
        B.ams_mass_segment_static(*args)
    else:
        B.ams_mass_segment(*args, workspace(p))
    for i in range(2):
        b_o, s_o, _ = oracle.segment_adaptive(m[i], delta, l_min, l_max, cap)
        np.testing.assert_array_equal(to_host(bounds)[i], b_o)
        assert_close_rel(to_host(mass)[i], s_o, rtol=1e-6, atol=0.0, what=f"seg_mass unit {i}")


@pytest.mark.parametrize("heads,T", [(2, 700), (130, 300)])     # the sweeps, the one-launch scorer
@pytest.mark.parametrize("D,G,W", [(128, 1, 8), (128, 2, 20), (128, 7, 16), (64, 4, 32)])
def test_fp32_keys_at_the_ends_of_the_range(oracle, heads, T, D, G, W):
    """fp32 products are formed from bf16 terms.  A key with an infinite entry against queries of one sign has logits of
    minus infinity and no share, and the keys next to it keep theirs (padded query columns multiply the infinity by zero:
    where there are any, the key's own usage may be no number); entries that round to infinity in bf16, and denormal ones,
    are ordinary numbers."""
    w = inputs.CONFIGS[0].scaled(L=1, H=heads, D=D, G=G, W=W, T=T, budget=50, S=4, n_spans=2, span_len=(8, 40))
    host = inputs.dense_cache(w, n_threads=8)
    host["Q"][..., 5] = -np.abs(host["Q"][..., 5]) - np.float32(1e-3)       # all negative in this channel
    k = host["K"]
    k[..., 7, 5] = np.inf
    k[..., T - 1, 5] = np.inf
    k[..., 40, 5] = np.finfo(np.float32).max
    k[..., 41, :] = np.float32(1e-41)
    k[..., 100, :] *= np.float32(2.0 ** -60)
    job = Job(w, host)
    job.step()
    u = to_host(job.intermediates().u)
    for h in range(0, heads, 43):
        want, _ = oracle.score(host["Q"][0, 0, h * G:(h + 1) * G].reshape(-1, D), k[0, 0, h], G, W)
        assert np.isfinite(want).all() and (want[[7, 40, T - 1]] == 0).all()
        plain = np.setdiff1d(np.arange(T), [7, T - 1] if G * W % 32 else [])
        assert_close_rel(u[h, plain], want[plain], what=f"u unit {h}")


@pytest.mark.parametrize("scorer", [B.SCORER_EXPECTED, B.SCORER_EXPECTED_VNORM])
@pytest.mark.parametrize("D,G,W,L", [(128, 1, 8, 1), (128, 4, 32, 1), (128, 4, 32, 130), (128, 3, 25, 130), (128, 7, 32, 1),
                                     (64, 1, 1, 1), (64, 1, 3, 1), (64, 2, 16, 1), (64, 7, 16, 1), (64, 7, 32, 1), (64, 8, 32, 1)])
def test_infinite_keys_next_to_the_expected_score(oracle, D, G, W, L, scorer):
    """A key with an infinite entry against queries of one sign has logits of minus infinity: no share in the usage, and the
    keys next to it keep theirs, whatever becomes of its own moment score (no number).  The largest finite number, whose
    logits are partly minus infinity, likewise.  In a full block, in two blocks of one wave, and in the ragged last one.
    (Padded query columns multiply the infinity by zero: where there are any, the key's own usage may be no number.)"""
    T = 1201                                                # (128 channels: the centred form from 512 workgroups on)
    w = inputs.CONFIGS[1].scaled(L=L, B=2, H=1, D=D, G=G, W=W, T=T, T_min=T, budget=50, S=4, n_spans=2, span_len=(8, 40))
    host = inputs.dense_cache(w, n_threads=8)
    q, k = inputs.as_f32(host["Q"]).copy(), inputs.as_f32(host["K"]).copy()
    q[..., 5] = -np.abs(q[..., 5]) - np.float32(0.01)       # all negative in this channel
    gone = [7, 140, 290, T - 1]
    k[0, 0, :, gone, 5] = np.inf
    k[..., 300, 5] = np.float32(3.3e38)
    host["Q"], host["K"] = inputs._store(q, "bf16"), inputs._store(k, "bf16")
    job = Job(w, host, scorer=scorer)
    job.step()
    inter = job.intermediates()
    u, g, m_used = to_host(inter.u), to_host(inter.g), to_host(inter.m_used)
    for i in range(2):                                      # the second sequence has ordinary keys (and one of 3.3e38)
        Q, K = host["Q"][0, i].reshape(-1, D), host["K"][0, i, 0]
        want, _ = oracle.score(Q, K, G, W)
        assert np.isfinite(want).all() and want[300] == 0 and (i or (want[gone] == 0).all())
        plain = np.setdiff1d(np.arange(T), gone + [300])
        assert_close_rel(u[i, plain], want[plain], what=f"u unit {i}")
        assert (G * W % 32 > 0 and i == 0) or not u[i, gone + [300]][want[gone + [300]] == 0].any()
        np.testing.assert_allclose(m_used[i, plain], oracle.ema(oracle.mass(want, w.eps), np.zeros(T, np.float32), w.lam, w.beta)[0][plain],
                                   rtol=1e-5)
        if scorer == B.SCORER_EXPECTED:
            assert np.isfinite(g[i, plain]).all() and (i or np.isnan(g[i, gone]).all())
            with np.errstate(all="ignore"):
                _, want_g = oracle.score(Q, K[plain], G, W, scorer=B.SCORER_EXPECTED)
                assert_close_terms(g[i, plain], want_g, score_term_magnitudes(scorer, Q, K[plain]), what=f"g unit {i}")


@pytest.mark.parametrize("scorer", [B.SCORER_MEAN_WINDOW, B.SCORER_EXPECTED])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("e", [-118, -110, -60, 60, 110, 118])
@pytest.mark.parametrize("heads,T,D", [(2, 700, 128), (2, 700, 64), (130, 300, 128)])     # the sweeps, the one-launch scorer
def test_scale_of_the_keys_moved_into_the_queries(oracle, heads, T, D, e, dtype, scorer):
    """Keys times a power of two and queries divided by it: the same logits, the same results."""
    G, W = 2, 20
    w = inputs.CONFIGS[0].scaled(L=1, H=heads, D=D, G=G, W=W, T=T, dtype=dtype, budget=50, S=4, n_spans=2, span_len=(8, 40))
    host = inputs.dense_cache(w, n_threads=8)
    plain = {n: inputs.as_f32(host[n]).copy() for n in ("Q", "K")}
    host["K"] = inputs._store((plain["K"] * np.float32(2.0 ** e)).astype(np.float32), dtype)
    host["Q"] = inputs._store((plain["Q"] * np.float32(2.0 ** -e)).astype(np.float32), dtype)
    job = Job(w, host, scorer=scorer)
    job.step()
    u, g = to_host(job.intermediates().u), to_host(job.intermediates().g)
    for h in range(0, heads, 43):
        Q, K = plain["Q"][0, 0, h * G:(h + 1) * G].reshape(-1, D), plain["K"][0, 0, h]
        want, want_g = oracle.score(inputs._store(Q, dtype), inputs._store(K, dtype), G, W, scorer=B.SCORER_EXPECTED)
        assert_close_rel(u[h, :T], want, what=f"u unit {h}")
        if scorer == B.SCORER_EXPECTED:
            assert_close_terms(g[h, :T], want_g, score_term_magnitudes(scorer, Q, K), what=f"g unit {h}")


@pytest.mark.parametrize("bits", [0x7F800001, 0x7F80FFFF, 0x7FC00000, 0x7FFFFFFF])
@pytest.mark.parametrize("heads,T", [(2, 700), (130, 300)])     # the sweeps, the one-launch scorer
@pytest.mark.parametrize("D,G,W", [(128, 1, 8), (128, 7, 16), (64, 4, 32)])
def test_fp32_key_that_is_no_number(heads, T, D, G, W, bits):
    """Whatever its bits, a key entry that is no number leaves no number in its unit's usage (and is not taken for an
    infinity, whose key would drop out against queries of one sign); the other units keep theirs."""
    w = inputs.CONFIGS[0].scaled(L=1, H=heads, D=D, G=G, W=W, T=T, budget=50, S=4, n_spans=2, span_len=(8, 40))
    host = inputs.dense_cache(w, n_threads=8)
    host["Q"][..., 5] = -np.abs(host["Q"][..., 5]) - np.float32(1e-3)
    host["K"].view(np.uint32)[0, 0, 0, 100, 5] = bits
    job = Job(w, host)
    job.step()
    u = to_host(job.intermediates().u)[:, :T]
    assert np.isnan(u[0]).all() and np.isfinite(u[1:]).all()
