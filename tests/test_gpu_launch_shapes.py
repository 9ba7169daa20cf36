"""Whole steps at the sizes where the split of the work changes: the edges of the chunks, tiles and groups that the
kernels cut a unit into.  Checked like every step (scores and masses within relative 1e-5 of the oracle, every later
stage exact on the GPU's own floats)."""
import numpy as np
import pytest

from paper_2605_23200_amd import binding as B
from paper_2605_23200_amd import inputs
from paper_2605_23200_amd.harness import Job
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
                                                ("bf16", 7, 32, 385, True), ("bf16", 2, 16, 8193, False)])
def test_few_units_are_cut_into_short_chunks(oracle, dtype, G, W, T, paged, causal):
    """Few units: chunks of 128 keys (one block per wave), up to one workgroup per CU; a ragged second sequence ends
    inside, on and before a chunk's edge."""
    w = inputs.CONFIGS[1].scaled(L=1, B=2, H=2, G=G, W=W, T=T, T_min=T, dtype=dtype, budget=min(64, T), S=4, n_spans=2,
                                 span_len=(4, 40), paged=paged, causal=causal)
    _run(oracle, w, lens=[T, max(1, T - 1 - (T % 128))])
