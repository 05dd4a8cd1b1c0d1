"""Launches with a team of waves per query against launches with one wave per
query and against the oracle, identical in ids, distances, widths and counts:
row widths around the slices that two helpers share, one row trip and several,
both kinds of visited set, query counts below and above what is resident at
once (where the launch for many queries takes over), every driver mode."""
import numpy as np
import pytest

import oracle
from helpers import random_arrays, random_index, random_queries
from test_gpu_parity import assert_parity, gpu_search

pytestmark = pytest.mark.gpu

MODES = {"phased": {}, "fused": {"fused": True}, "warm": {"fused": True, "warm": True}, "split": {"split": True},
         "plus": {"boa_plus": True, "sub_batches": 3}, "fixed": {"fixed_L": 70}}
SHAPES = [("f32", 4, 2, 1), ("f32", 64, 33, 2), ("f32", 128, 64, 3), ("f32", 768, 31, 4), ("f32", 1024, 64, 8),
          ("u8", 128, 32, 2), ("u8", 16, 63, 1), ("u8", 272, 5, 5)]


@pytest.mark.parametrize("dtype,d,R,m", SHAPES)
def test_team_equals_one_wave_and_oracle(dtype, d, R, m):
    import paper_2609_16175_amd as boa
    kw = dict(n=2000, d=d, m=m, R=R, dtype=dtype, seed=7, f32_col=m > 2)
    ref_ix = random_index(**kw)
    ix = boa.Index(*random_arrays(**kw))
    for nq in (1, 300, 1500):
        q, r = random_queries(ref_ix, nq, 60, nq, f32_col=m > 2)
        for name, mode in MODES.items():
            widths = [mode["fixed_L"]] if "fixed_L" in mode else [8, 24, 72, 200]
            if name == "warm":
                ref = oracle.boa_warm(ref_ix, q, r, 5, widths, 0.02)
            else:
                ref = oracle.boa(ref_ix, q, r, 5, widths, 0.02, threads=8)
            par = dict(k=5, eps=0.02, **mode) if "fixed_L" in mode else dict(k=5, eps=0.02, schedule=widths, **mode)
            for waves in (0, 1):
                for slots in (0, 64) if nq == 300 else (0,):
                    got = gpu_search(ix, q, r, escalation_waves=waves, lds_hash_slots=slots, **par)
                    assert_parity(got, ref, f"{name} nq={nq} escalation_waves={waves} slots={slots}")
    ix.close()


@pytest.mark.parametrize("dtype,d,R,M", [("f32", 36, 40, 18), ("f32", 96, 64, 32), ("u8", 272, 16, 34),
                                         ("f32", 768, 48, 192), ("f32", 512, 33, 256)])
def test_pq_team_equals_one_wave_and_oracle(dtype, d, R, M):
    """Product-quantised search: codes that end inside, at and past a 16-byte
    chunk, widths whose re-rank keys need more room than the distance table."""
    import paper_2609_16175_amd as boa
    from workloads import pq
    x, attrs, types, adj, entry = random_arrays(n=2000, d=d, m=2, R=R, dtype=dtype, seed=9)
    cb = pq.train(x, M, seed=2, sample=1000, iters=3)
    codes = pq.encode(x, cb)
    ref_ix = oracle.Index(x, attrs, types, adj, entry, cb, codes)
    ix = boa.Index(x, attrs, types, adj, entry)
    ix.set_pq(cb, codes)
    for nq in (3, 1500):
        q, r = random_queries(ref_ix, nq, 60, nq)
        for mode, ref in (({"fused": True}, oracle.boa(ref_ix, q, r, 5, [8, 40, 600], 0.02, threads=8)),
                          ({"fused": True, "warm": True}, oracle.boa_warm(ref_ix, q, r, 5, [8, 40, 600], 0.02))):
            for waves in (0, 1):
                got = gpu_search(ix, q, r, k=5, eps=0.02, schedule=[8, 40, 600], pq=True, escalation_waves=waves, **mode)
                assert_parity(got, ref, f"pq M={M} {mode} nq={nq} escalation_waves={waves}")
    ix.close()
