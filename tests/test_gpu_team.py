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
                    if nq == 300:   # the (first) launch is one of teams, 4 or 7 waves each, or is not
                        st = ix.stats()
                        team = st["waves_per_block"] in (4, 7) and st["blocks"] == (100 if name == "plus" else 300)
                        assert team == (waves == 0), (name, slots, st["waves_per_block"], st["blocks"])
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


def test_teams_with_tables_that_spill():
    """An index too large for the LDS bitmap over all ids (1.3 million points,
    162,500 bytes of a block's 163,840): teams, and the phased and split search
    in one launch, with the automatic hashed table, whose 16,384 slots a query of
    width 700 overflows into its team's HBM bitmap; and without allocation, where
    the scratch memory holds bitmaps for fewer teams than there are queries
    (64 MiB for 388 of 600)."""
    import paper_2609_16175_amd as boa
    n, d, R = 1_300_000, 16, 32
    g = np.random.default_rng(11)
    x = g.integers(0, 256, size=(n, d)).astype(np.uint8)
    attrs = g.integers(0, 100, size=(n, 1)).astype(np.int32)
    steps = np.stack([g.choice(n - 1, R, replace=False) + 1 for _ in range(64)])
    rows = np.arange(n)
    adj = ((rows[:, None] + steps[rows % 64]) % n).astype(np.uint32)   # mostly new to a query
    types = np.zeros(1, dtype=np.int32)
    ref_ix = oracle.Index(x, attrs, types, adj, 5)
    ix = boa.Index(x, attrs, types, adj, 5)
    widths = [8, 40, 700]
    for nq, eps in ((1, 0.0), (600, 0.05)):
        q, r = random_queries(ref_ix, nq, 60, nq)
        ref = oracle.boa(ref_ix, q, r, 5, widths, eps, threads=8)
        ref_warm = oracle.boa_warm(ref_ix, q, r, 5, widths, eps)
        assert ref.phases[2]["active"] > 0
        for name in ("phased", "fused", "warm", "split", "plus"):
            for no_alloc in (False, True):
                if name == "plus" and no_alloc:
                    continue   # (refused: it needs a second stream)
                ix.reset_counters()
                got = gpu_search(ix, q, r, k=5, eps=eps, schedule=widths, no_alloc=no_alloc, **MODES[name])
                assert_parity(got, ref_warm if name == "warm" else ref, f"{name} nq={nq} no_alloc={no_alloc}")
                if no_alloc:
                    continue
                st = ix.stats()
                assert st["spilled_queries"] > 0
                if name != "plus":   # one launch of teams of 4 waves
                    assert (st["waves_per_block"], st["blocks"], st["lds_hash_slots"]) == (4, nq, 16384)
                    assert st["cum_launches"] == 1
    ix.close()


def test_statistics_report_what_was_launched():
    """Shape and number of the launches in the statistics, for teams, for one
    wave per query, and where the number of a phase's queries is known on the
    device only and two kernels follow each other. An expansion takes 4 waves
    of a team here (R <= 32, rows of 128 bytes). Tables of 16,384 slots (32 KB)
    leave room for 4 teams per CU at width 8 and for 2 at width 2,048, by the
    160 KB of a CU: 800 queries are then teams in the first phase, and at most
    512 of them in the second."""
    import torch

    import paper_2609_16175_amd as boa
    kw = dict(n=2000, d=32, m=1, R=12, dtype="f32", seed=3)
    ref_ix = random_index(**kw)
    ix = boa.Index(*random_arrays(**kw))
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the capacities are those of 256 CUs")

    def run(nq, **par):
        q, r = random_queries(ref_ix, nq, 60, nq)
        ix.reset_counters()
        gpu_search(ix, q, r, k=5, **par)
        st = ix.stats()
        shape = (st["waves_per_block"], st["blocks"], st["lds_hash_slots"])
        launches = [p["launches"] for p in st["phases"]]
        assert st["cum_launches"] == sum(st["cum_phase_launches"])
        return shape, launches, st["cum_phase_launches"], st

    for mode in ({"fixed_L": 16}, {"schedule": [8], "fused": True}):
        assert run(300, **mode)[:3] == ((4, 300, 0), [1], [1])
    shape, launches, cum, _ = run(300, fixed_L=16, escalation_waves=1)
    assert shape[0] <= 4 and shape[0] * shape[1] >= 300 and shape[2] > 0 and launches == cum == [1]
    # modes 0 and 2 in one launch: its time under phase 0
    for mode in ({}, {"split": True}):
        shape, launches, cum, st = run(300, schedule=[8, 24], eps=0.0, **mode)
        assert shape == (4, 300, 0) and launches == [1, 1] and cum == [1, 0]
        assert st["phases"][0]["kernel_ms"] > 0 and st["phases"][1]["kernel_ms"] == 0
    # sub-batches of 100, then a pool of 200 and one of 100
    shape, launches, cum, _ = run(300, schedule=[8, 24], eps=0.0, boa_plus=True, sub_batches=3)
    assert shape == (4, 100, 0) and launches == cum == [3, 2]
    wide = dict(schedule=[8, 2048], eps=0.0, lds_hash_slots=16384)
    shape, launches, cum, _ = run(800, **wide)
    assert shape == (4, 800, 16384) and launches == cum == [1, 2]
    shape, launches, cum, _ = run(800, split=True, **wide)
    assert shape == (4, 800, 16384) and launches == cum == [1, 1]
    # more than fit at the narrow width, too
    shape, launches, cum, _ = run(1100, **wide)
    assert shape[0] < 4 and shape[2] == 16384 and launches == cum == [1, 2]
    ix.close()


def test_total_time_ends_with_the_last_device_work():
    """A split search without survivors ends with their compaction: one block
    over 2^18 flags, 256 steps of at least half a microsecond, beside 10 to
    20 us for what precedes the search launch."""
    import paper_2609_16175_amd as boa
    kw = dict(n=2000, d=16, m=1, R=8, dtype="f32", seed=5)
    ref_ix = random_index(**kw)
    ix = boa.Index(*random_arrays(**kw))
    q, r = random_queries(ref_ix, 1 << 18, 60, 1)
    r[:, :, 0], r[:, :, 1] = -2**31, 2**31 - 1
    rest = []
    for _ in range(3):
        gpu_search(ix, q, r, k=1, schedule=[4, 8], eps=1.0, split=True)
        st = ix.stats()
        assert [p["active"] for p in st["phases"]] == [1 << 18, 0]
        rest.append(st["total_ms"] - st["phases"][0]["kernel_ms"])
    assert min(rest) > 0.1, rest
    ix.close()
