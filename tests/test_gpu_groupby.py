"""Group-by on the GPU against the group-by oracle: group keys, counts and
per-column sums, for the hash-based and the partition-based algorithm, int32
and int64 keys and values, group counts from one to beyond an LDS table (the
spill path), the rule's HLL-guided choice, and the edge cases."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_04489_amd as eg
import synth

pytestmark = pytest.mark.gpu


def check(keys, vals, res):
    gk, cnt, sums = oracle.group_by(keys, vals)
    assert res.groups == len(gk)
    k = res.keys.cpu().numpy().astype(np.int64)
    order = np.argsort(k, kind="stable")
    assert np.array_equal(k[order], gk)
    assert np.array_equal(res.counts.cpu().numpy()[order], cnt)
    for got, want in zip(res.sums, sums):
        assert np.array_equal(got.cpu().numpy()[order], want)


def forced(keys, variant, bits=0):
    return eg.groupby_plan(eg.stats(keys), eg.SEL_FORCED, eg.make_groupby_plan(variant, bits))


# part2: 4 partitions of ~250,000 rows, each aggregated in 4 slices merged globally
VARIANTS = [("hash", eg.GB_HASH, 0), ("part2", eg.GB_PARTITION, 2), ("part4", eg.GB_PARTITION, 4),
            ("part8", eg.GB_PARTITION, 8), ("part12p2", eg.GB_PARTITION, 12)]


@pytest.mark.parametrize("variant", VARIANTS, ids=[v[0] for v in VARIANTS])
@pytest.mark.parametrize("groups", [1, 7, 1000, 50000, 300000])
def test_groupby_int32(gpu, variant, groups):
    keys, vals = synth.groupby_input(seed=groups, n=1_000_003, groups=groups, device=gpu)
    res = eg.groupby(keys, vals, forced(keys, variant[1], variant[2]))
    check(keys, vals, res)


@pytest.mark.parametrize("variant", VARIANTS[:3], ids=[v[0] for v in VARIANTS[:3]])
def test_groupby_int64_keys_and_values(gpu, variant):
    keys, vals = synth.groupby_input(seed=5, n=700_001, groups=200_000, key_dtype=torch.int64,
                                     val_dtype=torch.int64, device=gpu)
    vals = [vals[0], vals[1].to(torch.int32)]  # one 8-byte and one 4-byte value column
    res = eg.groupby(keys, vals, forced(keys, variant[1], variant[2]))
    check(keys, vals, res)


@pytest.mark.parametrize("key,val,nv,n", [(torch.int32, torch.int32, 2, 512 * 8192 + 3), (torch.int32, torch.int64, 2, 512 * 8192 + 3),
                                          (torch.int32, torch.int32, 0, 512 * 10240 + 3), (torch.int64, torch.int64, 2, 512 * 6144 + 3),
                                          (torch.int64, torch.int32, 1, 512 * 6144 - 1)])
def test_groupby_partition_tiles(gpu, key, val, nv, n):
    """Partition passes of rows of 0 to 4 value lanes (stride 1 and 2), on both sides
    of the row count from which they take the larger tiles."""
    keys, vals = synth.groupby_input(seed=n, n=n, groups=90_000, key_dtype=key, n_vals=nv, val_dtype=val, device=gpu)
    check(keys, vals, eg.groupby(keys, vals, forced(keys, eg.GB_PARTITION, 9)))


@pytest.mark.parametrize("vals", [(), (torch.int32,), (torch.int64,), (torch.int32, torch.int32), (torch.int32, torch.int64),
                                  (torch.int64, torch.int32), (torch.int64, torch.int64)],
                         ids=lambda v: "_".join(str(t)[6:] for t in v) or "count")
@pytest.mark.parametrize("groups", [1, 16, 17, 128, 600, 1024])
@pytest.mark.parametrize("key", [torch.int32, torch.int64])
def test_groupby_hash_shapes(gpu, key, groups, vals):
    """LDS tables of 64 to 2,048 slots with 32 to one accumulator a slot, every
    combination of value widths, a ragged last step, columns that start one row in."""
    keys, _ = synth.groupby_input(seed=groups, n=150_002, groups=groups, key_dtype=key, n_vals=0, device=gpu)
    cols = [synth.groupby_input(seed=groups + c, n=150_002, groups=1, n_vals=1, val_dtype=t, device=gpu)[1][0]
            for c, t in enumerate(vals)]
    keys, cols = keys[1:], [c[1:] for c in cols]
    check(keys, cols, eg.groupby(keys, cols, forced(keys, eg.GB_HASH)))


@pytest.mark.parametrize("value", [-(1 << 31), (1 << 31) - 1, -1])
def test_groupby_packed_sums_at_their_bounds(gpu, value):
    """Workgroups of more rows than a packed count holds, one group, the values at
    the ends of int32: exact sums known in closed form."""
    n = 768 * 65536 + 5
    keys = torch.full((n,), 3, dtype=torch.int32, device=gpu)
    keys[n // 2] = 4
    vals = torch.full((n,), value, dtype=torch.int32, device=gpu)
    res = eg.groupby(keys, [vals, vals], forced(keys, eg.GB_HASH))
    got = {int(k): (int(c), int(a), int(b)) for k, c, a, b in zip(res.keys, res.counts, *res.sums)}
    assert got == {3: (n - 1, (n - 1) * value, (n - 1) * value), 4: (1, value, value)}


@pytest.mark.parametrize("n", [2047, 2049, 5_000_011])
@pytest.mark.parametrize("vals", [(), (torch.int32, torch.int64), (torch.int64,)], ids=["count", "i32_i64", "i64"])
@pytest.mark.parametrize("order", ["random", "ascending", "late"])
@pytest.mark.parametrize("predicted,groups", [(0, 1000), (1, 33), (100, 513), (400, 1024), (1, 5000)])
def test_groupby_hash_with_a_low_estimate(gpu, n, vals, order, predicted, groups):
    """A plan kept for other data: the workgroups meet more groups than their LDS tables
    were shaped for, from the first rows on, one after another, or after most rows."""
    gid = torch.randint(0, groups, (n,), generator=torch.Generator().manual_seed(n))
    if order == "ascending":
        gid = gid.sort().values
    elif order == "late":
        gid[: n * 3 // 4] = 0
    keys = (gid * 2654435761 % (1 << 31)).to(torch.int32).to(gpu)
    cols = [synth.groupby_input(seed=c, n=n, groups=1, n_vals=1, val_dtype=t, device=gpu)[1][0] for c, t in enumerate(vals)]
    plan = forced(keys, eg.GB_HASH)
    plan.predicted_groups = predicted
    check(keys, cols, eg.groupby(keys, cols, plan, capacity=groups))


def best_time(*calls):
    """The fastest of ten runs of each call, in turn, in ms."""
    best = [float("inf")] * len(calls)
    for _ in range(11):
        for c, f in enumerate(calls):
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            f()
            stop.record()
            stop.synchronize()
            best[c] = min(best[c], start.elapsed_time(stop))
    return best


def test_groupby_hash_time_does_not_hang_on_the_estimate(gpu):
    """1,000 groups planned as one: each workgroup merges once more, rows do not go to
    global atomics one by one (which took 25 times as long)."""
    keys, vals = synth.groupby_input(seed=1, n=1 << 25, groups=1000, n_vals=2, device=gpu)
    plan = forced(keys, eg.GB_HASH)
    low = forced(keys, eg.GB_HASH)
    low.predicted_groups = 1
    t, t_low = best_time(lambda: eg.groupby(keys, vals, plan), lambda: eg.groupby(keys, vals, low, capacity=1000))
    assert t_low < 3 * t, (t_low, t)


@pytest.mark.parametrize("vals", [(), (torch.int32,), (torch.int64,), (torch.int32, torch.int32), (torch.int32, torch.int64),
                                  (torch.int64, torch.int32), (torch.int64, torch.int64)],
                         ids=lambda v: "_".join(str(t)[6:] for t in v) or "count")
@pytest.mark.parametrize("run", [3, 4, 8, 256, 257, 4096])
@pytest.mark.parametrize("key", [torch.int32, torch.int64])
def test_groupby_hash_clustered_rows(gpu, key, run, vals):
    """Runs of one key: rows of a lane, of a wave, or none alone in them; values at the
    ends of their type; tables of one and of two accumulators a slot, and one of two
    slots a group that has to grow; columns that start one row in."""
    n = 300_001
    keys = (torch.arange(n, device=gpu) // run * 7919 % 601 * 104729 - 3_000_000).to(key)
    cols = [synth.groupby_input(seed=c, n=n, groups=1, n_vals=1, val_dtype=t, device=gpu)[1][0] for c, t in enumerate(vals)]
    for c in cols:
        c[: n // 3] = torch.iinfo(c.dtype).min
        c[n // 3: n // 2] = torch.iinfo(c.dtype).max
    for first in (0, 1):
        k, v = keys[first:], [c[first:] for c in cols]
        for predicted in (601, 150):
            plan = forced(k, eg.GB_HASH)
            plan.predicted_groups = predicted
            check(k, v, eg.groupby(k, v, plan, capacity=601))


def test_groupby_hash_time_of_sorted_rows(gpu):
    """Sorted rows of 1,000 groups take no longer than shuffled ones (they took 1.3 times
    as long while every row was an atomic on its group's one word)."""
    keys, vals = synth.groupby_input(seed=1, n=1 << 25, groups=1000, n_vals=2, device=gpu)
    ordered = keys.sort().values
    plan = forced(keys, eg.GB_HASH)
    t, t_sorted = best_time(lambda: eg.groupby(keys, vals, plan), lambda: eg.groupby(ordered, vals, plan))
    assert t_sorted < t, (t_sorted, t)


def test_groupby_rule_follows_the_estimate(gpu):
    small, sv = synth.groupby_input(seed=1, n=2_000_000, groups=600, device=gpu)
    big, bv = synth.groupby_input(seed=2, n=2_000_000, groups=1_500_000, device=gpu)
    ps, pb = eg.groupby_plan(eg.stats(small)), eg.groupby_plan(eg.stats(big))
    assert ps.variant == eg.GB_HASH and pb.variant == eg.GB_PARTITION
    assert abs(ps.predicted_groups - 600) < 600 * 0.05
    check(small, sv, eg.groupby(small, sv, ps))
    check(big, bv, eg.groupby(big, bv, pb))


def test_groupby_spill_and_small_table_retry(gpu):
    keys, vals = synth.groupby_input(seed=3, n=400_000, groups=300_000, device=gpu)
    # two partitions of ~150,000 groups each: far beyond one LDS table, so every
    # partition spills into the global table
    check(keys, vals, eg.groupby(keys, vals, forced(keys, eg.GB_PARTITION, 1)))
    # a table far smaller than the groups: the library refuses, the wrapper retries larger
    p = forced(keys, eg.GB_HASH)
    p.slots = 1024
    check(keys, vals, eg.groupby(keys, vals, p))


def test_groupby_edges(gpu):
    e = torch.zeros(0, dtype=torch.int32, device=gpu)
    for v, b in ((eg.GB_HASH, 0), (eg.GB_PARTITION, 4)):
        r = eg.groupby(e, [e], forced(e, v, b))
        assert r.groups == 0
    same = torch.full((100_000,), -5, dtype=torch.int32, device=gpu)
    vals = [torch.arange(100_000, dtype=torch.int64, device=gpu)]
    for v, b in ((eg.GB_HASH, 0), (eg.GB_PARTITION, 6)):
        check(same, vals, eg.groupby(same, vals, forced(same, v, b)))
        check(same, [], eg.groupby(same, [], forced(same, v, b)))
    # int64 keys including INT64_MIN: the plan marks empty slots with INT64_MAX
    k = torch.tensor([-(2**63), 5, -(2**63), 7, 5], dtype=torch.int64, device=gpu)
    p = forced(k, eg.GB_HASH)
    assert p.sentinel == 2**63 - 1
    check(k, [k], eg.groupby(k, [k], p))
    both = torch.tensor([-(2**63), 2**63 - 1, 0], dtype=torch.int64, device=gpu)
    with pytest.raises(eg.EigerError) as err:
        eg.groupby(both, [], forced(both, eg.GB_HASH))
    assert err.value.code == eg.EIGER_ERR_UNSUPPORTED


# PARTITION over every lane count (0-4 value words: none, int32, two int32,
# int64 + int32, two int64) and one to three partitioning passes (digits of at
# most 8 bits, narrower for wide rows: 7 bits for 12-byte rows, 6 for 24-byte).
LANES = [("none", torch.int32, []), ("i32", torch.int32, [torch.int32]),
         ("2xi32", torch.int32, [torch.int32, torch.int32]), ("i64+i32", torch.int64, [torch.int64, torch.int32]),
         ("2xi64", torch.int64, [torch.int64, torch.int64])]


@pytest.mark.parametrize("lanes", LANES, ids=[x[0] for x in LANES])
@pytest.mark.parametrize("bits", [3, 9, 15, 18])
def test_groupby_partition_lanes_and_passes(gpu, lanes, bits):
    _, key_dtype, val_dtypes = lanes
    keys, vals = synth.groupby_input(seed=bits, n=1_500_007, groups=400_000, key_dtype=key_dtype, n_vals=2,
                                     val_dtype=torch.int64, device=gpu)
    vals = [v.to(d) for v, d in zip(vals, val_dtypes)]
    check(keys, vals, eg.groupby(keys, vals, forced(keys, eg.GB_PARTITION, bits)))


# 4-byte keys from 512 tiles of 10,240 rows on: 9 and 10 partition bits go in one
# pass of 10-bit digits; 8 and 11 bits and one row fewer take the 8-bit passes
@pytest.mark.parametrize("lanes", LANES[:3], ids=[x[0] for x in LANES[:3]])
@pytest.mark.parametrize("bits,n", [(8, 5_242_880), (9, 5_242_879), (9, 5_242_880), (10, 5_253_121), (11, 5_242_880)])
def test_groupby_partition_wide_digit(gpu, lanes, bits, n):
    _, key_dtype, val_dtypes = lanes
    keys, vals = synth.groupby_input(seed=bits, n=n, groups=300_000, key_dtype=key_dtype, n_vals=2,
                                     val_dtype=torch.int64, device=gpu)
    keys[: n // 2] = keys[0]  # one digit fills whole tiles
    vals = [v.to(d) for v, d in zip(vals, val_dtypes)]
    check(keys, vals, eg.groupby(keys, vals, forced(keys, eg.GB_PARTITION, bits)))


@pytest.mark.parametrize("key_dtype", [torch.int32, torch.int64])
def test_groupby_row_group_and_per_row_loads(gpu, key_dtype):
    # aligned columns are read four rows at a time, views one row in per row;
    # partitions start anywhere, so the four-row groups also mask rows before
    # a partition's start (odd lengths give ragged ends)
    keys, vals = synth.groupby_input(seed=9, n=300_001, groups=5000, key_dtype=key_dtype, n_vals=2,
                                     val_dtype=torch.int64, device=gpu)
    vals = [vals[0], vals[1].to(torch.int32)]
    for view in (0, 1):
        k, v = keys[view:], [x[view:] for x in vals]
        for variant, bits in ((eg.GB_HASH, 0), (eg.GB_PARTITION, 3), (eg.GB_PARTITION, 9)):
            check(k, v, eg.groupby(k, v, forced(k, variant, bits)))
