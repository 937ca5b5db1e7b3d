"""eiger_join on the GPU against the join oracle, for every variant and a spread
of knobs: canonical pair lists, counts and checksums must be identical."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_04489_amd as eg
import synth
from joincheck import SPECS, SPEC_IDS, assert_exact, forced_plan

pytestmark = pytest.mark.gpu


def run(inp, spec, **kw):
    plan = forced_plan(inp, spec)
    return eg.join(inp.build_keys, inp.build_payload, inp.probe_keys, inp.probe_payload, plan, **kw)


@pytest.mark.parametrize("spec", SPECS, ids=SPEC_IDS)
def test_plain_dense_small(gpu, spec):
    inp = synth.plain_dense(seed=3, n_build=4096, n_probe=100003, probe_range=5000, device=gpu)
    assert_exact(inp, run(inp, spec))


@pytest.mark.parametrize("spec", SPECS, ids=SPEC_IDS)
def test_plain_dense_full(gpu, spec):
    """The 65,536 x 1,048,576 plain join at full size, every variant."""
    inp = synth.plain_dense(seed=42, device=gpu)
    assert_exact(inp, run(inp, spec))


@pytest.mark.parametrize("spec", [s for s in SPECS if s[1] != eg.DIRECT], ids=[s[0] for s in SPECS if s[1] != eg.DIRECT])
def test_sparse_unique64(gpu, spec):
    inp = synth.sparse_unique64(seed=4, n_build=100000, n_probe=1000003, device=gpu)
    assert_exact(inp, run(inp, spec))


@pytest.mark.parametrize("key,bpay,ppay", [(torch.int32, torch.int32, torch.int32), (torch.int32, torch.int64, torch.int64),
                                           (torch.int64, torch.int32, torch.int32), (torch.int64, torch.int32, torch.int64)])
@pytest.mark.parametrize("order", ["sorted", "one key"])
def test_hash_probes_that_stay_near(gpu, order, key, bpay, ppay):
    """Probes in key order and probes of one key, all matching: every block fills a wave's
    stage by the same amount, in workgroups of each shape, one row short of and beyond
    their shares."""
    g = torch.Generator().manual_seed(9)
    keys = torch.randperm(400_000, generator=g) * 4999 - 77
    for n_probe in (7 * 256 * 3 - 1, 8 * 256 * 5 + 1, 3_000_001):
        hit = torch.randint(0, 400_000, (n_probe,), generator=g).sort().values if order == "sorted" else torch.full((n_probe,), 5)
        inp = synth.JoinInput("near", keys.to(key).to(gpu), torch.randint(-999, 999, (400_000,), generator=g).to(bpay).to(gpu),
                              (hit * 4999 - 77).to(key).to(gpu), torch.randint(-999, 999, (n_probe,), generator=g).to(ppay).to(gpu))
        res = run(inp, ("hash", eg.GLOBAL_HASH, 0, 0, 0.5))
        assert_exact(inp, res)
        cnt = run(inp, ("hash", eg.GLOBAL_HASH, 0, 0, 0.5), count_only=True)
        assert (cnt.count, cnt.checksum) == (res.count, res.checksum)


def test_hash_sorted_probes_of_wide_payloads_time(gpu):
    """Sorted probes, pairs: 8-byte payloads take no more over 4-byte ones than their
    share of the bytes, 20 to 16 a row (1.5 times while fewer waves staged fewer pairs)."""
    g = torch.Generator(device=gpu).manual_seed(1)
    n = 1 << 23
    bk = (torch.randperm(60_000, generator=g, device=gpu) * 4999 - 77).int()
    pk = bk[torch.randint(0, 60_000, (n,), generator=g, device=gpu)].sort().values
    pays, outs = [torch.ones(n, dtype=t, device=gpu) for t in (torch.int32, torch.int64)], [torch.empty_like(pk) for _ in range(2)]
    plan = eg.join_plan(eg.stats(bk), eg.stats(pk), eg.SEL_FORCED, eg.make_plan(eg.GLOBAL_HASH, 0, 0, 0.5))
    ws = torch.empty(eg.join_workspace_size(plan, bk, bk, pk, pays[1]), dtype=torch.uint8, device=gpu)

    def call(pp):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        assert eg.join(bk, bk, pk, pp, plan, workspace=ws, outputs=outs).count == n
        stop.record()
        stop.synchronize()
        return start.elapsed_time(stop)

    t = [[call(pp) for pp in pays] for _ in range(15)]
    narrow, wide = (min(x) for x in zip(*t))
    assert wide < 1.25 * narrow, (wide, narrow)


def test_hash_build_of_repeated_keys_time(gpu):
    """563,000 build rows: repeated keys take less than two and a half times as long as
    distinct ones (the walks over their copies; 3.5 while every wave raised the flag)."""
    g = torch.Generator(device=gpu).manual_seed(1)
    n = 562_928
    rep = torch.randint(0, n, (n,), generator=g, device=gpu).int() * 3
    pk, one = rep[:255], torch.ones(n, dtype=torch.int32, device=gpu)

    def build(keys):
        plan = eg.join_plan(eg.stats(keys), eg.stats(pk), eg.SEL_FORCED, eg.make_plan(eg.GLOBAL_HASH, 0, 0, 0.5))
        best = []
        for _ in range(11):
            eg.profile_enable(True)
            try:
                eg.join(keys, one, pk, one[:255], plan, count_only=True)
                torch.cuda.synchronize()
                best.append(eg.profile_read()["hash_build"][1])
            finally:
                eg.profile_enable(False)
        return min(best)

    assert build(rep) < 2.5 * build(torch.arange(n, device=gpu).int() * 3)


@pytest.mark.parametrize("key,pay", [(torch.int32, torch.int32), (torch.int32, torch.int64), (torch.int64, torch.int64)])
@pytest.mark.parametrize("repeats", [1, 40])
def test_hash_probe_of_small_sides(gpu, repeats, key, pay):
    """Probe sides around a wave's rows, a workgroup's and the sizes at which a wave takes
    twice as many, whole and half matching, of distinct and of repeated keys."""
    g = torch.Generator().manual_seed(2)
    keys = (torch.arange(120) * 7919 - 5000).repeat(repeats)
    waves = 2 * 256 * (8 if key == pay == torch.int32 else 7)
    for n_probe in (1, 63, 65, 448, 513, 64 * waves, 64 * waves + 1, 128 * waves + 1):
        if repeats > 1 and n_probe > 1000:
            continue
        inp = synth.JoinInput("small", keys.to(key).to(gpu), torch.randint(-999, 999, keys.shape, generator=g).to(pay).to(gpu),
                              (torch.randint(0, 240, (n_probe,), generator=g) * 7919 - 5000).to(key).to(gpu),
                              torch.randint(-999, 999, (n_probe,), generator=g).to(pay).to(gpu))
        res = run(inp, ("hash", eg.GLOBAL_HASH, 0, 0, 0.5))
        assert_exact(inp, res)
        cnt = run(inp, ("hash", eg.GLOBAL_HASH, 0, 0, 0.5), count_only=True)
        assert (cnt.count, cnt.checksum) == (res.count, res.checksum)


def test_hash_probe_of_few_rows_time(gpu):
    """256 probe rows of 64 matches each, pairs: less than half as long again as 64 of them,
    since other waves take the rest (2.5 times as long while one wave took them all)."""
    bk = torch.full((64,), 7, device=gpu)
    pk, one = bk.repeat(4), torch.ones(256, dtype=torch.int64, device=gpu)
    plan = eg.join_plan(eg.stats(bk), eg.stats(pk), eg.SEL_FORCED, eg.make_plan(eg.GLOBAL_HASH, 0, 0, 0.5))
    outs = [torch.empty(64 * 256, dtype=torch.int32, device=gpu) for _ in range(2)]

    def probe(n):
        best = []
        for _ in range(11):
            eg.profile_enable(True)
            try:
                assert eg.join(bk, one[:64], pk[:n], one[:n], plan, outputs=outs).count == 64 * n
                torch.cuda.synchronize()
                best.append(eg.profile_read()["hash_probe"][1])
            finally:
                eg.profile_enable(False)
        return min(best)

    assert probe(256) < 1.5 * probe(64)


@pytest.mark.parametrize("key,pay", [(torch.int32, torch.int32), (torch.int64, torch.int32), (torch.int64, torch.int64)])
@pytest.mark.parametrize("lf", [0.25, 0.9])
def test_hash_duplicate_check_finds_one_pair(gpu, lf, key, pay):
    """Keys at both ends of the domain, so that the build does not see duplicates itself:
    one key twice among distinct ones, first and last row or next to each other."""
    info = torch.iinfo(key)
    for n in (3, 30, 1021, 7373, 29491):
        keys = torch.arange(n) * 40009 - 3
        keys[0], keys[1] = info.min, info.max
        for a, b in ((0, n - 1), (n // 2, n // 2 + 1), (2, 2)):
            bk = keys.clone()
            bk[b] = bk[a]
            inp = synth.JoinInput("pair", bk.to(key).to(gpu), torch.arange(n).to(pay).to(gpu),
                                  bk[torch.arange(0, n, 7)].repeat(2).to(key).to(gpu), torch.arange(len(range(0, n, 7)) * 2).to(pay).to(gpu))
            assert_exact(inp, run(inp, ("hash", eg.GLOBAL_HASH, 0, 0, lf)))


def test_hash_duplicate_check_time(gpu):
    """30,000 rows, a tenth of them each of three keys at and between the ends of the
    domain: looking for duplicates takes a tenth of the build at most (0.22 of it while
    every row walked to its cluster's end)."""
    g = torch.Generator(device=gpu).manual_seed(1)
    info, n = torch.iinfo(torch.int64), 30_000
    m = torch.rand(n, generator=g, device=gpu)
    bk = torch.randint(0, n, (n,), generator=g, device=gpu)
    for k, at in enumerate((info.min, info.max, -1)):
        bk = torch.where((m >= k / 10) & (m < (k + 1) / 10), torch.full_like(bk, at), bk)
    plan = eg.join_plan(eg.stats(bk), eg.stats(bk[:9]), eg.SEL_FORCED, eg.make_plan(eg.GLOBAL_HASH, 0, 0, 0.5))
    t = []
    for _ in range(5):
        eg.profile_enable(True)
        try:
            eg.join(bk, bk.int(), bk[:9], bk[:9].int(), plan, count_only=True)
            torch.cuda.synchronize()
            prof = eg.profile_read()
            t.append((prof["hash_unique"][1], prof["hash_build"][1]))
        finally:
            eg.profile_enable(False)
    unique, build = (min(x) for x in zip(*t))
    assert unique < 0.1 * build, (unique, build)


# Build rows of which one more doubles the table at load factor 0.5. 16-byte slots: 2 to
# 16 MiB, from 16 on the probe loads two slots of a row at first; 32-byte slots: 4 to 32
# MiB, pairs of distinct keys by the rows' own probe, the others from 16 on two slots.
@pytest.mark.parametrize("n_build", [65535, 65536, 131071, 131072, 262143, 262144])
@pytest.mark.parametrize("key,pay", [(torch.int32, torch.int32), (torch.int32, torch.int64), (torch.int64, torch.int64)])
@pytest.mark.parametrize("shape", ["distinct", "repeated"])
def test_hash_probe_paths(gpu, n_build, key, pay, shape):
    """Distinct keys (one match per row) and repeated ones (keys of 3 rows, and two of
    300, so that a block of rows overflows a wave's stage), probe rows one short of and
    beyond whole blocks, pairs and count-only."""
    g = torch.Generator().manual_seed(n_build)
    for n_probe in (3 * 4096 - 1, 70001):
        i = torch.arange(n_build)
        keys = (i if shape == "distinct" else torch.where(i < 600, i % 2, i // 3)) * 7919 - 5000
        keys = keys[torch.randperm(n_build, generator=g)]
        pk = torch.randint(0, n_build + n_build // 4, (n_probe,), generator=g) * 7919 - 5000
        if shape == "repeated":
            pk[1000:1700] = -5000  # 700 rows of 300 matches each, together
        inp = synth.JoinInput("hash_paths", keys.to(key).to(gpu), torch.randint(-999, 999, (n_build,), generator=g).to(pay).to(gpu),
                              pk.to(key).to(gpu), torch.randint(-999, 999, (n_probe,), generator=g).to(pay).to(gpu))
        res = run(inp, ("hash", eg.GLOBAL_HASH, 0, 0, 0.5))
        assert_exact(inp, res)
        cnt = run(inp, ("hash", eg.GLOBAL_HASH, 0, 0, 0.5), count_only=True)
        assert (cnt.count, cnt.checksum) == (res.count, res.checksum)


@pytest.mark.parametrize("repeats", [1, 2])
def test_hash_probe_of_a_far_table(gpu, repeats):
    """A 4 GiB table of 32-byte slots: counted by the rows' probe, pairs by it (distinct
    keys) or by the waves (repeated ones). Count and checksum in closed form."""
    print(f"[far] {repeats}", flush=True)
    n, n_probe = (1 << 26) + 2, (1 << 20) + 77
    nd = n // repeats
    keys = torch.arange(nd, device=gpu).repeat(repeats) * 0x9E3779B97F4A7C1 - (1 << 60)
    bp = (torch.arange(nd, device=gpu) % 1009 - 500).repeat(repeats)
    hit = torch.randint(0, nd + nd // 4, (n_probe,), generator=torch.Generator().manual_seed(3)).to(gpu)
    pk, pp = hit * 0x9E3779B97F4A7C1 - (1 << 60), torch.arange(n_probe, device=gpu) % 777 - 300
    found = hit < nd
    want = (int(found.sum()) * repeats, int((pp * (hit % 1009 - 500))[found].sum()) * repeats)
    plan = eg.join_plan(eg.stats(keys), eg.stats(pk), eg.SEL_FORCED, eg.make_plan(eg.GLOBAL_HASH, 0, 0, 0.5))
    cnt = eg.join(keys, bp, pk, pp, plan, count_only=True)
    assert (cnt.count, cnt.checksum) == want
    res = eg.join(keys, bp, pk, pp, plan)
    assert (res.count, res.checksum) == want
    b, p = res.build_rowid.long(), res.probe_rowid.long()
    assert torch.equal(keys[b], pk[p])
    assert torch.unique((b << 32) | p).numel() == want[0]


def test_hash_pairs_of_repeated_keys_time(gpu):
    """1,000 keys of 16 rows: writing the pairs out takes no more than as long again as
    counting them (2.4 times as long while waves reserved output one by one)."""
    g = torch.Generator(device=gpu).manual_seed(1)
    keys = torch.arange(1000, device=gpu) * 1103515245 & ((1 << 31) - 1)
    bk = keys.repeat_interleave(16)[torch.randperm(16000, generator=g, device=gpu)].int()
    pk = keys[torch.randint(0, 1000, (1 << 20,), generator=g, device=gpu)].int()
    one, outs = torch.ones_like(pk), [torch.empty(1 << 24, dtype=torch.int32, device=gpu) for _ in range(2)]
    plan = eg.join_plan(eg.stats(bk), eg.stats(pk), eg.SEL_FORCED, eg.make_plan(eg.GLOBAL_HASH, 0, 0, 0.5))
    ws = torch.empty(eg.join_workspace_size(plan, bk, bk, pk, one), dtype=torch.uint8, device=gpu)

    def call(**kw):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        assert eg.join(bk, bk, pk, one, plan, workspace=ws, **kw).count == 1 << 24
        stop.record()
        stop.synchronize()
        return start.elapsed_time(stop)

    t = [(call(outputs=outs), call(count_only=True)) for _ in range(11)]
    pairs, count = (min(x) for x in zip(*t))
    assert pairs < 2 * count, (pairs, count)


def test_direct_refuses_sparse_range(gpu):
    inp = synth.sparse_unique64(seed=4, n_build=1000, n_probe=1000, device=gpu)
    with pytest.raises(eg.EigerError) as e:
        run(inp, SPECS[0])
    assert e.value.code == eg.EIGER_ERR_UNSUPPORTED


@pytest.mark.parametrize("s", [0.5, 1.0, 1.5])
@pytest.mark.parametrize("spec", [s for s in SPECS if s[1] != eg.DIRECT], ids=[s[0] for s in SPECS if s[1] != eg.DIRECT])
def test_skewed_dup32(gpu, spec, s):
    inp = synth.skewed_dup32(seed=5, n_distinct=20000, n_probe=300001, zipf_s=s, device=gpu)
    assert_exact(inp, run(inp, spec))


def test_skewed_dense_direct(gpu):
    """Duplicated build keys in a dense range: DIRECT's CSR runs."""
    inp = synth.random_small(11, 50000, 400000, -20000, 20000, device=gpu)
    assert_exact(inp, run(inp, SPECS[0]))


ADVERSARIAL = {
    "all_equal": lambda d: synth.JoinInput("all_equal", torch.full((1500,), 7, dtype=torch.int32, device=d),
                                           torch.arange(1500, dtype=torch.int32, device=d),
                                           torch.full((3000,), 7, dtype=torch.int32, device=d),
                                           torch.arange(3000, dtype=torch.int32, device=d) - 1500),
    "empty_build": lambda d: synth.random_small(1, 0, 1000, 0, 100, device=d),
    "empty_probe": lambda d: synth.random_small(1, 1000, 0, 0, 100, device=d),
    "one_build_row": lambda d: synth.random_small(2, 1, 5000, 0, 3, device=d),
    "narrow_dups": lambda d: synth.random_small(3, 3000, 20000, -5, 5, device=d),
    "int32_full_range": lambda d: synth.random_small(4, 20000, 50000, -(1 << 31), (1 << 31) - 1, device=d),
    "int64_full_range": lambda d: synth.random_small(5, 20000, 50000, -(1 << 63), (1 << 63) - 1,
                                                     dtype=torch.int64, payload_dtype=torch.int64, device=d),
    "mixed_payloads": lambda d: synth.random_small(6, 7000, 30000, 0, 9000, dtype=torch.int32,
                                                   payload_dtype=torch.int64, device=d),
}


def with_extremes(inp, dtype):
    info = torch.iinfo(dtype)
    ext = torch.tensor([info.min, info.max, info.min, 0, -1], dtype=dtype, device=inp.build_keys.device)
    return synth.JoinInput(inp.name + "+ext", torch.cat([inp.build_keys, ext]),
                           torch.cat([inp.build_payload, inp.build_payload[:5]]),
                           torch.cat([ext, inp.probe_keys, ext]),
                           torch.cat([inp.probe_payload[:5], inp.probe_payload, inp.probe_payload[:5]]))


@pytest.mark.parametrize("case", list(ADVERSARIAL))
@pytest.mark.parametrize("spec", SPECS, ids=SPEC_IDS)
def test_adversarial(gpu, case, spec):
    inp = ADVERSARIAL[case](gpu)
    if case.endswith("full_range"):
        inp = with_extremes(inp, inp.build_keys.dtype)
    if spec[1] == eg.DIRECT:
        st = eg.stats(inp.build_keys)
        if st.n and st.max - st.min + 1 > (1 << 30):
            pytest.skip("DIRECT needs a dense key range")
    assert_exact(inp, run(inp, spec))


@pytest.mark.parametrize("spec", SPECS, ids=SPEC_IDS)
def test_payload_dtype_mix(gpu, spec):
    inp = synth.random_small(8, 5000, 40000, 0, 7000, dtype=torch.int64, payload_dtype=torch.int32, device=gpu)
    inp.probe_payload = synth.rand64(8, 99, torch.arange(inp.n_probe, device=gpu))
    assert_exact(inp, run(inp, spec))


def test_misaligned_probe_view(gpu):
    inp = synth.random_small(9, 5000, 40001, 0, 6000, device=gpu)
    inp.probe_keys = inp.probe_keys[1:]
    inp.probe_payload = inp.probe_payload[1:]
    for spec in SPECS:
        assert_exact(inp, run(inp, spec))


@pytest.mark.parametrize("spec", SPECS, ids=SPEC_IDS)
def test_capacity_and_count_only(gpu, spec):
    inp = synth.random_small(10, 3000, 30000, 0, 2000, device=gpu)
    _, cnt, cs = oracle.join_sortmerge(inp.build_keys, inp.build_payload, inp.probe_keys,
                                       inp.probe_payload, with_pairs=False)
    plan = forced_plan(inp, spec)
    r = eg.join(inp.build_keys, inp.build_payload, inp.probe_keys, inp.probe_payload, plan, count_only=True)
    assert (r.count, r.checksum) == (cnt, cs)
    small = (torch.empty(cnt // 2, dtype=torch.int32, device=gpu), torch.empty(cnt // 2, dtype=torch.int32, device=gpu))
    with pytest.raises(eg.EigerError) as e:
        eg.join(inp.build_keys, inp.build_payload, inp.probe_keys, inp.probe_payload, plan, outputs=small)
    assert e.value.code == eg.EIGER_ERR_CAPACITY and e.value.count == cnt
    # the binding's retry path: a too-small capacity grows to the exact count
    r = eg.join(inp.build_keys, inp.build_payload, inp.probe_keys, inp.probe_payload, plan, capacity=10)
    assert_exact(inp, r)


def test_rule_plan_end_to_end(gpu):
    for inp in (synth.plain_dense(seed=1, device=gpu),
                synth.sparse_unique64(seed=2, n_build=300000, n_probe=2000000, device=gpu),
                synth.skewed_dup32(seed=3, n_distinct=30000, n_probe=400000, zipf_s=1.0, device=gpu)):
        plan = eg.join_plan(eg.stats(inp.build_keys), eg.stats(inp.probe_keys))
        assert_exact(inp, eg.join(inp.build_keys, inp.build_payload, inp.probe_keys, inp.probe_payload, plan))


def test_repeatable(gpu):
    inp = synth.skewed_dup32(seed=6, n_distinct=20000, n_probe=200000, zipf_s=1.5, device=gpu)
    for spec in SPECS[1:]:
        a, b = run(inp, spec), run(inp, spec)
        assert (a.count, a.checksum) == (b.count, b.checksum)
        from joincheck import gpu_canonical
        assert np.array_equal(gpu_canonical(a), gpu_canonical(b))
