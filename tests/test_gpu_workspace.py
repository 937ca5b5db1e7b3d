"""Calls in a workspace of exactly the size that was asked for, with guard bytes
behind it: results against the oracle, the guard untouched."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2607_04489_amd as eg
import synth
from joincheck import assert_exact, forced_plan

pytestmark = pytest.mark.gpu

GUARD = 1 << 20  # more than the count tables of any two tile sizes differ by


def guarded(size, device):
    buf = torch.full((size + GUARD,), 0xA5, dtype=torch.uint8, device=device)
    return buf[:size], buf[size:]


def groupby_size(plan, keys, vals):
    cols = (eg.Column * 2)(*[eg.column(v) for v in vals])
    size = ctypes.c_size_t()
    assert eg.lib().eiger_groupby_workspace_size(ctypes.byref(plan), eg.column(keys), cols, len(vals), ctypes.byref(size)) == 0
    return size.value


# Sides on either side of the row count from which the radix sort takes its large
# tiles (5,242,880 4-byte codes, 3,145,728 8-byte ones): the smaller side's sort needs
# the larger temporaries.
@pytest.mark.parametrize("key,bpay,n_build,n_probe", [
    (torch.int32, torch.int32, 5_242_879, 5_242_880), (torch.int32, torch.int32, 5_250_000, 5_200_000),
    (torch.int64, torch.int32, 3_145_727, 3_145_728), (torch.int64, torch.int64, 3_145_728, 3_145_727)])
def test_sort_merge_stays_in_its_workspace(gpu, key, bpay, n_build, n_probe):
    print(f"[workspace] sort-merge {n_build} x {n_probe} {key} {bpay}", flush=True)
    wide = key == torch.int64
    inp = synth.random_small(21, n_build, n_probe, -(1 << 40) if wide else 0, -(1 << 40) + 8_000_000 if wide else 8_000_000,
                             dtype=key, payload_dtype=torch.int32, device=gpu)
    if wide:  # codes of more than 32 bits: one build key far from the others
        inp.build_keys[7] = 1 << 41
    inp.build_payload = inp.build_payload.to(bpay)
    plan = forced_plan(inp, ("sort_merge", eg.SORT_MERGE, 0, 0, 0.0))
    args = (inp.build_keys, inp.build_payload, inp.probe_keys, inp.probe_payload)
    ws, guard = guarded(eg.join_workspace_size(plan, *args), gpu)
    res = eg.join(*args, plan, workspace=ws)
    assert bool((guard == 0xA5).all())
    assert_exact(inp, res)


@pytest.mark.parametrize("n", [8_000_000, 5_242_880, 5_242_879])
def test_groupby_in_a_workspace_sized_for_more_rows(gpu, n):
    """One pass of 10-bit digits for the larger inputs, two of 8-bit ones for the last,
    all in the workspace of the largest."""
    print(f"[workspace] group-by {n}", flush=True)
    keys, vals = synth.groupby_input(seed=5, n=8_000_000, groups=200_000, n_vals=2, device=gpu)
    plan = eg.groupby_plan(eg.stats(keys), eg.SEL_FORCED, eg.make_groupby_plan(eg.GB_PARTITION, 9))
    ws, guard = guarded(groupby_size(plan, keys, vals), gpu)
    keys, vals = keys[:n], [v[:n] for v in vals]
    assert groupby_size(plan, keys, vals) <= ws.numel()
    res = eg.groupby(keys, vals, plan, workspace=ws)
    assert bool((guard == 0xA5).all())
    gk, cnt, sums = oracle.group_by(keys, vals)
    order = torch.argsort(res.keys).cpu().numpy()
    for got, want in zip([res.keys, res.counts, *res.sums], [gk, cnt, *sums]):
        assert np.array_equal(got.cpu().numpy()[order], want)
