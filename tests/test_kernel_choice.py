"""Which kernel the library launches for a plan (on the CPU, behind a stand-in for the HIP runtime)."""
import numpy as np
import pytest

from helpers import GOING_ROUND, GOING_ROUND_OPTS, ROTATING, ROTATING_OPTS, going_round_forest, rotating_forest
from kernel_choice import case, launches, reduction_status
from plan_image import plan_image
from workloads import (Forest, HeadConfig, build_paged_kv, concat_forests, draft_masked_forest, two_level_forest, unshared_forest,
                       DTYPE_BF16, DTYPE_FP16)


def _case(f, head, layout="htd", **opts):
    return case(f, build_paged_kv(f, head, 1, layout=layout), head, **opts)


def test_reduction_forms_that_do_not_exist_are_refused():
    """A number of waves without a kernel is an error, not a reduction that never runs."""
    forms = [(d, w) for d in (64, 128, 256) for w in (-1, 3, 5, 7, 9, 16)] + [(96, 0), (96, 4)]
    assert all(status != 0 and not seen for status, seen in reduction_status(forms))
    for (d, w), (status, seen) in zip(good := [(d, w) for d in (64, 128, 256) for w in (0, 1, 2, 4, 8)],
                                      reduction_status(good)):
        kernel, args, dims = seen[0]
        assert status == 0 and len(seen) == 1 and args == (DTYPE_BF16, d, 1, w) and dims[:3] == (4, 1, 1)
        assert (kernel, dims[3]) == (("merge_kernel", 128) if w < 4 else ("merge_split_kernel", 64 * w))


@pytest.mark.parametrize("d,hq,hkv,wide", [(128, 32, 8, 2), (128, 7, 1, 1), (64, 16, 2, 4), (64, 6, 3, 1), (256, 10, 2, 1)])
def test_reduction_form_by_the_longest_list_and_the_launch(d, hq, hkv, wide):
    """One wave per list without the code behind fifteen rows, with rows sixteen to 23 beside them, or, in large launches,
    one after the other (more than 16383 waves); four or eight waves per list in launches of up to 6143 and 8191."""
    head = HeadConfig(hq, hkv, d, DTYPE_FP16)
    lists = [1, 2, 15, 16, 23, 24, 39, 40, 71, 72, 300]
    few = [_case(Forest(np.array([-1]), np.array([32 * n]), np.zeros(2, np.int64)), head, split_align=32, fixed_slices=n,
                 num_slots=4) for n in lists]
    for n, got in zip(lists, launches(few)):
        assert got["longest"] == n
        want = ("merge_kernel", 0) if n <= 15 else ("merge_kernel", 1) if n <= 23 else ("merge_split_kernel", 4 if n <= 39 else 8)
        (kernel, args, _), = got["reduction"]
        assert (kernel, args) == (want[0], (DTYPE_FP16, d, wide, want[1])), n
        assert got["decode"][1:] == (got["reduction"] if n > 1 else [])
    per_request = hq // wide
    many, want = [], []
    for n, waves, line, beyond in ((20, 1, 16383, 2), (30, 4, 6143, 1), (50, 8, 8191, 1), (30, 1, 16383, 2), (50, 1, 16383, 2)):
        most = line // (per_request * waves)
        for b, form in ((most, waves), (most + 1, beyond)):
            many.append(_case(Forest(np.array([-1]), np.array([32 * n]), np.zeros(b, np.int64)), head, split_align=32,
                              fixed_slices=n, num_slots=4))
            want.append(("merge_split_kernel" if form >= 4 else "merge_kernel", (DTYPE_FP16, d, wide, form)))
    assert [got["reduction"][0][:2] for got in launches(many)] == want


@pytest.mark.parametrize("opts", ROTATING_OPTS)
def test_rotating_kernels(opts):
    """The plans of the GPU parity test of the same name run the kernels whose stream tasks go round the KV heads, and most
    of their tasks do (those that alone read their slice, in a plan that reads little twice).  Heads that lie apart
    ([head][token] pools), one launch and 256 channels stay with the others; so do one KV head and short plans (below)."""
    cases, want = [], []
    for d, hq, hkv, dtype, nodes, requests, below, form in ROTATING:
        f, head = rotating_forest(nodes, requests, below), HeadConfig(hq, hkv, d, dtype)
        im = plan_image(f, head, **opts)
        recs = im["queue_recs" if im["schedule"] == 1 else "slot_recs"]
        assert (recs["flags"] & 1).mean() > 0.5 and (len(im["packs"]) > 0) == (d == 64 and form == 1)
        assert (form == 1 and d == 128) == (int(recs["n_req"].max()) * (hq // hkv) > (16 if d == 128 else 512))
        for layout, extra, args in (("thd", {}, (dtype, form, d, 1, 0)), ("htd", {}, (dtype, form, d, 0, 0)),
                                    ("thd", {"fused": 1}, (dtype, form, d, 0, 1))):
            cases.append(_case(f, head, layout, **opts, **extra))
            want.append(args)
    wide = HeadConfig(16, 8, 256, DTYPE_BF16)
    cases.append(_case(rotating_forest(120, 1, 0), wide, "thd", **opts))
    want.append((DTYPE_BF16, 0, 256, 0, 0))
    for got, args in zip(launches(cases), want):
        assert got["tasks"] * 8 >= 768 and got["makespan"] >= 60000
        assert got["decode"][0][:2] == ("pac_kernel", args)
        two = args[:-1] + (0,)
        assert got["attention"][0][:2] == ("pac_kernel", two if not args[-1] else args[:3] + (1, 0))


@pytest.mark.parametrize("opts", GOING_ROUND_OPTS)
def test_stream_tasks_go_round_the_heads(opts):
    """The same for the plans of that GPU parity test."""
    cases = []
    for d, hq, hkv, leaves in GOING_ROUND:
        f, head = going_round_forest(leaves), HeadConfig(hq, hkv, d, DTYPE_BF16)
        im = plan_image(f, head, **opts)
        assert (im["queue_recs" if im["schedule"] == 1 else "slot_recs"]["flags"] & 1).mean() > 0.5
        cases.append(_case(f, head, "thd", **opts))
    forms = [got["decode"][0][:2] for got in launches(cases)]
    assert [(k, a[0], *a[2:]) for k, a in forms] == [("pac_kernel", DTYPE_BF16, d, 1, 0) for d, _, _, _ in GOING_ROUND]
    assert {a[1] for _, a in forms} == {1}


@pytest.mark.parametrize("d", [64, 128])
def test_plans_whose_tasks_do_not_go_round(d):
    """By the plan's estimated time, its tasks of all heads and its KV heads: 60 us, 768, more than one."""
    head = HeadConfig(32, 8, d)
    f = unshared_forest([700] * 96)
    cases = [_case(f, head, "thd", num_slots=4, fixed_slices=n) for n in (1, 2)]
    cases += [_case(unshared_forest([700] * n), head, "thd", num_slots=2, fixed_slices=2) for n in (47, 48)]
    cases += [_case(f, head, "thd", num_slots=64, fixed_slices=2),
              _case(unshared_forest([700] * 400), HeadConfig(4, 1, d), "thd", num_slots=1, fixed_slices=2)]
    seen = launches(cases)
    forms = [got["attention"][0][1] for got in seen]
    assert [(c["tasks"] * k, a[3]) for c, a, k in zip(seen, forms, (8, 8, 8, 8, 8, 1))] == [
        (768, 1), (1536, 1), (752, 0), (768, 1), (1536, 0), (800, 0)]
    assert [c["makespan"] >= 60000 for c in seen] == [True, True, True, True, False, True]
    # finished rows: a kernel of its own (its tasks go round in any case), and nothing to reduce
    assert [a[:2] for a in (seen[0]["decode"][0],)] == [("pac_kernel", (DTYPE_BF16, 2, d, 0, 0))] and len(seen[0]["decode"]) == 1


@pytest.mark.parametrize("d,hq,hkv", [(64, 32, 8), (128, 32, 8)])
def test_plans_with_little_that_goes_round(d, hq, hkv):
    """Long plans with many tasks of which none goes round the heads (they read their slices several times: drafted tokens,
    flat plans of shared prefixes), or that read less than a tenth of the tokens, stay with the kernels that have no such
    tasks; from a tenth on they do not."""
    head = HeadConfig(hq, hkv, d)
    drafted = draft_masked_forest(900, [1800 + 100 * i for i in range(16)], 48, seed=3)
    flat = two_level_forest(2000, [100] * 100)
    # shared slices of 33 .. 256 rows (dense tasks, packed row tiles) beside contexts of one request
    shared = Forest(np.full(40, -1), np.full(40, 1500), np.repeat(np.arange(40), 16 if d == 128 else 24))
    few, many = (concat_forests(shared, unshared_forest([n] * 80)) for n in (60, 100))
    plans = [(drafted, dict(num_slots=4), 0), (flat, dict(num_slots=4, share=0), 0), (few, dict(num_slots=2), 0),
             (many, dict(num_slots=2), 1)]
    for (f, opts, turns), got in zip(plans, launches([_case(f, head, "thd", **opts) for f, opts, _ in plans])):
        recs = plan_image(f, head, **opts)["slot_recs"]
        rotating = (recs["flags"] & 1 == 1) & (recs["flags"] & 4 == 0) & (recs["n_req"] * (hq // hkv) <= (16 if d == 128 else 32))
        share = recs["kv_len"][rotating].sum() / recs["kv_len"].sum()
        assert got["makespan"] >= 60000 and got["tasks"] * hkv >= 768
        assert got["decode"][0][1][3] == turns == int(share >= 0.1), (share, got["decode"])
        assert share == 0 if f is drafted or f is flat else 0.05 < share < 0.15
