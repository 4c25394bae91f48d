"""Which kernel the library launches for a plan (on the CPU, behind a stand-in for the HIP runtime)."""
import numpy as np
import pytest

from kernel_choice import case, launches, reduction_status
from workloads import Forest, HeadConfig, build_paged_kv, DTYPE_BF16, DTYPE_FP16


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
    one after the other; four or eight waves per list.  Large: more than 16383 waves."""
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
    for n, waves in ((20, 1), (30, 4), (50, 8)):
        most = 16383 // (per_request * waves)
        for b, form in ((most, waves), (most + 1, 2)):
            many.append(_case(Forest(np.array([-1]), np.array([32 * n]), np.zeros(b, np.int64)), head, split_align=32,
                              fixed_slices=n, num_slots=4))
            want.append(("merge_split_kernel" if form >= 4 else "merge_kernel", (DTYPE_FP16, d, wide, form)))
    assert [got["reduction"][0][:2] for got in launches(many)] == want
