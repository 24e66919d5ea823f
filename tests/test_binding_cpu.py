"""The binding's short way through a call (one loop over the tensors) agrees with
its full checks: the sizes it reads from a descriptor, and that anything but
device tensors of the right size and type goes the long way, which raises."""
import pytest
import torch

import paper_2204_01701_amd as ql

DESCS = [ql.conv_desc(2, 16, 9, 8, 24, 3, 3, (2, 1), 1), ql.conv_desc(1, 3, 5, 5, 7, 1, 5, 3, (0, 2), ql.QL_F32),
         ql.conv_desc(2, 12, 7, 7, 12, 3, 3, 1, 1, ql.QL_F32, groups=12), ql.conv_desc(4, 1, 6, 6, 1, 3, 3, groups=1)]


@pytest.mark.parametrize("d", DESCS, ids=range(len(DESCS)))
def test_conv_sizes_agree(d):
    assert ql._conv_plan(d) == (*ql._conv_sizes(d), d.dtype)


def test_linear_sizes_agree():
    d = ql.linear_desc(5, 7, 9, ql.QL_F32)
    assert ql._linear_plan(d) == (*ql._linear_sizes(d), d.dtype)


def test_unusual_tensors_take_the_long_way():
    plan = ql._linear_plan(ql.linear_desc(4, 8, 8, ql.QL_F32))
    good = torch.empty(4, 8)
    for t in (good, 4096, good.double(), torch.empty(4, 9)):
        assert ql._pointers(plan, "x", (t,)) is None
    assert ql._pointers((*plan[:4], 7), "x", (good,)) is None      # unknown dtype code
    assert ql._pointers(None, "x", (good,)) is None                # a stride below 1
    assert ql._pointers(plan, "xb", (None, None)) is None          # no tensor: no device
    with pytest.raises(ValueError, match="CUDA device tensor"):
        ql.qlayer_linear_fwd(ql.linear_desc(4, 8, 8, ql.QL_F32), good, torch.empty(8, 8), None, None, y=torch.empty(4, 8))
