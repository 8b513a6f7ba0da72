"""The binding's descriptors follow their fields: assignments, replaced copies, lists changed in
place; cached axes keep refusing what they refused."""
import copy
import dataclasses

import pytest

import paper_1810_08723_amd as ocn


def _plan_size(t):
    out = ocn.Tensor(1 << 41, "float", t.sizes, tuple(t.strides), 0, 0)
    return ocn.plan_unary("neg", t, out)["size"]


def test_assigned_fields_reach_the_next_call():
    t = ocn.Tensor(1 << 40, "float", (4, 8), (64, 4))
    assert _plan_size(t) == (4, 8) and t.desc().base == 1 << 40
    t.sizes, t.strides = (4, 6), (64, 4)
    assert _plan_size(t) == (4, 6)
    t.base, t.offset, t.dtype, t.device, t.byteswapped = 1 << 39, 16, "int32", 1, True
    d = t.desc()
    assert (d.base, d.offset, d.dtype, d.device, d.byteswapped) == (1 << 39, 16, 3, 1, 1)
    other = dataclasses.replace(t, offset=32)
    assert other.desc().offset == 32 and t.desc().offset == 16 and other != t
    twin = copy.copy(t)
    assert twin == t
    twin.offset = 64
    assert twin.desc().offset == 64 and t.desc().offset == 16


def test_lists_changed_in_place_are_seen():
    t = ocn.Tensor(1 << 40, "float", [4, 8], [64, 4])
    assert t.desc().size[1] == 8
    t.sizes[1] = 5
    t.strides[0] = 128
    assert t.desc().size[1] == 5 and t.desc().stride[0] == 128


def test_axes_of_another_type_stay_refused():
    a, out = ocn.Tensor(1 << 40, "float", (4, 8), (32, 4)), ocn.Tensor(1 << 41, "float", (4,), (4,))
    assert ocn.plan_reduce("sum", a, [1], out)["red_size"] == (8,)
    assert ocn.plan_reduce("sum", a, (1,), out)["red_size"] == (8,)
    with pytest.raises(TypeError):
        ocn.plan_reduce("sum", a, [1.0], out)
    with pytest.raises(ocn.OcnError):
        ocn.plan_reduce("sum", a, [2], out)


def test_axes_that_are_not_plain_ints_are_read_at_every_call():
    np, torch = pytest.importorskip("numpy"), pytest.importorskip("torch")
    a, out = ocn.Tensor(1 << 40, "float", (4, 8), (32, 4)), ocn.Tensor(1 << 41, "float", (4,), (4,))
    assert ocn.plan_reduce("sum", a, [np.array(1)], out)["red_size"] == (8,)      # a 0-d array has an index, but no hash
    assert ocn.plan_reduce("sum", a, [np.int64(1)], out)["red_size"] == (8,)
    axis = torch.tensor(1)
    assert ocn.plan_reduce("sum", a, [axis], out)["red_size"] == (8,)
    axis.fill_(0)                                                                  # the same object, another value
    tall = ocn.Tensor(1 << 41, "float", (8,), (4,))
    assert ocn.plan_reduce("sum", a, [axis], tall)["red_size"] == (4,)
