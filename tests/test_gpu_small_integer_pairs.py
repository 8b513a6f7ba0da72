"""+, -, *, / of 8- and 16-bit integers with floats in the kernels that convert on load: every
layout the planner has for them, at ragged and whole sizes, against the oracle (bit-exact)."""
from dataclasses import replace

import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

SMALL = ("uint8", "int8", "uint16", "int16")


@pytest.mark.parametrize("small", SMALL)
@pytest.mark.parametrize("first", (True, False))
def test_small_integers_with_floats(small, first):
    import paper_1810_08723_amd as ocn
    rng = rng_for(26000 + SMALL.index(small) * 2 + first)
    da, db = (small, "float") if first else ("float", small)
    cases = []
    for shape in ((1, 1), (3, 5), (29, 63), (7, 257), (3, 5003), (64, 128)):
        a, b = random_view(rng, da, shape), random_view(rng, db, shape)
        cases += [(a, b, shape), (random_view(rng, da, shape[::-1]).permute(1, 0), b, shape),
                  (a, random_view(rng, db, (1, shape[1])), shape), (random_view(rng, da, (shape[0], 1)), b, shape),
                  (a.flip(1), replace(b, byteswapped=True), shape)]
    for op in ("add", "sub", "mul", "div"):
        for a, b, shape in cases:
            out = View.empty("float", shape)
            dv = H.DeviceViews()
            assert ocn.plan_binary(op, dv.tensor(a), dv.tensor(b), dv.tensor(out))["specialised"]
            print("small integers", op, da, db, shape, a.strides, b.strides, flush=True)
            H.check_binary(op, a, b, out)
