"""One-dimensional tensors whose length is not a multiple of the vector, in operations that take
several vectors per lane: the elements behind the last whole vector, at every workgroup edge."""
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", (1, 3, 4, 5, 255, 256, 257, 1023, 1024, 1025, 1027, 4099, 100003))
def test_flat_tails(n):
    rng = rng_for(27000 + n)
    for da, dout in (("double", "int16"), ("float", "uint8"), ("cdouble", "bool"), ("int64", "int8"), ("int8", "double")):
        print("flat tail", n, da, dout, flush=True)
        a, out = random_view(rng, da, (n,)), View.empty(dout, (n + 7,)).slice(0, 0, n, 1)     # (nothing behind it changes)
        H.check_unary("ident", a, out)
        H.check_unary("ident", random_view(rng, da, (1,)), out)
    for dt in ("float", "double", "int32", "cfloat"):
        a, b = random_view(rng, dt, (n,)), random_view(rng, dt, (n,))
        H.check_binary("eq", a, b, View.empty("bool", (n,)))
        H.check_binary("absgt", a, random_view(rng, dt, (1,)), View.empty("bool", (n,)))
    f = random_view(rng, "float", (n,))
    H.check_unary("ident", f.in_other_byte_order(), View.empty("half", (n,)))
