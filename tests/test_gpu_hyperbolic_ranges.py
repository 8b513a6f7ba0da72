"""Complex hyperbolic functions of floats from the smallest arguments to the last before overflow, where the
reciprocal of e^|x| goes from one to a subnormal number, in each pair of byte orders."""
import numpy as np
import pytest

from workloads.values import rng_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("swap_in,swap_out", ((False, False), (True, False), (False, True), (True, True)))
@pytest.mark.parametrize("op", ("sinh", "cosh"))
def test_each_component_over_the_range(op, swap_in, swap_out):
    import torch
    import paper_1810_08723_amd as ocn
    n = 4099
    rng = rng_for(26100 + len(op) + 2 * swap_in + swap_out)
    mag = np.concatenate([np.exp(rng.uniform(np.log(1e-30), np.log(88.0), n - 1001)), rng.uniform(86.5, 88.0, 1000), [88.0]])
    x = (mag * rng.choice((-1.0, 1.0), n)).astype(np.float32)
    y = rng.uniform(-3.0, 3.0, n).astype(np.float32)
    z = np.stack([x, y], axis=1)
    src = torch.from_numpy((z.byteswap() if swap_in else z).copy()).to("cuda:0")
    out = torch.zeros_like(src)
    print("hyperbolic", op, swap_in, swap_out, flush=True)
    ocn.unary(op, ocn.Tensor(src.data_ptr(), "cfloat", (n,), (8,), 0, 0, src, swap_in),
              ocn.Tensor(out.data_ptr(), "cfloat", (n,), (8,), 0, 0, out, swap_out))
    got = out.cpu().numpy()
    got = (got.byteswap() if swap_out else got).astype(np.float64)
    x, y = x.astype(np.float64), y.astype(np.float64)
    s, c = np.sinh(x), np.cosh(x)
    want = np.stack([s * np.cos(y), c * np.sin(y)] if op == "sinh" else [c * np.cos(y), s * np.sin(y)], axis=1)
    # e^|x| - 1, the sum behind it and sine or cosine are each within two units, the quotient, the halved sum and the
    # product within one rounding each: under eight units of 2^-23, relative to each component (numbers below the
    # normal ones, where a unit is 2^-149)
    assert (np.abs(got - want) <= 8 * 2.0 ** -23 * np.abs(want) + 8 * 2.0 ** -149).all()
