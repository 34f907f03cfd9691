"""FP32 operator: every coefficient is held to FP32's own rounding.

The error of one FP32 apply on uniform random values against the FP64 apply
(which the oracle tests pin to 1e-12) does not depend on the seed to more than
a few per cent: it is the sum of many roundings.  With coefficients rounded
once and plain sums it is 9.1e-8..9.6e-8 in 3-D (Q4..Q7) and 7.4e-8..7.7e-8 in 2-D;
the limits leave 15% for another order of the sums.  Mass coefficients one bit
coarser give 1.15e-7..1.41e-7 in 3-D."""
import sys

import pytest

from paper_2405_18982_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2405_18982_amd import dgmg  # noqa: E402

LIMIT = {2: 8.6e-8, 3: 1.1e-7}


@pytest.mark.parametrize("dim,k,L", [(2, 4, 3), (2, 5, 3), (2, 6, 3), (2, 7, 3), (3, 4, 2), (3, 5, 2), (3, 6, 2), (3, 7, 2)])
def test_fp32_apply_is_rounded_once(dim, k, L):
    print(f"fp32 apply error d={dim} k={k}", flush=True)
    sys.stdout.flush()
    prob = dgmg.Problem(dim, k, L)
    x = torch.from_numpy(inputs.uniform(101, (prob.ndofs(),))).to("cuda", torch.float32)
    ref = prob.apply(x.double())
    err = float((prob.apply(x).double() - ref).norm() / ref.norm())
    assert err <= LIMIT[dim], err
    prob.close()
